// Host-side check of the list kernels' plan against its plain definition (no GPU needed): the boundaries are those of the
// smallest bound under which a segment-by-segment greedy walk covers the line, found by halving from 0, for both cost
// models; and planning, which every call does on the host, takes less than 0.7 of that plain search's time on the lists of a
// decoder block.  Prints "OK <plans> <worst share of the plain search's time, in percent>" or the first violation.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <vector>

#include "launch.hpp"

using namespace qlora;

struct Costs { int tail, stage, item; };
static const Costs kCosts[2][2] = {{{30, 70, 40}, {70, 200, 120}}, {{3, 4, 4}, {2, 4, 6}}};   // [backward][compact]

// Fills q from the shapes in P (n_slabs, ups, unit0, total_units, adapters).
static void plain(bool bwd, bool compact, const ListPlan& P, int n, ListPart* q, int* max_contrib) {
  const Costs c = kCosts[bwd][compact];
  const int units = P.total_units, adapters = P.part.n_adapter;
  std::vector<int> slab_end;
  for (int l = 0; l < n; ++l)
    for (int s = 0; s < P.n_slabs[l]; ++s) slab_end.push_back(P.unit0[l] + (s + 1) * P.ups[l]);
  auto walk = [&](int grid, long long T, int* start) {
    int u = 0, next = 0;
    for (int rho = 0; rho < grid; ++rho) {
      if (start) start[rho] = u;
      long long budget = T - (long long)c.item * (rho < adapters ? (adapters - rho + grid - 1) / grid : 0);
      for (bool took = false; u < units && budget > 0; took = true) {
        while (slab_end[next] <= u) ++next;
        const long long overhead = c.tail + (u == (next ? slab_end[next - 1] : 0) ? c.stage : 0);
        if (budget <= overhead) { u += !took; break; }
        const int take = (int)std::min<long long>(budget - overhead, slab_end[next] - u);
        u += take; budget -= overhead + take;
      }
    }
    if (start) start[grid] = units;
    return u >= units;
  };
  for (int grid = std::min(kListGridMax, units); grid >= 1; grid = grid > 32 ? grid - 32 : grid - 1) {
    long long lo = 0, hi = units + (long long)(c.tail + c.stage) * P.total_slabs + (long long)c.item * adapters + 1;
    while (hi - lo > 1) { const long long mid = (lo + hi) / 2; if (walk(grid, mid, nullptr)) hi = mid; else lo = mid; }
    q->grid = grid;
    walk(grid, hi, q->start);
    int worst = 1;
    for (int l = 0; l < n; ++l) {
      max_contrib[l] = 1;
      for (int s = 0; s < P.n_slabs[l]; ++s) {
        const int U0 = P.unit0[l] + s * P.ups[l];
        max_contrib[l] = std::max(max_contrib[l], list_rho_of(*q, U0 + P.ups[l] - 1) - list_rho_of(*q, U0) + 1);
      }
      worst = std::max(worst, max_contrib[l]);
    }
    if (worst <= 23) return;
  }
}

static int check(bool bwd, bool compact, int M, int n, const int* h, const int* o, const int* r) {
  const ListPlan P = fewlist_plan(bwd, M, n, h, o, r, compact);
  if (!P.ok) return -1;
  ListPart q{};
  int mc[kListMax];
  plain(bwd, compact, P, n, &q, mc);
  if (P.part.grid != q.grid || std::memcmp(P.part.start, q.start, (q.grid + 1) * sizeof(int)) || std::memcmp(P.max_contrib, mc, n * sizeof(int))) {
    std::printf("FAIL %s compact %d n %d: grid %d, plain search %d\n", bwd ? "bwd" : "fwd", compact, n, P.part.grid, q.grid);
    return 1;
  }
  return 0;
}

int main() {
  int plans = 0;
  unsigned long long state = 0x9E3779B97F4A7C15ull;
  auto rnd = [&](int m) { state = state * 6364136223846793005ull + 1442695040888963407ull; return (int)((state >> 33) % (unsigned)m); };
  for (int it = 0; it < 4000; ++it) {
    int h[kListMax], o[kListMax], r[kListMax];
    const int n = 1 + rnd(kListMax), M = 1 + rnd(16);
    for (int l = 0; l < n; ++l) {
      const int big = rnd(4);
      h[l] = 64 * (1 + rnd(big == 0 ? 400 : big == 1 ? 40 : 4));
      o[l] = 64 * (1 + rnd(big == 0 ? 4 : big == 1 ? 40 : 400));
      r[l] = 16 * rnd(5);
    }
    const int rc = check(it & 1, it & 2, M, n, h, o, r);
    if (rc > 0) return rc;
    plans += rc == 0;
  }
  double worst = 0;
  for (int d : {4096, 5120, 8192})
    for (int bwd = 0; bwd < 2; ++bwd) {
      const int f = d == 4096 ? 11008 : d == 5120 ? 13824 : 22016;
      const int h[7] = {d, d, d, d, d, d, f}, o[7] = {d, d, d, d, f, f, d}, r[7] = {64, 64, 64, 64, 64, 64, 64};
      const ListPlan P = fewlist_plan(bwd, 4, 7, h, o, r);
      double best[2] = {1e9, 1e9};
      for (int rep = 0; rep < 400; ++rep)
        for (int k = 0; k < 2; ++k) {
          ListPart q{};
          int mc[kListMax];
          const auto t = std::chrono::steady_clock::now();
          if (k) plain(bwd, false, P, 7, &q, mc); else (void)fewlist_plan(bwd, 4, 7, h, o, r);
          best[k] = std::min(best[k], std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t).count());
        }
      worst = std::max(worst, best[0] / best[1]);
    }
  if (worst > 0.7) { std::printf("FAIL planning takes %.0f %% of the plain search\n", 100 * worst); return 1; }
  std::printf("OK %d %.0f\n", plans, 100 * worst);
  return 0;
}
