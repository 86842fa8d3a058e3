"""The skinny products' loop over K holds what it needs of a job in registers: in the generated code no scalar load may
stand inside a loop that issues MFMAs (a job is read through an index into the kernel's arguments, and the compiler would
load its fields again in front of every predicated load).
Usage: small_loop_check.py file.s -> "OK <kernels checked>" or the first violation."""
import re
import sys


def main(path):
    text, checked = open(path).read(), 0
    for name, body in re.findall(r"^(_ZN\S*small_jobs?_kernel\S*):.*?\n(.*?)\.Lfunc_end", text, re.S | re.M):
        lines = [l.split(";")[0].strip() for l in body.split("\n")]
        label = {l[:-1]: i for i, l in enumerate(lines) if l.startswith(".LBB") and l.endswith(":")}
        loops = 0
        for i, l in enumerate(lines):
            m = re.match(r"s_c?branch\S*\s+(\.LBB\S+)", l)
            if not m or label.get(m[1], i) >= i:
                continue                                     # a backward branch closes a loop
            loop = [x for x in lines[label[m[1]] + 1:i] if x]
            if loop and loop[0] == "s_endpgm":
                continue                                     # or leads to the kernel's one exit
            if not any(x.startswith("v_mfma") for x in loop):
                continue
            loops += 1
            bad = [x for x in loop if x.startswith("s_load")]
            if bad:
                print(f"FAIL {name}: {len(bad)} scalar loads in the loop, '{bad[0]}'")
                return 1
        if not loops:
            print(f"FAIL {name}: no loop with MFMAs found")
            return 1
        checked += 1
    print(f"OK {checked}")
    return 0


if __name__ == "__main__":
    sys.exit(main(sys.argv[1]))
