"""The mid-token kernels issue their MFMAs as inline asm, which the compiler's hazard recogniser does not see: in the
generated code no vector-ALU instruction may write an A or B operand register of such an MFMA within the two
instructions in front of it, and within a basic block no accumulator may be read within 18 wait states behind one.
Usage: mfma_operand_check.py file.s -> "OK <mfmas checked>" or the first violation."""
import re
import sys


def regs(op):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", op) or re.fullmatch(r"v(\d+)", op)
    if not m:
        return set()
    g = m.groups()
    return set(range(int(g[0]), int(g[-1]) + 1))


def main(path):
    text, checked = open(path).read(), 0
    for name, body in re.findall(r"^(_ZN\S*mid_main_kernelILi\d+ELi4E\S*):.*?\n(.*?)\.Lfunc_end", text, re.S | re.M):
        recent, since_mfma = [], 99                           # (instruction, registers it writes), newest last
        for line in body.split("\n"):
            if line.startswith(".LBB"):
                since_mfma = 99                               # what came before in execution is not what stands above
            line = line.split(";")[0].strip()
            if not line or line.startswith("."):
                continue
            op, _, rest = line.partition(" ")
            args = [a.strip() for a in rest.split(",")]
            if op == "s_nop":
                recent += [("s_nop", set())] * (int(args[0]) + 1)
                since_mfma += int(args[0]) + 1
                continue
            if op.startswith("v_mfma") and args[0].startswith("a["):
                src = regs(args[1]) | regs(args[2])
                for prev, wrote in recent[-2:]:
                    if wrote & src:
                        print(f"FAIL {name}: '{prev}' right in front of '{line}'")
                        return 1
                checked += 1
                since_mfma = 0
            else:
                since_mfma += 1
                if op.startswith("v_accvgpr_read") and since_mfma < 18:
                    print(f"FAIL {name}: '{line}' {since_mfma} wait states behind an MFMA")
                    return 1
            recent.append((line, regs(args[0]) if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp")) else set()))
            recent = recent[-4:]
    print(f"OK {checked}")
    return 0


if __name__ == "__main__":
    sys.exit(main(sys.argv[1]))
