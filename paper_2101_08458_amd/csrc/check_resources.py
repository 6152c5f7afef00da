#!/usr/bin/env python3
"""Build-time check of the register-spill precondition of the main kernel's inline-assembly LDS reads.

The direct-read variants of igemm_kernel (B source 2, 3 or 5) issue their transposing LDS reads as inline
assembly and wait for them themselves; a fragment register the compiler spilled between such a read and the
kernel's own wait would be saved before its data has arrived.  Those variants must therefore compile to zero
scratch.  This script reads the compiler's kernel-resource-usage remarks (one file per kernel translation
unit, written by the Makefile) and fails when a variant that uses the inline-assembly reads reports scratch
or spilled vector registers.  Variants that keep the compiler's builtins (32-byte fragments on wave windows of eight or more
MFMA tiles: igemm.hpp, ASM_TR) may spill and are only listed.

The tiles of 128 rows and more with 16x16 accumulators issue their MFMAs as inline assembly, whose operands must not be written by
vector instructions just before; a spilled register would be copied there, so those kernels must not spill either, and in the
instructions of the object beside each FILE.res (llvm-objdump, where it is installed) no vector instruction may write an operand of
such an MFMA within the FAR wait states before it, also around a loop.

usage: check_resources.py FILE.res [FILE.res ...]      exit status 1 on a violation
"""
import glob
import os
import re
import shutil
import subprocess
import sys
import tempfile

NAME = re.compile(r"Function Name: _ZN4unit12igemm_kernelI((?:Li\d+E)+)EEvNS_9IgemmArgsE")
FIELD = re.compile(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\S+) \[-Rpass-analysis")
DIRECT = (2, 3, 5)                     # BSRC_NCHW, BSRC_NCHWS, BSRC_NCHWE


def kernels(path):
    cur = None
    for line in open(path, errors="replace"):
        m = NAME.search(line)
        if m:
            cur = {"args": [int(v) for v in re.findall(r"Li(\d+)E", m.group(1))]}
            yield cur
            continue
        if cur is not None:
            f = FIELD.search(line)
            if f:
                cur[f.group(1).strip()] = f.group(2)


OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
FAR = 4
INST = re.compile(r"^\s+(\S+)(.*?)\s*// ([0-9A-F]+): ")
REGS = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])")


def disassembled(obj):
    """(kernel's template arguments, [(address, mnemonic, operands)]) of every igemm_kernel of 16x16 MFMAs and 128 rows or more."""
    with tempfile.TemporaryDirectory() as tmp:
        local = shutil.copy(obj, tmp)
        subprocess.run([OBJDUMP, "--offloading", os.path.basename(local)], cwd=tmp, check=True, stdout=subprocess.DEVNULL)
        for part in glob.glob(os.path.join(tmp, "*gfx950*")):
            text = subprocess.run([OBJDUMP, "-d", part], check=True, capture_output=True, text=True).stdout
            for chunk in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
                name = chunk[:chunk.index(">")]
                args = [int(v) for v in re.findall(r"Li(\d+)E", name)] if "igemm_kernel" in name and not name.endswith(".kd") else []
                if len(args) == 12 and args[7] == 16 and args[1] >= 128:
                    yield args, [(int(m.group(3), 16), m.group(1), m.group(2)) for m in map(INST.match, chunk.splitlines()) if m]


def registers(operand):
    return {(k, r) for k, one, lo, hi in REGS.findall(operand) for r in range(int(one or lo), int(one or hi) + 1)}


def late_writes(code):
    """MFMAs with an operand that a vector instruction wrote fewer than FAR wait states before."""
    at, found = {a: i for i, (a, _, _) in enumerate(code)}, []

    def step(i, ages):              # ages: register -> wait states since it was written
        addr, op, operands = code[i]
        if op.startswith("v_mfma") and any(ages.get(r, FAR) < FAR for r in registers(operands.split(",", 1)[1])):
            found.append(hex(addr))
        wait = int(operands.split()[0], 0) + 1 if op == "s_nop" else 1
        ages = {r: n + wait for r, n in ages.items() if n + wait < FAR}
        if op.startswith("v_") and not op.startswith("v_mfma"):
            ages.update((r, 0) for r in registers(operands.split(",", 1)[0]))
        return ages

    ages = {}
    for i, (addr, op, operands) in enumerate(code):
        ages = step(i, ages)
        if op.startswith(("s_cbranch", "s_branch")):
            jump = int(operands.split()[0], 0)
            j = at.get(addr + 4 + 4 * (jump - 65536 if jump > 32767 else jump))
            ahead = dict(ages)
            while j is not None and j < len(code) and ahead:
                ahead = step(j, ahead)
                j += 1
    return found


def main(paths):
    late, checked = [], 0
    for p in paths:
        obj = os.path.splitext(p)[0] + ".o"
        if not (os.path.exists(OBJDUMP) and os.path.exists(obj)):
            continue
        for args, code in disassembled(obj):
            checked += 1
            late += [(p, args, w) for w in [late_writes(code)] if w]
    bad, quad, seen, spilled_builtin = [], [], 0, 0
    for p in paths:
        for k in list(kernels(p)):
            dt, bm, bn, bkb, wgm, wgn, wgk, mf, nst, occ, bsrc, epi = k["args"]
            if mf == 16 and bm >= 128 and int(k.get("VGPRs Spill", "0")):
                quad.append((p, k["args"], int(k["VGPRs Spill"])))
            if bsrc not in DIRECT:
                continue
            fw = 2 if dt == 5 else 1
            asm_tr = not (fw == 2 and (bm // wgm // mf) * (bn // wgn // mf) >= 8)
            scratch = int(k.get("ScratchSize", "0"))
            # (spilled SGPRs live in lanes of a reserved VGPR: they never touch the fragment registers)
            spills = int(k.get("VGPRs Spill", "0"))
            seen += 1
            if asm_tr and (scratch or spills):
                bad.append((p, k["args"], scratch, spills))
            elif scratch or spills:
                spilled_builtin += 1
    if not seen:
        print("check_resources: no direct-read igemm_kernel variant found in", paths, file=sys.stderr)
        return 1
    for p, args, scratch, spills in bad:
        print(f"check_resources: {p}: igemm_kernel<{', '.join(map(str, args))}> uses inline-assembly LDS reads but "
              f"has {scratch} bytes of scratch per lane and {spills} spilled vector registers", file=sys.stderr)
    for p, args, spills in quad:
        print(f"check_resources: {p}: igemm_kernel<{', '.join(map(str, args))}> issues its MFMAs as inline assembly but has "
              f"{spills} spilled vector registers", file=sys.stderr)
    print(f"check_resources: {seen} direct-read variants, {len(bad)} violations, "
          f"{spilled_builtin} builtin-read variants with spills (allowed)")
    for p, args, where in late:
        print(f"check_resources: {p}: igemm_kernel<{', '.join(map(str, args))}>: operands of inline-assembly MFMAs written just before "
              f"them, at {', '.join(where[:5])}", file=sys.stderr)
    print(f"check_resources: operands of {checked} kernels with inline-assembly MFMAs looked through, {len(late)} written too late")
    return 1 if bad or quad or late else 0


if __name__ == "__main__":
    sys.exit(main(sys.argv[1:]))
