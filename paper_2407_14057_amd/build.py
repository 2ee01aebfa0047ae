"""Builds the C-ABI library (csrc/*.hip -> liblazyllm.so) for gfx950 with hipcc."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblazyllm.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep hipcc from forming packed-fp32 VALU ops out of scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


# Sources whose kernels keep their accumulators in accumulation registers by name (see csrc/gemm_w4.h)
NAMED_ACCUMULATORS = ("gemm_w4.hip", "gemm_w4_fp8.hip")


def _registers(kind: str, operand: str) -> set:
    """Numbers of the vector (kind "v") or accumulation ("a") registers that an operand names."""
    m = re.fullmatch(r"-?\|?%s(?:(\d+)|\[(\d+):(\d+)\])\|?" % kind, operand.strip())
    if m is None:
        return set()
    return {int(m.group(1))} if m.group(1) else set(range(int(m.group(2)), int(m.group(3)) + 1))


def accumulator_faults(asm: str) -> list:
    """What in the AMD assembly of kernels with named accumulators could corrupt them.

    The compiler does not know what a0 .. a255 hold, nor that the products in the inline assembly read their
    operands as matrix instructions do.  So: outside the inline assembly no instruction may name an
    accumulation register; no kernel may have vector spills or scratch memory; and no vector
    instruction may write an operand of a product less than two wait states in front of it."""
    faults = []
    kernel, in_asm, written = "?", False, []          # written: (wait states ago, registers) of recent vector writes
    for number, line in enumerate(asm.split("\n"), 1):
        text = line.strip()
        if "#ASMSTART" in text or "#ASMEND" in text:
            in_asm = "#ASMSTART" in text
            continue
        label = re.match(r"(\w+):", line)
        if label:
            if not label.group(1).startswith("."):
                kernel = label.group(1)
            written = []
            continue
        code = text.split(";")[0].strip()
        if not code or code.startswith("."):
            spill = re.match(r"\.(vgpr_spill_count|private_segment_fixed_size):\s*(\d+)", code)
            if spill and int(spill.group(2)) != 0:
                faults.append("line %d: %s is %s" % (number, spill.group(1), spill.group(2)))
            continue
        op, _, rest = code.partition(" ")
        operands = re.split(r",\s*", rest.strip()) if rest else []
        if not in_asm and any(_registers("a", x.split(" ")[0]) for x in operands):
            faults.append("line %d, %s: the compiler uses an accumulation register: %s" % (number, kernel, code))
        if op.startswith("v_mfma"):
            reads = set().union(*(_registers("v", x.split(" ")[0]) for x in operands[1:3]))
            for ago, regs in written:
                if ago < 2 and reads & regs:
                    faults.append("line %d, %s: an operand is written %d wait states ahead: %s" % (number, kernel, ago, code))
        states = int(operands[0], 0) + 1 if op == "s_nop" else 1
        written = [(ago + states, regs) for ago, regs in written if ago + states < 2]
        if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp", "v_readlane", "v_readfirstlane", "v_accvgpr_write")):
            written.append((0, _registers("v", operands[0].split(" ")[0])))
    return faults


def _check_accumulators(source: str) -> None:
    stem = os.path.basename(source)[:-4]
    found = glob.glob(os.path.join(CSRC, stem + "-hip-amdgcn-amd-amdhsa-*.s"))
    if len(found) != 1:
        raise RuntimeError("%s: one assembly file expected, found %s" % (source, found))
    for path in found:
        with open(path) as f:
            faults = accumulator_faults(f.read())
        if faults:
            raise RuntimeError("%s: the accumulators are not safe\n%s" % (source, "\n".join(faults[:20])))


def build(verbose: bool = True) -> str:
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    objs = []
    procs = []
    for s in srcs:
        o = os.path.join(CSRC, os.path.basename(s)[:-4] + ".o")
        objs.append(o)
        keep = ["-save-temps=obj", "-Wno-array-bounds"] if os.path.basename(s) in NAMED_ACCUMULATORS else []
        procs.append((s, subprocess.Popen([HIPCC, *FLAGS, *keep, "-c", s, "-o", o],
                                          stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    for s, p in procs:
        out = p.communicate()[0].decode()
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (s, out))
        if os.path.basename(s) in NAMED_ACCUMULATORS:
            _check_accumulators(s)
            for path in glob.glob(os.path.join(CSRC, os.path.basename(s)[:-4] + "-h*")) + glob.glob(s + "-hip-*"):
                os.remove(path)
        if verbose:
            print("compiled", os.path.basename(s), flush=True)
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    if verbose:
        print("linked", LIB, flush=True)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
