"""Build the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libguard_hip.so")
SCORE_SOURCES = ["score.hip", "score_z.hip"]
RAGGED_SOURCES = ["score_ragged_few.hip", "score_ragged_few_z.hip", "score_ragged_many.hip",
                  "score_ragged_many_z.hip", "score_ragged_columns.hip", "score_ragged_columns_z.hip"]
SOURCES = [*RAGGED_SOURCES, *SCORE_SOURCES, "api.hip", "window.hip", "topk.hip", "severity.hip", "sweep.hip", "ledger.hip", "membership.hip"]

# One rounding per written operation (no FMA contraction), IEEE divide,
# denormals kept, and no packed-fp32 instructions.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # atomics as they are written: the optimiser would reduce the operands of the active lanes
    # first, in a loop or a scan, where mostly one lane or a few of a wave have one (scoring 1 to 2 %
    # slower with it, the ledger up to 2 %, the 64 slowest of 8 192 equal scores 11.3 us instead of
    # 9.3, severity of 8 192 nodes 10.9 instead of 10.4).  Where every lane adds to one word the
    # kernels reduce by hand, unless that is seldom.
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    "-Wall", "-Wno-unused-command-line-argument",
    # the compiler's own account of registers, spills and LDS per kernel (kept as text
    # beside the objects and checked below)
    "-Rpass-analysis=kernel-resource-usage",
]

# The scoring kernel keeps a whole column in registers and is laid out for 16 waves per
# CU (20 in the 256-thread tilings of up to eight rows): every instantiation must stay within
# 128 vector registers, and those named below may spill none of them.
VGPR_BUDGET = 128


def resource_file(src: str) -> str:
    return os.path.join(HERE, "_build", src.replace(".hip", ".resources.txt"))


def parse_resources(text: str) -> dict:
    """{kernel symbol: {field: int}} from -Rpass-analysis=kernel-resource-usage remarks."""
    out, cur = {}, None
    for line in text.splitlines():
        m = re.search(r"remark:\s+Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+([A-Za-z][A-Za-z /\[\]]*?):\s+(-?\d+|True|False)\s", line)
        if m and cur is not None:
            v = m.group(2)
            cur[m.group(1).strip()] = int(v) if v.lstrip("-").isdigit() else (v == "True")
    return out


def tiling_of(symbol: str):
    """(NT, ROWS, LOG_NB, FULL, SPLIT, WANT_Z) of a mangled score_kernel<...> symbol, or None."""
    m = re.search(r"score_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb([01])ELb([01])ELb([01])E", symbol)
    return tuple(int(g) for g in m.groups()) if m else None


def waves_of(symbol: str) -> int:
    """Waves per SIMD that the launcher counts on for a scoring kernel (waves_of in score.hip)."""
    m = re.search(r"score_(?:ragged_)?kernelILi(\d+)ELi(\d+)ELi\d+E(?:Lb[01]E)+?Lb([01])EE", symbol)
    return 5 if m and (int(m.group(1)), m.group(3)) == (256, "0") and int(m.group(2)) <= 8 else 4


def is_ragged(symbol: str) -> bool:
    """A score_ragged_kernel<...> symbol: a rank count that fills no tiling exactly."""
    return "score_ragged_kernelILi" in symbol


# Ragged tilings (rank counts that do not fill the register tile: bounds checks on the last
# rows), the one-wave tilings of up to 4 096 ranks and the per-column route
# of short batches (latency-bound: one column per workgroup) may keep a few registers in
# scratch memory; the exact-fit batch tilings of 256 threads and more may not.
RAGGED_SCRATCH_LIMIT = 128     # bytes per lane


def check_register_budget(resources: dict) -> list:
    """Violations among the score_kernel instantiations (empty = within budget)."""
    bad = []
    for name, r in resources.items():
        t = tiling_of(name)
        if t is None and not is_ragged(name):
            continue
        full = t is not None and bool(t[3]) and t[0] >= 256 and not t[4]
        if r.get("VGPRs", 0) + r.get("AGPRs", 0) > VGPR_BUDGET:
            bad.append(f"{name}: {r.get('VGPRs')} VGPRs + {r.get('AGPRs')} AGPRs > {VGPR_BUDGET}")
        scratch = r.get("ScratchSize [bytes/lane]", 0)
        if r.get("Dynamic Stack", False) or scratch > (0 if full else RAGGED_SCRATCH_LIMIT) or \
                (full and r.get("VGPRs Spill", 0)):
            bad.append(f"{name}: {r.get('VGPRs Spill')} vector registers spilled, {scratch} bytes of scratch per lane")
        if r.get("Occupancy [waves/SIMD]", 0) < waves_of(name):
            bad.append(f"{name}: occupancy {r.get('Occupancy [waves/SIMD]')} waves per SIMD < {waves_of(name)}")
    return bad


def build(verbose: bool = False, extra=()) -> str:
    """Compile every source and link libguard_hip.so; always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stderr=subprocess.PIPE, text=True)))
        objs.append(obj)
    for src, p in procs:
        _, err = p.communicate()
        remarks = [l for l in err.splitlines() if "-Rpass-analysis=kernel-resource-usage" in l]
        with open(resource_file(src), "w") as f:
            f.write("\n".join(remarks) + "\n")
        err = "\n".join(l for l in err.splitlines()
                        if "packed-fp32-ops" not in l and "-Rpass-analysis=kernel-resource-usage" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
    bad = []
    for src in [*SCORE_SOURCES, *RAGGED_SOURCES]:
        with open(resource_file(src)) as f:
            res = parse_resources(f.read())
        if not any(is_ragged(k) if src in RAGGED_SOURCES else tiling_of(k) for k in res):
            bad.append(f"{src}: the compiler reported no instantiation of the scoring kernel")
        bad += check_register_budget(res)
    if bad:
        raise RuntimeError("register budget of the scoring kernel exceeded:\n  " + "\n  ".join(bad))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
