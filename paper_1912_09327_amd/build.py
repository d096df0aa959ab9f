"""Build ``liblbt1.so`` (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

Usage: ``python -m paper_1912_09327_amd.build`` (or ``build()``); it always
recompiles.  The sources compile in parallel and link into one shared library
next to this file.
"""
import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblbt1.so")
SOURCES = ["lbt1_kernels.hip", "lbt1_runtime.hip", "lbt1_batch.hip", "lbt1_probe.hip", "lbt1_3d.hip"]
# sources compiled once per storage precision (LBT1_PREC), the longest to compile first
PREC_SOURCES = ["lbt1_step_kernels.hip", "lbt1_batch_step_kernels.hip", "lbt1_tile_kernels.hip"]
UNITS = [(s, p) for s in PREC_SOURCES for p in (1, 2, 3, 0)] + [(s, None) for s in SOURCES]
# sources whose kernels must neither spill registers nor use scratch memory
CHECKED = PREC_SOURCES + ["lbt1_kernels.hip", "lbt1_3d.hip"]
# ... except scalar registers, kept in lanes of vector registers instead of scratch memory, by
# these kernels (a part of the mangled name: most of them): the FP64 march, whose 64-bit weights
# take pairs of scalar registers and whose blocks of 8 wavefronts have vector ones to spare
SGPR_SPILLS = {"k_step3_marchILi0E": 48}

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
# -ffp-contract=off: every kernel rounds exactly as its source is written, which
# keeps the kernel families bitwise identical.  Packed FP32 instructions are
# disabled for the device code.
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", "-I", os.path.join(ROOT, "include"),
]


def _resources(text):
    """Per-kernel (scratch bytes, SGPR spills, VGPR spills) from the compiler's
    kernel-resource-usage remarks."""
    res, name = {}, None
    for ln in text.splitlines():
        if "Function Name:" in ln:
            name = ln.split("Function Name:")[1].split("[")[0].strip()
            res[name] = [0, 0, 0]
        elif name and "ScratchSize [bytes/lane]:" in ln:
            res[name][0] = int(ln.split("ScratchSize [bytes/lane]:")[1].split("[")[0])
        elif name and "SGPRs Spill:" in ln:
            res[name][1] = int(ln.split("SGPRs Spill:")[1].split("[")[0])
        elif name and "VGPRs Spill:" in ln:
            res[name][2] = int(ln.split("VGPRs Spill:")[1].split("[")[0])
    return res


def spills(name, res):
    """Whether (scratch bytes, SGPR spills, VGPR spills) of a kernel are more than it may have."""
    allowed = max((n for part, n in SGPR_SPILLS.items() if part in name), default=0)
    return res[0] > 0 or res[1] > allowed or res[2] > 0


def _compile(src, prec, out, verbose):
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", out]
    if prec is not None:
        cmd.append(f"-DLBT1_PREC={prec}")
    if src in CHECKED:
        cmd.append("-Rpass-analysis=kernel-resource-usage")
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    lines = [ln for ln in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in ln]
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n" + "\n".join(lines))
    if src in CHECKED:
        # No step kernel may spill registers or use scratch memory: the strip
        # kernels are sized to stay in registers, and a spilling variant is a
        # design error (it is not built).
        bad = {k: v for k, v in _resources(r.stdout + r.stderr).items() if spills(k, v)}
        if bad:
            raise RuntimeError("kernels spill or use scratch (scratch B/lane, SGPR, VGPR spills): "
                               + "; ".join(f"{k}: {v}" for k, v in sorted(bad.items())))
        lines = [ln for ln in lines if "kernel-resource-usage" not in ln]
    return "\n".join(lines)


def build(verbose: bool = False) -> str:
    tmp = tempfile.mkdtemp(prefix="lbt1_build_")
    try:
        objs = [os.path.join(tmp, f"{s}.{p}.o") for s, p in UNITS]
        with cf.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
            for msg in ex.map(lambda a: _compile(*a[0], a[1], verbose), zip(UNITS, objs)):
                if msg.strip() and verbose:
                    print(msg)
        cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", LIB + ".tmp"] + objs
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        os.replace(LIB + ".tmp", LIB)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
