"""Build libmsc.so (host C++ + HIP kernels for gfx950) in-tree.

Every source is compiled by hipcc for --offload-arch=gfx950 with packed
FP32 instructions disabled, then linked into
paper_2609_19116_amd/libmsc.so.  Run ``python -m paper_2609_19116_amd.build``.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
CSRC = PKG / "csrc"
OUT = PKG / "libmsc.so"
BUILD = ROOT / "_build"

SOURCES = [
    CSRC / "host" / "circuit.cpp",
    CSRC / "host" / "prescreen_compile.cpp",
    CSRC / "host" / "sampler.cpp",
    CSRC / "host" / "stats.cpp",
    CSRC / "host" / "order.cpp",
    CSRC / "host" / "camps.cpp",
    CSRC / "host" / "capi.cpp",
    CSRC / "kernels" / "mps.hip",
    CSRC / "kernels" / "mps_fast.hip",
    CSRC / "kernels" / "prescreen.hip",
    CSRC / "kernels" / "sampler.hip",
    CSRC / "kernels" / "batch.hip",
    CSRC / "kernels" / "camps.hip",
    CSRC / "kernels" / "twosite.hip",
    CSRC / "kernels" / "lx.hip",
]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
COMMON = ["-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
          f"-I{ROOT / 'include'}", f"-I{CSRC}"]
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang",
          "-packed-fp32-ops"]

# Kernels whose registers the build checks: source, name, and the wavefronts
# per SIMD that the launch counts on, with no vector register spilled.
RESOURCES = {
    "mps_fast.hip": {"mps_fast_wave_kernel": 3, "mps_fast_mid_kernel": 2,
                     "mps_fast_group_kernel": 2},
    "camps.hip": {"camps_kernel": 2},
}


def kernel_resources(asm: str) -> dict:
    """Per kernel (mangled name) of a device assembly text the wavefronts per
    SIMD and the spilled vector registers."""
    waves, out, fn = {}, {}, None
    for ln in asm.splitlines():
        m = re.match(r"(_Z\w+):", ln)
        fn = m[1] if m else fn
        if (m := re.match(r"; Occupancy: (\d+)", ln)):
            waves[fn] = int(m[1])
        elif (m := re.match(r"\s+\.name:\s+(_Z\w+)", ln)):
            fn = m[1]
        elif (m := re.match(r"\s+\.vgpr_spill_count:\s+(\d+)", ln)):
            out[fn] = {"waves": waves[fn], "vgpr_spills": int(m[1])}
    return out


def check_resources(source: str, asm: str) -> None:
    """Raise if a kernel of RESOURCES[source] spills vector registers, has
    fewer resident wavefronts than its launch counts on, or is not there."""
    seen = kernel_resources(asm)
    for name, waves in RESOURCES.get(source, {}).items():
        found = {k: r for k, r in seen.items() if re.search(rf"\d{name}(?![a-z_])", k)}
        if not found:
            raise RuntimeError(f"{source}: no kernel {name}")
        for k, r in found.items():
            if r["vgpr_spills"] > 0 or r["waves"] < waves:
                raise RuntimeError(f"{source}: {k} needs {waves} wavefronts per SIMD and no "
                                   f"spilled vector registers, the compiler gives it {r}")


def lost_lanes(asm: str) -> list:
    """(kernel, instructions) per place in a device assembly text where vector
    instructions stand between a join of divergent paths and the restore of the
    execution mask.

    The register allocator puts copies and spills at a block's start behind the
    mask's restore, but takes the block to start earlier where scalar registers
    are spilled there too (v_writelane); such copies run for the lanes of one
    path only and the others keep stale values.  An earlier form of the
    one-wavefront shot kernel gave wrong FP32 results that way (12 instructions
    before the restore that ends the search for overlapping pairs, found in its
    assembly); register pressure decides where it happens, so every build looks.
    """
    joins = set(re.findall(r"s_cbranch_execz\s+(\S+)", asm))
    found, kernel, pending = [], None, None
    for ln in asm.splitlines():
        ins = ln.split(";")[0].strip()
        label = re.match(r"(\S+):$", ins)
        if label:
            if not label[1].startswith("."):
                kernel = label[1]
            pending = [] if label[1] in joins else None
            continue
        op = ins.split()[0] if ins else ""
        if op == "s_cbranch_execnz":
            pending = []                   # falls through with no lane left
        elif pending is None or not op:
            continue
        elif re.match(r"s_or_b64 exec, exec", ins):
            if pending:
                found.append((kernel, pending))
            pending = None
        elif ("saveexec" in op or re.match(r"s_\w+ exec\b", ins)
              or op.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_setpc"))):
            pending = None
        elif (op.startswith(("v_", "ds_", "scratch_", "global_", "flat_", "buffer_"))
              and not op.startswith(("v_writelane", "v_readlane", "v_readfirstlane", "v_nop"))):
            pending.append(ins)
    return found


def device_assembly(src: Path, out: Path) -> str:
    """Compile a kernel source to the object `out`; its device assembly."""
    with tempfile.TemporaryDirectory(dir=out.parent) as tmp:
        obj = Path(tmp) / out.name
        _run([HIPCC, "-x", "hip", *DEVICE, *COMMON, "-save-temps=obj", "-c", str(src), "-o",
              str(obj)])
        asm = "".join(f.read_text() for f in Path(tmp).glob(f"*-{ARCH}.s"))
        os.replace(obj, out)
    return asm


def _compile(src: Path) -> Path:
    obj = BUILD / (src.stem + (".hip.o" if src.suffix == ".hip" else ".o"))
    if src.suffix == ".hip":
        asm = device_assembly(src, obj)
        check_resources(src.name, asm)
        lost = lost_lanes(asm)
        if not asm or lost:
            raise RuntimeError(f"{src.name}: vector instructions ahead of the execution mask's "
                               f"restore: {lost or 'no device assembly'}")
    else:
        # host-only sources still include the HIP runtime headers
        _run([HIPCC, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *COMMON, "-c",
              str(src), "-o", str(obj)])
    return obj


def _run(cmd: list) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    warn = [ln for ln in r.stderr.splitlines()
            if "packed-fp32-ops" not in ln and ln.strip()]
    if warn:
        sys.stderr.write("\n".join(warn) + "\n")


def build(verbose: bool = True) -> Path:
    if shutil.which(HIPCC) is None and not Path(HIPCC).exists():
        raise RuntimeError("hipcc not found")
    BUILD.mkdir(exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = OUT.with_suffix(".so.tmp")
    cmd = [HIPCC, "-shared", f"--offload-arch={ARCH}", "-o", str(tmp), *map(str, objs),
           "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, OUT)
    if verbose:
        print(f"built {OUT}")
    return OUT


if __name__ == "__main__":
    build()
