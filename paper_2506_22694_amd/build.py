"""Builds libvocabtrim.so (the HIP kernels + C ABI) in-tree for gfx950 with hipcc."""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig
import warnings

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libvocabtrim.so")
BIND = os.path.join(PKG, "_vt_bind" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
BIND_STAMP = os.path.join(OBJ, "vt_bind.command")      # how BIND was built
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


# The draft-step kernels issue their loads from inline assembly and wait for them by hand; the compiler
# does not know that such a register is still in flight, so a spill of one would save a value that
# has not arrived yet.  Their sources must therefore compile without any scratch memory.
NO_SCRATCH = ("vt_head_", "vt_row_select")
# For the same reason nothing may touch such a register between its load and the wait that covers it (a
# copy at the join of a branch, a split live range): the device assembly of these sources is checked
# path by path, see inflight_lint.py.
# The check recognises hand-issued loads by the markers the compiler puts around inline assembly and by their
# mnemonics; if a compiler update changed either it would find no loads and pass everything.  So the number of
# hand-issued loads it followed must reach a floor per source: two thirds of today's counts (vt_head_mfma.hip 818,
# vt_head_gemv_np1/2/4/8.hip 344 / 344 / 300 / 72; vt_row_select.hip none, its loads are the compiler's own), so that no more
# than a kernel or two can go unseen.  The model was validated against the assembly of AMD clang 20 (ROCm 7.2.0), -O3, gfx950.
MIN_HAND_LOADS = {"vt_head_mfma.hip": 540, "vt_head_gemv_np1.hip": 230, "vt_head_gemv_np2.hip": 230,
                  "vt_head_gemv_np4.hip": 200, "vt_head_gemv_np8.hip": 48}
# Likewise the hand-written loads straight into LDS, which are checked for the wait state behind the write of M0
# (2929 today).
MIN_LDS_LOADS = {"vt_head_mfma_rows.hip": 1950}

# The sources with buffer loads, which are checked for scalar offsets that the descriptor's size may not cover.
BUFFER_LOADS = ("vt_count.hip",)


def _scratch_users(remarks: str):
    """(kernel, bytes per lane) for every kernel the resource-usage remarks report with scratch memory."""
    out, name = [], None
    for line in remarks.splitlines():
        if "remark: Function Name:" in line:
            name = line.split("Function Name:")[1].split("[")[0].strip()
        elif "ScratchSize [bytes/lane]:" in line and name is not None:
            n = int(line.split("ScratchSize [bytes/lane]:")[1].split("[")[0])
            if n != 0:
                out.append((name, n))
    return out


def device_assembly(src: str) -> str:
    """The gfx950 assembly of src, compiled with the flags of the object."""
    r = subprocess.run([HIPCC] + FLAGS + ["--cuda-device-only", "-S", src, "-o", "-"], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc -S failed on {src}:\n{r.stderr}")
    return r.stdout


def _lint():
    try:
        from . import inflight_lint
    except ImportError:      # run as a script
        import inflight_lint
    return inflight_lint


def _check_buffer_loads(src: str):
    bad, loads = _lint().check_buffer_offsets(device_assembly(src))
    if loads == 0:
        raise RuntimeError(f"{os.path.basename(src)}: no buffer load found, the check of their offsets would pass anything")
    if bad:
        raise RuntimeError(f"{os.path.basename(src)}: buffer loads with a scalar offset that the descriptor's size may not "
                           f"cover (kernel, line in the device assembly, text): {bad[:5]}")


def _inflight_violations(src: str):
    """Runs the in-flight register check on the gfx950 assembly of src."""
    inflight_lint, text = _lint(), device_assembly(src)
    bad, followed = inflight_lint.check_asm(text)
    hazards, into_lds = inflight_lint.check_m0(text)
    floor = MIN_HAND_LOADS.get(os.path.basename(src), 0)
    if followed < floor:
        raise RuntimeError(f"{os.path.basename(src)}: the in-flight register check followed {followed} hand-issued "
                           f"loads, fewer than the {floor} this source is known to hold: it no longer recognises "
                           "them (compiler output changed?) and would pass anything")
    if into_lds < MIN_LDS_LOADS.get(os.path.basename(src), 0):
        raise RuntimeError(f"{os.path.basename(src)}: {into_lds} hand-written loads into LDS found, fewer than the "
                           f"{MIN_LDS_LOADS[os.path.basename(src)]} this source is known to hold")
    if hazards:
        raise RuntimeError(f"{os.path.basename(src)}: loads into LDS directly behind the write of M0 they read "
                           f"(kernel, line in the device assembly, text): {hazards[:5]}")
    return bad


def _compile(src: str, force: bool) -> str:
    base = os.path.basename(src)
    obj = os.path.join(OBJ, base[:-4] + ".o")
    headers = glob.glob(os.path.join(CSRC, "*.h")) + \
        glob.glob(os.path.join(ROOT, "include", "*.h"))
    if force or _stale(obj, [src] + headers):
        check = base.startswith(NO_SCRATCH)
        extra = ["-Rpass-analysis=kernel-resource-usage"] if check else []
        r = subprocess.run([HIPCC] + FLAGS + extra + ["-c", src, "-o", obj], capture_output=True, text=True)
        if check:
            bad = _scratch_users(r.stderr)
            if bad:
                if os.path.exists(obj):
                    os.remove(obj)
                raise RuntimeError(f"{base}: kernels with hand-issued loads must not spill: {bad}")
            if r.returncode == 0:
                touched = _inflight_violations(src)
                if touched:
                    os.remove(obj)
                    raise RuntimeError(f"{base}: registers of hand-issued loads are touched before their wait "
                                       f"(kernel, line of the load, line and text of the instruction in the "
                                       f"device assembly): {touched[:5]}")
        if base in BUFFER_LOADS and r.returncode == 0:
            try:
                _check_buffer_loads(src)
            except RuntimeError:
                os.remove(obj)
                raise
        lines = r.stderr.splitlines()
        if check and r.returncode == 0:
            lines = []      # the remarks (and their source excerpts) are not diagnostics
        err = "\n".join(l for l in lines if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if err.strip():
            sys.stderr.write(err + "\n")
    return obj


def _binding_command(src: str) -> list[str]:
    import torch
    from torch.utils.cpp_extension import include_paths

    from .binding import BIND_ABI
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return [os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-fPIC", "-shared", f'-DVT_BUILT_FOR="{BIND_ABI}"',
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + os.path.join(ROOT, "include"),
            *("-I" + p for p in include_paths()), "-I" + sysconfig.get_paths()["include"], src, "-o", BIND,
            "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10"]


def _binding_stamp(cmd) -> str:
    return "\n".join(c.replace(ROOT, ".") for c in cmd)      # (a tree may be moved)


def _binding_stale(cmd, deps) -> bool:
    """The sources are newer, or it was built by another command: for another torch or interpreter."""
    if _stale(BIND, deps) or not os.path.exists(BIND_STAMP):
        return True
    with open(BIND_STAMP) as f:
        return f.read() != _binding_stamp(cmd)


def build_binding(force: bool = False) -> str:
    """The native part of the Python binding: host code against torch's headers, no GPU code in it."""
    src = os.path.join(CSRC, "vt_bind.cpp")
    cmd = _binding_command(src)
    if force or _binding_stale(cmd, [src] + glob.glob(os.path.join(ROOT, "include", "*.h"))):
        # (a build that fails leaves none behind, and none of the name without the interpreter's tag that it once had)
        for old in (BIND, BIND_STAMP, os.path.join(PKG, "_vt_bind.so")):
            if os.path.exists(old):
                os.remove(old)
        try:
            r = subprocess.run(cmd, capture_output=True, text=True)
            failure = r.stderr if r.returncode != 0 else None
        except OSError as e:
            failure = str(e)
        if failure is not None:
            warnings.warn(f"the native part of the binding is left out (plain calls go through Python): {cmd[0]} failed on {src}:\n{failure}")
            return BIND
        with open(BIND_STAMP, "w") as f:
            f.write(_binding_stamp(cmd))
    return BIND


def build_library(force: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = _sources()
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as ex:
        binding = ex.submit(build_binding, force)
        objs = list(ex.map(lambda s: _compile(s, force), srcs))
        binding.result()
    if force or _stale(LIB, objs):
        r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs,
                           capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stderr)
    return LIB


if __name__ == "__main__":
    print(build_library(force="--force" in sys.argv))
