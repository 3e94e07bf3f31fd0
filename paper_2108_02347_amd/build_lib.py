"""Builds libfmm_attn.so in-tree with hipcc for gfx950, and, where torch is
installed, _fmm_torch.so, the torch.autograd functions over it, with the host
compiler.

Usage: python -m paper_2108_02347_amd.build_lib   (or call build(); without
torch, which the package needs, run this file by its path)
"""

from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libfmm_attn.so")
TORCH_EXT = os.path.join(PKG, "_fmm_torch.so")
SOURCES = ["fmm_kernels.hip", "fmm_wide.hip", "fmm_wide128.hip", "fmm_bwd.hip", "fmm_pair.hip",
           "fmm_causal.hip", "fmm_noalloc.hip", "fmm_layer.hip", "fmm_fastweight.hip", "fmm_api.cpp"]
# translation units compiled again with other options: (source, object name,
# extra flags, whether MFMA results are forced into vector registers)
VARIANTS = [
    # the backward's fp32 passes
    ("fmm_bwd.hip", "fmm_bwd_f32", ["-DFMM_BWD_F32"], True),
    # and those at d = 128: one workgroup per CU, with the accumulation
    # registers beside the vector registers
    ("fmm_bwd.hip", "fmm_bwd_f32_d128", ["-DFMM_BWD_F32_D128"], False),
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; the HIP library cannot be built")


def _flags(vgpr_form: bool = True):
    f = [
        "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
        # keep the compiler from forming packed fp32 instructions
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    ]
    if vgpr_form:
        # keep MFMA accumulators in ordinary VGPRs: the kernels scale and
        # blend them with VALU code, which would otherwise copy them out of
        # and back into AGPRs
        f += ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
    return f + ["-Wno-unused-result", "-I", os.path.join(ROOT, "include")]


def _torch_ext_cmds(obj: str):
    """Compile and link commands of the extension module (host code only), or
    None without torch: the library itself needs hipcc alone."""
    import sysconfig

    try:
        import torch
    except ImportError:
        return None
    tdir = os.path.dirname(torch.__file__)
    cxx = os.environ.get("CXX") or shutil.which("g++") or "g++"
    inc = [os.path.join(tdir, "include"),
           os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
           "/opt/rocm/include", sysconfig.get_paths()["include"]]
    compile_ = [cxx, "-O2", "-std=c++17", "-fPIC", "-c",
                f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                "-DTORCH_EXTENSION_NAME=_fmm_torch", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"]
    for i in inc:
        compile_ += ["-isystem", i]
    compile_ += [os.path.join(CSRC, "fmm_torch.cpp"), "-o", obj]
    link = [cxx, "-shared", obj, "-o", TORCH_EXT + ".tmp", "-L" + os.path.join(tdir, "lib"),
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python", "-L" + PKG,
            "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"]
    return compile_, link


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 into LIB (always recompiles).  The
    translation units are compiled in parallel, then linked."""
    cc = hipcc()
    tmpdir = tempfile.mkdtemp(prefix="fmm_build_")
    ext_proc = None
    try:
        objs, procs = [], []
        units = [(src, src, [], True) for src in SOURCES] + VARIANTS
        for src, name, extra, vgpr_form in units:
            obj = os.path.join(tmpdir, name + ".o")
            cmd = [cc] + _flags(vgpr_form) + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((name, subprocess.Popen(cmd, stdout=subprocess.PIPE,
                                                 stderr=subprocess.STDOUT, text=True)))
            objs.append(obj)
        ext_obj = os.path.join(tmpdir, "fmm_torch.o")
        ext = _torch_ext_cmds(ext_obj)
        if ext:
            if verbose:
                print(" ".join(ext[0]), flush=True)
            ext_proc = subprocess.Popen(ext[0], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                        text=True)
        failed = []
        for src, pr in procs:
            out, _ = pr.communicate()
            if pr.returncode != 0:
                sys.stderr.write(out)
                failed.append(src)
            elif verbose and out.strip():
                sys.stderr.write(out)
        if failed:
            raise RuntimeError(f"hipcc failed on {', '.join(failed)}")
        # rocBLAS serves the attention layer's projections
        cmd = ([cc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs +
               ["-L/opt/rocm/lib", "-lrocblas", "-Wl,-rpath,/opt/rocm/lib", "-o", LIB + ".tmp"])
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError(f"hipcc link failed with status {res.returncode}")
        os.replace(LIB + ".tmp", LIB)
        if not ext:
            print("torch is not installed: _fmm_torch.so is not built", file=sys.stderr)
            return LIB
        # the extension links against the library just built
        out, _ = ext_proc.communicate()
        if ext_proc.returncode != 0:
            sys.stderr.write(out)
            raise RuntimeError("compiling fmm_torch.cpp failed")
        if verbose:
            print(" ".join(ext[1]), flush=True)
        res = subprocess.run(ext[1], capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError(f"linking _fmm_torch.so failed with status {res.returncode}")
        os.replace(TORCH_EXT + ".tmp", TORCH_EXT)
    finally:
        if ext_proc is not None and ext_proc.returncode is None:
            ext_proc.kill()
            ext_proc.wait()
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
