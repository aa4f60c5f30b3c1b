"""Builds libmixdq.so (gfx950) in-tree with hipcc, and _mqhost.so (host code over torch's C++ interface) with g++.  Object
files are cached per source; pass force=True to rebuild everything."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.environ.get("MQ_CSRC_DIR", os.path.join(HERE, "csrc"))
OBJ = os.environ.get("MQ_OBJ_DIR", os.path.join(HERE, "_build"))
LIB = os.environ.get("MQ_LIB_OUT", os.path.join(HERE, "libmixdq.so"))
HOST = os.path.join(os.path.dirname(LIB), "_mqhost.so")
EXTRA = os.environ.get("MQ_EXTRA_FLAGS", "").split()
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
          "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]
# The quantisers decide integer codes: every fp32 operation must round once.
PER_FILE = {
    "quant_pack.hip": ["-ffp-contract=off"],
    "act_quant.hip": ["-ffp-contract=off"],
    "alloc.cpp": ["-ffp-contract=off"],  # budgets are floors of double products: no fused multiply-add
    # The epilogue converts four results per lane to 16 bits; the SLP vectoriser pairs the middle two and then needs
    # three more instructions per four values to put the halves where the store wants them.
    "gemm.hip": ["-fno-slp-vectorize"],
    "gemm_solo.hip": ["-fno-slp-vectorize"],
    "gemm_panel.hip": ["-fno-slp-vectorize", "-ffp-contract=off"],
}
SOURCES = ["api.hip", "quant_pack.hip", "act_quant.hip", "gemm.hip", "gemm_solo.hip", "gemm_panel.hip", "bos.hip", "prof.hip", "peaks.hip", "alloc.cpp"]


def _compile(src: str, force: bool) -> str:
    path = os.path.join(CSRC, src)
    obj = os.path.join(OBJ, src + ".o")
    deps = [path, os.path.join(CSRC, "mq_common.h"), os.path.join(CSRC, "bos_rows.h"), os.path.join(CSRC, "gemm_core.h"), os.path.join(CSRC, "act_range.h"),
            os.path.join(HERE, "..", "include", "mixdq.h"), __file__]
    if not force and os.path.exists(obj) and all(os.path.getmtime(obj) >= os.path.getmtime(d) for d in deps):
        return obj
    cmd = [HIPCC, *COMMON, *EXTRA, *PER_FILE.get(src, []), "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        errs = [l for l in (r.stdout + r.stderr).splitlines() if "error" in l]
        sys.stderr.write("\n".join(errs[:20]) + "\n")
        raise RuntimeError(f"hipcc failed on {src}")
    warn = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    if warn:
        sys.stderr.write("\n".join(warn) + "\n")
    return obj


def _host_made_for() -> str:
    """What _mqhost.so is compiled against, beside its source: it reads torch's and Python's object layouts."""
    import torch

    return f"torch {torch.__version__}, hip {torch.version.hip}, {sysconfig.get_config_var('SOABI')}"


def _build_host(force: bool) -> None:
    src, stamp, made_for = os.path.join(CSRC, "host.cpp"), os.path.join(OBJ, "mqhost.made_for"), _host_made_for()
    if not force and os.path.exists(HOST) and os.path.exists(stamp) and open(stamp).read() == made_for and \
            all(os.path.getmtime(HOST) >= os.path.getmtime(d) for d in (src, __file__)):
        return
    import torch
    from torch.utils import cpp_extension

    tmp = f"{HOST}.{os.getpid()}"
    inc = [a for d in (*cpp_extension.include_paths(), "/opt/rocm/include", sysconfig.get_paths()["include"]) for a in ("-isystem", d)]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-Wno-missing-field-initializers",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f'-DMQ_MADE_FOR="{made_for}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", *inc, src, "-o", tmp,
           *(f"-L{d}" for d in cpp_extension.library_paths()), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.stderr:
        sys.stderr.write(r.stdout + r.stderr)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on host.cpp")
    os.replace(tmp, HOST)
    with open(stamp, "w") as f:
        f.write(made_for)


def build(force: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        host = ex.submit(_build_host, force)
        objs = list(ex.map(lambda s: _compile(s, force), SOURCES))
        host.result()
    if force or not os.path.exists(LIB) or any(os.path.getmtime(o) > os.path.getmtime(LIB) for o in objs):
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("link failed")
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
