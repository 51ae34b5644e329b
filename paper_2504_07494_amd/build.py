"""Build libapt_hybrid.so (gfx950) in-tree with hipcc: every source is compiled by itself, side by side, then linked; and, where there is
what it takes, the CPython extension that calls it (host only; without it the binding calls through ctypes)."""
import os
import platform
import shlex
import shutil
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libapt_hybrid.so")
CALL = os.path.join(PKG, "_apt_call" + sysconfig.get_config_var("EXT_SUFFIX"))     # another Python version does not load it
SOURCES = ["apt_mfma_f16.hip", "apt_mfma_bf16.hip", "apt_mfma_dealt_f16.hip", "apt_mfma_dealt_bf16.hip",
           "apt_kernels.hip", "apt_raw16.hip", "apt_raw32.hip", "apt_absorb16.hip", "apt_absorb_pv16.hip", "apt_absorb_out16.hip", "apt_plan.cpp", "apt_pool.cpp", "apt_sched.cpp"]


def extension_command():
    """The compiler's command for the extension; None without a host compiler, without Python's headers, or on another architecture than
    the one whose calling convention the extension relies on."""
    cc, include = shlex.split(os.environ.get("CC", "gcc")), sysconfig.get_paths()["include"]
    if platform.machine() != "x86_64" or not cc or not shutil.which(cc[0]) or not os.path.exists(os.path.join(include, "Python.h")):
        return None
    return [*cc, "-O2", "-fPIC", "-shared", "-I", include, os.path.join(CSRC, "apt_call.c"), "-o", CALL]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
             # packed-fp32 instruction forms are kept out of the device code
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-inline-asm", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    if verbose:
        flags += ["-Rpass-analysis=kernel-resource-usage"]

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            sys.stderr.write("\n".join(l for l in out.splitlines() if "error" in l)[:4000] + "\n")
            raise RuntimeError(f"{cmd[0]} failed")
        return out

    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        for old in (CALL, os.path.join(PKG, "_apt_call.so")):        # (no older one is loaded in place of one that is not built)
            if os.path.exists(old):
                os.remove(old)
        command = extension_command()
        call = ex.submit(run, command) if command else None
        if not command:
            sys.stderr.write("no host compiler or Python headers: calls go through ctypes\n")
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        cmds = [[hipcc, *flags, "-x", "hip", "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
        outs = list(ex.map(run, cmds))
        if call:
            outs.append(call.result())
        outs.append(run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", LIB]))
    if verbose:
        print("\n".join(outs))
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
