"""Compile the sources under csrc/ (HIP kernels and the host-only policy core) for gfx950 into paper_2605_06472_amd/libpbkv.so, and
csrc/calls.cpp into the Python extension _calls, named for the interpreter that builds it.

Every call recompiles (objects go to _build/, which is not committed).  Packed fp32
instructions are disabled for all device code.
"""
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpbkv.so")
SOURCES = ["pbkv_api.hip", "attn_bf16.hip", "attn_f32.hip", "scatter.hip", "decode_bf16.hip", "predictor.hip", "policy.cpp"]
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))    # the binding's argument marshalling, a Python extension
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the device-only feature flag; that remark is expected
    out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        print(out)
    return obj


def _build_calls() -> None:
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + sysconfig.get_paths()["include"],
                    os.path.join(CSRC, "calls.cpp"), "-o", CALLS], check=True)


def build() -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        calls = ex.submit(_build_calls)
        objs = list(ex.map(_compile, SOURCES))
        calls.result()
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,--no-undefined",
                    *objs, "-o", LIB], check=True)
    return LIB


if __name__ == "__main__":
    print(build())
