"""Build libfitnll.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_1710_08826_amd.build        # or build() from Python

Every .hip file under csrc/ is compiled to an object and linked into
paper_1710_08826_amd/libfitnll.so.  Objects go to paper_1710_08826_amd/_build/.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libfitnll.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
    # packed-FP32 instructions stay off (device code here is FP64 anyway)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics",
]


# Device headers compiled again at run time (hipRTC) with a model's structure
# as compile-time constants; their text is embedded in the library.
EMBEDDED = ["model.hpp", "fastmath.hpp", "device_common.hpp", "philox.hpp",
            "accept_device.hpp", "gram_device.hpp", "dalitz_device.hpp", "td4_types.hpp", "td4_device.hpp",
            "tddp_device.hpp"]
DELIM = "FNSRC"


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _embedded_source() -> str:
    """C++ source defining the embedded header table (name, text)."""
    names, texts = [], []
    for name in EMBEDDED:
        with open(os.path.join(CSRC, name)) as fh:
            text = fh.read()
        if f"){DELIM}\"" in text:
            raise RuntimeError(f"{name} contains the raw-string delimiter")
        names.append(f'"{name}"')
        texts.append(f'R"{DELIM}({text}){DELIM}"')
    return ("// generated by build.py: device headers for runtime compilation\n"
            "namespace fn {\n"
            f"extern const int kEmbeddedCount = {len(EMBEDDED)};\n"
            f"extern const char* const kEmbeddedNames[] = {{{', '.join(names)}}};\n"
            f"extern const char* const kEmbeddedTexts[] = {{\n{(',' + chr(10)).join(texts)}}};\n"
            "}  // namespace fn\n")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def _compile_embedded() -> str:
    src = os.path.join(BUILD, "embedded_headers.cpp")
    with open(src, "w") as fh:
        fh.write(_embedded_source())
    obj = src + ".o"
    r = subprocess.run(["g++", "-O1", "-fPIC", "-std=c++17", "-c", src, "-o", obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"embedding the device headers failed:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    objs.append(_compile_embedded())
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs,
           "-L/opt/rocm/lib", "-lhiprtc", "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
