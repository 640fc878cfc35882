"""Build libpsf.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import struct
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OUT = os.path.join(HERE, "libpsf.so")
SOURCES = ["psf_api.hip", "psf_kernels.hip", "psf_partition.hip", "psf_paths.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
READELF = os.environ.get("LLVM_READELF", "/opt/rocm/llvm/bin/llvm-readelf")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", f"-I{INCLUDE}", f"-I{CSRC}",
]


def kernel_resources(lib: str = OUT) -> dict:
    """What the compiler recorded of every kernel in a built library: mangled
    name -> {"private_segment_fixed_size": scratch bytes a lane,
    "group_segment_fixed_size": static LDS bytes, "vgpr_count": ...}."""
    blob = open(lib, "rb").read()
    out: dict = {}
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for m in re.finditer(re.escape(magic), blob):
        at = m.start() + len(magic)
        (count,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(count):
            offset, size, width = struct.unpack_from("<QQQ", blob, at)
            triple = blob[at + 24:at + 24 + width].decode("ascii", "replace")
            at += 24 + width
            if "amdgcn" not in triple or size == 0:
                continue
            with tempfile.NamedTemporaryFile(suffix=".elf") as f:
                f.write(blob[m.start() + offset:m.start() + offset + size])
                f.flush()
                notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
            # one "- " list item per kernel, its arguments nested deeper
            kernels = notes.partition("amdhsa.kernels:")[2].partition("amdhsa.target:")[0]
            for item in re.split(r"^  - ", kernels, flags=re.M)[1:]:
                fields = dict(re.findall(r"^(?:    )?\.(\w+):[ ]+(\S+)", item, flags=re.M))
                if "name" in fields:  # (an object without kernels has an empty list)
                    out[fields["name"]] = {k: int(v) for k, v in fields.items() if v.isdigit()}
    return out


def check_resources(kernels: dict) -> None:
    """The binning kernels keep a thread's records in registers across the
    sort.  One instantiation that the compiler made to spill to scratch lost a
    row of every tile, so none may; and their dynamic LDS holds 16-byte values,
    so it has to start at a multiple of 16 behind the static part."""
    binning = {n: k for n, k in kernels.items() if "k_bin" in n}
    if not binning:
        raise RuntimeError("no binning kernels in the library")
    for name, k in binning.items():
        if k["private_segment_fixed_size"] or k["vgpr_spill_count"]:
            raise RuntimeError(f"{name} spills registers to scratch")
        if k["group_segment_fixed_size"] % 16:
            raise RuntimeError(f"{name}: dynamic LDS starts at {k['group_segment_fixed_size']}, not a multiple of 16")


def build(verbose: bool = False) -> str:
    objs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        if not os.path.exists(path):
            raise FileNotFoundError(f"listed HIP source is missing: {path}")
        obj = os.path.join(bdir, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, "-c", path, "-o", obj]
        if verbose:
            print(" ".join(cmd), file=sys.stderr)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
        objs.append(obj)
    tmp = OUT + ".tmp"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    check_resources(kernel_resources(tmp))
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
