"""The built library's kernels as its own build describes them: the hot kernels
of either index width keep everything in registers."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1711_07793_amd as rb
from paper_1711_07793_amd import build as hip_build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel name -> bytes of scratch a lane, from the notes of the code objects in the library."""
    if not os.path.exists(rb.LIB_PATH):
        hip_build.build()
    if not os.path.exists(READELF) or not shutil.which("c++filt"):
        pytest.skip("needs ROCm's llvm-readelf and c++filt")
    data = open(rb.LIB_PATH, "rb").read()
    at = [m.start() for m in re.finditer(b"\x7fELF\x02\x01\x01\x40", data)]  # OS ABI 64: AMDGPU HSA
    found = {}
    for k, pos in enumerate(at):
        path = tmp_path_factory.mktemp("co") / f"{k}.co"
        path.write_bytes(data[pos:at[k + 1] if k + 1 < len(at) else len(data)])
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True).stdout
        for rec in re.split(r"\n +- \.agpr_count", notes)[1:]:
            name = re.search(r"\.name: +(\S+)", rec).group(1)
            found[name] = int(re.search(r"\.private_segment_fixed_size: +(\d+)", rec).group(1))
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True).stdout.split("\n")
    return {n: found[m] for n, m in zip(names, found)}


@pytest.mark.parametrize("family", ["tile_kernel", "tile_persistent_kernel", "batch_kernel", "batch_persistent_kernel",
                                    "batch_arg_kernel", "batch_arg_queue_kernel", "serve_kernel", "serve_view_kernel",
                                    "frag_kernel", "sm_kernel", "raster_kernel"])
def test_no_scratch(kernels, family):
    of_family = {n: s for n, s in kernels.items() if re.search(rf"\b{family}<", n)}
    assert of_family
    assert {n.split("(")[0]: s for n, s in of_family.items() if s > 0} == {}
