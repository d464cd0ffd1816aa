"""Registers and scratch of the built kernels, from the code object's own metadata (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2308_02494_amd.build import LIB

LLVM = "/opt/rocm/llvm/bin/"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: (vector registers per lane, scratch bytes per lane)} of the library."""
    d = str(tmp_path_factory.mktemp("co"))
    fat, co = os.path.join(d, "fat"), os.path.join(d, "co")
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout
    run(LLVM + "llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", LIB, os.path.join(d, "lib"))
    target = next(t for t in run(LLVM + "clang-offload-bundler", "--type=o", "--list", f"--input={fat}").split()
                  if "gfx950" in t)
    run(LLVM + "clang-offload-bundler", "--type=o", "--unbundle", f"--targets={target}", f"--input={fat}",
        f"--output={co}")
    out, fields = {}, {}
    for entry in run(LLVM + "llvm-readelf", "--notes", co).split(".agpr_count:")[1:]:
        fields = dict(re.findall(r"\.(\w+):\s+(\S+)", entry))
        out[fields["name"]] = (int(fields["vgpr_count"]), int(fields["private_segment_fixed_size"]))
    names = run("c++filt", *out).splitlines()
    return {n.split("(")[0].replace("void ", ""): v for n, v in zip(names, out.values())}


def test_forward_kernels_use_no_scratch(kernels):
    fwd = {n: s for n, (_, s) in kernels.items() if n.startswith(("apmg::k_forward<", "apmg::k_forward_small<"))}
    assert len(fwd) > 100
    assert not {n: s for n, s in fwd.items() if s}
