"""Registers and scratch of the built kernels, from the code object's own metadata (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2308_02494_amd.build import LIB

LLVM = "/opt/rocm/llvm/bin/"


def run(*a):
    return subprocess.run(a, check=True, capture_output=True, text=True).stdout


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    """The gfx950 code object of the library, as a file."""
    d = str(tmp_path_factory.mktemp("co"))
    fat, co = os.path.join(d, "fat"), os.path.join(d, "co")
    run(LLVM + "llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", LIB, os.path.join(d, "lib"))
    target = next(t for t in run(LLVM + "clang-offload-bundler", "--type=o", "--list", f"--input={fat}").split()
                  if "gfx950" in t)
    run(LLVM + "clang-offload-bundler", "--type=o", "--unbundle", f"--targets={target}", f"--input={fat}",
        f"--output={co}")
    return co


def plain(names):
    """Demangled kernel names without their arguments."""
    return [n.split("(")[0].replace("void ", "") for n in run("c++filt", *names).splitlines()]


@pytest.fixture(scope="module")
def kernels(code_object):
    """{kernel: (vector registers per lane, scratch bytes per lane)} of the library."""
    out = {}
    for entry in run(LLVM + "llvm-readelf", "--notes", code_object).split(".agpr_count:")[1:]:
        fields = dict(re.findall(r"\.(\w+):\s+(\S+)", entry))
        out[fields["name"]] = (int(fields["vgpr_count"]), int(fields["private_segment_fixed_size"]))
    return dict(zip(plain(out), out.values()))


def test_forward_kernels_use_no_scratch(kernels):
    fwd = {n: s for n, (_, s) in kernels.items() if n.startswith(("apmg::k_forward<", "apmg::k_forward_small<"))}
    assert len(fwd) > 100
    assert not {n: s for n, s in fwd.items() if s}


def test_brick_forward_keeps_four_waves_per_simd(kernels):
    # 512 vector registers per SIMD lane, handed out in eights; the weights staged in LDS, four-wave blocks
    few = {}
    for C in (1, 2):
        for f16 in ("true", "false"):
            for bf16 in ("true", "false"):
                name = f"apmg::k_forward<{C}, 64, {f16}, {bf16}, true, 0, 4, true>"
                waves = 512 // (-(-kernels[name][0] // 8) * 8)
                if waves < (3 if (C, f16, bf16) == (2, "false", "true") else 4):
                    few[name] = waves
    assert not few


def test_one_channel_half_forward_takes_the_registers_of_four_waves(kernels):
    # more than the 98 it is squeezed into under a bound, at most the 128 of four waves
    for bf16 in ("true", "false"):
        assert 104 < kernels[f"apmg::k_forward<1, 64, true, {bf16}, true, 0, 4, false>"][0] <= 128


def test_waves_per_simd_of_the_one_channel_gather(kernels):
    # <C, binary16, transform gradient, time slices, four waves a block, six waves per SIMD>
    pull = {n: v for n, (v, _) in kernels.items() if n.startswith("apmg::k_block_pull<1, ")}
    assert len(pull) == 10
    for n, v in pull.items():
        assert 512 // (-(-v // 8) * 8) >= (6 if n.endswith("true>") else 4), n
        assert n.endswith("true>") or ", true, 1, " in n and v > 80, n


def test_one_channel_half_grids_load_pairs_at_once(code_object):
    # the two binary16 values of an x-adjacent vertex pair come in one 4-byte load
    syms = [ln.split()[-1] for ln in run(LLVM + "llvm-readelf", "-sW", code_object).splitlines() if " FUNC " in ln]
    fwd = sorted({s for s, n in zip(syms, plain(syms)) if re.match(r"apmg::k_forward<1, \d+, true,", n)})
    assert len(fwd) >= 8
    for s in fwd:
        code = run(LLVM + "llvm-objdump", "-d", f"--disassemble-symbols={s}", code_object)
        assert "global_load_dword" in code and "_ushort" not in code, s
