"""What the built kernels hold of a CU, read from the library's own code
objects: the launches are planned for these numbers, and a kernel that grows
past one of them is right but slow."""
import os
import re
import struct
import subprocess

import pytest

from paper_1808_06194_amd import build, cfog

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: {resource: value}} of every gfx950 code object."""
    if not os.path.exists(cfog.LIB_PATH):
        build.build()
    with open(cfog.LIB_PATH, "rb") as f:
        lib = f.read()
    out, at = {}, lib.find(MAGIC)
    while at >= 0:
        n, p = struct.unpack_from("<Q", lib, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, ln = struct.unpack_from("<3Q", lib, p)
            name, p = lib[p + 24:p + 24 + ln], p + 24 + ln
            if b"gfx950" not in name:
                continue
            elf = tmp_path_factory.mktemp("co") / "k.elf"
            elf.write_bytes(lib[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(elf)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n  - \.agpr_count", notes)[1:]:
                mangled = re.search(r"\.name:\s+(\S+)", k).group(1)
                name = subprocess.run(["c++filt", mangled], capture_output=True, text=True, check=True).stdout.strip()
                name = name.removeprefix("void ").replace("cfog::", "").split("(")[0]
                out[name] = {m: int(v) for m, v in re.findall(r"\.(\w+):\s+(\d+)", k)}
        at = lib.find(MAGIC, at + 1)
    assert out
    return out


def test_two_reduce_workgroups_share_a_cu(kernels):
    """32 waves of 1024-thread workgroups: 64 VGPRs, 96 SGPRs (with VCC), half of LDS at the largest surface."""
    k = kernels["split_reduce_kernel"]
    assert k["vgpr_count"] <= 64 and k["sgpr_count"] <= 96 and k["private_segment_fixed_size"] == 0
    largest = max((2 * r + 1) ** 2 for r in range(96) if cfog.fft_size(1, r))
    assert 4 * largest + 16 * 16 + k["group_segment_fixed_size"] <= 64 * 1024


def _lane(kernels, head, team):
    return kernels["match_lane_kernel<LaneCfg<%s, %s>, false>" % (head, team)]


def test_lane_workgroups_of_80_and_100(kernels):
    """Two full workgroups of 512 threads to a CU (128 VGPRs), and no spills at P = 80 and in the spread forms."""
    for head, team in (("80, 10, 8, 10, 8, 10, 8", "512, 1, 2, 1"), ("80, 10, 8, 10, 8, 10, 8", "768, 1, 3, 1"),
                       ("100, 10, 10, 5, 20, 10, 10", "768, 2, 3, 1")):
        k = _lane(kernels, head, team)
        assert k["private_segment_fixed_size"] == 0 and k["vgpr_count"] <= (128 if "512" in team else 168)
    assert _lane(kernels, "100, 10, 10, 5, 20, 10, 10", "512, 1, 4, 1")["vgpr_count"] <= 128


@pytest.mark.parametrize("team", ["1, 4, false", "1, 5, false", "1, 6, false", "2, 4, false", "1, 4, true", "2, 4, true"])
def test_two_bf16_workgroups_share_a_cu(kernels, team):
    """Where a launch takes one template buffer for two workgroups of eight waves to a CU: 128 VGPRs."""
    k = kernels["match_direct_kernel<%s>" % team]
    assert k["vgpr_count"] <= 128 and k["private_segment_fixed_size"] == 0
