"""Registers of the hot kernels in the built library, from the metadata the
compiler writes beside each kernel: none of them may spill to scratch memory
(the extra traffic and latency show in no result)."""
import os
import re
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2607_01757_amd", "liblkmi.so")


@pytest.fixture(scope="module")
def kernels():
    """Mangled name -> metadata of every kernel (ELF notes named AMDGPU)."""
    raw, out, at = open(LIB, "rb").read(), {}, 0
    while (at := raw.find(b"AMDGPU\0\0", at)) >= 0:
        namesz, descsz, kind = struct.unpack_from("<III", raw, at - 12)
        if (namesz, kind) == (7, 32):
            meta = msgpack.unpackb(raw[at + 8:at + 8 + descsz])
            out.update((k[".name"], k) for k in meta["amdhsa.kernels"])
        at += 8
    assert len(out) > 20
    return out


def spills(kernels, pattern):
    hit = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert hit, pattern
    return {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in hit.items()
            if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}


# a wavefront per keypoint, one per workgroup (windows up to 21) or four (31)
@pytest.mark.parametrize("kernel", ["k_track", "k_track_batched"])
@pytest.mark.parametrize("storage", [0, 1])
@pytest.mark.parametrize("geo", ["ILi1ELi7ELi21ELi1ELi6ELb1E", "ILi1ELi7ELi21ELi1ELi4ELb0E", "ILi1ELi16ELi31ELi4ELi2ELb0E"])
def test_tracker_does_not_spill(kernels, kernel, storage, geo):
    assert spills(kernels, r"\d%sILi%dENS0_3Geo%s" % (kernel, storage, geo)) == {}


@pytest.mark.parametrize("kernel", ["k_gftt_select", "k_gftt_peaks_pair", "k_gftt_compact", "k_gftt_bucket"])
def test_detector_does_not_spill(kernels, kernel):
    assert spills(kernels, r"\d" + kernel) == {}


def test_epipolar_fills_a_cu(kernels):
    """Three workgroups of four wavefronts share a CU (LDS holds three): a SIMD
    has 512 registers for one wavefront of each, granted eight at a time."""
    assert spills(kernels, r"\dk_epi_(hypotheses|best)") == {}
    (k,) = [k for n, k in kernels.items() if "k_epi_hypotheses" in n]
    assert 3 * (-(-k[".vgpr_count"] // 8) * 8) <= 512 and 3 * k[".group_segment_fixed_size"] <= 160 * 1024


def test_no_level_kernel_without_a_launch(kernels):
    """The launch by levels exists for the default shapes only: no kernel of it
    is built for the 2 and 4 keypoints a workgroup that a program can ask for."""
    names = [n for n in kernels if "k_track_batched_levels" in n]
    assert len(names) == 6                     # three layouts, two storages
    assert not [n for n in names if re.search(r"ILi1ELi7ELi21ELi[24]E", n)]
