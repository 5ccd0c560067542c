"""The compiler's report on the kernels of the in-tree build: no kernel of the streaming paths may
keep data in scratch memory (a stack object or a register spill there costs a large part of the
bandwidth these kernels are bound by)."""
import json
import os

from paper_2405_12591_amd import build as B


def _resources():
    if not os.path.exists(B.RESOURCES_PATH):
        B.build_library()
    with open(B.RESOURCES_PATH) as f:
        return json.load(f)


def test_no_scratch_in_the_streaming_kernels():
    res = _resources()
    decode = {k: v for k, v in res.items() if "decode_mfma_kernel" in k}
    assert len(decode) >= 100            # every (bits, groups, heads, waves, tail mode, tensors, head pairing) instance
    for name, r in res.items():
        if any(s in name for s in ("decode_mfma_kernel", "decompose16_kernel", "quantize_tiles_kernel",
                                   "quantize_pack_kernel", "split3_kernel", "stream_read_kernel")):
            assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0, (name, r)


def test_occupancy_the_launch_shapes_count_on():
    import re
    res = _resources()
    seen = 0
    for name, r in res.items():
        m = re.search(r"decode_mfma_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELb([01])ELb([01])E", name)
        if not m:
            continue
        seen += 1
        bits, _, _, waves, _, _, _ = (int(x) for x in m.groups())
        assert r["LDS Size"] <= 160 * 1024, (name, r)
        if bits < 8 and waves == 4:
            # these workgroups run two to a compute unit: two waves per SIMD share its 512 registers
            assert r["VGPRs"] + r["AGPRs"] <= 256 and r["LDS Size"] <= 80 * 1024, (name, r)
    assert seen >= 100


def test_resident_waves_of_the_launch_shape_estimate():
    """choose_mfma_shape (dq_api.hip) counts on so many waves of the 4-wave kernels per SIMD; the built
    kernels must hold at least as many (launches in several splits; those in one split hold the tail's
    rows in more registers)."""
    import re

    def resident(bits, heads, two_groups, three, tail):
        if bits == 8:
            return 2 if heads == 1 or (heads == 2 and not three and not tail) else 1
        if bits == 4:
            return 3 if not three and (heads == 1 or (heads == 2 and not tail and not two_groups)) else 2
        return {1: 3 if three else 4, 2: 2 if three else 3, 4: 2}[heads]

    seen = 0
    for name, r in _resources().items():
        m = re.search(r"decode_mfma_kernelILi(\d)ELi(\d)ELi(\d)ELi4ELi([02])ELb([01])ELb([01])E", name)
        if m:
            bits, groups, heads, tail, three, pair = (int(x) for x in m.groups())
            seen += 1
            want = resident(bits, heads, groups == 2, three == 1, tail == 2)
            # (two kinds of launch with two step groups hold one wave less; the estimate does not tell them apart)
            less = groups == 2 and ((bits, heads, tail, three, pair) == (2, 2, 2, 0, 0) or (bits, heads, three) == (8, 1, 1))
            assert r["Occupancy"] >= want - less, (name, r, want)
    assert seen >= 40
