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


def test_resident_waves_of_the_launch_shape_estimate(dq):
    """choose_mfma_shape (dq_api.hip) counts on so many waves of the 4-wave kernels per SIMD (launches in several splits; those in
    one split hold the tail's rows in more registers): exactly what the built kernels hold, but for the launches in which
    the last wave is left out on purpose, with the measurements beside the rule."""
    import re
    # (bits, step groups, heads, tail, three tensors, pair): holds one more than is counted
    fewer = {(4, 1, 4, 0, 0, 0), (2, 1, 4, 0, 0, 0), (4, 2, 2, 0, 0, 0), (2, 2, 4, 0, 0, 1), (2, 1, 2, 0, 1, 0), (2, 1, 2, 1, 1, 0),
             (2, 1, 2, 0, 0, 0)}
    seen, met = 0, set()
    for name, r in _resources().items():
        m = re.search(r"decode_mfma_kernelILi(\d)ELi(\d)ELi(\d)ELi4ELi([02])ELb([01])ELb([01])ELi([12])E", name)
        if not m:
            continue
        bits, groups, heads, tail, three, pair, sets = (int(x) for x in m.groups())
        seen += 1
        if sets == 2 and groups == 1:
            heads = 8                        # (of both sets; with two step groups the instance's name counts both)
        want = dq.lib.dq_debug_resident_waves(bits, heads, groups == 2, three, sets == 2, tail == 2)
        holds = min(r["Occupancy"], 160 * 1024 // r["LDS Size"])
        key = (bits, groups, heads, tail // 2, three, pair)
        if sets == 1 and key in fewer:
            met.add(key)
            want += 1
        assert holds == want, (name, r, want)
    assert seen >= 70 and met == fewer
