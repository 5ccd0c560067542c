"""64-channel heads with grouped query heads: the library's choice (the matrix-core kernel, two
neighbouring kv heads per workgroup with one or two query heads of each) against the oracle and
against the plain kernel, at the edges of the head groups, splits, tails and code widths."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV
from test_gpu_pairs import _say, _w64
from test_gpu_parity import _decode_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,batch,q_heads,kv_heads,tb,lens,shape", [
    (4, 2, 8, 4, 128, [640, 129], 0),                                  # two heads per kv head: one group
    (4, 1, 6, 2, 128, [1000], 0),                                      # three: 2 + 1
    (2, 2, 8, 2, 256, [768, 1], 0),                                    # four: two groups
    (8, 1, 16, 2, 128, [515], 0),                                      # eight: four groups
    (4, 3, 4, 2, 128, [384, 0, 77], dq.decode_flags(splits=3)),        # an empty sequence, forced splits
    (4, 1, 10, 2, 128, [2300], dq.decode_flags(splits=5, waves=8)),    # five: 2 + 2 + 1
    (4, 1, 64, 2, 128, [300], 0),                                      # thirty-two: sixteen groups, the most
    (4, 1, 66, 2, 128, [130], 0),                                      # thirty-three: the plain kernel's
])
def test_grouped_pairs_against_the_oracle(bits, batch, q_heads, kv_heads, tb, lens, shape):
    cap = -(-max(lens) // tb) * tb
    w = _w64(bits=bits, batch=batch, q_heads=q_heads, kv_heads=kv_heads, block_tokens=tb, max_seq=cap)
    _say("grouped pairs: %s" % ((bits, batch, q_heads, kv_heads, tb, lens, shape),))
    worst = _decode_case(w, lens, dq.DECODE_AUTO | shape)
    _say("  worst fp32 abs err %.3g" % worst)


@pytest.mark.parametrize("q_heads,kv_heads,tail_lens,shape", [
    (8, 4, [5, 100], 0), (6, 2, [0, 128], dq.decode_flags(splits=2)), (8, 2, [1, 33], dq.decode_flags(waves=8)),
])
def test_grouped_pairs_with_a_tail_match_the_plain_kernel(q_heads, kv_heads, tail_lens, shape):
    """Same call through both kernels; fp32 outputs agree to the accuracy either is held to (a garbage
    partner's rows past the tail's length are never used)."""
    _say("grouped pairs with a tail: %s" % ((q_heads, kv_heads, tail_lens, shape),))
    fmt = dq.Format(4, 64, 64, 8, 8, 128)
    g = torch.Generator(device=DEV).manual_seed(5)
    b, n = 2, 640
    cache = dq.alloc_cache(fmt, b, kv_heads, n // 128, DEV)
    k, v = (torch.randn(b, kv_heads, n, 64, device=DEV, generator=g).half() for _ in "kv")
    dq.compress_kv_blocks(cache, k, v, torch.zeros(b, dtype=torch.int32, device=DEV), None,
                          dq.compress_workspace(fmt, b, kv_heads, DEV, t_new=n))
    lens = torch.tensor([n, 130], dtype=torch.int32, device=DEV)
    tail = [torch.randn(b, kv_heads, 128, 64, device=DEV, generator=g).half() for _ in "kv"]
    for i, m in enumerate(tail_lens):
        for t in tail:
            t[i, :, m:] = float("nan")
    tail.append(torch.tensor(tail_lens, dtype=torch.int32, device=DEV))
    q = torch.randn(b, q_heads, 64, device=DEV, generator=g).half()
    outs = []
    for flags in (dq.DECODE_AUTO | shape, dq.DECODE_FORCE_GENERIC):
        ws = dq.decode_workspace(fmt, b, q_heads, kv_heads, n, DEV)
        o32 = torch.empty(b, q_heads, 64, dtype=torch.float32, device=DEV)
        first = dq.attn_decode(cache, q, lens, n, ws, out_f32=o32, flags=flags, tail=tuple(tail)).clone()
        again = dq.attn_decode(cache, q, lens, n, ws, flags=flags, tail=tuple(tail))      # tickets left clean
        assert torch.equal(first, again)
        outs.append(o32)
    # (the two kernels round differently: had the library's choice been the plain one, the bits would agree)
    assert not torch.equal(outs[0], outs[1])
    # both kernels are within 1e-4 of |out| < 4 of the exact result (fp32 sums over 770 rows)
    assert torch.isfinite(outs[0]).all()
    assert (outs[0] - outs[1]).abs().max().item() < 2e-4


@pytest.mark.parametrize("bits,q_heads,kv_heads,plain", [
    (4, 8, 4, False), (2, 6, 2, False), (8, 16, 2, False), (4, 64, 2, False), (4, 66, 2, True), (4, 6, 3, True),
])
def test_which_kernel_grouped_heads_get(bits, q_heads, kv_heads, plain):
    """The library's choice gives the plain kernel's bits exactly where it is the plain kernel: more than
    32 query heads per kv head, an odd number of kv heads."""
    _say("kernel of grouped pairs: %s" % ((bits, q_heads, kv_heads, plain),))
    fmt = dq.Format(bits, 64, 64, 8, 8, 128)
    g = torch.Generator(device=DEV).manual_seed(6)
    cache = dq.alloc_cache(fmt, 1, kv_heads, 3, DEV)
    k, v = (torch.randn(1, kv_heads, 384, 64, device=DEV, generator=g).half() for _ in "kv")
    dq.compress_kv_blocks(cache, k, v, torch.zeros(1, dtype=torch.int32, device=DEV), None,
                          dq.compress_workspace(fmt, 1, kv_heads, DEV, t_new=384))
    q = torch.randn(1, q_heads, 64, device=DEV, generator=g).half()
    lens = torch.tensor([380], dtype=torch.int32, device=DEV)
    outs = []
    for flags in (dq.DECODE_AUTO, dq.DECODE_FORCE_GENERIC):
        o32 = torch.empty(1, q_heads, 64, dtype=torch.float32, device=DEV)
        dq.attn_decode(cache, q, lens, 384, dq.decode_workspace(fmt, 1, q_heads, kv_heads, 384, DEV), out_f32=o32, flags=flags)
        outs.append(o32)
    assert torch.equal(*outs) == plain
