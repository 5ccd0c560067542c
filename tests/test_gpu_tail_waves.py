"""The fp16 tail in the matrix-core kernel is dealt over all waves of all splits: tail lengths at the edges
of a load, of a wave's batch and of the capacity, over launch shapes, against the plain kernel."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q_heads,kv_heads,i3", [(4, 4, 1), (8, 4, 1), (8, 2, 1), (14, 2, 1), (8, 2, 8)])
@pytest.mark.parametrize("shape", [0, dq.decode_flags(splits=1, waves=4), dq.decode_flags(splits=1, waves=8),
                                   dq.decode_flags(splits=5, waves=4), dq.decode_flags(splits=3, waves=8)])
def test_tail_lengths_against_the_plain_kernel(q_heads, kv_heads, i3, shape):
    print("tail waves: heads %d/%d i3=%d shape=%#x" % (q_heads, kv_heads, i3, shape), flush=True)
    fmt = dq.Format(4, 128, 128, 16, 8, 1024, i3)
    tails = [0, 1, 3, 4, 5, 63, 64, 65, 127, 128, 129, 511, 1023, 1024]
    b, n = len(tails), 1024
    g = torch.Generator(device=DEV).manual_seed(9)
    cache = dq.alloc_cache(fmt, b, kv_heads, 1, DEV)
    k, v = (torch.randn(b, kv_heads, n, 128, device=DEV, generator=g).half() for _ in "kv")
    dq.compress_kv(cache, k, v, torch.zeros(b, dtype=torch.int32, device=DEV), None,
                   dq.compress_workspace(fmt, b, kv_heads, DEV))
    lens = torch.tensor([[n, 0, 700][i % 3] for i in range(b)], dtype=torch.int32, device=DEV)
    tail = [torch.randn(b, kv_heads, 1024, 128, device=DEV, generator=g).half() for _ in "kv"]
    for i, m in enumerate(tails):
        for t in tail:
            t[i, :, m:] = float("nan")        # rows past the length may hold anything
    tail.append(torch.tensor(tails, dtype=torch.int32, device=DEV))
    q = torch.randn(b, q_heads, 128, device=DEV, generator=g).half()
    outs = []
    for flags in (dq.DECODE_FORCE_MFMA | shape, dq.DECODE_FORCE_GENERIC):
        ws = dq.decode_workspace(fmt, b, q_heads, kv_heads, n, DEV)
        o32 = torch.empty(b, q_heads, 128, dtype=torch.float32, device=DEV)
        dq.attn_decode(cache, q, lens, n, ws, out_f32=o32, flags=flags, tail=tuple(tail))
        outs.append(o32)
    # each kernel is within 1e-4 of the exact result at |out| < 5 (fp32 sums over at most 2048 rows)
    assert torch.isfinite(outs[0]).all()
    assert (outs[0] - outs[1]).abs().max().item() < 2e-4


@pytest.mark.parametrize("dim,q_heads,kv_heads,shape", [
    (128, 4, 4, 0), (128, 8, 2, dq.decode_flags(splits=1, waves=8)), (128, 8, 4, dq.decode_flags(splits=3, waves=4)),
    (64, 4, 4, 0), (64, 8, 4, dq.decode_flags(splits=2, waves=8)),
])
def test_rows_that_score_minus_infinity_weigh_nothing(dim, q_heads, kv_heads, shape):
    """A key of -inf against a positive query component masks its row.  Whole loads, whole waves and whole
    tails of such rows must leave the result that the tail without them gives."""
    print("tail waves, infinite keys: %s" % ((dim, q_heads, kv_heads, shape),), flush=True)
    fmt = dq.Format(4, min(dim, 128), dim, dim // 8, 8, 128)
    n, cap = 256, 128
    masked = [[], range(4), range(4, 8), range(60), range(64), [7], range(0, 64, 2), range(32, 64)]   # of 64 rows
    b = len(masked)
    g = torch.Generator(device=DEV).manual_seed(21)
    cache = dq.alloc_cache(fmt, b, kv_heads, 2, DEV)
    k, v = (torch.randn(b, kv_heads, n, dim, device=DEV, generator=g).half() for _ in "kv")
    dq.compress_kv_blocks(cache, k, v, torch.zeros(b, dtype=torch.int32, device=DEV), None,
                          dq.compress_workspace(fmt, b, kv_heads, DEV, t_new=n))
    lens = torch.full((b,), n, dtype=torch.int32, device=DEV)
    q = torch.randn(b, q_heads, dim, device=DEV, generator=g).half()
    q[..., 3] = q[..., 3].abs() + 0.5
    kt, vt = (torch.randn(b, kv_heads, cap, dim, device=DEV, generator=g).half() for _ in "kv")
    kt_without, vt_without, left = kt.clone(), vt.clone(), []
    for i, rows in enumerate(masked):
        keep = [r for r in range(64) if r not in rows]
        kt_without[i, :, :len(keep)], vt_without[i, :, :len(keep)] = kt[i][:, keep], vt[i][:, keep]
        kt[i, :, list(rows), 3] = float("-inf")
        left.append(len(keep))
    outs = []
    for keys, values, tl in ((kt, vt, [64] * b), (kt_without, vt_without, left)):
        ws = dq.decode_workspace(fmt, b, q_heads, kv_heads, n, DEV)
        o32 = torch.empty(b, q_heads, dim, dtype=torch.float32, device=DEV)
        tail = (keys, values, torch.tensor(tl, dtype=torch.int32, device=DEV))
        dq.attn_decode(cache, q, lens, n, ws, out_f32=o32, flags=shape, tail=tail)
        outs.append(o32)
    # the two differ in the order of fp32 sums over 320 rows only: each is within 1e-4 of the exact result
    assert torch.isfinite(outs[0]).all()
    assert (outs[0] - outs[1]).abs().max().item() < 2e-4
