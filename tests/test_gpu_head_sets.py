"""Launches of more than four query heads per kv head (more than two with two step groups) that are large enough go to the matrix-core
kernel with two sets of columns a workgroup.  It is compared with the plain kernel: on both sides of the line, with missing heads in
either set (5 = 4 + 1, 13 = 8 + 4 + 1 of sixteen; 3 = 2 + 1, 7 = 4 + 2 + 1), every merge path, lengths at the edges of tiles, codes and steps of any
content past the end, NaN and infinities in the small tensors of blocks past the end.  Calls with a fp16 tail or three local
tensors stay with one set, beyond the line as well.  Which kernel a launch takes is asked of the library."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV
from test_launch_shape import shape

pytestmark = pytest.mark.gpu


# (the last entry: whether the launch is large enough for two sets)
@pytest.mark.parametrize("bits,group,rep,batch,tiles,wide", [
    (4, 128, 8, 17, 4, 1), (4, 128, 8, 16, 4, 0), (4, 128, 5, 17, 5, 1), (4, 128, 13, 17, 4, 1), (4, 128, 8, 33, 3, 0), (2, 128, 8, 17, 4, 1),
    (2, 128, 7, 17, 4, 1), (8, 128, 8, 17, 1, 1), (8, 128, 8, 17, 4, 1), (8, 128, 6, 5, 33, 1), (4, 128, 8, 2, 513, 1),
    (4, 64, 4, 17, 4, 1), (4, 64, 4, 16, 4, 0), (4, 64, 3, 17, 5, 1), (4, 64, 7, 17, 4, 1), (2, 64, 4, 17, 4, 1), (2, 64, 8, 17, 4, 1), (8, 64, 4, 17, 1, 1),
    (8, 64, 3, 17, 4, 1), (8, 64, 8, 17, 2, 0), (8, 64, 8, 17, 4, 1), (4, 64, 4, 2, 313, 1), (4, 64, 2, 5, 5, 0), (2, 64, 2, 5, 5, 0), (8, 64, 2, 5, 5, 0)])
def test_two_sets_of_heads_a_workgroup(bits, group, rep, batch, tiles, wide):
    most = 4 if group == 128 else 2
    assert shape(dq, bits, group, rep, batch, tiles)[3] == (2 * most if wide else most)
    _compare(bits, group, rep, batch, tiles)


@pytest.mark.parametrize("bits,group,rep,batch,tiles", [(4, 128, 8, 17, 4), (8, 128, 5, 17, 4), (2, 64, 4, 17, 4), (4, 64, 7, 17, 4)])
@pytest.mark.parametrize("i3,tail", [(1, 1), (8, 0), (8, 1)])
def test_large_launches_with_a_tail_or_three_tensors_keep_one_set(bits, group, rep, batch, tiles, i3, tail):
    most = 4 if group == 128 else 2
    assert shape(dq, bits, group, rep, batch, tiles)[3] == 2 * most
    assert shape(dq, bits, group, rep, batch, tiles, i3=i3, tail=tail)[3] == most
    _compare(bits, group, rep, batch, tiles, i3, tail)


def _compare(bits, group, rep, batch, tiles, i3=1, tail=0):
    print("two sets of heads: %s" % ((bits, group, rep, batch, tiles, i3, tail),), flush=True)
    heads, dim = 8, 128
    fmt = dq.Format(bits, group, dim, 16, 8, 128, i3)
    g = torch.Generator(device=DEV).manual_seed(100 * bits + rep)
    cache = dq.alloc_cache(fmt, batch, heads, tiles, DEV, fill=None)
    for name, x in cache.t.items():
        if "codes" in name:
            x.random_(0, 256, generator=g)
        elif "scales" in name:
            x.copy_(torch.rand(x.shape, device=DEV, generator=g) * 0.02 + 0.002)
        else:
            x.copy_(torch.randn(x.shape, device=DEV, generator=g) * 0.25)      # (a column has a norm of about one)
    n = tiles * 128
    lens = torch.tensor([(n, n - 1, 0, 1, 128, n - 127, 127, n)[i % 8] for i in range(batch)], dtype=torch.int32, device=DEV).clamp_(max=n)
    # |v| <= step * |code| * sum over sixteen rows of the small tensor: what a weight's 22 bits of the largest step (half a unit a token, the
    # signs at random: four deviations of the root of n tokens), the scores' and both kernels' fp32 sums are relative to
    code = {2: 2, 4: 8, 8: 128}[bits]
    vmax = 0.022 * code * float(cache.t["v_small"].float().abs().reshape(-1, 16, 16).sum(-1).max())
    bound = vmax * (4 * (min(n, 4096) ** 0.5) * 2.0 ** -23 + 16 * 2.0 ** -24)
    if i3 == 8:   # (a run's rows mixed by the third tensors: sums of eight, of scores and of values)
        for name in ("k_small3", "v_small3"):
            bound *= float(cache.t[name].float().abs().sum((-1, -2)).max()) / 8 ** 0.5
    # what lies past the end counts for nothing: steps NaN (three tensors: from the end of the last run on), small tensors of blocks that
    # hold no token NaN and infinite
    run = -(-lens // i3) * i3
    past = torch.arange(n, device=DEV)[None, :] >= run[:, None]
    empty = torch.arange(tiles, device=DEV)[None, :] * 128 >= lens[:, None]
    for name, x in cache.t.items():
        if "scales" in name:
            x.view(batch, heads, n, 128 // group).masked_fill_(past[:, None, :, None], float("nan"))
        elif "small" in name:
            x.masked_fill_(empty[:, None, :, None, None], float("nan"))
            x[..., 0, :].masked_fill_(empty[:, None, :, None], float("inf"))
    q = torch.randn(batch, heads * rep, dim, device=DEV, generator=g).half()
    rows = None
    if tail:      # rows within the cache's range, so that the bound holds; past the tail's end anything
        kt, vt = (torch.randn(batch, heads, 128, dim, device=DEV, generator=g).mul_(0.2 * min(vmax, 1.0)).half() for _ in "kv")
        tl = torch.tensor([(77, 128, 0, 1, 5, 64, 127, 16)[i % 8] for i in range(batch)], dtype=torch.int32, device=DEV)
        gone = (torch.arange(128, device=DEV)[None, :] >= tl[:, None])[:, None, :, None]
        rows = (kt.masked_fill_(gone, float("nan")), vt.masked_fill_(gone, float("inf")), tl)
    ws = dq.decode_workspace(fmt, batch, heads * rep, heads, n, DEV)
    want = torch.empty(batch, heads * rep, dim, dtype=torch.float32, device=DEV)
    dq.attn_decode(cache, q, lens, n, ws, out_f32=want, flags=dq.DECODE_FORCE_GENERIC, tail=rows)
    for splits, waves in ((0, 0), (1, 4), (1, 8), (3, 4), (3, 8)):
        got = torch.empty_like(want)
        out = dq.attn_decode(cache, q, lens, n, ws, out_f32=got, flags=dq.decode_flags(splits=min(splits, tiles), waves=waves), tail=rows)
        torch.cuda.synchronize()
        assert torch.isfinite(got).all() and torch.equal(out, got.half())
        err = float((got - want).abs().max())
        print("  splits %d waves %d: error %.2e of %.2e, output up to %.2e" % (splits, waves, err, bound, float(want.abs().max())), flush=True)
        assert err <= bound, (splits, waves, err, bound)
        if not tail:
            assert (got[lens == 0] == 0).all()
