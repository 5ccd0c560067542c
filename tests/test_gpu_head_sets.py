"""Launches of more than four query heads per kv head (more than two with two step groups) that are large enough go to the matrix-core
kernel with two sets of columns a workgroup.  It is compared with the plain kernel: on both sides of the line, with missing heads in
either set (5 = 4 + 1, 13 = 8 + 4 + 1 of sixteen; 3 = 2 + 1, 7 = 4 + 2 + 1), every merge path, lengths at the edges of tiles, and codes, steps and small tensors of any content past the end."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,group,rep,batch,tiles", [
    (4, 128, 8, 17, 4), (4, 128, 8, 16, 4), (4, 128, 5, 17, 5), (4, 128, 13, 17, 4), (4, 128, 8, 33, 3), (2, 128, 8, 17, 4),
    (2, 128, 7, 17, 4), (8, 128, 8, 17, 1), (8, 128, 8, 17, 4), (8, 128, 6, 5, 33), (4, 128, 8, 2, 513),
    (4, 64, 4, 17, 4), (4, 64, 4, 16, 4), (4, 64, 3, 17, 5), (4, 64, 7, 17, 4), (2, 64, 4, 17, 4), (2, 64, 8, 17, 4), (8, 64, 4, 17, 1),
    (8, 64, 3, 17, 4), (4, 64, 4, 2, 313), (4, 64, 2, 5, 5), (2, 64, 2, 5, 5), (8, 64, 2, 5, 5)])
def test_two_sets_of_heads_a_workgroup(bits, group, rep, batch, tiles):
    print("two sets of heads: %s" % ((bits, group, rep, batch, tiles),), flush=True)
    heads, dim = 8, 128
    fmt = dq.Format(bits, group, dim, 16, 8, 128)
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
    # steps past the end: NaN (what lies there counts for nothing)
    past = torch.arange(n, device=DEV)[None, :] >= lens[:, None]
    for name in ("k_scales", "v_scales"):
        x = cache.t[name].view(batch, heads, n, 128 // group)
        x.masked_fill_(past[:, None, :, None], float("nan"))
    q = torch.randn(batch, heads * rep, dim, device=DEV, generator=g).half()
    ws = dq.decode_workspace(fmt, batch, heads * rep, heads, n, DEV)
    want = torch.empty(batch, heads * rep, dim, dtype=torch.float32, device=DEV)
    dq.attn_decode(cache, q, lens, n, ws, out_f32=want, flags=dq.DECODE_FORCE_GENERIC)
    # |v| <= step * |code| * sum over sixteen rows of the small tensor: what a weight's 22 bits of the largest step (half a unit a token, the
    # signs at random: four deviations of the root of n tokens), the scores' and both kernels' fp32 sums are relative to
    code = {2: 2, 4: 8, 8: 128}[bits]
    vmax = 0.022 * code * float(cache.t["v_small"].float().abs().reshape(-1, 16, 16).sum(-1).max())
    bound = vmax * (4 * (min(n, 4096) ** 0.5) * 2.0 ** -23 + 16 * 2.0 ** -24)
    for splits, waves in ((0, 0), (1, 4), (1, 8), (3, 4), (3, 8)):
        got = torch.empty_like(want)
        out = dq.attn_decode(cache, q, lens, n, ws, out_f32=got, flags=dq.decode_flags(splits=min(splits, tiles), waves=waves))
        torch.cuda.synchronize()
        assert torch.isfinite(got).all() and torch.equal(out, got.half())
        err = float((got - want).abs().max())
        print("  splits %d waves %d: error %.2e of %.2e, output up to %.2e" % (splits, waves, err, bound, float(want.abs().max())), flush=True)
        assert err <= bound, (splits, waves, err, bound)
        assert (got[lens == 0] == 0).all()
