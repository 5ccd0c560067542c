"""Value steps that no compression writes, within a sequence's length, in every build of the matrix-core kernel with two local tensors: an
infinite step counts as the largest that a tile's weights can hold (1 - 2^-11: the tile's scale is one then), a NaN step's
token has no weight.  Compared with the plain kernel on the same cache with that step in their place."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV
from test_launch_shape import shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [4, 2, 8])
@pytest.mark.parametrize("group,dim,rep,batch", [(128, 128, 1, 2), (128, 128, 2, 2), (128, 128, 4, 2), (128, 128, 8, 17), (64, 128, 1, 2), (64, 128, 2, 2),
                                                 (64, 128, 4, 17), (64, 64, 1, 2), (64, 64, 2, 2)])
def test_an_infinite_and_a_nan_value_step(bits, group, dim, rep, batch):
    print("special steps: %s" % ((bits, group, dim, rep, batch),), flush=True)
    heads, tiles = 8, 4
    assert shape(dq, bits, group, rep, batch, tiles, dim=dim)[3] == (2 if dim == 64 and rep > 1 else rep)
    fmt = dq.Format(bits, group, dim, dim // 8, 8, 128)
    g = torch.Generator(device=DEV).manual_seed(bits + rep)
    cache = dq.alloc_cache(fmt, batch, heads, tiles, DEV, fill=None)
    for name, x in cache.t.items():
        if "codes" in name:
            x.random_(0, 256, generator=g)
        elif "scales" in name:
            x.copy_(torch.rand(x.shape, device=DEV, generator=g) * 0.02 + 0.002)
        else:
            x.copy_(torch.randn(x.shape, device=DEV, generator=g) * 0.25)
    n = tiles * 128 - 3
    lens = torch.full((batch,), n, dtype=torch.int32, device=DEV)
    q = torch.randn(batch, heads * rep, dim, device=DEV, generator=g).half()
    ws = dq.decode_workspace(fmt, batch, heads * rep, heads, n, DEV)
    steps = cache.t["v_scales"].view(batch, heads, tiles * 128, dim // group)
    places = [(0, 1, 5, 0), (batch - 1, 6, 200, dim // group - 1), (batch - 1, 2, n - 1, 0)]   # (in the first, a middle and the last tile)
    want, got = (torch.empty(batch, heads * rep, dim, dtype=torch.float32, device=DEV) for _ in "wg")
    for written, counts_as in ((float("inf"), 1 - 2.0 ** -11), (float("nan"), 0.0)):
        for at in places:
            steps[at] = counts_as
        dq.attn_decode(cache, q, lens, n, ws, out_f32=want, flags=dq.DECODE_FORCE_GENERIC)
        for at in places:
            steps[at] = written
        # half a unit of 22 bits of a step of one, in each of a tile's tokens (signs at random: four deviations), at most 128 of them under that
        # scale, times the largest code and a sum of small-tensor entries; sums in fp32
        code = {2: 2, 4: 8, 8: 128}[bits]
        vmax = code * float(cache.t["v_small"].float().abs().sum(-1).max())
        bound = vmax * (4 * 128 ** 0.5 * 2.0 ** -23 + 16 * 2.0 ** -24)
        for splits, waves in ((0, 0), (1, 8), (2, 4)):
            dq.attn_decode(cache, q, lens, n, ws, out_f32=got, flags=dq.decode_flags(splits=splits, waves=waves))
            torch.cuda.synchronize()
            err = float((got - want).abs().max())
            print("  %s splits %d waves %d: error %.2e of %.2e, output up to %.2e" % (written, splits, waves, err, bound, float(want.abs().max())), flush=True)
            assert torch.isfinite(got).all() and err <= bound
