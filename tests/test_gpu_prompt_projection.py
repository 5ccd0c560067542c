"""The prompt path's projection runs on the fp16 matrix cores and settles in fp64 only what lies within its
error bound of a decision: codes, steps and small tensors must be those of the fp64 projection (the
path that keeps the fp32 rows), bit for bit, also where the decisions are hard: tokens of very
different size (steps down to fp16 subnormals and zero), empty tokens, values on a coarse grid (many
equal magnitudes), strong outliers, short blocks."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _rows(kind, b, h, n, d, g):
    x = torch.randn(b, h, n, d, device=DEV, generator=g)
    if kind == "sizes":
        x *= 10.0 ** (-7.5 * torch.rand(b, h, n, 1, device=DEV, generator=g))
        x[:, :, ::9] = 0
    elif kind == "grid":
        x = (2 * x).round() / 2
    elif kind == "outliers":
        x[..., ::17] *= 3000
    return x.clamp(-60000, 60000).half()


@pytest.mark.parametrize("kind", ["normal", "sizes", "grid", "outliers"])
@pytest.mark.parametrize("bits,group,dim,levels,tb", [
    (4, 128, 128, 0, 128), (4, 64, 128, 1, 256), (2, 64, 128, 0, 128), (2, 128, 128, 1, 128), (4, 64, 64, 0, 128),
    (2, 64, 64, 1, 256), (4, 32, 128, 0, 128),
])
def test_prompt_projection_is_that_of_the_fp64_path(kind, bits, group, dim, levels, tb):
    print("prompt projection: %s" % ((kind, bits, group, dim, levels, tb),), flush=True)
    fmt = dq.Format(bits, group, dim, dim // 8, 8, tb, 1, levels)
    g = torch.Generator(device=DEV).manual_seed(3)
    b, h, n = 4, 6, 5 * tb - 37
    k, v = _rows(kind, b, h, n, dim, g), _rows(kind, b, h, n, dim, g)
    first = torch.tensor([0, 1, -1, 0], dtype=torch.int32, device=DEV)
    valid = torch.tensor([n, 2 * tb + 5, n, tb + 1], dtype=torch.int32, device=DEV)
    out = []
    # the fp32 rows kept (fp64 projection); not kept (waves=1: the three launches of a prompt on few blocks)
    for kw in (dict(keep_large=True), dict(keep_large=True, waves=1), dict(keep_large=False, waves=1)):
        cache = dq.alloc_cache(fmt, b, h, 5, DEV, fill=0xA5)
        ws = dq.compress_workspace(fmt, b, h, DEV, t_new=n)
        dq.compress_kv_blocks(cache, k, v, first, valid, ws, **kw)
        out.append((cache, ws[:8].clone()))
    for cache, status in out[1:]:
        for name in cache.t:
            assert torch.equal(cache.t[name], out[0][0].t[name]), name
        assert torch.equal(status, out[0][1])
