"""The prompt path's projection runs on the fp16 matrix cores and takes only the tokens within its error
bound of a decision through fp64: codes, steps and small tensors must be those of the fp64 projection (the
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
    (2, 64, 64, 1, 256), (4, 128, 128, 1, 128),
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


def _hard_rows(kind, b, h, n, d, g):
    """Blocks that an error bound of the fp16 pass has to know about."""
    j1 = d // 8
    x = torch.randn(b, h, n, d, device=DEV, generator=g)
    if kind == "subnormal":        # most tokens among fp16's subnormals, some ordinary: W is of the ordinary ones' size
        x *= torch.where(torch.arange(n, device=DEV) % 16 == 0, 1.0, 1e-6)[:, None]
    elif kind == "one_row":        # every column of the regrouped matrix has one entry: a diagonal Gram matrix
        at = torch.randint(j1, (b, h, n, 1, 8), device=DEV, generator=g)
        x = (x.view(b, h, n, j1, 8) * torch.zeros(b, h, n, j1, 8, device=DEV).scatter_(3, at, 1.0)).flatten(-2)
    elif kind.startswith("mixed"):       # singular values over so many decades, in general position
        q, _ = torch.linalg.qr(torch.randn(b, h, j1, j1, device=DEV, generator=g, dtype=torch.float64))
        size = 1000 * 10.0 ** (-float(kind[5:]) * torch.arange(j1, device=DEV) / (j1 - 1))
        x = (q.float()[:, :, None] @ (x.view(b, h, n, j1, 8) * size[:, None])).flatten(-2)
    elif kind.startswith("channels"):    # the same, along the channels
        x = 1000 * x * 10.0 ** (-float(kind[8:]) * torch.arange(d, device=DEV) / (d - 1))
    elif kind == "low_rank":       # four directions, and small tokens that have more
        x = torch.randn(b, h, 1, 4, d, device=DEV, generator=g) * torch.randn(b, h, n, 4, 1, device=DEV, generator=g)
        x = 100 * x.sum(3)
        x[:, :, 5::7] = 1e-4 * torch.randn(b, h, len(range(5, n, 7)), d, device=DEV, generator=g)
    elif kind == "dropped":        # tokens that live in a direction under the cut-off alone
        x = 300 * x
        x[..., 8:16] *= 3e-7
        x[:, :, 3::11, :8] = x[:, :, 3::11, 16:] = 0
    return x.clamp(-60000, 60000).half()


@pytest.mark.parametrize("kind", ["subnormal", "one_row", "mixed1", "mixed2", "mixed4", "mixed6", "channels3", "channels6",
                                  "low_rank", "dropped"])
@pytest.mark.parametrize("bits,group,dim,levels", [(4, 128, 128, 0), (4, 64, 128, 1), (2, 64, 128, 0), (4, 64, 64, 0)])
def test_prompt_projection_on_blocks_that_strain_its_bound(kind, bits, group, dim, levels):
    """2048 blocks (half as many pairs of 64-channel heads) each."""
    print("strained prompt projection: %s" % ((kind, bits, group, dim, levels),), flush=True)
    fmt = dq.Format(bits, group, dim, dim // 8, 8, 128, 1, levels)
    g = torch.Generator(device=DEV).manual_seed(7)
    b, h, n = 8, 32, 4 * 128
    k, v = _hard_rows(kind, b, h, n, dim, g), _hard_rows(kind, b, h, n, dim, g)
    first = torch.zeros(b, dtype=torch.int32, device=DEV)
    caches = []
    for keep in (True, False):
        cache = dq.alloc_cache(fmt, b, h, 4, DEV, fill=0xA5)
        ws = dq.compress_workspace(fmt, b, h, DEV, t_new=n)
        dq.compress_kv_blocks(cache, k, v, first, None, ws, keep_large=keep, waves=1)
        caches.append(cache)
    for name in caches[0].t:
        assert torch.equal(caches[1].t[name].view(torch.uint8), caches[0].t[name].view(torch.uint8)), name


@pytest.mark.parametrize("groups", [2048, 2050, 2816, 2818, 6144, 6146, 8192, 8194])
@pytest.mark.parametrize("bits,group,dim,levels", [(4, 128, 128, 0), (2, 64, 128, 1), (4, 64, 64, 1), (2, 64, 64, 0)])
def test_prompt_projection_on_both_sides_of_its_launch_rules(bits, group, dim, levels, groups):
    """Calls of up to 2048, 2816, 6144, 8192 and more workgroups take different builds: sequences of whole
    and of ragged length, easy tokens and blocks that are settled in fp64 as a whole, against the rows kept."""
    print("projection launch rules: %s" % ((bits, group, dim, levels, groups),), flush=True)
    fmt = dq.Format(bits, group, dim, dim // 8, 8, 128, 1, levels)
    g = torch.Generator(device=DEV).manual_seed(11)
    nb, b, h = groups // 2, 1, 1 if dim == 128 else 2   # keys and values; a workgroup takes a pair of 64-channel heads
    n = nb * 128
    k = torch.cat([_rows("normal", b, h, n - 256 * 128, dim, g), _hard_rows("mixed3", b, h, 256 * 128, dim, g)], 2)
    v = torch.cat([_hard_rows("channels3", b, h, 256 * 128, dim, g), _rows("outliers", b, h, n - 256 * 128, dim, g)], 2)
    first = torch.zeros(b, dtype=torch.int32, device=DEV)
    for valid in (n, n - 128 * 3 - 37):
        caches = []
        for keep in (True, False):
            cache = dq.alloc_cache(fmt, b, h, nb, DEV, fill=0xA5)
            ws = dq.compress_workspace(fmt, b, h, DEV, t_new=n)
            dq.compress_kv_blocks(cache, k, v, first, torch.tensor([valid], dtype=torch.int32, device=DEV), ws, keep_large=keep)
            caches.append(cache)
        for name in caches[0].t:
            assert torch.equal(caches[1].t[name].view(torch.uint8), caches[0].t[name].view(torch.uint8)), name
