"""The eigen-solver over the spectra it may meet: rows of T_L orthonormal and spanning the block's rows to the rounding
of the fp32 T_L, for spectra from flat to five decades in general position, few rows, few directions, empty channels, and
pairs of 64-channel heads of very different size; the same bits through every number of blocks a solver wave holds; and
all sweeps reported (an iteration that starts from the Gram matrix itself, in double precision throughout, takes four
to seventeen on blocks whose channels are mixed)."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV

pytestmark = pytest.mark.gpu

FULL_RANK = ("normal", "outliers", "graded1", "graded2.5", "graded3")   # no direction is near the cut-off


def _rows(kind, h, dim, g):
    j1 = dim // 8
    x = torch.randn(h, 128, dim, device=DEV, generator=g)
    if kind == "outliers":
        x[..., 3::29] *= 20
    elif kind.startswith("graded"):
        q, _ = torch.linalg.qr(torch.randn(h, j1, j1, device=DEV, generator=g, dtype=torch.float64))
        size = 1000 * 10.0 ** (-float(kind[6:]) * torch.arange(j1, device=DEV) / (j1 - 1))
        x = (q.float()[:, None] @ (x.view(h, 128, j1, 8) * size[:, None])).flatten(-2)
    elif kind == "three_rows":
        x[:, 3:] = 0
    elif kind == "empty_channels":
        x[..., dim // 2:] = 0
    elif kind == "unlike_heads":
        x[1::2] *= 1e-5
    return x.half()


@pytest.mark.parametrize("dim", [128, 64])
@pytest.mark.parametrize("kind", ["normal", "outliers", "graded1", "graded2.5", "graded3", "graded5", "three_rows",
                                  "empty_channels", "unlike_heads"])
def test_blocks_come_out_orthonormal_whatever_they_start_from(kind, dim):
    print("solver start: %s, d=%d" % (kind, dim), flush=True)
    fmt = dq.Format(4, 128 if dim == 128 else 64, dim, dim // 8, 8, 128)
    g = torch.Generator(device=DEV).manual_seed(9)
    h, j1 = 10, dim // 8
    k, v = _rows(kind, h, dim, g), _rows(kind, h, dim, g)
    first = torch.zeros(1, dtype=torch.int32, device=DEV)
    seen = []
    # 2 and 4 waves: one block per solver wave; 1: two; many copies of the heads: four (8220 blocks) and eight (16400)
    for waves, copies in ((4, 1), (2, 1), (1, 1), (0, 411), (0, 820)):
        kk, vv = (t.repeat(copies, 1, 1)[None].contiguous() for t in (k, v))
        if dim == 64 and copies > 1:
            kk, vv = (t.repeat(1, 2, 1, 1) for t in (kk, vv))
        hh = kk.shape[1]
        cache = dq.alloc_cache(fmt, 1, hh, 1, DEV)
        ws = dq.compress_workspace(fmt, 1, hh, DEV)
        dq.compress_kv(cache, kk, vv, first, None, ws, keep_large=True, waves=waves)
        torch.cuda.synchronize()
        sweeps = int(ws[4:8].view(torch.int32).item())
        assert sweeps <= 24, (kind, sweeps)
        if kind in FULL_RANK:
            assert sweeps >= 4, (kind, sweeps)
        seen.append(([cache.t[n][0, :h].clone() for n in ("k_codes", "v_codes", "k_scales", "v_scales", "k_small", "v_small")],
                     ws[256:256 + 2 * h * 128 * dim * 4].view(torch.float32).view(h, 2, 128, j1, 8).clone()))
    large = seen[0][1].double()
    for which, src in enumerate((k, v)):
        t = large[:, which].permute(0, 2, 1, 3).reshape(h, j1, -1)
        m = src.double().view(h, 128, j1, 8).permute(0, 2, 1, 3).reshape(h, j1, -1)
        gram = t @ t.transpose(1, 2)
        kept = torch.diagonal(gram, dim1=1, dim2=2) > 0.5            # (a dropped direction has a zero row)
        want = torch.diag_embed(kept.double())
        # 1024 products of entries rounded to fp32 (2^-24 each, of rows of norm one): 2 * 2^-24 along a row
        assert (gram - want).abs().max() < 2.0 ** -22, kind
        rest = (m - (m @ t.transpose(1, 2)) @ t).norm(dim=(1, 2)) / m.norm(dim=(1, 2))
        if kind in FULL_RANK:
            # every row of T_L is a combination of the block's rows, as many as these are: what a projection on them leaves
            # is their distance from orthonormal and the rounding of their entries (2^-24 each way, sixteen rows of norm one)
            assert kept.all(), kind
            off = torch.linalg.matrix_norm(gram - want, 2)
            assert (rest <= off + 2.0 ** -21).all(), (kind, rest.max().item(), off.max().item())
        else:
            # directions under the cut-off (1e-6 of the largest singular value) are dropped; the rest is rounding
            assert rest.max() < 4e-6, kind
    for arrays, rows in seen[1:]:
        assert torch.equal(rows, seen[0][1])
        for x, y in zip(arrays, seen[0][0]):
            assert torch.equal(x, y)
