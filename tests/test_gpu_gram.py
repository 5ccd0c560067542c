"""The Gram matrix of a block is an exact sum rounded once: fp16 rows cut into integer digits, int8 matrix products.
A prompt's launches leave it at the head of the block's part of the workspace, where it is compared with
Python integers: values on both sides of 127.5 (where the fifth digit begins) and of 32256 (where the digits end
and the fp64 instructions take over), fp16 subnormals, short blocks, pairs of 64-channel heads.  The builds of small
calls, several waves per block, must come to the same cache."""
import numpy as np
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV

pytestmark = pytest.mark.gpu

EDGES = [127.4375, 127.5, 128.0, 254.0, 381.0, 512.0, 1000.0, 2.0 ** -24, 3 * 2.0 ** -24, 2.0 ** -14, 0.0, 1.0]


def _rows(kind, shape, g):
    x = torch.randn(shape, device=DEV, generator=g)
    if kind == "outliers":
        x[..., 3::29] *= 100
    elif kind == "edges":
        pick = torch.tensor(EDGES, device=DEV)[torch.randint(len(EDGES), shape, device=DEV, generator=g)]
        x = pick * x.sign()
    elif kind == "equal":          # the largest value without a fifth digit, everywhere: a block of rank one
        x = torch.full(shape, -127.4375, device=DEV)
    elif kind == "last":
        x[..., 5] = 32256
        x[..., 1, 77 % shape[-1]] = -32256
    elif kind == "beyond":
        x[..., 0, 9] = 32272
        x[..., 1, 40] = -65504
    return x.half()


def _exact(x, j1):
    """x fp16 [T, d] -> the Gram matrix of its regrouped rows, every entry rounded once."""
    v = (x.astype(np.float64) * 2.0 ** 24).astype(np.int64).astype(object)
    m = v.reshape(-1, j1, 8).transpose(1, 0, 2).reshape(j1, -1)
    return np.array([[float(e) * 2.0 ** -48 for e in row] for row in m @ m.T])


@pytest.mark.parametrize("kind", ["normal", "outliers", "edges", "equal", "last", "beyond"])
@pytest.mark.parametrize("dim,tb", [(128, 128), (128, 256), (64, 128)])
def test_gram_matrix_is_the_exact_sum_rounded_once(kind, dim, tb):
    print("gram: %s" % ((kind, dim, tb),), flush=True)
    fmt = dq.Format(4, 128 if dim == 128 else 64, dim, dim // 8, 8, tb)
    g = torch.Generator(device=DEV).manual_seed(5)
    valid = [2 * tb, tb + 1, tb + 5, 37, tb - 1]
    b, h, j1 = len(valid), 2, dim // 8
    k, v = _rows(kind, (b, h, 2 * tb, dim), g), _rows(kind, (b, h, 2 * tb, dim), g)
    first = torch.zeros(b, dtype=torch.int32, device=DEV)
    n = torch.tensor(valid, dtype=torch.int32, device=DEV)
    caches = []
    for waves in (1, 2, 4):
        cache = dq.alloc_cache(fmt, b, h, 2, DEV)
        ws = dq.compress_workspace(fmt, b, h, DEV, t_new=2 * tb)
        dq.compress_kv_blocks(cache, k, v, first, n, ws, keep_large=False, waves=waves)
        torch.cuda.synchronize()
        caches.append(cache)
        if waves == 1:
            # [batch, head, block, K|V]: the block's part of the workspace
            part = ws[256:256 + b * h * 2 * 2 * tb * dim * 4].view(torch.float64).view(b, h, 2, 2, -1)[..., :256].cpu().numpy()
    for i in range(b):
        for j in range(2):
            rows = min(max(valid[i] - j * tb, 0), tb)
            for which, src in enumerate((k, v)):
                if rows == 0:
                    continue
                want = [_exact(src[i, hh, j * tb:j * tb + rows].cpu().numpy(), j1) for hh in range(h)]
                if dim == 64:      # one matrix for the pair, no products across the heads
                    pair = np.zeros((16, 16))
                    pair[:8, :8], pair[8:, 8:] = want
                    want = [pair]
                for hh, w in enumerate(want):
                    got = part[i, hh, j, which].reshape(16, 16)
                    size = np.sqrt(np.outer(np.diag(w), np.diag(w)))
                    if kind == "beyond":   # 8 * tb exact products, each sum rounds
                        assert (np.abs(got - w) <= 8 * tb * 2.0 ** -53 * size).all(), (i, hh, j, which)
                    elif kind == "last":   # the high half has bits from 2^39 * 2^16 (sums of squares near 2^39) down to
                        # 2^-7 and rounds where its terms are added, three times, before the last rounding
                        assert (np.abs(got - w) <= 4 * 2.0 ** -53 * size).all(), (i, hh, j, which)
                    else:
                        assert (got == w).all(), (i, hh, j, which)
    if kind != "beyond":
        for other in caches[1:]:
            for name in other.t:
                assert torch.equal(other.t[name], caches[0].t[name]), name


def _exact_long(x, j1):
    """_exact for long blocks: the products of upper and lower halves of the values in 64-bit integers
    (2^20 * 2^20 * 2^17 columns), joined as Python integers."""
    v = (x.astype(np.float64) * 2.0 ** 24).astype(np.int64)
    m = v.reshape(-1, j1, 8).transpose(1, 0, 2).reshape(j1, -1)
    hi, lo = m >> 20, m & (2 ** 20 - 1)
    top, mid, low = hi @ hi.T, hi @ lo.T, lo @ lo.T
    mid = mid + mid.T
    return np.array([[float((int(top[p, q]) << 40) + (int(mid[p, q]) << 20) + int(low[p, q])) * 2.0 ** -48
                      for q in range(j1)] for p in range(j1)])


@pytest.mark.parametrize("tokens", [257, 8191, 16512])
@pytest.mark.parametrize("kind", ["half", "tiny", "wide", "top", "small_by_large", "normal", "edges"])
def test_gram_matrix_of_long_blocks(kind, tokens):
    """The products of digits are summed in 32 bits.  One digit of -128 throughout (a half) passes 2^31 at 16384
    tokens of a wave, other values later; a block may have any multiple of 128 tokens.  257 tokens: the first that a
    wave alone adds up in two parts."""
    print("gram of a long block: %s, %d tokens" % (kind, tokens), flush=True)
    tb = -(-tokens // 128) * 128
    fmt = dq.Format(4, 128, 128, 16, 8, tb)
    g = torch.Generator(device=DEV).manual_seed(6)
    shape = (1, 2, tokens, 128)
    fill = {"half": 0.5,                      # the third digit is -128
            "tiny": -32896 * 2.0 ** -24,      # the two lowest digits are
            "wide": 126.5,                    # the third -128, the fourth 127
            "top": 31872.0}                   # the fifth 125, the fourth 122
    if kind in fill:
        k = torch.full(shape, fill[kind], device=DEV)
    elif kind == "small_by_large":            # the two products of the middle weight at their largest together
        k = torch.full(shape, 126.5, device=DEV)
        k[..., :64] = -32896 * 2.0 ** -24
    else:
        k = _rows(kind, shape, g)
    k = k.half()
    v = k * torch.randn(shape, device=DEV, generator=g).sign().half()   # (the off-diagonal sums cancel)
    first = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = dq.compress_workspace(fmt, 1, 2, DEV, t_new=tokens)
    caches = []
    for waves in (1, 2, 4):
        cache = dq.alloc_cache(fmt, 1, 2, 1, DEV)
        dq.compress_kv(cache, k, v, first, None, ws, keep_large=False, waves=waves)
        torch.cuda.synchronize()
        caches.append(cache)
        if waves == 1:
            part = ws[256:256 + 2 * 2 * tb * 128 * 4].view(torch.float64).view(2, 2, -1)[..., :256].cpu().numpy()
    for h in range(2):
        for which, src in enumerate((k, v)):
            want = _exact_long(src[0, h].cpu().numpy(), 16)
            got = part[h, which].reshape(16, 16)
            if kind in ("edges", "top"):   # rows with values beyond 127.5: every part of 256 tokens may round three times
                size = np.sqrt(np.outer(np.diag(want), np.diag(want)))
                assert (np.abs(got - want) <= (3 * -(-tokens // 256) + 1) * 2.0 ** -53 * size).all(), (h, which)
            else:
                assert (got == want).all(), (h, which)
    if kind == "normal":
        for other in caches[1:]:
            for name in other.t:
                assert torch.equal(other.t[name], caches[0].t[name]), name
