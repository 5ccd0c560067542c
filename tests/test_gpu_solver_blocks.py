"""The eigen-solver of a prompt works two, four or eight blocks a wave and passes matrices and factors through LDS: on both
sides of the lines between them, with blocks that are skipped beside live ones in a wave and a last wave that is not full,
every block comes out with the bits of a call of its own."""
import pytest
import torch

import paper_2405_12591_amd as dq
from gpu_util import DEV

pytestmark = pytest.mark.gpu


# blocks (keys and values) of the call that is compared; sequences beside the first are skipped
@pytest.mark.parametrize("dim,heads,batch", [(128, 1024, 1), (128, 1025, 1), (128, 683, 3), (128, 6144, 1), (128, 6145, 1),
                                             (128, 2050, 3), (64, 2050, 1), (64, 1366, 10)])
def test_every_number_of_blocks_a_wave(dim, heads, batch):
    print("solver blocks: %s" % ((dim, heads, batch),), flush=True)
    fmt = dq.Format(4, 128 if dim == 128 else 64, dim, dim // 8, 8, 128)
    g = torch.Generator(device=DEV).manual_seed(13)
    few = 6
    size = 10.0 ** (-3 * torch.rand(few, 1, dim, device=DEV, generator=g))     # graded channels: unlike numbers of sweeps
    k, v = ((torch.randn(few, 128, dim, device=DEV, generator=g) * size * 50).half() for _ in range(2))
    at = torch.arange(heads, device=DEV) // 2 % (few // 2) * 2 + torch.arange(heads, device=DEV) % 2   # (pairs stay together)
    first = torch.tensor([0] + [-1] * (batch - 1), dtype=torch.int32, device=DEV)
    caches = []
    for kk, vv, f, waves in ((k[at].expand(batch, -1, -1, -1), v[at].expand(batch, -1, -1, -1), first, 0),
                             (k[None], v[None], first[:1], 4)):
        cache = dq.alloc_cache(fmt, kk.shape[0], kk.shape[1], 1, DEV, fill=0x5A)
        ws = dq.compress_workspace(fmt, kk.shape[0], kk.shape[1], DEV)
        dq.compress_kv(cache, kk.contiguous(), vv.contiguous(), f, None, ws, keep_large=False, waves=waves)
        torch.cuda.synchronize()
        caches.append(cache)
    for name in ("k_codes", "v_codes", "k_scales", "v_scales", "k_small", "v_small"):
        many, one = caches[0].t[name], caches[1].t[name]
        assert torch.equal(many[0], one[0][at]), name
        if batch > 1:
            assert (many[1:].view(torch.uint8) == 0x5A).all(), name           # nothing is written for a skipped block
