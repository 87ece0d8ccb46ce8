"""Masks under the Gaussian-weighted window: a masked plan runs the tiles that its heights were chosen for."""
import numpy as np
import pytest

import synth
from gpu_util import announce, dev, to_dev

pytestmark = pytest.mark.gpu


def _mask(H, W):
    y, x = np.mgrid[0:H, 0:W]
    m = (x >= 7) & (y < H - 5) & ((x - W // 2) ** 2 + (y - H // 2) ** 2 > (min(H, W) // 4) ** 2)
    return m.astype(np.uint8)


@pytest.mark.parametrize("r", [0, 1, 4, 8, 9])
@pytest.mark.parametrize("shape", [(97, 129), (256, 300)])
def test_masked_gaussian_tiles(gpu_lib, r, shape):
    """Default tiles under a mask (up to r = 8 one-band tiles of 16 or 32 columns with flags of their
    own) give the bits of the narrow variant and of taller tiles, masked pixels zero."""
    import torch
    ofmi = gpu_lib
    announce(f"masked gaussian tiles r={r} {shape}")
    I1, I2, _, _ = synth.make_pair("c2", 4)
    H, W = shape
    d1, d2 = (to_dev(np.ascontiguousarray(f[:H, :W])) for f in (I1, I2))
    mask = to_dev(_mask(H, W))
    plan = ofmi.Plan(H, W, 2, r, 2, gaussian_window=True, device=dev())
    plan.set_mask(mask)

    def flow(bands=None, variant=None):
        if bands:
            plan.set_config({"bands": [bands] * 2, "variant": [variant] * 2})
        u, v = plan.compute(d1, d2)
        torch.cuda.synchronize()
        return torch.stack([u, v])

    ref = flow(2, 0)
    assert bool((ref[:, mask == 0] == 0).all()) and bool((ref[:, mask != 0] != 0).any())
    for bands, variant in [(1, 1), (1, 0), (3, 1)]:
        assert torch.equal(flow(bands, variant).view(torch.int32), ref.view(torch.int32)), (bands, variant)
    plan.close()
    plan = ofmi.Plan(H, W, 2, r, 2, gaussian_window=True, device=dev())
    plan.set_mask(mask)
    assert torch.equal(flow().view(torch.int32), ref.view(torch.int32))
    plan.close()


def test_mask_of_ones_takes_the_tiles_of_no_mask(gpu_lib):
    """A small level's iterations take the same time with a mask of ones (5.7 us at 128^2, r = 8; at the
    same height in 64-column strips, for which it was not chosen, 9.5 us)."""
    import torch
    ofmi = gpu_lib
    I1, I2, _, _ = synth.make_pair("c2", 4)
    d1, d2 = (to_dev(np.ascontiguousarray(f[:128, :128])) for f in (I1, I2))
    plan = ofmi.Plan(128, 128, 1, 8, 8, gaussian_window=True, device=dev())
    times = []
    for masked in (False, True):
        announce(f"gaussian level time, mask of ones: {masked}")
        if masked:
            plan.set_mask(torch.ones((128, 128), dtype=torch.uint8, device=dev()))
        for _ in range(10):
            plan.compute(d1, d2)
        torch.cuda.synchronize()
        best = 1e9
        for _ in range(10):
            plan.set_timing(ofmi.OF_TIMING_LEVEL)
            for _ in range(10):
                plan.compute(d1, d2)
            torch.cuda.synchronize()
            ms, launches = plan.read_timing(ofmi.OF_KERNEL_LEVEL(0))[:2]
            plan.set_timing(0)
            best = min(best, ms / launches)
        times.append(best)
    plan.close()
    print(times)
    assert times[1] <= 1.25 * times[0], times
