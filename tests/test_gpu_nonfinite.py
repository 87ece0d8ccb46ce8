"""Float frames with pixels that are not finite: the pixels a value that is not a number reaches follow
from the method alone, whatever kernels and tiles a call runs on."""
import numpy as np
import pytest

import oracle
from gpu_util import announce, dev, to_dev

pytestmark = pytest.mark.gpu


def _frames(shape, seed, spots, value):
    rng = np.random.default_rng(seed)
    I1, I2 = (rng.integers(0, 256, size=shape).astype(np.float32) for _ in range(2))
    for y, x in spots:
        I1[y, x] = value
    return I1, I2


def _reached(I1, levels, r):
    """Pixels of one-iteration levels that a NaN of frame 1 reaches: the products at its position (or
    at a position whose field is NaN) and every window that holds one; the prolongation reads its
    base row and column and those after them, with a weight of zero too."""
    P = oracle.pyramid(I1, levels)
    nan = None
    for p in reversed(P):
        bad = ~np.isfinite(p)
        if nan is not None:
            up = np.isnan(oracle.upsample_flow(np.where(nan, np.nan, 0.0), *p.shape))
            bad |= up
        nan = oracle.box_sum(bad.astype(np.float64), r) > 0
    return nan


def _bits(u, v):
    """Bits of a field, with every NaN alike."""
    import torch
    f = torch.stack([u, v])
    return torch.where(torch.isnan(f), torch.full_like(f, float("nan")), f).cpu().numpy().view(np.int32)


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("r,levels", [(0, 2), (1, 3), (2, 3), (4, 2), (5, 3), (8, 2), (9, 2), (12, 2)])
def test_reach_of_a_pixel_that_is_not_finite(gpu_lib, r, levels, value):
    import torch
    ofmi = gpu_lib
    N = 2 * r + 1
    shape = (5 * N + 22, 150)
    I1, I2 = _frames(shape, 3, [(2 * N + 7, 40), (N + 5, 101), (0, 146), (shape[0] - 1, 20)], value)
    want = _reached(I1, levels, r)
    announce(f"not finite r={r} L={levels} {value}")
    d1, d2 = to_dev(I1), to_dev(I2)
    plan = ofmi.Plan(*shape, levels, r, 1, input_f32=True, device=dev())

    def flow(bands=None, variant=None):
        if bands:
            plan.set_config({"bands": [bands] * levels, "variant": [variant] * levels})
        u, v = plan.compute(d1, d2)
        torch.cuda.synchronize()
        return _bits(u, v)

    ref = flow()
    assert np.array_equal(~np.isfinite(ref[0].view(np.float32)), want)
    for variant in range(8):
        if variant > 4 and r > 8:
            continue
        for bands in (1, 2, 3):
            assert np.array_equal(flow(bands, variant), ref), (variant, bands)
    plan.close()
    for fp16 in (False, True):
        plan = ofmi.Plan(*shape, levels, r, 1, input_f32=True, fp16=fp16, device=dev())
        ref = flow()
        plan.close()
        b = ofmi.Batch([shape], levels, r, 1, input_f32=True, fp16=fp16, device=dev())
        for bands in (None, 1, 2, 4):
            for variant in (0, 1):
                if bands:
                    b.set_config({"bands": [bands] * levels, "variant": [variant] * levels, "grid": [0] * levels})
                us, vs = b.compute([d1], [d2])
                torch.cuda.synchronize()
                assert np.array_equal(_bits(us[0], vs[0]), ref), (fp16, bands, variant)
        b.close()


@pytest.mark.parametrize("shape", [(40, 70), (1, 40), (40, 1), (2, 3)])
@pytest.mark.parametrize("r", [0, 2, 8])
def test_8_bit_frames_under_a_field_that_is_not_finite(gpu_lib, r, shape):
    """One iteration from a caller's field that holds NaNs and infinities: 8-bit frames give what float
    frames of the same values give, next to those pixels too (their samples come from the clamped
    position, that of a NaN from the first pixel of its axis)."""
    import torch
    ofmi = gpu_lib
    announce(f"8-bit frames, field not finite r={r} {shape}")
    rng = np.random.default_rng(7)
    H, W = shape
    I = [to_dev(rng.integers(0, 256, size=shape).astype(np.uint8)) for _ in range(2)]
    f = rng.uniform(-3, 3, size=(2, *shape)).astype(np.float32)
    for k, value in enumerate([np.nan, np.inf, -np.inf, np.nan]):
        f[k % 2, (5 + 9 * k) % H, (11 + 17 * k) % W] = value
    f[:, H - 1, W - 1] = np.nan
    got = []
    for f32 in (False, True):
        plan = ofmi.Plan(H, W, 1, r, 1, input_f32=f32, device=dev())
        for variant in range(8) if r <= 8 else range(5):
            plan.set_config({"bands": [1], "variant": [variant]})
            un = torch.empty(shape, dtype=torch.float32, device=dev())
            vn = torch.empty_like(un)
            ofmi.debug_stage(plan, ofmi.OF_STAGE_ITERATE, 0,
                             [i.float() if f32 else i for i in I] + [to_dev(f[0]), to_dev(f[1])], [un, vn])
            torch.cuda.synchronize()
            got.append(_bits(un, vn))
        plan.close()
    for g in got:
        assert np.array_equal(g, got[-1])
