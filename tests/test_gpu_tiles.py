"""The iteration kernel at the edges of its tiles, for every radius: thread groups per column,
rows per thread and pass structure all follow from the radius, the strip width and the bands per
pass, so each radius is a kernel shape of its own."""
import numpy as np
import pytest

import floor_util
import oracle
import synth
from gpu_util import announce, dev, flow_error, to_dev

pytestmark = pytest.mark.gpu

TOL32 = 1e-3


def _frames(H, W):
    I1, I2, _, _ = synth.make_pair("c1", 11)
    I1, I2 = np.tile(I1, (2, 2)), np.tile(I2, (2, 2))
    return np.ascontiguousarray(I1[30:30 + H, 20:20 + W]), np.ascontiguousarray(I2[30:30 + H, 20:20 + W])


@pytest.mark.parametrize("r", range(13))
def test_every_radius_at_tile_edges(gpu_lib, r):
    """Frames one row past a whole number of bands and one column past a strip, two levels: the
    default tiles on every pixel against the oracle (tolerance, or where an FP32 evaluation departs
    from FP64 further, the floor computed here), the same with float frames of the same values and
    with every tile variant at one to three bands, bit for bit."""
    import torch
    ofmi = gpu_lib
    N = 2 * r + 1
    H, W, L, K = max(3 * N + 1, 4), 129, 2, 2
    I1, I2 = _frames(H, W)
    announce(f"tile edges r={r} {H}x{W}")
    plan = ofmi.Plan(H, W, L, r, K, device=dev())
    d1, d2 = to_dev(I1), to_dev(I2)
    u, v = plan.compute(d1, d2)
    torch.cuda.synchronize()
    u0, v0 = u.cpu().numpy(), v.cpu().numpy()
    floor, (ou, ov) = floor_util.ensemble_floor(I1, I2, L, r, K)
    print(floor_util.check_all_pixels(flow_error(u0, v0, ou, ov), TOL32, floor, f"r={r}"))
    f32 = ofmi.Plan(H, W, L, r, K, input_f32=True, device=dev())
    u, v = f32.compute(d1.float(), d2.float())
    torch.cuda.synchronize()
    assert np.array_equal(u.cpu().numpy(), u0) and np.array_equal(v.cpu().numpy(), v0)
    f32.close()
    for variant in range(8):
        if variant > 4 and r > 8:
            continue
        for nb in (1, 2, 3):
            plan.set_config({"bands": [nb, 1], "variant": [variant, variant]})
            u, v = plan.compute(d1, d2)
            torch.cuda.synchronize()
            assert np.array_equal(u.cpu().numpy(), u0) and np.array_equal(v.cpu().numpy(), v0), (variant, nb)
    plan.close()


@pytest.mark.parametrize("shape", [(40, 70), (200, 210), (2, 2), (2, 90), (90, 2), (1, 50), (50, 1)])
@pytest.mark.parametrize("reach", [3.0, 1e3, 1e7, 4e9])
def test_samples_past_the_image(gpu_lib, shape, reach):
    """Displacements that leave the image by a little, by a lot, and past the range of a 32-bit
    integer: 8-bit frames (two taps from a base clamped to n - 2) give the bits of float frames of
    the same values (taps clamped one by one)."""
    import torch
    ofmi = gpu_lib
    H, W = shape
    rng = np.random.default_rng(5)
    I1 = rng.integers(0, 256, size=shape).astype(np.uint8)
    I2 = rng.integers(0, 256, size=shape).astype(np.uint8)
    u = (reach * rng.uniform(-1, 1, size=shape)).astype(np.float32)
    v = (reach * rng.uniform(-1, 1, size=shape)).astype(np.float32)
    u[0, 0], v[-1, -1] = -0.0, 0.0
    got = []
    for f32 in (False, True):
        announce(f"samples past the image {shape} reach {reach} f32={f32}")
        plan = ofmi.Plan(H, W, 1, 2, 1, input_f32=f32, device=dev())
        cast = (lambda a: to_dev(a).float()) if f32 else to_dev
        un = torch.empty(shape, dtype=torch.float32, device=dev())
        vn = torch.empty_like(un)
        ofmi.debug_stage(plan, ofmi.OF_STAGE_ITERATE, 0, [cast(I1), cast(I2), to_dev(u), to_dev(v)], [un, vn])
        torch.cuda.synchronize()
        got.append((un.cpu().numpy(), vn.cpu().numpy()))
        plan.close()
    assert np.array_equal(got[0][0], got[1][0], equal_nan=True)
    assert np.array_equal(got[0][1], got[1][1], equal_nan=True)


@pytest.mark.parametrize("sizes", [[(1024, 1024)], [(1024, 1024)] * 3 + [(200, 333)], [(33, 40)] * 40])
def test_batch_default_heights(gpu_lib, sizes):
    """Default tile heights of a batch (from one band to taller than the shorter frames) give each
    pair the bits of its own plan."""
    import torch
    ofmi = gpu_lib
    announce(f"batch default heights {len(sizes)} x {sizes[0]}")
    big1, big2, _, _ = synth.make_pair("c2", 1)
    b = ofmi.Batch(sizes, 3, 6, 2, device=dev())
    d1 = [to_dev(np.ascontiguousarray(big1[i:i + h, :w] if h < 1000 else big1)) for i, (h, w) in enumerate(sizes)]
    d2 = [to_dev(np.ascontiguousarray(big2[i:i + h, :w] if h < 1000 else big2)) for i, (h, w) in enumerate(sizes)]
    us, vs = b.compute(d1, d2)
    torch.cuda.synchronize()
    assert all(1 <= n <= 64 for n in b.config()["bands"])
    for i in {0, len(sizes) - 1}:
        plan = ofmi.Plan(*sizes[i], 3, 6, 2, device=dev())
        u, v = plan.compute(d1[i], d2[i])
        torch.cuda.synchronize()
        assert torch.equal(u, us[i]) and torch.equal(v, vs[i]), i
        plan.close()
    b.close()


@pytest.mark.parametrize("r", range(13))
@pytest.mark.parametrize("shape", [(1, 1), (37, 18), (97, 129), (300, 390)])
def test_gaussian_one_band_tiles(gpu_lib, r, shape):
    """The Gaussian window's default tiles (up to r = 8 two-band passes on 16 or 32 columns on small
    levels), tiles of one band and taller ones give the bits of the narrow variant, also under a mask
    of ones (whose tiles keep 64 columns)."""
    import torch
    ofmi = gpu_lib
    announce(f"gaussian one-band tiles r={r} {shape}")
    I1, I2 = (to_dev(np.ascontiguousarray(np.pad(f, ((0, 140), (0, 200)), mode="reflect")[:shape[0], :shape[1]]))
              for f in _frames(220, 220))
    plan = ofmi.Plan(*shape, 1, r, 3, gaussian_window=True, device=dev())

    def flow(bands=None, variant=None):
        if bands:
            plan.set_config({"bands": [bands], "variant": [variant]})
        u, v = plan.compute(I1, I2)
        torch.cuda.synchronize()
        return torch.stack([u, v]).cpu().numpy().view(np.int32)

    default = flow()
    ref = flow(2, 0)
    assert np.array_equal(default, ref)
    for bands, variant in [(1, 1), (1, 2), (3, 1), (1, 0)]:
        assert np.array_equal(flow(bands, variant), ref), (bands, variant)
    plan.set_mask(torch.ones(shape, dtype=torch.uint8, device=dev()))
    assert np.array_equal(flow(1, 1), ref)
    plan.close()


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("r", range(13))
def test_batch_field_from_coarser_level(gpu_lib, r, f32):
    """First iterations of a batch, which hand the field of a coarser level on within the tile, against
    plans, which read it again: the same bits for every radius, odd sizes and tiles of 1 .. 5 bands."""
    import torch
    ofmi = gpu_lib
    announce(f"batch field from the coarser level r={r} f32={f32}")
    sizes = [(4 * (2 * r + 1) + 3, 201), (max(2 * r + 1, 5), 66), (150, 131)]
    frames = [[to_dev(np.ascontiguousarray(f[:h, :w])) for f in _frames(150, 201)] for h, w in sizes]
    if f32:
        frames = [[f.float() * 0.75 for f in p] for p in frames]
    b = ofmi.Batch(sizes, 3, r, 1, input_f32=f32, device=dev())
    for nb in (None, 1, 2, 5):
        if nb:
            b.set_config({"bands": [nb] * 3, "variant": [1] * 3, "grid": [0] * 3})
        us, vs = b.compute([p[0] for p in frames], [p[1] for p in frames])
        for i, s in enumerate(sizes):
            plan = ofmi.Plan(*s, 3, r, 1, input_f32=f32, device=dev())
            u, v = plan.compute(*frames[i])
            torch.cuda.synchronize()
            assert torch.equal(u.view(torch.int32), us[i].view(torch.int32)), (nb, i)
            assert torch.equal(v.view(torch.int32), vs[i].view(torch.int32)), (nb, i)
            plan.close()
    b.close()
