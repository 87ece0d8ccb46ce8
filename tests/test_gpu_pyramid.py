"""The pyramid step of 8-bit frames (eight-byte row windows and byte permutations per lane) against
the one of float frames of the same values (one thread per output): the same bits."""
import numpy as np
import pytest

from gpu_util import announce, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp16", [False, True])
@pytest.mark.parametrize("H", [2, 3, 17, 63, 64, 66, 130])
def test_u8_reduction_at_edges(gpu_lib, H, fp16):
    """Widths below, at and past the eight-byte window and the 256 input columns of a wave, odd and
    even (unaligned rows and output pairs), frames at odd addresses."""
    import torch
    ofmi = gpu_lib
    g = torch.Generator().manual_seed(H)
    for W in (2, 3, 5, 7, 8, 9, 10, 31, 254, 255, 256, 257, 258, 259, 513):
        announce(f"u8 reduction {H}x{W} fp16={fp16}")
        flat = torch.randint(0, 256, (H * W + 3,), generator=g, dtype=torch.uint8).to(dev())
        got = []
        for off, f32 in [(0, True), (0, False), (1, False), (3, False)]:
            frame = flat[off:off + H * W].view(H, W)
            if f32:
                frame = frame.float()
            elif off:
                flat[off:off + H * W] = flat0   # the same values at an odd address
            else:
                flat0 = frame.clone().flatten()
            plan = ofmi.Plan(H, W, 2, 2, 1, fp16=fp16, input_f32=f32, device=dev())
            out = torch.full(((H + 1) // 2, (W + 1) // 2), -1.0, dtype=torch.float16 if fp16 else torch.float32,
                             device=dev())
            ofmi.debug_stage(plan, ofmi.OF_STAGE_REDUCE, 0, [frame], [out])
            torch.cuda.synchronize()
            got.append(out.cpu().numpy())
            plan.close()
        for o in got[1:]:
            assert np.array_equal(o, got[0]), W


@pytest.mark.parametrize("shape,L", [((513, 515), 4), ((1030, 1027), 4), ((1921, 1923), 3), ((1024, 1024), 2)])
def test_chain_and_single_levels(gpu_lib, shape, L):
    """Either side of the sizes from which the first level of 8-bit frames is reduced by itself: the
    flow of float frames of the same values (chains up to larger sizes)."""
    import torch
    ofmi = gpu_lib
    announce(f"pyramid forms {shape} L={L}")
    g = torch.Generator().manual_seed(L)
    I1 = torch.randint(0, 256, shape, generator=g, dtype=torch.uint8).to(dev())
    I2 = torch.roll(I1, (1, 2), (0, 1))
    flows = []
    for f32 in (False, True):
        plan = ofmi.Plan(*shape, L, 4, 1, input_f32=f32, device=dev())
        u, v = plan.compute(I1.float() if f32 else I1, I2.float() if f32 else I2)
        torch.cuda.synchronize()
        flows.append(torch.stack([u, v]).cpu())
        plan.close()
    assert torch.equal(flows[0], flows[1])
