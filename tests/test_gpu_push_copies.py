"""A push's frames and arguments are copied together, sixteen copies per launch."""
import numpy as np
import pytest

import synth
from gpu_util import announce, dev, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 14, 15, 16, 17, 33])
def test_push_copies_every_frame(gpu_lib, n):
    """Pushes below, at and past the copies of one launch, frames of different sizes: every stream's
    flow equals its own plan's, bit for bit."""
    import torch
    from paper_1306_2461_amd.serve import GpuExecutor, Server
    ofmi = gpu_lib
    announce(f"push of {n} frames")
    a, b, _, _ = synth.make_pair("c1", 4)
    srv = Server(GpuExecutor(2, 3, 2, device=dev()))
    sizes = [(40 + 3 * i, 77 - i) for i in range(n)]
    pairs = [(np.ascontiguousarray(a[i:i + h, :w]), np.ascontiguousarray(b[i:i + h, :w]))
             for i, (h, w) in enumerate(sizes)]
    for k in (0, 1):
        reqs = [srv.submit(i, torch.from_numpy(p[k]).pin_memory()) for i, p in enumerate(pairs)]
        assert srv.step() == n
        srv.drain()
    for r, p in zip(reqs, pairs):
        plan = ofmi.Plan(*p[0].shape, 2, 3, 2, device=dev())
        u, v = plan.compute(to_dev(p[0]), to_dev(p[1]))
        torch.cuda.synchronize()
        assert torch.equal(u, r.u) and torch.equal(v, r.v), r.stream_id
        plan.close()
    srv.ex.close_all()
