"""The motion update fused into the force path's last kernel, and streamed after it."""
import numpy as np
import pytest

from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, api.PAIR_PREDICATED, api.PAIR_FULL_SHELL])
@pytest.mark.parametrize("n,box", [(1, (30.0, 30.0, 30.0)), (257, (26.0, 30.0, 28.0)),
                                   (3000, (30.0, 30.0, 30.0)),
                                   (131072, (110.0, 110.0, 109.0)),    # the last to be fused
                                   (131073, (110.0, 110.0, 109.0))])   # the first to be streamed
def test_run_equals_single_steps(gpu, n, box, flags):
    """Five steps in one call and one at a time: the same bits of positions, velocities, forces
    and potential energy (each step's arithmetic is the same wherever the kicks are done);
    kinetic energies to 1e-13 of each other and 1e-6 of sums with m = 1/(1/m in float32)."""
    import torch
    if flags and n > 3000:
        pytest.skip("the larger systems run the default path only")
    print("case:", n, box, flags, flush=True)
    s = W.liquid_system(n, box) if n > 1 else W.gen_system(1, box, 3)
    v0, im = W.velocities(s.types) if n > 1 else (np.full((1, 3), 1e-3, np.float32), np.ones(1, np.float32))
    im[0] = 0.0 if n > 1 else im[0]          # no acceleration, no kinetic energy
    p = api.Params.from_dict(s.params(flags=flags))
    t, q = torch.as_tensor(s.types).to(gpu), torch.as_tensor(s.charges).to(gpu)
    inv = torch.as_tensor(im).to(gpu)
    m = torch.where(inv > 0, 1.0 / inv.double().clamp(min=1e-30), torch.zeros_like(inv, dtype=torch.float64))

    def state():
        x, v = torch.as_tensor(s.pos).to(gpu), torch.as_tensor(v0).to(gpu)
        f, _ = api.forces(p, x, t, q)
        return x, v, f
    a, b = state(), state()
    ea = api.run_vv(p, a[0], a[1], t, q, inv, a[2], 0.5, 5)
    for k in range(5):
        eb = api.run_vv(p, b[0], b[1], t, q, inv, b[2], 0.5, 1)
        assert ea[k, 0].item() == eb[0, 0].item()
        ke = float((0.5 * m[:, None] * b[1].double() ** 2).sum()) / float(np.float32(4.184e-4))
        assert ea[k, 1].item() == pytest.approx(ke, rel=1e-6)
        assert eb[0, 1].item() == pytest.approx(ea[k, 1].item(), rel=1e-13)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
