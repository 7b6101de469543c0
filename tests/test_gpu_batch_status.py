"""A system that a call of its own accepts is accepted in a batch too, also where forces near the bounds
of the fixed-point sums: a batch has fewer workgroups per cell, so each gathers more of a neighbour's share.
One heavily charged atom just above a cell face, pushed by ever more partners below it, whose cell adds
their shares to it."""
import numpy as np
import pytest

from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

pytestmark = pytest.mark.gpu


# the other systems of the batch: large ones leave one part per cell, small ones some of them
@pytest.mark.parametrize("n,box,others", [
    (3000, (30.0, 30.0, 30.0), (120000, 106.3)), (9001, (60.5, 48.3, 30.9), (120000, 106.3)),
    (16000, (73.5, 73.5, 30.0), (120000, 106.3)), (3000, (30.0, 30.0, 30.0), (9001, 45.1)),
    (9001, (60.5, 48.3, 30.9), (9001, 45.1))])
def test_accepted_alone_accepted_in_a_batch(gpu, n, box, others):
    import torch
    print("case: bounds of the fixed-point sums in a batch", n, box, others, flush=True)
    s = W.gen_system(n, box, 31)
    p = api.Params.from_dict(dict(s.params(), epsilon=np.zeros(len(s.epsilon))))
    rng = np.random.default_rng(3)
    big = W.gen_system(others[0], (others[1],) * 3, 32)
    dev_big = [torch.as_tensor(x).to(gpu) for x in (big.pos, big.types, (0.01 * big.charges).astype(np.float32))]

    def out(m):   # the workspace without times of a call before: the launch order is that of the atom counts
        return dict(force=torch.zeros((m, 3), dtype=torch.float32, device=gpu),
                    energy=torch.zeros(1, dtype=torch.float64, device=gpu), workspace=api.alloc_workspace(p, m, gpu).zero_())

    filler = [dict(params=p, pos=dev_big[0], types=dev_big[1], charges=dev_big[2], **out(big.n)) for _ in range(3)]
    seen = set()
    for partners in range(1, 60, 2):
        pos, q = s.pos.copy(), np.zeros(n, np.float32)
        pos[0] = (5.0, 5.0, box[2] / 2 + 1.0)
        q[0] = 1.0e6
        at = 1 + np.arange(partners)          # each pushes with about 0.2 x 2^27 kcal/mol/A
        # spread along x, so that they are in different groups of home atoms
        pos[at] = pos[0] + np.stack([rng.uniform(-4, 4, partners), rng.uniform(-1, 1, partners),
                                     rng.uniform(-4.5, -3.5, partners)], 1)
        q[at] = 0.2 * 2.0 ** 27 * 16.0 / (W.COULOMB_K * 1.0e6)
        dev = [torch.as_tensor(x).to(gpu) for x in (pos.astype(np.float32), s.types, q)]
        one, in_batch = out(n), out(n)
        api.forces(p, *dev, **one)
        api.forces_batched([dict(params=p, pos=dev[0], types=dev[1], charges=dev[2], **in_batch)] + filler)
        torch.cuda.synchronize()
        st = [api.read_status(d["workspace"]) for d in (one, in_batch)]
        print(partners, "partners: status", st, "force", float(one["force"][0, 2]), flush=True)
        seen.add(st[0])
        if st[0] == 0:
            assert st[1] == 0, partners
            assert torch.equal(one["force"].view(torch.int32), in_batch["force"].view(torch.int32))
            assert torch.equal(one["energy"].view(torch.int64), in_batch["energy"].view(torch.int64))
    assert seen == {0, api.STATUS_FIXED_OVERFLOW}
