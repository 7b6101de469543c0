"""The one-launch binning of small systems against the general one, which a batched call takes:
the same cell starts, order of atoms, status, forces and energy, bit for bit."""
import numpy as np
import pytest

from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case,n,box", [
    ("one atom", 1, (24.5, 24.5, 24.5)),
    ("a round of loads and one atom", 4097, (40.0, 31.0, 52.0)),
    ("256 cells, most of them empty", 301, (97.0, 97.0, 49.0)),
    ("257 cells or more: the general form", 301, (97.0, 97.0, 62.0)),
    ("the most atoms", 9216, (49.0, 50.0, 51.0)),
    ("one atom more: the general form", 9217, (49.0, 50.0, 51.0)),
    ("1,500 atoms in one cell", 3000, (37.0, 37.0, 37.0)),
    ("images of the box, faces and negative zeros", 2500, (37.0, 49.0, 30.0)),
    ("a NaN, an atom far outside and a bad type", 2500, (37.0, 49.0, 30.0)),
])
def test_one_launch_matches_general(gpu, case, n, box):
    import torch
    print("case:", case, n, box, flush=True)
    s = W.gen_system(n, box, 23)
    p = api.Params.from_dict(s.params())
    pos, typ = s.pos.copy(), s.types.copy()
    rng = np.random.default_rng(6)
    L = np.asarray(box, np.float32)
    if case.startswith("1,500"):
        pos[rng.choice(n, 1500, replace=False)] = rng.uniform(0.2, 12.0, (1500, 3)).astype(np.float32)
    if case.startswith("images"):
        pos[::3] -= L
        pos[1::3, 0] += L[0]
        pos[2::5, 1] = np.float32(-0.0)
        pos[3::7, 2] = L[2]
        pos[4::11, 0] = np.float32(12.333333)
    if case.startswith("a NaN"):
        pos[7, 1] = np.nan
        pos[n - 1, 0] = 5 * L[0]
        typ[1234] = 77
    dev = [torch.as_tensor(x).to(gpu) for x in (pos, typ, s.charges)]
    lay = api.workspace_layout(p, n)

    def system():
        return dict(params=p, pos=dev[0], types=dev[1], charges=dev[2],
                    force=torch.zeros((n, 3), dtype=torch.float32, device=gpu),
                    energy=torch.zeros(1, dtype=torch.float64, device=gpu),
                    workspace=api.alloc_workspace(p, n, gpu))

    def table(d):
        ws = d["workspace"]
        start = ws[lay["cell_start"]: lay["cell_start"] + 4 * (lay["n_cells"] + 1)].view(torch.int32)
        perm = ws[lay["perm"]: lay["perm"] + 4 * n].view(torch.int32)
        return start.cpu().numpy(), perm.cpu().numpy()

    one, many = system(), [system(), system()]
    for _ in range(2):   # the second time in the order of the measured times
        api.forces(p, *dev, force=one["force"], energy=one["energy"], workspace=one["workspace"])
        api.forces_batched(many)
        torch.cuda.synchronize()
        start, perm = table(one)
        assert np.array_equal(np.sort(perm), np.arange(n)) and start[-1] == n
        for d in many:
            assert all(np.array_equal(x, y) for x, y in zip((start, perm), table(d)))
            assert api.read_status(d["workspace"]) == api.read_status(one["workspace"])
            if api.read_status(one["workspace"]) & api.STATUS_FIXED_OVERFLOW:
                continue   # sums past the fixed point's range have no defined value
            assert torch.equal(d["force"].view(torch.int32), one["force"].view(torch.int32))
            assert torch.equal(d["energy"].view(torch.int64), one["energy"].view(torch.int64))
    status = api.read_status(one["workspace"])
    if case.startswith("a NaN"):
        assert status == api.STATUS_NAN | api.STATUS_OUT_OF_BOX | api.STATUS_BAD_TYPE
    else:   # atoms put next to each other at random may overflow
        assert status & ~api.STATUS_FIXED_OVERFLOW == 0
