"""The one-launch binning of a cell of more than 1,024 atoms (its members listed by a second pass over
all atoms) against the general form, which a batched call takes: cell starts, order, z split, status,
forces and energy, bit for bit. No Lennard-Jones term and small charges, so that no sum overflows."""
import numpy as np
import pytest

from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("double", [False, True])
@pytest.mark.parametrize("crowd", [1024, 1025, 1500, 2600])
def test_crowded_cell(gpu, crowd, double):
    import torch
    n, box = 3000, (37.0, 37.0, 37.0)          # 3^3 cells of 12.33 A
    print("case:", crowd, "atoms in one cell, double", double, flush=True)
    s = W.gen_system(n, box, 29)
    rng = np.random.default_rng(8)
    # crowd atoms on a jittered lattice inside cell (1, 1, 1), the others in other cells
    pos = s.pos.copy()
    other = np.array([c for c in np.ndindex(3, 3, 3) if c != (1, 1, 1)])
    pos[:] = (other[rng.integers(0, 26, n)] * 12.3333 + rng.uniform(0.1, 12.2, (n, 3))).astype(np.float32)
    m = int(np.ceil(crowd ** (1 / 3)))
    site = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:crowd]
    at = rng.choice(n, crowd, replace=False)
    pos[at] = (12.5 + (site + 0.5 + rng.uniform(-0.2, 0.2, (crowd, 3))) * (12.0 / m)).astype(np.float32)
    p = api.Params.from_dict(dict(s.params(), epsilon=np.zeros(len(s.epsilon))))
    real = torch.float64 if double else torch.float32
    dev = [torch.as_tensor(pos).to(gpu, real), torch.as_tensor(s.types).to(gpu),
           (0.1 * torch.as_tensor(s.charges)).to(gpu, real)]
    lay = api.workspace_layout(p, n, double)

    def table(ws):
        def ints(off, k):
            return ws[off: off + 4 * k].view(torch.int32).cpu().numpy()
        return [ints(lay["cell_start"], lay["n_cells"] + 1), ints(lay["perm"], n),
                ints(lay["z_split"], lay["n_cells"])]

    one = dict(force=torch.zeros((n, 3), dtype=real, device=gpu),
               energy=torch.zeros(1, dtype=torch.float64, device=gpu),
               workspace=api.alloc_workspace(p, n, gpu, double))
    for _ in range(2):
        api.forces(p, *dev, **one)
        torch.cuda.synchronize()
        assert api.read_status(one["workspace"]) == 0
        start, perm, low = table(one["workspace"])
        assert np.array_equal(np.sort(perm), np.arange(n)) and start[-1] == n
        counts = np.diff(start)
        assert counts[13] == crowd
        # the order within each cell: (z half, x, index), its lower half as long as z_split says
        for c in range(27):
            a = perm[start[c]: start[c + 1]]
            x, half = dev[0][:, 0].float().cpu().numpy()[a], np.arange(len(a)) >= low[c]
            assert np.array_equal(np.lexsort((a, x, half)), np.arange(len(a)))
    if double:      # a batch is float32: the float64 order and forces against float32's
        q = api.Params.from_dict(dict(s.params(), epsilon=np.zeros(len(s.epsilon))))
        f, _ = api.forces(q, *[d.float() if d.is_floating_point() else d for d in dev])[:2]
        scale = one["force"].abs().max()
        assert float((f.double() - one["force"]).abs().max() / scale) <= 1e-5
        return
    many = [dict(params=p, pos=dev[0], types=dev[1], charges=dev[2],
                 force=torch.zeros((n, 3), dtype=real, device=gpu),
                 energy=torch.zeros(1, dtype=torch.float64, device=gpu),
                 workspace=api.alloc_workspace(p, n, gpu)) for _ in range(2)]
    api.forces_batched(many)
    torch.cuda.synchronize()
    for d in many:
        assert api.read_status(d["workspace"]) == 0
        assert all(np.array_equal(x, y) for x, y in zip(table(d["workspace"]), (start, perm, low)))
        assert torch.equal(d["force"].view(torch.int32), one["force"].view(torch.int32))
        assert torch.equal(d["energy"].view(torch.int64), one["energy"].view(torch.int64))
