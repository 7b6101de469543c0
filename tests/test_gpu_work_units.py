"""How the force path's work is shared out over workgroups, at the sizes where it changes.

Bars as in test_gpu_parity.py: float64 1e-12 and exact partner counts, float32 1e-5 on the
conditioning-normalised and RMS errors, energy 1e-6."""
import numpy as np
import pytest

import oracle
from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

from _gpu import run
from _metrics import force_errors

pytestmark = pytest.mark.gpu


def _system(n, box, seed):
    s = W.gen_system(n, box, seed)
    return s, s.params()


@pytest.mark.parametrize("double", [False, True])
@pytest.mark.parametrize("n,box", [
    (1, (24.5, 24.5, 24.5)),      # 8 cells, most slices of every list empty
    (65, (24.5, 40.0, 30.0)),     # lists about one 64-atom slice long
    (3000, (30.0, 30.0, 30.0)),   # 8 cells of more groups than one workgroup's waves
    (4001, (97.0, 97.0, 49.0)),   # 8 x 8 x 4 = 256 cells: the largest grid that is cut
    (4001, (97.0, 97.0, 62.0)),   # 8 x 8 x 5 = 320 cells: the shortest 64 in two parts
    (4003, (73.5, 73.5, 61.5)),   # 180 cells: the longest 76 in two parts
    (4003, (121.0, 97.0, 37.0)),  # 240 cells: the longest 16
    (4003, (133.0, 97.0, 37.0)),  # 11 x 8 x 3 = 264 cells: the shortest 8 in six parts
    (6007, (97.0, 97.0, 85.0)),   # 448 cells: the longest 64
    (20000, (205.0, 193.0, 97.0)),  # 17 x 16 x 8 = 2176 cells: all whole
])
def test_units_match_oracle(gpu, n, box, double):
    """Slices of the neighbour list and parts of the home atoms, from one atom to 2,176 cells:
    the oracle's forces, energy and partner counts, and the same bits however the home atoms
    are split."""
    print("case:", n, box, "double", double, flush=True)
    s, p = _system(n, box, 3)
    pos = s.pos.astype(np.float64) if double else s.pos
    q = s.charges.astype(np.float64) if double else s.charges
    f, e, ws, cnt = run(p, pos, s.types, q, gpu, double=double, flags=api.DIAG_COUNTERS)
    r = oracle.forces(p, s.pos, s.types, s.charges, "bruteforce" if n < 5000 else "celllist")
    err = force_errors(f, r.force, r.abs_sum)
    tol = 1e-12 if double else 1e-5
    assert err["max_norm"] <= tol and err["rms"] <= tol, err
    assert e == pytest.approx(r.energy, rel=1e-12 if double else 1e-6, abs=1e-9)
    if double:
        assert np.array_equal(cnt, r.count)
    assert api.read_status(ws) == 0
    for split in (1, 4):
        f2, e2 = run(p, pos, s.types, q, gpu, double=double, flags=api.PAIR_SPLIT(split))[:2]
        assert np.array_equal(f, f2) and e == e2


@pytest.mark.parametrize("n", [2040, 6000, 16384, 16385])
def test_crowded_sort_order(gpu, n):
    """Cells whose atoms lie in planes of x, so that the in-cell sort's buckets overflow their
    lists, gathered from 1, 3, 8 and 9 histogram blocks (the last past the block-by-block
    gather): every cell ordered by (z half, x, index), ties in x included."""
    print("case: crowded sort,", n, "atoms", flush=True)
    from test_gpu_parity import _check_binning
    s, p = _system(n, (60.0, 37.0, 97.0), 8)
    pos = s.pos.copy()
    pos[: n // 2, 0] = np.float32(2.5) * np.round(pos[: n // 2, 0] / np.float32(2.5))
    pos[:, 0] = np.clip(pos[:, 0], 0, 59.5)
    f, e, ws, _ = run(p, pos, s.types, s.charges, gpu)
    _check_binning(p, pos, ws, n)


@pytest.mark.parametrize("sizes", [
    [2000, 2500],                          # few cells in all: the systems keep their splits
    [2001, 90000, 3000, 40000, 1700],      # mixed: small systems' cells whole, costliest first
    [1600 + 37 * k for k in range(130)],   # more systems than one launch takes
])
def test_batch_units_same_bits(gpu, sizes):
    """A batch shares its systems out over fewer workgroups than they would take alone; every
    system's forces and energy are the bits of its own call."""
    import torch
    print("case: batch of", len(sizes), "sizes", sizes[:5], flush=True)
    systems, alone = [], []
    table = W.draw_type_table(np.random.default_rng(2))
    for k, n in enumerate(sizes):
        L = W.cube_for(n)
        s = W.gen_system(n, (max(L, 24.5),) * 3, 100 + k, type_table=table)
        p = api.Params.from_dict(s.params())
        d = dict(params=p, pos=torch.as_tensor(s.pos).to(gpu), types=torch.as_tensor(s.types).to(gpu),
                 charges=torch.as_tensor(s.charges).to(gpu),
                 force=torch.empty(n, 3, device=gpu),
                 energy=torch.empty(1, dtype=torch.float64, device=gpu),
                 workspace=api.alloc_workspace(p, n, gpu))
        alone.append([t.clone() for t in api.forces(p, d["pos"], d["types"], d["charges"])])
        systems.append(d)
    for _ in range(2):
        api.forces_batched(systems)
        torch.cuda.synchronize()
        for d, (f, e) in zip(systems, alone):
            assert torch.equal(d["force"], f) and torch.equal(d["energy"], e)


def test_batched_energy_partials(gpu):
    """A batched call may take fewer workgroups for a system than a call of its own: the energy
    partials in its workspace still add up to the energy, all of them."""
    import torch
    systems = []
    for k, (n, box) in enumerate([(3000, (30.0, 30.0, 30.0)), (4003, (73.5, 73.5, 61.5)),
                                  (20000, (58.5, 58.5, 58.5)), (30000, (97.0, 97.0, 85.0))]):
        s, p = _system(n, box, 3 + k)
        P = api.Params.from_dict(p)
        d = dict(params=P, pos=s.pos, types=s.types, charges=s.charges)
        d = dict(d, **{x: torch.as_tensor(d[x]).to(gpu) for x in ("pos", "types", "charges")})
        systems.append(dict(d, force=torch.empty((n, 3), dtype=torch.float32, device=gpu),
                            energy=torch.empty(1, dtype=torch.float64, device=gpu),
                            workspace=api.alloc_workspace(P, n, gpu)))

    def check(d):
        lay = api.workspace_layout(d["params"], d["pos"].shape[0])
        at, m = lay["energy_partials"], lay["n_energy_partials"]
        part = d["workspace"][at: at + 8 * m].view(torch.int64).cpu().numpy()
        assert int(part.sum()) * 2.0 ** -24 == d["energy"].item()

    for d in systems:   # alone first: what a batch leaves unwritten would be these
        api.forces(d["params"], d["pos"], d["types"], d["charges"], force=d["force"], energy=d["energy"],
                   workspace=d["workspace"])
        check(d)
    api.forces_batched(systems)
    for d in systems:
        check(d)
