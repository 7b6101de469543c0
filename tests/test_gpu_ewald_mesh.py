"""The grid form of the Ewald reciprocal sum (md_ewald_mesh.hip) against the oracle's plain sum
over wave vectors, at the sizes where it can go wrong.

Bars as in test_gpu_ewald.py (RMS and largest force error 1e-5); the energy to 1e-6 of the
sizes of its reciprocal, self and background terms, which partly cancel."""
import numpy as np
import pytest

import oracle
from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

from test_gpu_ewald import _recip_errors, _recip_gpu, ewald_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case,n,box,kmax,crowd", [
    ("few atoms, many wave vectors", 300, (26.0, 29.0, 31.0), (60, 55, 64), 0),
    ("fewest tiles per axis, unequal", 30000, (50.0, 62.0, 40.0), (8, 9, 46), 0),
    ("one axis without modes", 60001, (70.0, 76.0, 90.0), (60, 0, 50), 0),
    ("a bin of hundreds, bit map over two index ranges", 40000, (74.0, 71.0, 73.0), (14, 16, 15), 900),
    ("long axis: two column tiles a workgroup, the last one alone", 4000, (260.0, 22.0, 40.0), (170, 5, 20), 0),
    ("long axis: three column tiles, three row tiles", 300, (100.0, 30.0, 30.0), (150, 40, 40), 0),
    ("over 24,576 tiles", 100, (30.0, 31.0, 32.0), (90, 90, 90), 0),
    ("outside the box, net charge", 12000, (48.0, 51.0, 50.0), (18, 18, 18), 0),
])
def test_mesh_matches_oracle(gpu, case, n, box, kmax, crowd):
    print("case:", case, n, box, kmax, flush=True)
    s = W.gen_system(n, box, 17)
    p = ewald_params(s, 0.3)
    if crowd:      # atoms of all index ranges packed into a 2 A cube
        rng = np.random.default_rng(4)
        at = rng.choice(n, crowd, replace=False)
        s.pos[at] = (0.01 + rng.uniform(0, 2.0, (crowd, 3))).astype(np.float32)
    if case.startswith("outside"):
        s.pos[::3] -= np.asarray(box, np.float32)
        s.charges = (s.charges + np.float32(0.01)).astype(np.float32)
    # it is the grid form that runs: the direct sum's phase tables alone would take more (for a
    # few atoms or a long axis the grid is larger than these)
    tables = 8 * n * ((kmax[0] + 1) + (2 * kmax[1] + 1) + (2 * kmax[2] + 1))
    f, e, ws = _recip_gpu(p, s, kmax, gpu)
    if n > 4000:
        assert api.ewald_workspace_bytes(api.Params.from_dict(p), n, kmax) < tables + 16 * n
    ref_f, er, es, eb = oracle.ewald_recip(p, s.pos, s.charges, kmax)
    err = _recip_errors(f.double().cpu().numpy(), e, ref_f, er + es + eb)
    print("errors", err, "energy", e, er, es, eb, flush=True)
    assert err["rms"] <= 1e-5 and err["max_rel_to_largest"] <= 1e-5
    assert abs(e - (er + es + eb)) <= 1e-6 * (abs(er) + abs(es) + abs(eb))
    assert api.read_status(ws) == 0
    # the same bits again, and added onto what the force buffer holds
    f2, e2, _ = _recip_gpu(p, s, kmax, gpu)
    assert e2 == e and bool((f2 == f).all())
    base = f.new_full(f.shape, 0.25)
    f3, _, _ = _recip_gpu(p, s, kmax, gpu, force=base.clone(), accumulate=True)
    assert bool((f3 == base + f).all())


def test_mesh_nan(gpu):
    """A NaN position or charge sets the status bit, as in the direct sum."""
    import torch
    s = W.gen_system(12000, (50.0, 50.0, 50.0), 2)
    p = api.Params.from_dict(ewald_params(s, 0.3))
    for what in (0, 1):
        pos, q = torch.as_tensor(s.pos).to(gpu), torch.as_tensor(s.charges).to(gpu)
        if what:
            q[77] = float("nan")
        else:
            pos[77, 2] = float("nan")
        _, _, ws = api.ewald_recip(p, pos, q, (18, 18, 18))
        assert api.read_status(ws) & api.STATUS_NAN
