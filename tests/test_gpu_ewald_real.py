"""The real-space Ewald term over its argument's range, pair by pair: pairs of charges alone in
their surroundings (no Lennard-Jones term), so that each atom's force is one pair's. The charges are
such that every pair's force is about 100 kcal/mol/A, where the sums' fixed-point units (2^-28 and, for
the neighbour's share, 2^-24 kcal/mol/A) are 1e-9 of it and do not count.

Bars. The force factor k q q (erfc(x)/r + (2 alpha/sqrt(pi)) exp(-x^2))/r^2 with x = alpha r goes
through about eight float32 roundings (u, its reciprocal root and the root's powers, the two functions,
their sum and products), 2^-24 at most each; three of them (u, the root, alpha r) reach the functions too,
where the term's own slope, at most 2 x^2 + 1 of its value, multiplies them. So at most
2^-24 (8 + 3 (2 x^2 + 1)) relative, and a third of that RMS."""
import numpy as np
import pytest
from scipy.special import erfc

from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

pytestmark = pytest.mark.gpu


def lone_pairs(alpha, r_lo, r_hi, seed=11, r_cut=6.0):
    """1,000 pairs 18 A apart in a 180 A cube, at separations over [r_lo, r_hi) in random directions."""
    rng = np.random.default_rng(seed)
    n = 1000
    site = (np.stack(np.meshgrid(*[np.arange(10)] * 3, indexing="ij"), -1).reshape(-1, 3) * 18.0 + 9.0)
    r = r_lo + (r_hi - r_lo) * (np.arange(n) + rng.uniform(0, 1, n)) / n
    d = rng.normal(size=(n, 3))
    d *= (0.5 * r / np.linalg.norm(d, axis=1))[:, None]
    pos = np.concatenate([site + d, site - d]).astype(np.float32)
    x = alpha * r
    unit = W.COULOMB_K * (erfc(x) / r + 2 * alpha / np.sqrt(np.pi) * np.exp(-x * x)) / r
    q = np.tile(np.sqrt(100.0 / unit).astype(np.float32), 2)
    params = dict(W.gen_system(8, (180.0,) * 3, 1).params(r_cut=r_cut, r_switch=r_cut - 2.0,
                                                         flags=api.COULOMB_EWALD), ewald_alpha=alpha)
    params["epsilon"] = np.zeros_like(np.asarray(params["epsilon"], dtype=np.float64))
    return params, pos, q


def run(gpu, params, pos, q):
    import torch
    p = api.Params.from_dict(params)
    dev = [torch.as_tensor(x).to(gpu) for x in (pos, np.zeros(len(pos), np.int32), q)]
    f, e = api.forces(p, *dev, workspace=(ws := api.alloc_workspace(p, len(pos), gpu)))
    torch.cuda.synchronize()
    return f.double().cpu().numpy(), float(e.item()), api.read_status(ws)


@pytest.mark.parametrize("alpha,r_lo,r_hi", [(0.15, 0.5, 6.0), (0.3, 1.0, 6.0), (0.6, 0.8, 6.0), (1.0, 0.5, 6.0),
                                             (1.4, 4.0, 6.0)])
def test_lone_pairs(gpu, alpha, r_lo, r_hi):
    print("case: lone pairs", alpha, r_lo, r_hi, flush=True)
    params, pos, q = lone_pairs(alpha, r_lo, r_hi)
    f, _, status = run(gpu, params, pos, q)
    n = len(q) // 2
    d = pos[:n].astype(np.float64) - pos[n:].astype(np.float64)
    r = np.linalg.norm(d, axis=1)
    x = float(np.float32(alpha)) * r
    qq = params["coulomb_k"] * q[:n].astype(np.float64) ** 2
    k = qq * (erfc(x) / r + 2 * alpha / np.sqrt(np.pi) * np.exp(-x * x)) / r ** 2
    inside = r < params["r_cut"]
    ref = np.where(inside, k, 0.0)[:, None] * d
    assert status == 0 and inside.sum() > 0.99 * n
    err = np.linalg.norm(f - np.concatenate([ref, -ref]), axis=1).reshape(2, n)[:, inside]
    rel = err / (2.0 ** -24 * (8 + 3 * (2 * x ** 2 + 1)) * np.linalg.norm(ref, axis=1))[inside]
    print("largest error over its bar", rel.max(), "RMS", np.sqrt((rel ** 2).mean()), flush=True)
    assert rel.max() <= 1.0 and np.sqrt((rel ** 2).mean()) <= 1.0 / 3.0


@pytest.mark.parametrize("alpha", [30.0, 1.0e10, 1.0e20, 3.0e37])
def test_large_alpha_leaves_nothing(gpu, alpha):
    """erfc and the exponential of an argument from 9 on to beyond the root of the largest float32 are 0 (or
    under the sums' units), never NaN."""
    print("case: large alpha", alpha, flush=True)
    params, pos, q = lone_pairs(1.0, 0.5, 6.0)
    f, e, status = run(gpu, dict(params, ewald_alpha=alpha), pos, np.full_like(q, 0.5))
    assert status == 0 and e == 0.0 and not f.any()
