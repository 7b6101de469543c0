"""Accuracy of the Ewald reciprocal sum against a plain float64 sum over wave vectors, as tight as
float32 storage allows.

Bars for the grid form. A force passes through about twelve float32 roundings (three windows and
the charge's grid, three intermediates of the transforms each way, the window derivative, the
product and the output), each 2^-24/sqrt(3) RMS of its own value, so 1.2e-7; those on the potential
grow with the grid's points per wavelength, so up to twice that, 2^-22, with twice the wave numbers that
the splitting parameter needs. The energy's terms are tens of thousands of squares with independent
errors, so only a bias would be left: a quarter of a float32 rounding unit, 2^-25, of the reciprocal
part."""
import math

import numpy as np
import pytest

from paper_1611_04474_amd import api
from paper_1611_04474_amd import workloads as W

from test_ewald_forms import takes_grid
from test_gpu_ewald import _recip_gpu, ewald_params

pytestmark = pytest.mark.gpu


def recip_reference(s, alpha, kmax, device):
    """Forces and the reciprocal, self and background energies in float64, the sum over wave
    vectors as written (mx >= 0: -k gives the same term as k)."""
    import torch
    L = torch.as_tensor(np.asarray(s.box, np.float32)).double().to(device)
    x = torch.as_tensor(s.pos).double().to(device)
    q = torch.as_tensor(s.charges).double().to(device)
    V, kc = float(L.prod()), W.COULOMB_K
    g = [2.0 * math.pi / float(v) for v in L]
    m = [torch.arange(lo, hi + 1, device=device, dtype=torch.float64)
         for lo, hi in ((0, kmax[0]), (-kmax[1], kmax[1]), (-kmax[2], kmax[2]))]
    kv = [g[d] * m[d] for d in range(3)]
    k2 = kv[0][:, None, None] ** 2 + kv[1][None, :, None] ** 2 + kv[2] ** 2
    w = torch.where(k2 > 0, torch.exp(-k2 / (4 * alpha ** 2)) / k2.clamp(min=1e-300), 0.0 * k2)
    w = (w * torch.where(m[0] > 0, 2.0, 1.0)[:, None, None]).reshape(-1, len(m[2]))
    step = max(1, 4_000_000 // w.shape[0])

    def phases(b):
        e = [torch.polar(torch.ones_like(p), p) for p in (x[b, d, None] * kv[d] for d in range(3))]
        return (e[0][:, :, None] * e[1][:, None, :]).reshape(-1, w.shape[0]), e[2]

    parts = [slice(b, b + step) for b in range(0, len(x), step)]
    S = torch.zeros(w.shape, dtype=torch.complex128, device=device)
    for b in parts:
        xy, z = phases(b)
        S += (xy * q[b, None]).t().contiguous() @ z
    e_rec = float(2.0 * math.pi * kc / V * (w * S.abs() ** 2).sum())
    e_self = float(-kc * alpha / math.sqrt(math.pi) * (q * q).sum())
    e_back = float(-kc * math.pi * q.sum() ** 2 / (2.0 * V * alpha ** 2))
    G = (4.0 * math.pi * kc / V * w) * S.conj()
    Gt, Gz = G.t().contiguous(), (G * kv[2]).t().contiguous()
    kx = kv[0][:, None].expand(-1, len(m[1])).reshape(-1)
    ky = kv[1][None, :].expand(len(m[0]), -1).reshape(-1)
    F = torch.zeros_like(x)
    for b in parts:
        xy, z = phases(b)
        t = (xy * (z @ Gt)).imag
        F[b, 0], F[b, 1], F[b, 2] = (t * kx).sum(1), (t * ky).sum(1), (xy * (z @ Gz)).imag.sum(1)
    return F * q[:, None], e_rec, e_self, e_back


def errors(gpu, n, box, alpha, kmax, seed=3):
    """RMS force error over the RMS force, and the energy's error over its reciprocal part."""
    s = W.gen_system(n, box, seed)
    f, e, ws = _recip_gpu(ewald_params(s, alpha), s, kmax, gpu)
    ref, er, es, eb = recip_reference(s, alpha, kmax, gpu)
    assert api.read_status(ws) == 0
    return float((f.double() - ref).norm() / ref.norm()), abs(e - (er + es + eb)) / er


@pytest.mark.parametrize("case,n,box,alpha,kmax", [
    ("the wave numbers that alpha needs", 9001, (44.82,) * 3, 0.3, (16,) * 3),
    ("twice as many", 9001, (44.82,) * 3, 0.3, (32,) * 3),
    ("fewer atoms", 5000, (38.2,) * 3, 0.4, (19, 19, 20)),
    ("fewer still, twice the wave numbers", 3000, (30.0,) * 3, 0.3, (23,) * 3),
    ("unconverged: every wave number with the same weight", 9001, (44.82,) * 3, 6.0, (16,) * 3),
    ("a slab, unequal axes", 20000, (70.0, 75.0, 39.0), 0.3, (25, 27, 14)),
])
def test_grid_form_keeps_float32_accuracy(gpu, case, n, box, alpha, kmax):
    print("case:", case, n, box, alpha, kmax, flush=True)
    assert takes_grid(n, kmax)
    rms, e = errors(gpu, n, box, alpha, kmax)
    print("RMS force error", rms, "energy", e, flush=True)
    assert rms <= 2.0 ** -22
    assert e <= 2.0 ** -25


@pytest.mark.parametrize("case,n,box,kmax", [
    ("fewest tiles per axis, unequal", 30000, (50.0, 62.0, 40.0), (8, 9, 46)),
    ("one axis without modes", 60001, (70.0, 76.0, 90.0), (60, 0, 50)),
    ("long axis: two column tiles a workgroup, the last one alone", 22880, (260.0, 22.0, 40.0), (170, 5, 20)),
    ("long axis: two column tiles, three row tiles", 9000, (100.0, 30.0, 30.0), (150, 40, 40)),
    ("over 4,096 tiles: bins scanned by a kernel of their own", 2000, (30.0, 31.0, 32.0), (50, 50, 50)),
    ("over 24,576 tiles: four waves a tile", 2100, (30.0, 31.0, 32.0), (90, 90, 90)),
    ("the longest axis: over 64 KB of LDS in the last transform", 33880, (22.0, 22.0, 700.0), (7, 7, 255)),
])
def test_grid_form_branches(gpu, case, n, box, kmax):
    """The grid form's launch shapes, at sizes that take it. The bar grows with the wave numbers
    beyond twice what alpha needs (exp(-k^2/4 alpha^2) = 1e-6), as the potential's share does."""
    print("case:", case, n, box, kmax, flush=True)
    assert takes_grid(n, kmax)
    alpha = 0.3
    beyond = max(k * math.pi / (alpha * L * math.sqrt(-math.log(1e-6))) for k, L in zip(kmax, box))
    rms, e = errors(gpu, n, box, alpha, kmax)
    print("RMS force error", rms, "energy", e, "kmax over need", beyond, flush=True)
    assert rms <= 2.0 ** -22 * max(1.0, beyond / 2)
    assert e <= 2.0 ** -25
