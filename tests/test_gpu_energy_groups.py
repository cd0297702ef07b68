"""Energy and gradients over batch sizes and lattices that change how a call
is split: configurations per work item (2 to 32), one or many tiles, dE/dB
from one block or from the configurations' sums, several passes.  Reference:
the same formulas in torch, double precision, on the same inputs; FP64 to
1e-12 of the scale of what is summed, FP32 within the bounds of _fp32.py."""
import numpy as np
import pytest
import torch

import synth
from _fp32 import U32, grad_bounds, site_scale
from paper_1803_07030_amd import hsim
from paper_1803_07030_amd.energy import heisenberg_energy

pytestmark = pytest.mark.gpu


def _reference(lat, S, J, k, axis, B, w):
    i, j, _ = (torch.tensor(np.asarray(v), device="cuda") for v in lat.bonds())
    S, J, k, axis = S.double(), J.double(), k.double(), axis.double()
    a = (S * axis).sum(1)
    dots = (S[:, :, i] * S[:, :, j]).sum(1)
    E = -(dots * J).sum(1) - B * S[:, 2].sum(1) - (k * a * a).sum(1)
    g = torch.zeros_like(S)
    g.index_add_(2, i, -J * S[:, :, j])
    g.index_add_(2, j, -J * S[:, :, i])
    g[:, 2] -= B
    g -= 2.0 * (k * a)[:, None] * axis
    return (E, w[:, None, None] * g, -(w[:, None] * dots).sum(0), -(w[:, None] * a * a).sum(0),
            -(w * S[:, 2].sum(1)).sum())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("kind,L,batch", [("sc", 4, 1), ("sc", 4, 3), ("sc", 9, 33), ("film", 23, 70), ("sc", 16, 65),
                                          ("sc", 20, 300), ("sc", 3, 2100), ("sc", 13, 2050), ("tree", 900, 40)])
def test_splits_match_the_formulas(dtype, kind, L, batch):
    if kind == "sc":
        lat = synth.gradient_lattice(L=L, seed=4)
    elif kind == "film":
        lat = synth.diluted_film(L, 3, seed=5)
    else:
        lat = synth.random_tree(L, seed=6, max_degree=12)      # rows beyond 8: the CSR walk
        lat.k, lat.axis = 0.2 * synth.uniform01(6, lat.n, tag=1), synth.unit_vectors(6, lat.n, tag=2)
    plan = hsim.Plan(lat)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(L + batch)
    S = torch.randn(batch, 3, lat.n, generator=gen, device="cuda", dtype=torch.float64)
    S = (S / S.norm(dim=1, keepdim=True)).to(dtype).requires_grad_(True)
    J = torch.tensor(lat.bonds()[2], dtype=dtype, device="cuda", requires_grad=True)
    k = torch.tensor(lat.k, dtype=dtype, device="cuda", requires_grad=True)
    B = torch.tensor(0.5, dtype=torch.float64, device="cuda", requires_grad=True)
    axis = torch.tensor(lat.axis.T.copy(), dtype=dtype, device="cuda")
    w = torch.rand(batch, generator=gen, device="cuda", dtype=torch.float64) + 0.5
    E = heisenberg_energy(S, J, k, B, plan, axis)
    gS, gJ, gk, gB = torch.autograd.grad(E, (S, J, k, B), w)
    rE, rS, rJ, rk, rB = _reference(lat, S.detach(), J.detach(), k.detach(), axis, 0.5, w)
    si = torch.tensor(site_scale(lat, 0.5), device="cuda")
    scale, sw = float(si.sum()), float(w.sum())
    if dtype == torch.float64:
        bE, bS, bJ, bk, bB = 1e-12 * scale, 1e-12 * si, 1e-12 * sw, 1e-12 * sw, 1e-12 * lat.n * sw
    else:
        bS, bJ, bk, bB = grad_bounds(lat, 0.5, w.cpu().numpy())
        bE, bS = 34 * U32 * scale, torch.tensor(bS, device="cuda")
    assert float((E - rE).abs().max()) <= bE
    assert bool(((gS.double() - rS).abs() <= bS * w[:, None, None]).all())
    assert float((gJ.double() - rJ).abs().max()) <= bJ
    assert float((gk.double() - rk).abs().max()) <= bk
    assert abs(float(gB) - float(rB)) <= bB


# From 192 tiles of 256 sites on (96 on rows beyond 6) groups are formed by the
# blocks that run at once: ragged batches of one group to several, and past
# two rounds of them.
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("batch", [3, 17, 50, 170])
@pytest.mark.parametrize("kind,L,degree", [("sc", 37, 6), ("tree", 25000, 8), ("tree", 25000, 12)])
def test_groups_of_many_tiles_match_the_formulas(monkeypatch, dtype, kind, L, degree, batch):
    tree = synth.random_tree
    monkeypatch.setattr(synth, "random_tree", lambda n, seed, max_degree: tree(n, seed=seed, max_degree=degree))
    test_splits_match_the_formulas(dtype, kind, L, batch)
