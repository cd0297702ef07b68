"""Double-precision block layout at the sizes where its kernels change (one or
two classes of up to 256 sites, at and past the edges of the waves): spins,
accept bitmap and accepted moves equal the site layout's bit for bit, E and M
to 1e-12 of the energy scale, over several steps, a resumed call and step-end
states, for replicas of different lattices in one batch, one of them empty."""
import numpy as np
import pytest
import torch

import synth
from paper_1803_07030_amd import hsim

pytestmark = pytest.mark.gpu


def _with_terms(lat, seed):
    lat.k = 0.3 * synth.uniform01(seed, lat.n, tag=1)
    lat.axis = synth.unit_vectors(seed, lat.n, tag=2)
    lat.ndir = synth.unit_vectors(seed, lat.n, tag=3)
    return lat


CASES = {
    "one_site": lambda: [synth.isolated(1)],
    "one_class": lambda: [synth.isolated(200)],
    "classes_64": lambda: [synth.sc_periodic(4, 4, 8)],
    "classes_65": lambda: [synth.open_chain(130)],
    "classes_256": lambda: [synth.sc_periodic(8)],
    "classes_257": lambda: [synth.open_chain(513)],
    "per_site_terms": lambda: [_with_terms(synth.sc_periodic(6), 4)],
    "degree_8": lambda: [synth.random_tree(200, seed=7, max_degree=8)],
    "batch": lambda: [synth.open_chain(130), synth.isolated(0), synth.open_chain(9), synth.open_chain(400)],
}


@pytest.mark.parametrize("case", CASES)
def test_block_layout_equals_site_layout(case):
    lats = CASES[case]()
    R, S, M = len(lats), 3, 5
    T = np.array([1.5, 0.0, 0.7]) * np.ones((R, 1))
    B = np.array([0.3, -0.2, 0.0])
    plans = [hsim.Plan(lat) for lat in lats]
    got = []
    for layout in (hsim.LAYOUT_BLOCK, hsim.LAYOUT_SITE):
        b = hsim.Batch(plans, seed=11, precision=hsim.FP64_EXACT, layout=layout).bind(S, M)
        b.bind_outputs(snapshots=True)
        b.init_spins(hsim.INIT_RANDOM)
        trace = b.new_trace(2), b.new_trace(1)
        b.run(T[:, :2], B[:2], recompute_every=3, trace=trace[0], launch=hsim.LAUNCH_PLAIN)
        b.run(T[:, 2:], B[2:], first_step=2, recompute_every=3, trace=trace[1], launch=hsim.LAUNCH_PLAIN)
        torch.cuda.synchronize()
        assert b.status() == 0
        got.append((b.history, b.snapshots, *trace, [b.spins_user(r) for r in range(R)]))
    (h0, s0, a0, c0, u0), (h1, s1, a1, c1, u1) = got
    assert torch.equal(s0, s1) and torch.equal(a0, a1) and torch.equal(c0, c1)
    assert all(torch.equal(x, y) for x, y in zip(u0, u1))
    assert torch.equal(h0[..., 4], h1[..., 4])
    for r, lat in enumerate(lats):
        scale = np.abs(lat.J).sum() / 2 + 2.0 * lat.n + 1.0
        assert float((h0[r, ..., :4] - h1[r, ..., :4]).abs().max()) <= 1e-12 * scale


# Classes of 65 to 128 sites change the kernel beyond three replicas per CU.
@pytest.mark.parametrize("more", [0, 1])
def test_many_replicas_equal_site_layout(more):
    R = 3 * torch.cuda.get_device_properties(0).multi_processor_count + more
    plan = hsim.Plan(_with_terms(synth.sc_periodic(6), 4))
    T = np.linspace(0.4, 2.5, R)[:, None]
    got = []
    for layout in (hsim.LAYOUT_BLOCK, hsim.LAYOUT_SITE):
        b = hsim.Batch([plan] * R, seed=5, precision=hsim.FP64_EXACT, layout=layout).bind(1, 4)
        b.bind_outputs(snapshots=True)
        b.init_spins(hsim.INIT_RANDOM)
        b.run(T, 0.2, recompute_every=2)
        torch.cuda.synchronize()
        assert b.status() == 0
        got.append((b.history, b.snapshots))
    (h0, s0), (h1, s1) = got
    assert torch.equal(s0, s1) and torch.equal(h0[..., 4], h1[..., 4])
    assert float((h0 - h1)[..., :4].abs().max()) <= 1e-12 * (4 * 216 + 1.0)   # bonds, k, B and M of 216 sites
