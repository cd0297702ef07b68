"""Replica layout: the per-type magnetisation, summed chunk by chunk into a
window of MCS, equals the per-type sums of the spins after every MCS (steps of
one MCS, whose end states are recorded), for lattices with one and several
sites per lane group in a chunk, one and two columns of replicas, a type
without sites, and windows shorter than the run.  The adaptive widths, whose
accepted moves one block or several sum, equal the site layout's."""
import numpy as np
import pytest
import torch

import synth
from paper_1803_07030_amd import hsim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,R,n_types", [(5, 20, 1), (5, 100, 4), (21, 33, 3), (26, 100, 8)])
@pytest.mark.parametrize("launch", [hsim.LAUNCH_PLAIN, hsim.LAUNCH_GRAPH])
def test_type_sums_equal_sums_of_the_states(L, R, n_types, launch):
    lat = synth.sc_periodic(L)
    plan = hsim.Plan(lat)
    types = (np.arange(lat.n) * 7 // 3) % n_types
    if n_types == 4:
        types[types == 1] = 2                    # a type without sites
    plan.set_types(types.astype(np.int32))
    S = 70 if L == 5 else 20
    T = np.linspace(0.5, 2.5, R)[:, None] * np.ones((1, S))
    b = hsim.Batch([plan] * R, seed=8, layout=hsim.LAYOUT_REPLICA).bind(S, 1)
    b.bind_outputs(type_mag_types=n_types, snapshots=True)
    b.init_spins(hsim.INIT_COLD_Z)
    b.run(T, 0.1, launch=launch)
    torch.cuda.synchronize()
    assert b.status() == 0
    t = torch.tensor(types, device="cuda")
    for k in range(n_types):
        ref = b.snapshots[:, :, t == k].sum(dim=2)
        # n terms of at most 1, summed in double in another order
        assert torch.allclose(b.type_mag[:, :, 0, k], ref, rtol=0, atol=1e-15 * lat.n)


@pytest.mark.parametrize("L,R", [(8, 24), (24, 40), (24, 100)])
def test_adaptive_widths_equal_the_site_layouts(L, R):
    lat = synth.sc_periodic(L)
    plan = hsim.Plan(lat)
    plan.set_types((np.arange(lat.n) % 3 == 0).astype(np.int32))
    T = np.linspace(0.5, 1.4, R)[:, None]
    got = []
    for layout in (hsim.LAYOUT_REPLICA, hsim.LAYOUT_SITE):
        b = hsim.Batch([plan] * R, seed=3, layout=layout).bind(1, 6)
        b.set_policies([(hsim.POLICY_ADAPTIVE, 0.5), (hsim.POLICY_RANDOM, 0.0)])
        b.init_spins(hsim.INIT_COLD_Z)
        b.run(T, 0.0, launch=hsim.LAUNCH_PLAIN)
        got.append(b.sigma())
        assert b.status() == 0
    assert np.array_equal(got[0], got[1])


# Just below and above the number of tiles one block adds by itself, and many
# chunks of tiles, over one to three columns of replicas.
@pytest.mark.parametrize("L,R", [(18, 70), (19, 33), (20, 150), (40, 66)])
@pytest.mark.parametrize("launch", [hsim.LAUNCH_PLAIN, hsim.LAUNCH_GRAPH])
def test_adaptive_widths_over_chunks_of_tiles(L, R, launch):
    plan = hsim.Plan(synth.sc_periodic(L))
    T = np.linspace(0.5, 1.4, R)[:, None] * np.ones((1, 2))
    got = []
    for layout in (hsim.LAYOUT_REPLICA, hsim.LAYOUT_SITE):
        b = hsim.Batch([plan] * R, seed=3, layout=layout).bind(2, 3)
        b.set_policies([(hsim.POLICY_ADAPTIVE, 0.5)])
        b.init_spins(hsim.INIT_COLD_Z)
        b.run(T, 0.0, launch=launch if layout == hsim.LAYOUT_REPLICA else hsim.LAUNCH_PLAIN)
        got.append(b.sigma())
        assert b.status() == 0
    assert np.array_equal(got[0], got[1])
