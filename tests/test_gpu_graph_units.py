"""Graph launches replay a recompute period, a whole step, or pieces of a long
step: for steps and periods on both sides of those rules they give the spins,
histories, per-type magnetisation and step-end states of plain launches, bit
for bit, with the adaptive move among the policies."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import synth
from paper_1803_07030_amd import hsim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout,R", [(hsim.LAYOUT_REPLICA, 20), (hsim.LAYOUT_SITE, 3)])
@pytest.mark.parametrize("steps,M,P", [(3, 1, 100), (3, 7, 100), (4, 6, 3), (2, 10, 4), (3, 70, 20), (2, 8, 0),
                                       (2, 512, 100), (1, 600, 300), (1, 515, 200), (1, 514, 0)])
def test_graph_units_equal_plain_launches(layout, R, steps, M, P):
    lat = synth.sc_periodic(4)
    lat.k = 0.2 * synth.uniform01(3, lat.n, tag=1)
    plan = hsim.Plan(lat)
    plan.set_types((np.arange(lat.n) % 3 == 0).astype(np.int32))
    T = np.linspace(0.6, 2.0, R)[:, None] * np.ones((1, steps))
    got = []
    for launch in (hsim.LAUNCH_PLAIN, hsim.LAUNCH_GRAPH):
        b = hsim.Batch([plan] * R, seed=4, layout=layout).bind(steps, M)
        b.set_policies([(hsim.POLICY_RANDOM, 0.0), (hsim.POLICY_ADAPTIVE, 0.5)])
        b.bind_outputs(type_mag_types=2, snapshots=True)
        b.init_spins(hsim.INIT_RANDOM)
        for _ in range(2):                       # the second run replays the first one's graph
            b.run(T, 0.1, recompute_every=P, launch=launch)
        torch.cuda.synchronize()
        assert b.status() == 0
        got.append([b.history, b.type_mag, b.snapshots, torch.cat([b.spins_user(r) for r in range(R)]),
                    torch.tensor(b.sigma())])
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.parametrize("M,P,graphs", [(130, 100, 1), (512, 0, 1), (127, 0, 0)])
def test_loop_of_one_step_calls_replays_its_graph(M, P, graphs):
    # a call of one step goes plain; the same call again replays the step
    plan = hsim.Plan(synth.sc_periodic(6))
    T = np.linspace(0.6, 2.0, 20)[:, None]
    got = []
    for launch in (hsim.LAUNCH_PLAIN, hsim.LAUNCH_GRAPH):
        b = hsim.Batch([plan] * 20, seed=4, layout=hsim.LAYOUT_REPLICA).bind(1, M)
        b.init_spins(hsim.INIT_RANDOM)
        for _ in range(2):
            b.run(T, 0.1, recompute_every=P, launch=launch)
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
            b.run(T, 0.1, recompute_every=P, launch=launch)
            torch.cuda.synchronize()
        seen = {e.key: e.count for e in p.key_averages()}
        if "hipLaunchKernel" not in seen:
            pytest.skip("the profiler records no launches here")
        assert seen.get("hipGraphLaunch", 0) == (graphs if launch == hsim.LAUNCH_GRAPH else 0), seen
        assert b.status() == 0
        got.append([b.history, torch.cat([b.spins_user(r) for r in range(20)])])
    for x, y in zip(*got):
        assert torch.equal(x, y)
