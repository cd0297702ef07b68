"""Sites per wave of the replica layout's tiles on both sides of each line of
the rule (host only: batches are created, not bound)."""
import pytest

import synth
from paper_1803_07030_amd import hsim


# 12 L^3 x (replicas padded to 32 or a multiple of 64) bytes of spins; below
# the first line a phase of two blocks per CU or more takes 32 sites.
@pytest.mark.parametrize("L,R,spw", [(66, 64, 32), (67, 64, 8), (34, 500, 8), (28, 1024, 8), (30, 1024, 32),
                                     (22, 2048, 8), (24, 2048, 32), (66, 20, 32), (68, 20, 8), (68, 32, 8)])
def test_sites_per_wave(L, R, spw):
    plan = hsim.Plan(synth.sc_periodic(L))
    b = hsim.Batch([plan] * R, seed=1, layout=hsim.LAYOUT_REPLICA)
    assert b.info.sites_per_wave == spw
