"""Analysis kernels at the sizes where their paths change: series that stay in
registers or in LDS, longer ones, temperature tables in the arguments or in
device memory, and one or several samples per thread of the multiple-histogram
launches, whose block sums are added by every block or by a launch of their
own.  The reference forms the same sums in numpy; both sides round every term
in double precision, so they agree to 1e-9 relative."""
import numpy as np
import pytest
import torch
from scipy.special import logsumexp

from oracle import analysis as A
from paper_1803_07030_amd import hsim

pytestmark = pytest.mark.gpu


def _history(R, S, M, seed, N=64.0):
    """Correlated samples with the energies of a Gaussian density of states,
    whose neighbouring temperatures overlap."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((R * S, M, 4))
    x[:, 1:] += 0.7 * x[:, :-1]
    h = np.zeros((R * S, M, 5))
    beta = 0.3 + 0.05 * np.arange(R * S) / max(R * S - 1, 1)
    h[..., 0] = -beta[:, None] * N + np.sqrt(N) * x[..., 0]
    h[..., 1:4] = 0.2 * N + np.sqrt(N) * x[..., 1:]
    return h.reshape(R, S, M, 5), beta.reshape(R, S)


def _close(got, ref, rel=1e-9, floor=1e-12):
    got, ref = np.asarray(got), np.asarray(ref)
    assert np.all(np.abs(got - ref) <= rel * np.abs(ref) + floor), np.max(np.abs(got - ref))


@pytest.mark.parametrize("R,S,n,evals", [(1, 1, 2, 1), (3, 2, 1025, 2), (1, 1, 4096, 1), (1, 2, 4097, 3),
                                         (1, 1, 12288, 2), (2, 1, 12289, 1), (40, 5, 33, 1), (97, 1, 40, 3)])
def test_thermal_sizes(R, S, n, evals):
    h, beta = _history(R, S, n + 1, seed=n)
    ev = None if evals == 1 else beta[..., None] * np.linspace(0.97, 1.02, evals)
    out = hsim.hsim_analysis_thermal(torch.tensor(h, device="cuda"), 1, 64, beta, ev).cpu().numpy()
    for r in range(R):
        for s in range(S):
            E, Mv = h[r, s, 1:, 0], h[r, s, 1:, 1:4]
            for j in range(evals):
                b = beta[r, s] if ev is None else ev[r, s, j]
                _close(out[r, s, j], A.thermal_array(A.reweight(E, Mv, 64, beta[r, s], b)))


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 255, 258, 1023, 4097, 12290, 18432, 18433, 30001])
@pytest.mark.parametrize("obs", [0, 1])
def test_tau_sizes(n, obs):
    """Windows from a few lags to several batches of them, up to the half
    length (a slow wave added to one series)."""
    h, _ = _history(1, 3, n + 2, seed=n + 1)
    slow = 30.0 * np.cos(np.arange(n + 2) * 2 * np.pi / max(0.15 * n, 4.0))
    h[0, 1, :, 0] += slow
    h[0, 1, :, 3] += slow
    if n < 10000:
        h[0, 2, :, 0] = 1.5                      # constant series: tau 1/2, window 0
        h[0, 2, :, 1:4] = 2.0
    tau, win = hsim.hsim_analysis_tau(torch.tensor(h, device="cuda"), 2, obs)
    for s in range(3):
        E, Mv = h[0, s, 2:, 0], h[0, s, 2:, 1:4]
        x = E if obs == 0 else np.sqrt((Mv * Mv).sum(axis=1))
        if np.ptp(x) == 0.0:
            # 1.5 n is exact, so the deviations are 0; n sqrt(12) is not, and
            # the rounded mean leaves a residue of no meaning on either side
            assert obs == 1 or (float(tau[0, s]) == 0.5 and int(win[0, s]) == 0)
            continue
        ref, w = A.tau_int(x)
        assert int(win[0, s]) == w
        _close(float(tau[0, s]), ref)


@pytest.mark.parametrize("K,n,iters", [(1, 2, 5), (2, 2, 5), (3, 257, 5000), (70, 30, 40), (16, 1000, 7),
                                       (3, 50000, 5), (16, 9000, 5), (300, 20, 5)])
def test_multihist_sizes(K, n, iters):
    h, beta = _history(K, 1, n, seed=K)
    bk, tol = beta[:, 0], 1e-9
    ev = np.array([bk.min(), 0.5 * (bk.min() + bk.max())])
    f, it, out = hsim.hsim_analysis_multihist(torch.tensor(h, device="cuda"), 0, 64,
                                              [(k, 0) for k in range(K)], bk, ev, max_iter=iters, tol=tol)
    e, Mv = h[:, 0, :, 0].reshape(-1), h[:, 0, :, 1:4].reshape(-1, 3)
    f_ref, it_ref = np.zeros(K), 0
    while it_ref < iters:
        it_ref += 1
        logd = logsumexp(np.log(n) + f_ref - bk * e[:, None], axis=1)
        fn = -logsumexp(-bk * e[:, None] - logd[:, None], axis=0)
        fn -= fn[0]
        done = np.max(np.abs(fn - f_ref)) < tol
        f_ref = fn
        if done:
            break
    assert it == it_ref
    _close(f, f_ref, floor=1e-9)
    logd = logsumexp(np.log(n) + f_ref - bk * e[:, None], axis=1)
    for j, b in enumerate(ev):
        _close(out[j].cpu().numpy(), A.thermal_array(A.thermal(e, Mv, 64, b, logw=-b * e - logd)), rel=1e-8,
               floor=1e-10)


# Around the numbers of series that have four lanes per sample, and around the
# samples of a block.
@pytest.mark.parametrize("K,n,iters", [(8, 32, 40), (9, 57, 40), (12, 64, 40), (31, 33, 40), (32, 120, 40),
                                       (32, 129, 3),
                                       (33, 31, 40)])
def test_multihist_lanes_per_sample(K, n, iters):
    test_multihist_sizes(K, n, iters)


# More series than a wave has lanes, their block sums added by a launch of
# their own, stopped by the number of iterations: the last iteration's f is
# complete for every series, the same in every call.
@pytest.mark.parametrize("K,n,iters", [(65, 300, 6), (100, 200, 1), (100, 200, 7), (257, 17, 4)])
def test_multihist_stopped_by_iterations(K, n, iters):
    test_multihist_sizes(K, n, iters)
    h, beta = _history(K, 1, n, seed=K)
    args = (torch.tensor(h, device="cuda"), 0, 64, [(k, 0) for k in range(K)], beta[:, 0], beta[:1, 0])
    f = [hsim.hsim_analysis_multihist(*args, max_iter=iters, tol=1e-9)[0] for _ in range(20)]
    assert all(np.array_equal(f[0], x) for x in f)


# On a card that is nearly full, energies and |M| are read in the history
# instead of from copies: a call that has room for 8 bytes per sample and no
# more gives the same bits.  The same series stands for every temperature, so
# the samples outnumber the history.
@pytest.mark.parametrize("K", [8, 9])
def test_multihist_without_room_for_copies(K):
    n, room = 1 << 22, 500 << 20                 # 268 or 302 MB for ln D, three times as much with copies
    g = torch.Generator(device="cuda").manual_seed(3)
    h = torch.randn(1, 1, n, 5, generator=g, device="cuda", dtype=torch.float64) * 8.0 + 20.0
    bk = 0.3 + 0.01 * np.arange(K)
    args = (h, 0, 64, [(0, 0)] * K, bk, bk[:3])
    want = hsim.hsim_analysis_multihist(*args, max_iter=3, tol=1e-30)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    try:
        while (left := torch.cuda.mem_get_info()[0] - room) > 1 << 20:
            held.append(torch.empty(min(left, 16 << 30), dtype=torch.uint8, device="cuda"))
        got = hsim.hsim_analysis_multihist(*args, max_iter=3, tol=1e-30)
        torch.cuda.synchronize()
    finally:
        held.clear()
        torch.cuda.empty_cache()
    assert got[1] == want[1] == 3
    assert np.array_equal(got[0], want[0]) and torch.equal(got[2], want[2])


# Around the series lengths and numbers of series at which the blocks change
# their size (64, 256 or 1024 threads).
@pytest.mark.parametrize("R,S,n", [(1, 1, 256), (1, 1, 257), (2, 1, 1024), (1, 2, 1025), (301, 2, 50), (300, 1, 128),
                                   (300, 1, 129), (300, 1, 257), (300, 1, 2048), (300, 1, 2049)])
def test_block_sizes(R, S, n):
    h, beta = _history(R, S, n + 1, seed=n)
    slow = 20.0 * np.cos(np.arange(n + 1) * 2 * np.pi / max(0.3 * n, 4.0))
    h[::2, ..., 0] += slow                       # windows up to the half length beside short ones
    h[::2, ..., 3] += slow
    d = torch.tensor(h, device="cuda")
    out = hsim.hsim_analysis_thermal(d, 1, 64, beta, beta[..., None] * np.array([0.98, 1.0])).cpu().numpy()
    taus = [hsim.hsim_analysis_tau(d, 1, obs) for obs in (0, 1)]
    for r in range(0, R, max(1, R // 7)):
        for s in range(S):
            E, Mv = h[r, s, 1:, 0], h[r, s, 1:, 1:4]
            for j, q in enumerate((0.98, 1.0)):
                _close(out[r, s, j], A.thermal_array(A.reweight(E, Mv, 64, beta[r, s], q * beta[r, s])))
            for (tau, win), x in zip(taus, (E, np.sqrt((Mv * Mv).sum(axis=1)))):
                ref, w = A.tau_int(x)
                assert int(win[r, s]) == w
                _close(float(tau[r, s]), ref)


# A series whose mean is exact and whose deviations are 0: tau 1/2, window 0.
@pytest.mark.parametrize("n", [2, 65, 300, 5000])
@pytest.mark.parametrize("obs", [0, 1])
def test_tau_of_a_constant_series(n, obs):
    h = np.zeros((1, 2, n, 5))
    h[..., 0], h[..., 1], h[..., 3] = 1.5, 3.0, 4.0            # |M| = 5
    tau, win = hsim.hsim_analysis_tau(torch.tensor(h, device="cuda"), 0, obs)
    assert torch.all(tau == 0.5) and torch.all(win == 0)
