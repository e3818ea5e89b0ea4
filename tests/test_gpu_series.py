"""Window means, window maxima, tail probabilities, lineages and AMS selection at the sizes where
their kernels cut the work: around the runs of 16 samples, the 4096 samples of a workgroup, the
samples and ancestors that fit in LDS, waves of 64 slots, and windows of one sample and of the row.

The references are FP64 sums in another order: an FP32 result may differ by its last rounding
(2^-23 relative), an FP64 one by len * 2^-53 relative to the sum of magnitudes (samples are O(1)
and positive, so to the mean itself); copies and selections are equal.
"""
import numpy as np
import pytest
import torch

from oracle import ams as oams
from paper_2005_09323_amd import rare

pytestmark = pytest.mark.gpu


def _series(rows, length, seed):
    return np.random.default_rng(seed).uniform(0.5, 1.5, (rows, length)).astype(np.float32)


def _means(x, w):
    c = np.cumsum(np.pad(x.astype(np.float64), ((0, 0), (1, 0))), axis=1)
    return (c[:, w:] - c[:, :-w]) / w


@pytest.mark.parametrize("length,window", [(1, 1), (16, 16), (17, 2), (100, 33), (4096, 512), (4097, 4097),
                                           (9000, 4096), (9000, 1), (14000, 13000), (8193, 100)])
def test_window_means_and_maxima(length, window):
    from paper_2005_09323_amd.ensemble import window_mean
    x = _series(3, length, length + window)
    ref = _means(x, window)
    dev = torch.from_numpy(x).cuda()
    got = window_mean(dev, window).cpu().numpy()
    assert np.all(np.isneginf(got[:, :window - 1]))
    assert np.abs(got[:, window - 1:] / ref - 1.0).max() <= 2.0 ** -23
    fmax = rare.window_maxima(dev, window).cpu().numpy()
    assert np.abs(fmax / ref.max(axis=1) - 1.0).max() <= 2 * length * 2.0 ** -53 * (length / window)


def test_a_sample_that_is_not_finite_stays_in_its_windows():
    from paper_2005_09323_amd.ensemble import window_mean
    x = _series(2, 5000, 1)
    x[0, 1000] = np.nan
    x[1, 4095] = np.inf
    w = 64
    got = window_mean(torch.from_numpy(x).cuda(), w).cpu().numpy()
    clean = np.isfinite(got)
    for r, at in ((0, 1000), (1, 4095)):
        assert not clean[r, at:at + w].any()
        # runs of 16 outputs slide: at most the rest of the run behind the last such window
        assert clean[r, w - 1:at].all() and clean[r, (at + w + 15) // 16 * 16:].all()


@pytest.mark.parametrize("n,levels", [(1, 1), (255, 3), (1024, 2), (1025, 5), (5000, 33)])
def test_tail_probability_in_index_order(n, levels):
    rng = np.random.default_rng(n)
    fmax, lw = rng.uniform(0, 1, n), rng.normal(0, 2, n)
    lw[fmax < 0.2] = 800.0           # exp overflows: must not enter a level above
    lev = np.linspace(0.2, 1.1, levels)
    got = rare.tail_probability(torch.from_numpy(fmax).cuda(), torch.from_numpy(lw).cuda(), lev)
    ref = np.array([np.exp(lw[fmax >= q]).sum() / n for q in lev])
    assert np.allclose(got, ref, rtol=n * 2.0 ** -52 + 2.0 ** -50, atol=0.0)


@pytest.mark.parametrize("n,periods,tau", [(1, 1, 1), (7, 300, 3), (256, 32, 5), (256, 33, 5)])
def test_lineages(n, periods, tau):
    class Ens:                       # what rebuild reads of an ensemble
        device = torch.device("cuda")
    rng = np.random.default_rng(n + periods)
    anc = np.sort(rng.integers(0, n, (periods, n)), axis=1).astype(np.int32)
    ints, lnr = rng.normal(size=(periods, n)), rng.normal(size=periods)
    x = _series(n, periods * tau + 3, 5)
    ens = Ens()
    ens.n, ens.capacity, ens.series = n, x.shape[1], torch.from_numpy(x).cuda()
    run = rare.GktlRun(0.5, tau, periods, 2, torch.from_numpy(anc).cuda(), torch.from_numpy(ints).cuda(),
                       torch.from_numpy(lnr).cuda())
    tr = rare.rebuild(run, ens)
    slot, traj, integ = np.arange(n), np.empty((n, periods * tau), np.float32), np.zeros(n)
    order = []
    for i in range(periods - 1, -1, -1):
        slot = anc[i][slot]
        traj[:, i * tau:(i + 1) * tau] = x[slot, 2 + i * tau:2 + (i + 1) * tau]
        order.append(slot)
    for i, s in enumerate(order[::-1]):
        integ = integ + ints[i][s]
    assert np.array_equal(tr.series.cpu().numpy(), traj)
    assert np.array_equal(tr.integral.cpu().numpy(), integ)     # added in period order on both sides
    lz = 0.0
    for v in lnr:
        lz += v
    assert np.allclose(tr.log_weight.cpu().numpy(), lz - 0.5 * integ, rtol=0, atol=4 * 2.0 ** -53 * np.abs(lz - 0.5 * integ).max() + 1e-15)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 2047, 2048])
def test_ams_selection_sizes(n):
    from paper_2005_09323_amd.ensemble import ams_score_kill_branch
    x = _series(n, 65, n)
    x[::3] = x[0]                    # ties
    kill = max(1, n // 5)
    sel = ams_score_kill_branch(torch.from_numpy(x).cuda(), kill, 9, 4)
    ref = oams.kill_branch(x.astype(np.float64), kill, 9, 4)
    assert sel["level"] == ref.level
    assert np.array_equal(sel["killed"].cpu().numpy(), ref.killed)
    assert np.array_equal(sel["parents"].cpu().numpy(), ref.parents)
    assert np.array_equal(sel["branch_t"].cpu().numpy(), ref.branch_t)
