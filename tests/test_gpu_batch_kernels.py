"""Which kernel steps a batch, asked (Ensemble.batch_kernel) and set (set_batch_kernel): the lattices of the
resident and the sweep kernel's own tests, each stepped by that kernel in every batch, against the one-step
shape 0 (the arithmetic of a cell is the same: the tolerance is zero), and the cut that the estimates
choose for each."""
import pytest
import torch

import workloads
from test_gpu_resident import LATTICES as RESIDENT
from test_gpu_resident import OPEN
from test_gpu_sweep import LATTICES as SWEEP

pytestmark = pytest.mark.gpu


def _ensemble(members, tile, kernel=None, collision=None, opened=None):
    from paper_2005_09323_amd.ensemble import Ensemble
    ens = Ensemble(members, series_capacity=90)
    ens.pop_a.zero_()  # solid cells are never written
    ens.pop_b.zero_()
    ens.set_tile(tile)
    ens.set_batch_kernel(kernel)
    if collision is not None:
        ens.set_collision("central", *collision)
    if opened is not None:
        grid, bar, sponge, outlet = opened
        ens.set_open_channel(0.05, grid, bar, sponge, 0.9, outlet_density=outlet)
    return ens


def _steps(ens, kernel):
    n = ens.n
    ens.init(7, 1e-2)
    for mask, steps in ((None, 13), ([j % 2 == 0 for j in range(n)], 7), ([j % 2 == 1 or j == 2 for j in range(n)], 2),
                        (None, 65)):
        ens.set_active(mask)
        if kernel is not None:
            assert ens.batch_kernel(steps)["kernel"] == kernel, steps
        ens.step(steps)
    torch.cuda.synchronize()
    out = [ens.series.clone(), ens.accum.clone()] + [ens.state(i).clone() for i in range(n)]
    ens.close()
    return out


def _same(got, want, what):
    for k, (a, b) in enumerate(zip(got, want)):
        assert torch.equal(a, b), (what, k)


@pytest.mark.parametrize("collision", [None, (1.0, 1.0, 1.0), (1.2, 0.9, 1.4)])
@pytest.mark.parametrize("lattices", sorted(RESIDENT))
def test_resident_in_every_batch(lattices, collision):
    from paper_2005_09323_amd import native
    members = RESIDENT[lattices]
    want = _steps(_ensemble(members, 0, None, collision), "plain")
    for wait in (None, 0) if len(members) < 8 else (None,):
        ens = _ensemble(members, 20, "resident", collision)
        if wait is not None:
            native.check(ens.lib.lbm_set_wait_limit(ens._ctx, wait))
        _same(_steps(ens, "resident"), want, wait)


@pytest.mark.parametrize("collision", [None, (1.0, 1.0, 1.0), (1.2, 0.9, 1.4)])
@pytest.mark.parametrize("lattices", sorted(OPEN))
def test_open_resident_in_every_batch(lattices, collision):
    from paper_2005_09323_amd import native
    members, opened = OPEN[lattices]
    want = _steps(_ensemble(members, 0, None, collision, opened), "plain")
    for wait in (None, 0) if len(members) < 8 else (None,):
        ens = _ensemble(members, 20, "resident", collision, opened)
        if wait is not None:
            native.check(ens.lib.lbm_set_wait_limit(ens._ctx, wait))
        _same(_steps(ens, "resident"), want, wait)


@pytest.mark.parametrize("collision", [None, (1.0, 1.0, 1.0), (1.2, 0.9, 1.4)])
@pytest.mark.parametrize("lattices", sorted(SWEEP))
def test_sweep_in_every_batch(lattices, collision):
    members = SWEEP[lattices]
    want = _steps(_ensemble(members, 0, None, collision), "plain")
    for rows in (None, 0, 7, 1):
        ens = _ensemble(members, 20, "sweep", collision)
        if rows is not None:
            ens.set_run_rows([rows] * ens.run_count())
        _same(_steps(ens, "sweep"), want, rows)


def _m(nx, ny, square):
    return workloads.Member(nx, ny, 0.56, 2e-5, square)


# (columns per lane, rows per wave): lattices that the estimates cut so, their squares over seams of waves and rows
CUTS = {
    (2, 1): [_m(256, 64, (124, 20, 9))],
    (2, 2): [_m(128, 101, (60, 40, 9))] * 20,
    (2, 3): [_m(200, 101, (95, 40, 9))] * 20,
    (2, 4): [_m(200, 128, (95, 60, 9))] * 24,
    (2, 6): [_m(512, 101, (250, 40, 13))] * 20,
    (3, 2): [_m(330, 101, (160, 40, 9))] * 14,
    (3, 3): [_m(330, 101, (160, 40, 9))] * 20,
    (3, 4): [_m(330, 128, (160, 60, 9))] * 24,
}


@pytest.mark.parametrize("collision", [None, (1.0, 1.0, 1.0), (1.2, 0.9, 1.4)])
@pytest.mark.parametrize("cut", sorted(CUTS))
def test_each_cut_of_the_resident_kernel(cut, collision):
    members = CUTS[cut]

    def run(tile):
        ens = _ensemble(members, tile, None, collision)
        ens.init(7, 1e-2)
        if tile == 20 and (collision is None or collision == (1.0, 1.0, 1.0)):
            k = ens.batch_kernel(64)
            assert k["kernel"] == "resident" and (k["columns"], k["rows"]) == cut, k
        ens.step(13)
        ens.step(65)
        torch.cuda.synchronize()
        out = [ens.series.clone(), ens.accum.clone()] + [ens.state(i).clone() for i in range(len(members))]
        ens.close()
        return out

    _same(run(20), run(0), cut)


@pytest.mark.parametrize("lattices,cut", [("odd_widths", (2, 2)), ("three_rows", (2, 3)), ("several_launches", (2, 4)),
                                          ("six_rows", (2, 6)), ("three_columns_two_rows", (3, 2)),
                                          ("four_rows", (3, 3))])
def test_cuts_of_open_channels(lattices, cut):
    members, opened = OPEN[lattices]
    ens = _ensemble(members, 20, None, (1.0, 1.0, 1.0), opened)
    k = ens.batch_kernel(64)
    ens.close()
    assert k["kernel"] == "resident" and (k["columns"], k["rows"]) == cut, k


def test_a_kernel_that_cannot_step_the_ensemble_is_passed_over():
    """Asked for the sweep in an open channel, or for either in a channel of more than 1024 columns, the others
    step it; values outside the range are refused and change nothing."""
    from paper_2005_09323_amd import native
    for members, opened in (([_m(1300, 20, None)], None), ([_m(256, 20, (100, 4, 5))], (20, 3, 200, 0))):
        for asked in ("sweep", "resident", "plain"):
            ens = _ensemble(members, 20, asked, None, opened)
            can = asked == "resident" and opened is not None
            assert ens.batch_kernel(13)["kernel"] == ("resident" if can else "plain"), asked
            for bad in (-2, 3):
                assert ens.lib.lbm_set_batch_kernel(ens._ctx, bad) == native.LBM_EINVAL
            assert ens.batch_kernel(13)["kernel"] == ("resident" if can else "plain"), asked
            assert ens.lib.lbm_batch_kernel(ens._ctx, 0, None) == native.LBM_EINVAL
            ens.close()


@pytest.mark.parametrize("members,rows,swept", [
    ([_m(256, 64, (124, 20, 9))], 32, False),                # 64 steps: 429 us with one step per launch, 1752 swept
    ([_m(1024, 256, (500, 100, 32))] * 8, 64, False),        # 1869 and 5273
    ([_m(512, 128, (250, 60, 9))] * 64, 128, False),         # 3667 and 6209
    ([_m(1024, 256, (500, 100, 32))] * 128, 0, False),       # two steps per launch 15 852, swept 18 805
    ([_m(1024, 256, (500, 100, 32))] * 128, 64, True),       # 16 818 and 11 373
])
def test_row_ranges_do_not_force_the_sweep(members, rows, swept):
    """Row ranges given by the caller are the two-step strips' and the sweep's; the faster of these steps the
    batch, and the sweep never steps batches of one to three."""
    ens = _ensemble(members, 20)
    ens.set_run_rows([rows])
    assert ens.batch_kernel(64)["kernel"] == ("sweep" if swept else "plain")
    assert [ens.batch_kernel(n)["kernel"] for n in (1, 2, 3)] == ["plain"] * 3
    ens.close()


@pytest.mark.parametrize("members,collision,opened,n_steps,us", [
    # us with the kernel that the estimates chose once, and with the one- and two-step kernels
    ([_m(768, 306, (300, 100, 9))] * 16, (1.2, 0.9, 1.4), None, 8, (604, 492)),
    ([_m(512, 163, (300, 50, 9))] * 3, None, None, 2, (27.9, 21.1)),
    ([_m(399, 68, (300, 30, 9))] * 97, None, None, 2, (111, 79)),
    ([_m(512, 37, (300, 20, 5))] * 5, (1.0, 1.0, 1.0), (20, 3, 400, 0), 1, (26.4, 19.6)),
    ([_m(601, 58, (300, 20, 5))] * 437, (1.2, 0.9, 1.4), (20, 3, 400, 0), 3, (1144, 949)),
])
def test_batches_that_the_one_and_two_step_kernels_step_faster(members, collision, opened, n_steps, us):
    """Short batches, whose resident launches mostly load and store the state, and central moments with three
    rates, whose sweeps take half as long again as other collisions', go to the one- or two-step kernel."""
    ens = _ensemble(members, 20, None, collision, opened)
    assert ens.batch_kernel(n_steps)["kernel"] == "plain", us
    ens.close()
