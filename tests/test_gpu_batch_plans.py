"""The host side of lbm_step_batch with the default shape: what it works out and allocates per call."""
import time

import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def _ensemble(members, capacity=90, tile=20):
    from paper_2005_09323_amd.ensemble import Ensemble
    ens = Ensemble(members, series_capacity=capacity)
    ens.pop_a.zero_()  # solid cells are never written
    ens.pop_b.zero_()
    ens.set_tile(tile)
    return ens


def test_short_batches_of_a_tall_channel_cost_the_host_little():
    """How a batch is stepped is worked out once for a set of members, not in each call, and not by trying
    every height of a tall channel: ten batches of one step are enqueued in less time than the heights of
    six million rows alone take to be counted once."""
    ens = _ensemble([workloads.Member(4, 6_000_000, 0.6, 1e-6, None)], capacity=20)
    ens.init(7, 1e-3)
    ens.step(1)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(10):
        ens.step(1)
    spent = time.perf_counter() - t0
    torch.cuda.synchronize()
    ens.close()
    assert spent < 0.02, spent


@pytest.mark.parametrize("change", ["active", "collision", "tile", "open", "rows", "init"])
def test_a_plan_is_worked_out_afresh_after_a_change(change):
    """Batches before and after each call that decides how members are stepped, against the one-step shape 0
    (bit for bit: the arithmetic of a cell is the same in every kernel)."""
    members = [workloads.Member(257, 40, 0.56, 2e-5, (120, 12, 9))] * 6

    def run(tile):
        ens = _ensemble(members, 120, tile)
        ens.init(7, 1e-2)
        ens.step(9)
        if change == "active":
            ens.set_active([1, 0, 0, 1, 0, 0])
        elif change == "collision":
            ens.set_collision("central", 1.2, 0.9, 1.4)
        elif change == "tile":
            ens.set_tile(0)
            ens.step(5)
            ens.set_tile(tile)
        elif change == "open":
            ens.set_open_channel(0.05, 20, 3, 200, 0.9)
            ens.init(3, 1e-2)
        elif change == "rows":
            ens.set_run_rows([7] * ens.run_count())
            ens.step(5)
            ens.set_run_rows(None)
        else:
            ens.set_active([1, 0, 0, 1, 0, 0])
            ens.step(9)
            ens.init(5, 1e-2)
        ens.step(9)
        ens.set_active(None)
        ens.step(70)
        torch.cuda.synchronize()
        out = ens.series.clone(), [ens.state(i).clone() for i in range(len(members))]
        ens.close()
        return out

    drag0, states0 = run(0)
    drag, states = run(20)
    assert torch.equal(drag, drag0)
    for i, (a, b) in enumerate(zip(states, states0)):
        assert torch.equal(a, b), i


def test_batches_allocate_nothing():
    """lbm_step_batch enqueues: what it needs on the device is allocated with the context, for every set of
    active members (24 x 512 x 128 needs 25 MB of words between workgroups)."""
    members = [workloads.Member(512, 128, 0.56, 2e-5, (250, 60, 9))] * 24

    def steps(ens):
        ens.init(7, 1e-3)
        ens.set_active([j == 0 for j in range(24)])
        ens.step(8)
        ens.set_active(None)
        ens.step(64)
        ens.set_active([j % 2 == 0 for j in range(24)])
        ens.step(7)
        torch.cuda.synchronize()

    ens = _ensemble(members)
    steps(ens)  # (every kernel loaded)
    ens.close()
    ens = _ensemble(members)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    steps(ens)
    assert abs(free - torch.cuda.mem_get_info()[0]) < 4 << 20
    ens.close()


def test_contexts_of_two_threads_take_turns():
    """Two contexts that do not fit on the device together, each stepped by its own thread on its own stream:
    a long batch, then a smaller plan while the larger one's launches are still queued, against the same
    batches alone (bit for bit)."""
    import threading

    members = [workloads.Member(256, 203, 0.56, 2e-5, (124, 100, 13))] * 28
    few = [j < 3 for j in range(28)]

    def batches(ens):
        ens.step(64 * 20 + 9)
        ens.set_active(few)
        ens.step(64)
        ens.set_active(None)
        ens.step(130)

    def made():
        ens = _ensemble(members, 1600)
        ens.init(7, 1e-2)
        return ens

    ens = made()
    batches(ens)
    torch.cuda.synchronize()
    want = [ens.series.clone()] + [ens.state(i).clone() for i in (0, 27)]
    ens.close()
    streams = [torch.cuda.Stream() for _ in range(2)]
    pair = []
    for st in streams:
        with torch.cuda.stream(st):
            pair.append(made())
    torch.cuda.synchronize()
    failed = []

    def work(st, e):
        try:
            with torch.cuda.stream(st):
                batches(e)
        except Exception as err:  # noqa: BLE001 (reported below)
            failed.append(err)

    threads = [threading.Thread(target=work, args=a) for a in zip(streams, pair)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for e in pair:
        got = [e.series] + [e.state(i) for i in (0, 27)]
        for a, b in zip(got, want):
            assert torch.equal(a, b)
        e.close()


def test_tuning_makes_about_the_steps_asked_for():
    """lbm_autotune(n) makes n launches of each shape (of up to two steps), or of the default shape n steps or two
    chunks of 64 if these are more, and two launches more: with n = 200 at most 404 steps each.  The steps are
    untracked, but a body force F adds F to every cell's momentum in each of them (the walls take less than a
    tenth of it back: their layers grow to sqrt(nu T) = 6 of 256 rows)."""
    force = 1e-9
    members = [workloads.Member(256, 256, 0.51, force, None)] * 8
    ens = _ensemble(members)
    ens.init(7, 0.0)
    ens.autotune(200)
    torch.cuda.synchronize()
    d = ens.state(3).double()
    jx = (d[1] - d[3] + d[5] - d[6] - d[7] + d[8]).mean().item()
    shapes = ens.lib.lbm_tile_count()
    ens.close()
    assert 16 * 200 * 0.9 < jx / force < shapes * 404, jx / force


def test_row_ranges_of_ragged_widths_read_back():
    """Row ranges given for the default shape's sweep are what run_rows returns, for widths that no two-step
    shape takes too, and setting what was read changes nothing; where no kernel uses them it returns -1."""
    members = [workloads.Member(250, 40, 0.56, 2e-5, (116, 12, 9))] * 2 + [workloads.Member(330, 24, 0.56, 2e-5, None)]
    ens = _ensemble(members)
    assert ens.run_rows() == [-1, -1]
    for given, read in (([7, -1], [7, -1]), ([0, 3], [0, 3]), ([40, 25], [0, 0]), ([39, 23], [39, 23])):
        ens.set_run_rows(given)
        assert ens.run_rows() == read, given
        ens.set_run_rows(ens.run_rows())
        assert ens.run_rows() == read, given
    ens.set_tile(0)
    assert ens.run_rows() == [-1, -1]
    ens.set_tile(20)
    assert ens.run_rows() == [39, 23]
    ens.set_open_channel(0.05, 20, 3, 200, 0.9)
    assert ens.run_rows() == [-1, -1]
    ens.set_open_channel(None)
    ens.set_run_rows(None)
    assert ens.run_rows() == [-1, -1]
    ens.close()
    # two-step launches: the ranges in use, given or not
    ens = _ensemble([workloads.Member(256, 64, 0.56, 2e-5, None)] * 2)
    assert ens.run_rows() == [32]
    ens.set_run_rows([16])
    assert ens.run_rows() == [16]
    ens.close()
