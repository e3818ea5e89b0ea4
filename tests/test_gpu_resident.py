"""The resident kernel (the default shape on an ensemble that fits in the device's registers: a chunk
of steps per launch) against the one-step shape 0.

Both collide every cell with the same arithmetic on the same FP32 inputs, so states and drag are
equal bit for bit: the tolerance is zero.  Sizes sit where the cutting can go wrong: widths around the
128 columns of a wave and odd ones (a last lane with one cell), one to eight waves per row, heights
that end inside a wave's rows, workgroups beside one another within and across members, squares across
wave and row seams and beside the walls and the periodic edge, every number of columns per lane and
rows per wave, more members than one launch holds, runs of lattices cut alike or each its own way,
chunks of one step up to the longest, and inactive members.  With a wait limit below zero every member
of more than one workgroup is given up and stepped by the kernel that waits for nothing; with a limit of
zero a chunk may be given up anywhere in it.
"""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def _m(nx, ny, square):
    return workloads.Member(nx, ny, 0.56, 2e-5, square)


LATTICES = {
    "wave_seams": [_m(256, 24, (124, 8, 8)), _m(256, 24, (1, 1, 3)), _m(256, 24, (250, 18, 5))],
    "widths": [_m(1024, 11, (127, 3, 4)), _m(600, 10, (594, 4, 3)), _m(330, 9, (128, 3, 4))],
    "ragged": [_m(201, 33, (60, 12, 6)), _m(257, 11, (125, 4, 4)), _m(130, 21, (1, 1, 3)), _m(127, 6, None)],
    "smallest": [_m(4, 4, (1, 1, 2)), _m(5, 7, (2, 2, 2)), _m(128, 4, (60, 1, 2)), _m(129, 5, None)],
    "two_rows": [_m(384, 61, (127, 30, 9))] * 12,
    "three_rows": [_m(384, 61, (250, 30, 9))] * 17,
    "four_rows": [_m(512, 131, (250, 60, 9))] * 12,
    "several_launches": [_m(512, 128, (250, 60, 9))] * 25 + [_m(130, 40, (124, 20, 5))] * 3,
    "six_rows": [_m(256, 203, (124, 100, 13))] * 28,
    "three_columns_two_rows": [_m(575, 101, (190, 40, 9))] * 13,
    "three_columns_three_rows": [_m(331, 110, (188, 60, 9))] * 24,
    "three_columns_four_rows": [_m(701, 200, (187, 100, 13))] * 8,
    "runs_apart": [_m(332, 109, (321, 2, 9))] * 22 + [_m(201, 75, (99, 30, 9))] * 35,
}


# open channels: (members, grid column and bar, sponge column, outlet density)
OPEN = {
    "one_wave": ([_m(128, 21, (60, 8, 4)), _m(67, 9, None), _m(9, 4, None)], (1, 1, 40, 0)),
    "odd_widths": ([_m(201, 33, (120, 12, 6)), _m(129, 30, (100, 13, 5)), _m(257, 14, (250, 4, 4))], (20, 3, 96, 1)),
    "eight_waves": ([_m(1024, 37, (130, 10, 9)), _m(769, 19, (600, 4, 3))], (64, 4, 500, 0)),
    "no_sponge": ([_m(330, 50, (80, 20, 8))] * 3, (0, 0, 1 << 30, 1)),
    "three_rows": ([_m(512, 81, (250, 30, 9))] * 18, (31, 5, 300, 1)),
    "four_rows": ([_m(513, 129, (250, 60, 9))] * 8, (31, 5, 300, 0)),
    "six_rows": ([_m(256, 203, (124, 100, 13))] * 28, (100, 7, 200, 1)),
    "several_launches": ([_m(512, 128, (250, 60, 9))] * 25 + [_m(130, 40, (122, 20, 5))] * 3, (9, 4, 100, 0)),
    "three_columns_two_rows": ([_m(640, 100, (190, 40, 9))] * 10, (62, 5, 300, 1)),
    "three_columns_three_rows": ([_m(512, 129, (188, 60, 9))] * 11, (31, 5, 300, 0)),
    "three_columns_odd": ([_m(514, 129, (500, 60, 9))] * 11, (31, 5, 190, 1)),
}


def _run(members, tile, collision, wait=None, opened=None):
    from paper_2005_09323_amd import native
    from paper_2005_09323_amd.ensemble import Ensemble
    ens = Ensemble(members, series_capacity=90)
    ens.pop_a.zero_()  # solid cells are never written
    ens.pop_b.zero_()
    ens.set_tile(tile)
    if collision is not None:
        ens.set_collision("central", *collision)
    if opened is not None:
        grid, bar, sponge, outlet = opened
        ens.set_open_channel(0.05, grid, bar, sponge, 0.9, outlet_density=outlet)
    if wait is not None:
        native.check(ens.lib.lbm_set_wait_limit(ens._ctx, wait))
    ens.init(7, 1e-2)
    ens.step(13)
    ens.set_active([j % 2 == 0 for j in range(len(members))])
    ens.step(7)
    ens.set_active([j % 2 == 1 or j == 2 for j in range(len(members))])
    ens.step(2)
    ens.set_active(None)
    ens.step(65)                      # a whole chunk and one step
    torch.cuda.synchronize()
    out = ens.series.clone(), [ens.state(i).clone() for i in range(len(members))], ens.accum.clone()
    ens.close()
    return out


@pytest.mark.parametrize("collision", [None, (1.0, 1.0, 1.0), (1.2, 0.9, 1.4)])
@pytest.mark.parametrize("lattices", sorted(LATTICES))
def test_resident_bit_identical_to_one_step(lattices, collision):
    members = LATTICES[lattices]
    drag0, states0, accum0 = _run(members, 0, collision)
    for wait in (None, -1, 0) if len(members) < 8 else (None,):
        drag, states, accum = _run(members, 20, collision, wait)
        assert torch.equal(drag, drag0) and torch.equal(accum, accum0), wait
        for i, (a, b) in enumerate(zip(states, states0)):
            assert torch.equal(a, b), (wait, i)


@pytest.mark.parametrize("collision", [None, (1.0, 1.0, 1.0), (1.2, 0.9, 1.4)])
@pytest.mark.parametrize("lattices", sorted(OPEN))
def test_open_resident_bit_identical_to_one_step(lattices, collision):
    members, opened = OPEN[lattices]
    drag0, states0, accum0 = _run(members, 0, collision, None, opened)
    for wait in (None, -1, 0) if len(members) < 8 else (None,):
        drag, states, accum = _run(members, 20, collision, wait, opened)
        assert torch.equal(drag, drag0) and torch.equal(accum, accum0), wait
        for i, (a, b) in enumerate(zip(states, states0)):
            assert torch.equal(a, b), (wait, i)


def test_contexts_on_two_streams():
    """Two contexts that do not fit on the device together, stepped from two streams in turn."""
    from paper_2005_09323_amd.ensemble import Ensemble
    members = LATTICES["six_rows"]
    _, states0, _ = _run(members, 0, None)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    ens = []
    for st in streams:
        with torch.cuda.stream(st):
            e = Ensemble(members, series_capacity=90)
            e.pop_a.zero_()
            e.pop_b.zero_()
            e.init(7, 1e-2)
            ens.append(e)
    half = [j % 2 == 0 for j in range(len(members))]
    other = [j % 2 == 1 or j == 2 for j in range(len(members))]
    for mask, n in ((None, 13), (half, 7), (other, 2), (None, 65)):
        for st, e in zip(streams, ens):
            with torch.cuda.stream(st):
                e.set_active(mask)
                e.step(n)
    torch.cuda.synchronize()
    for st, e in zip(streams, ens):
        with torch.cuda.stream(st):
            for i, b in enumerate(states0):
                assert torch.equal(e.state(i), b), i
        e.close()
