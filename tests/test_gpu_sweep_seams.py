"""The sweep kernel against the one-step shape 0 where a
width gives a wave fewer than 64 lanes and the square lies over the seam between two waves.

The lanes of a wave beyond its columns run over the next wave's; what they work out there is wrong in
the last ones (one column more with each of the four steps) and belongs to no cell.  The squares below
reach these columns: they end inside a lane's two cells, hold them, or have their ring of fluid cells
there.  Both kernels collide every cell with the same arithmetic on the same FP32 inputs, so the
tolerance is zero.
"""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def _m(nx, ny, square):
    return workloads.Member(nx, ny, 0.56, 2e-5, square)


# lanes per wave: 60, 63, 63, 62, 60, 63, 56, 63 (the seam's column, the last that a surplus lane holds)
LATTICES = {
    "two_waves": [_m(240, 24, (116, 6, 8)), _m(240, 24, (123, 8, 7)), _m(250, 24, (120, 6, 8))],        # 120 (127), 126 (127)
    "four_waves": [_m(500, 24, (120, 6, 7)), _m(500, 24, (125, 5, 12)), _m(490, 29, (122, 6, 15))],     # 126 (127), 124 (127)
    "six_waves": [_m(720, 24, (235, 4, 12)), _m(720, 24, (596, 9, 11))],                                # 240 (247), 600 (607)
    "eight_waves": [_m(1000, 44, (234, 6, 32)), _m(1000, 44, (246, 6, 7))],                             # 252 (253)
    "odd_width": [_m(333, 26, (111, 6, 14)), _m(333, 26, (230, 8, 9)), _m(497, 24, (120, 6, 6))],       # 112 (127), 224 (239), 126 (127)
}


def _run(members, tile, rows, collision):
    from paper_2005_09323_amd.ensemble import Ensemble
    ens = Ensemble(members, series_capacity=80)
    ens.pop_a.zero_()  # solid cells are never written
    ens.pop_b.zero_()
    ens.set_tile(tile)
    if collision is not None:
        ens.set_collision("central", *collision)
    if rows is not None:
        ens.set_batch_kernel("sweep")
        ens.set_run_rows([rows] * ens.run_count())
        assert ens.batch_kernel(13)["kernel"] == "sweep"
    ens.init(7, 1e-2)
    ens.step(13)                      # 4 + 4 + 4 + 1
    ens.step(66)                      # a captured chunk, then 2
    torch.cuda.synchronize()
    out = ens.series.clone(), ens.accum.clone(), [ens.state(i).clone() for i in range(len(members))]
    ens.close()
    return out


@pytest.mark.parametrize("collision", [None, (1.0, 1.0, 1.0), (1.2, 0.9, 1.4)])
@pytest.mark.parametrize("lattices", sorted(LATTICES))
def test_squares_over_ragged_seams(lattices, collision):
    members = LATTICES[lattices]
    drag0, accum0, states0 = _run(members, 0, None, collision)
    for rows in (0, 7, 1):
        drag, accum, states = _run(members, 20, rows, collision)
        for i, (a, b) in enumerate(zip(states, states0)):
            assert torch.equal(a, b), (rows, i)
        assert torch.equal(drag, drag0) and torch.equal(accum, accum0), rows
