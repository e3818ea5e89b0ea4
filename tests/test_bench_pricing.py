"""The benchmark prices a launch by the kernel that the library says it takes."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("kernel, collision, steps, said, unsaid", [
    (dict(kernel="plain", steps=2, launches=1), "bgk", 2, None, None),
    (dict(kernel="plain", steps=1, launches=1), "central", 1, None, None),
    (dict(kernel="sweep", steps=4, launches=1), "bgk", 4, "4.0 of 4.4 us", "workgroups"),
    (dict(kernel="sweep", steps=4, launches=1), "central", 4, "4 steps per pass", "4.0 of 4.4 us"),
    (dict(kernel="sweep", steps=2, launches=1), "bgk", 2, "2 steps per pass", "4.0 of 4.4 us"),
    (dict(kernel="resident", steps=64, launches=3), "bgk", 64, "64 steps per pass", "4.0 of 4.4 us"),
    (dict(kernel="resident", steps=20, launches=1), "central", 20, "20 steps per pass", "4.0 of 4.4 us"),
])
def test_steps_per_pass_and_note(kernel, collision, steps, said, unsaid):
    per_pass, note = bench.pass_pricing(kernel, collision)
    assert per_pass == steps
    assert (note is None) == (said is None)
    if said:
        assert said in note and unsaid not in note


@pytest.mark.gpu
@pytest.mark.parametrize("members, kernel", [(128, "sweep"), (1, "resident")])
def test_the_library_names_the_kernel_of_the_timed_batch(members, kernel):
    """The benchmark's own lattice: the full ensemble is swept, one member stays in registers."""
    import workloads
    from paper_2005_09323_amd.ensemble import Ensemble
    ens = Ensemble(workloads.ensemble_1024().members[:members], series_capacity=66)
    ens.set_tile(20)
    assert ens.batch_kernel(20)["kernel"] == kernel
    ens.close()
