"""GPU tests of the no-allocation entry point at its 64 MiB of scratch.

Reference: the device entry point on the same handle. Both solve each of a few
steps to 1e-12, so signals agree to about steps x 1e-12 x (condition of the
step operator, < 10); the tests allow 1e-9.
"""

import numpy as np
import pytest

import dmri_inputs as di

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SEQ = di.Sequence(1000.0, 1000.0, 200.0, 0.5)


def _arrays(pid, pairs):
    rng = np.random.default_rng(5)
    b = rng.uniform(100.0, 4000.0, pairs)
    q = rng.standard_normal((pairs, 3))
    q /= np.linalg.norm(q, axis=1)[:, None]
    return (torch.full((pairs,), pid, dtype=torch.int32, device="cuda"),
            torch.from_numpy(b).cuda(), torch.from_numpy(q).cuda(),
            torch.zeros((pairs, 2), dtype=torch.float64, device="cuda"))


@pytest.fixture(scope="module")
def Sim():
    from paper_1908_01719_amd import Simulator
    return Simulator


# 7,128 rows x 64 systems leave 0.4 MB of the 64 MiB: the solver's exchange finds
# room only with fewer blocks of the step start. 7,200 rows are refused.
def test_just_under_and_over(Sim):
    with Sim(0) as sim:
        sim.set_sequence(SEQ)
        sim.set_options(rtol=1e-12)
        for r, rows in ((4.5, 7128), (5.4, 7200)):
            pid = sim.add_problem(di.cylinder_box(n=18, half=6.0, r=r, kappa=1e-3, D_in=1e-3))
            assert sim.dmri_problem_info(pid)[0] == rows
            ids, b, q, sig = _arrays(pid, 64)
            sim.dmri_run_device(ids, b, q, sig)
            ref = sig.cpu().numpy().copy()
            sig.zero_()
            if rows == 7200:
                with pytest.raises(Exception, match="DMRI_E_INVALID.*scratch"):
                    sim.dmri_run_device_noalloc(ids, b, q, sig)
                continue
            for _ in range(2):
                st = sim.dmri_run_device_noalloc(ids, b, q, sig)
                assert st["status"] == "DMRI_OK"
                got = sig.cpu().numpy()
                assert np.abs(got - ref).max() < 1e-9 * np.abs(ref).max()


# A mesh whose tile no persistent solver could address (128^3 rows x 64 systems x
# 16 B = 2^31) is refused for its scratch, like every other that is too large.
def test_far_over(Sim):
    with Sim(0) as sim:
        sim.set_sequence(SEQ)
        pid = sim.add_problem(di.free_box(n=128))
        sim.set_options(rtol=1e-3, n_steps=1, sys_tile=8, signal=0)
        ids, b, q, sig = _arrays(pid, 1)
        sim.dmri_run_device(ids, b, q, sig)
        sim.set_options(sys_tile=64)
        with pytest.raises(Exception, match="DMRI_E_INVALID.*scratch"):
            sim.dmri_run_device_noalloc(ids, b, q, sig)
