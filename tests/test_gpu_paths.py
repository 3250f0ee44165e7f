"""GPU tests of launch rules and kernel paths at the sizes where they can go wrong.

Reference: the FP64 oracle's exact solves. A run at per-step tolerance 1e-12
over 15 steps accumulates at most about 15 x 1e-12 x (condition of the step
operator, < 10 here) in a signal; the tests allow 1e-9 as the parity suite
does.
"""

import numpy as np
import pytest

import dmri_inputs as di

pytestmark = pytest.mark.gpu

TOL = 1e-9
SEQ = di.Sequence(2000.0, 4000.0, 400.0, 0.5)  # 15 steps


def _pairs(n, seed=3):
    rng = np.random.default_rng(seed)
    b = rng.uniform(100.0, 4000.0, n)
    b[0] = 0.0
    q = rng.standard_normal((n, 3))
    return b, q / np.linalg.norm(q, axis=1)[:, None]


def _err(sig, ref):
    return np.max(np.abs(sig - ref) / np.maximum(np.abs(ref), 1e-8 * np.abs(ref).max()))


@pytest.fixture(scope="module")
def case():
    """A two-compartment mesh with 130 pairs and the oracle's signals."""
    from oracle import timestep
    prob = di.cylinder_box(n=6, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3)
    b, q = _pairs(130)
    return prob, b, q, timestep.signals(prob, SEQ, b, q, solver="splu")


@pytest.fixture(scope="module")
def Sim():
    from paper_1908_01719_amd import Simulator
    return Simulator


# Tile widths are powers of two from 8 to 64: each side of every step, in the
# chunked and the persistent solver.
@pytest.mark.parametrize("persistent", [0, 2])
@pytest.mark.parametrize("pairs", [1, 8, 9, 16, 17, 32, 33, 63, 64, 65])
def test_tile_rule(Sim, case, pairs, persistent):
    prob, b, q, ref = case
    with Sim(0) as sim:
        sim.set_sequence(SEQ)
        sim.set_options(rtol=1e-12, persistent=persistent)
        pid = sim.add_problem(prob)
        sig, st = sim.dmri_run([pid] * pairs, b[:pairs], q[:pairs])
    assert st["status"] == "DMRI_OK"
    assert _err(sig, ref[:pairs]) < TOL


# Finalize slices (8 or 16 systems a block) and partial counts: every tile width,
# ragged last slices, one block, several, and more partials than one round of a
# finalize block loads; FP64, and mixed precision with 128-system tiles. A rerun
# is bitwise identical (fixed summation order).
@pytest.mark.parametrize("precision,pairs,tile", [(0, 5, 8), (0, 13, 16), (0, 37, 32), (0, 67, 64),
                                                  (1, 67, 64), (1, 130, 64)])
@pytest.mark.parametrize("blocks", [None, 1, 3, 512])
def test_finalize_slices(Sim, case, precision, pairs, tile, blocks):
    prob, b, q, ref = case
    with Sim(0) as sim:
        sim.set_sequence(SEQ)
        sim.set_options(rtol=1e-12, precision=precision, sys_tile=tile, persistent=0,
                        sort_systems=0)
        if blocks:
            sim.set_options(blocks_per_xcd=blocks)
        pid = sim.add_problem(prob)
        sig, st = sim.dmri_run([pid] * pairs, b[:pairs], q[:pairs])
        again, _ = sim.dmri_run([pid] * pairs, b[:pairs], q[:pairs])
    assert st["status"] == "DMRI_OK"
    assert _err(sig, ref[:pairs]) < TOL
    assert np.array_equal(sig, again)


# The persistent solver: one element per lane (4 and 8 wavefronts a block), rows
# in memory (more rows than lanes), both exchanges (every block reading every
# word, one block per value), rows longer than the entries kept in registers,
# more than one tile, both forms, FP64 and the FP32 inner solves; repeated runs
# are bitwise identical.
@pytest.mark.parametrize("n,pairs,tile,precision", [
    (6, 1, 8, 0), (6, 13, 16, 0), (6, 13, 8, 1), (6, 64, 64, 0), (6, 33, 32, 1), (12, 20, 8, 0),
    (16, 24, 32, 0), (16, 60, 64, 1), (20, 40, 64, 0)])
@pytest.mark.parametrize("mask", [7, 0])
def test_persistent_solver(Sim, n, pairs, tile, precision, mask):
    prob = di.cylinder_box(n=n, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3, periodic_mask=mask)
    b, q = _pairs(pairs)
    seq = di.Sequence(1000.0, 1000.0, 200.0, 0.5)
    out = []
    with Sim(0) as sim:
        sim.set_sequence(seq)
        pid = sim.add_problem(prob)
        # the chunked solver (checked against the oracle by test_finalize_slices)
        for persistent in (0, 1, 1):
            sim.set_options(rtol=1e-12, persistent=persistent, sys_tile=tile, precision=precision,
                            sort_systems=0)
            sig, st = sim.dmri_run([pid] * pairs, b, q)
            assert st["status"] == "DMRI_OK"
            out.append(sig)
    assert _err(out[1], out[0]) < TOL
    assert np.array_equal(out[1], out[2])


# Row slots: tiles of up to 32 systems take one per wavefront and chunk, wider
# ones two. Row counts with ragged last chunks, in one block and in many.
@pytest.mark.parametrize("n", [3, 4, 7])
@pytest.mark.parametrize("pairs,tile", [(3, 8), (16, 16), (20, 32), (40, 64)])
@pytest.mark.parametrize("blocks", [1, 512])
def test_row_slots(Sim, n, pairs, tile, blocks):
    from oracle import timestep
    prob = di.cylinder_box(n=n, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3)
    b, q = _pairs(pairs)
    seq = di.Sequence(1000.0, 1000.0, 200.0, 0.5)
    ref = timestep.signals(prob, seq, b, q, solver="splu")
    with Sim(0) as sim:
        sim.set_sequence(seq)
        sim.set_options(rtol=1e-12, sys_tile=tile, persistent=0, blocks_per_xcd=blocks)
        pid = sim.add_problem(prob)
        sig, st = sim.dmri_run([pid] * pairs, b, q)
    assert st["status"] == "DMRI_OK"
    assert _err(sig, ref) < TOL


# COCG (the U-form) in paired tiles keeps FP32 directions whatever dir_bf16 says.
@pytest.mark.parametrize("pairs", [65, 130])
def test_cocg_directions(Sim, pairs):
    from oracle import timestep
    prob = di.cylinder_box(n=6, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3, periodic_mask=0)
    b, q = _pairs(pairs)
    seq = di.Sequence(1000.0, 1000.0, 200.0, 0.5)
    ref = timestep.signals(prob, seq, b, q, solver="splu")
    out = []
    with Sim(0) as sim:
        sim.set_sequence(seq)
        pid = sim.add_problem(prob)
        for d in (0, 1):
            sim.set_options(rtol=1e-12, precision=1, persistent=0, sort_systems=0, dir_bf16=d)
            sig, st = sim.dmri_run([pid] * pairs, b, q)
            assert st["status"] == "DMRI_OK"
            assert _err(sig, ref) < TOL
            out.append(sig)
    assert np.array_equal(out[0], out[1])


# Persistent solves of several handles at once, of both block sizes (256 threads,
# two blocks a CU; 512) and of block counts that do not divide among the XCDs:
# the same signals as one after the other.
def test_persistent_solves_in_threads(Sim):
    import threading
    seq = di.Sequence(1000.0, 1000.0, 100.0, 0.5)
    sims, args, ref = [], [], []
    for n, pairs in ((10, 3), (14, 13), (18, 16), (10, 5), (20, 40), (14, 11)):
        sim = Sim(0)
        sim.set_sequence(seq)
        sim.set_options(rtol=1e-12, persistent=1)
        pid = sim.add_problem(di.cylinder_box(n=n, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3))
        sims.append(sim)
        args.append(([pid] * pairs, *_pairs(pairs)))
        ref.append(sim.dmri_run(*args[-1])[0])
    got = [[] for _ in sims]

    def run(k):
        for _ in range(3):
            got[k].append(sims[k].dmri_run(*args[k])[0])

    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(sims))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for sim in sims:
        sim.close()
    for k in range(len(sims)):
        assert len(got[k]) == 3
        for sig in got[k]:
            assert np.array_equal(sig, ref[k])


# GMRES's kernels take four row slots per wavefront and chunk whatever the tile:
# row counts with ragged last chunks, one block and many, several tiles.
@pytest.mark.parametrize("n", [3, 4, 7])
@pytest.mark.parametrize("pairs,tile", [(3, 8), (20, 16), (20, 32), (40, 64)])
@pytest.mark.parametrize("blocks", [1, 512])
def test_gmres_row_slots(Sim, n, pairs, tile, blocks):
    from oracle import timestep
    prob = di.cylinder_box(n=n, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3)
    b, q = _pairs(pairs)
    seq = di.Sequence(1000.0, 1000.0, 200.0, 0.5)
    ref = timestep.signals(prob, seq, b, q, solver="splu")
    with Sim(0) as sim:
        sim.set_sequence(seq)
        sim.set_options(rtol=1e-12, krylov=3, sys_tile=tile, blocks_per_xcd=blocks)
        pid = sim.add_problem(prob)
        sig, st = sim.dmri_run([pid] * pairs, b, q)
    assert st["status"] == "DMRI_OK"
    assert _err(sig, ref) < TOL


# Option blocks_per_xcd reads back as a value that means the same when it is set:
# writing it back changes nothing, and another value changes the launches.
def test_blocks_option_round_trip(Sim):
    prob = di.cylinder_box(n=24, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3)
    b, q = _pairs(40)
    with Sim(0) as sim:
        sim.set_sequence(di.Sequence(1000.0, 1000.0, 200.0, 0.5))
        sim.set_options(rtol=1e-10, persistent=0, n_steps=3, signal=0, sort_systems=0)
        pid = sim.add_problem(prob)
        out = []
        for blocks in (None, sim.dmri_get_option("blocks_per_xcd"), 300):
            if blocks:
                sim.set_options(blocks_per_xcd=blocks)
                assert sim.dmri_get_option("blocks_per_xcd") == blocks
            out.append(sim.dmri_run([pid] * 40, b, q)[0])
    assert np.array_equal(out[0], out[1])
    assert not np.array_equal(out[0], out[2])  # sums of 300 blocks round differently
    assert _err(out[2], out[0]) < TOL


# The persistent solver's remaining kernels (elements per lane in 512-thread
# blocks, rows in memory with either exchange; tests/rules/rules_driver.cpp holds
# the table) and that it is what runs: one Krylov launch a step.
@pytest.mark.parametrize("n,pairs,tile", [(6, 13, 16), (20, 8, 8), (18, 16, 16), (18, 13, 8),
                                          (18, 20, 8), (26, 5, 8), (20, 40, 64)])
@pytest.mark.parametrize("mask", [7, 0])
def test_persistent_kernels_run(Sim, n, pairs, tile, mask):
    prob = di.cylinder_box(n=n, half=6.0, r=4.0, kappa=1e-3, D_in=1e-3, periodic_mask=mask)
    b, q = _pairs(pairs)
    out, launches = [], []
    with Sim(0) as sim:
        sim.set_sequence(di.Sequence(1000.0, 1000.0, 200.0, 0.5))
        pid = sim.add_problem(prob)
        for persistent in (0, 1):
            sim.set_options(rtol=1e-12, persistent=persistent, sys_tile=tile, sort_systems=0,
                            time_kernel=1)
            sig, st = sim.dmri_run([pid] * pairs, b, q)
            assert st["status"] == "DMRI_OK"
            out.append(sig)
            launches.append((st["n_kernel_launches"], st["n_steps"]))
    assert _err(out[1], out[0]) < TOL
    assert launches[1][0] == launches[1][1]
    assert launches[0][0] > 4 * launches[0][1]


# COCG's inner solves of mixed precision near a breakdown of the bilinear form
# (walls; the residual grows past what FP32 can take back): the step is taken
# back and the refinement goes on, so runs end converged and with the FP64
# solver's signals. Both solve each of 4 steps to 1e-10; 1e-8 allowed. Paired
# tiles, 64-system tiles, narrow tiles, the persistent solver; seeds in which
# such solves occurred.
@pytest.mark.parametrize("n,pairs,opts", [
    (16, 128, {}), (12, 100, {}), (20, 198, {}), (16, 128, dict(pair_lanes=0)),
    (12, 100, dict(pair_lanes=0)), (12, 40, {}), (12, 40, dict(persistent=1)),
    (16, 16, dict(persistent=1)), (10, 5, dict(persistent=1))])
def test_cocg_inner_breakdown(Sim, n, pairs, opts):
    prob = di.cylinder_box(n=n, half=6.0, r=4.0, kappa=1e-4, periodic_mask=0)
    with Sim(0) as sim:
        sim.set_sequence(di.Sequence(2000.0, 3000.0, 250.0, 0.5))
        pid = sim.add_problem(prob)
        for seed in range(1, 7):
            rng = np.random.default_rng(seed)
            b = rng.uniform(0.05, 1.0, pairs) * 4000.0
            b[::7] = 0.0
            q = rng.standard_normal((pairs, 3))
            q /= np.linalg.norm(q, axis=1)[:, None]
            sim.set_options(rtol=1e-10, n_steps=4, signal=0, precision=0, persistent=0, guess=1)
            ref, st = sim.dmri_run([pid] * pairs, b, q)
            assert st["status"] == "DMRI_OK"
            for guess in (0, 1):
                sim.set_options(precision=1, guess=guess, **opts)
                sig, st = sim.dmri_run([pid] * pairs, b, q)
                assert st["status"] == "DMRI_OK", (seed, guess)
                assert np.abs(sig - ref).max() < 1e-8 * np.abs(ref).max(), (seed, guess)
