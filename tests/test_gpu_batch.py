"""Batches of independent problems (mvpf_create_batch): lockstep FGMRES with
the V-cycles of all problems in one captured HIP graph, one launch per
V-cycle operator for all problems.

* Every problem's result is bitwise the one of solving it alone under the
  same tuning (same kernels in the same order), on every replay of the graph, with eager work on the
  same stream between the replays.
* A rotated-crystal problem of the batch matches the oracle (right-hand side
  <= 1e-12, increment at rtol 1e-12 vs the oracle's direct solve <= 1e-9)."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import OracleCase, check_entries, rel, say, seeded_state

pytestmark = pytest.mark.gpu


def small_batch():
    """The batched workload's recipe (own size, rotation, seed and depth per
    problem) at sizes the oracle handles: 8^3 / 16^3 / 8^3 with 3, 4 and 2
    levels."""
    out = []
    for i, (n, levels) in enumerate([(8, 3), (16, 4), (8, 2)]):
        s = synth.BASE_SEED + 100 + i
        Q = synth.random_rotation(s)
        out.append(synth.Problem(n, n, n, n_levels=levels, patch=2, depth_increment=0.005 + 0.005 * i, seed=s,
                                 material=synth.config_material(Q=tuple(Q.ravel()))))
    return out


def _state(gp):
    u, e, en, d = gp.get_state()
    return np.concatenate([u.cpu().numpy(), e.cpu().numpy()], 1)


def test_batch_bitwise_long_arnoldi_cycles():
    """A weak smoother (V(1,1), damping 0.3) and rtol 1e-11 make every
    problem take many FGMRES iterations (at least one more than 30), so the Arnoldi steps reach
    all register tiers of the single-problem Gram-Schmidt kernels (basis sizes
    up to 31, the first pass's update fused with the second pass's
    projections) and a restart: the batched solve, which keeps the separate
    passes, gives bitwise the same states and iteration counts."""
    from paper_2011_08802_amd import mvpf
    probs = small_batch()
    states = [seeded_state(p, 1e-3) for p in probs]
    opts = dict(nu_pre=1, nu_post=1, omega=0.3, rtol=1e-11)
    B = mvpf.Batch(probs, "mixed", **opts)
    say("[batch long cycles] single-problem references")
    ref = []
    for i, (p, (U, En)) in enumerate(zip(probs, states)):
        gp = mvpf.Problem(p, "mixed", **opts)
        gp.set_tuning("small_grid_nodes", 0, B.problem(i).get_tuning("small_grid_nodes"))
        gp.set_state(U[:, :3], U[:, 3:], En, 0.0)
        gp.newton_system(p.depth_increment)
        _, st = gp.solve(want_x=False)
        gp.newton_update()
        say(f"    problem {i}: {st.iterations} FGMRES iterations, {st.restarts} restarts")
        ref.append((_state(gp), st.iterations))
        gp.close()
    assert max(r[1] for r in ref) > 30
    for i, (U, En) in enumerate(states):
        B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
    B.newton_system([p.depth_increment for p in probs])
    stats = B.solve()
    B.newton_update()
    for i in range(len(probs)):
        assert stats[i].converged and stats[i].iterations == ref[i][1], (i, stats[i].iterations, ref[i][1])
        assert np.array_equal(_state(B.problem(i)), ref[i][0]), i
    B.close()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_batch_bitwise_equals_single_solves(precision):
    from paper_2011_08802_amd import mvpf
    probs = small_batch()
    states = [seeded_state(p, 1e-3) for p in probs]
    B = mvpf.Batch(probs, precision)
    say(f"[batch {precision}] single-problem references (the batch's tuning)")
    ref = []
    for i, (p, (U, En)) in enumerate(zip(probs, states)):
        gp = mvpf.Problem(p, precision)
        gp.set_tuning("small_grid_nodes", 0, B.problem(i).get_tuning("small_grid_nodes"))
        gp.set_state(U[:, :3], U[:, 3:], En, 0.0)
        gp.newton_system(p.depth_increment)
        _, st = gp.solve(want_x=False)
        gp.newton_update()
        ref.append((_state(gp), st.iterations))
        gp.close()
    x = torch.randn(9 * probs[0].n_nodes, dtype=torch.float64, device="cuda")
    for replay in range(3):
        say(f"[batch {precision}] replay {replay}")
        for i, (U, En) in enumerate(states):
            B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
        B.newton_system([p.depth_increment for p in probs])
        stats = B.solve()
        B.newton_update()
        for i in range(len(probs)):
            assert stats[i].converged and stats[i].iterations == ref[i][1], (i, stats[i].iterations, ref[i][1])
            assert np.array_equal(_state(B.problem(i)), ref[i][0]), i
        # eager work on the same stream between replays
        B.problem(0).newton_system(probs[0].depth_increment)
        B.problem(0).jacobian_apply(0, x)
        B.problem(0).solve(want_x=False)
    B.close()


def test_batch_problem_matches_oracle():
    from paper_2011_08802_amd import mvpf
    probs = small_batch()
    states = [seeded_state(p, 5e-4) for p in probs]
    B = mvpf.Batch(probs, "mixed", rtol=1e-12)
    for i, (U, En) in enumerate(states):
        B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
    B.newton_system([p.depth_increment for p in probs])
    stats = B.solve()
    i = 0  # 8^3, rotated card
    p = probs[i]
    U, En = states[i]
    say("[batch oracle] oracle system + direct solve")
    oc = OracleCase(p, U, En, p.depth_increment, build_mg=False)
    b = B.problem(i).get_rhs().cpu().numpy()
    check_entries(b, oc.sys.b, 1e-12, "rhs", oc.abs_scales()[1])
    assert stats[i].converged and stats[i].rel_residual <= 1e-12
    B.newton_update()
    dx = _state(B.problem(i)) - U
    assert rel(dx, oc.x) <= 1e-9, rel(dx, oc.x)
    B.close()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_batch_contact_and_assembled_finest_bitwise(precision):
    """A batch mixing a sphere-contact problem (its contact terms are
    per-problem launches inside the batched chains), a problem on the
    assembled finest level (tuning matrix_free = 0: half-stencil sweeps and
    operator product) and a matrix-free patch problem tuned to 16 elements per
    workgroup (the largest problem, so the batched element launches take 16
    elements per workgroup): every problem bitwise as solved alone under the
    same tuning, on two replays."""
    from paper_2011_08802_amd import mvpf
    sb = small_batch()
    probs = [synth.Problem(8, 8, 4, lz=0.5, n_levels=3, kind="sphere", radius=0.5, seed=synth.BASE_SEED + 7),
             sb[0], sb[1]]
    depths = [0.03, sb[0].depth_increment, sb[1].depth_increment]
    states = [seeded_state(p, 1e-3) for p in probs]
    B = mvpf.Batch(probs, precision)
    B.problem(2).set_tuning("matrix_free", 0, 0)
    B.problem(1).set_tuning("mf_elements_per_block", 0, 16)  # the largest problem: sets the batch's launches
    say(f"[batch mixed kinds {precision}] single-problem references")
    ref = []
    for i, (p, (U, En)) in enumerate(zip(probs, states)):
        gp = mvpf.Problem(p, precision)
        for key in ("small_grid_nodes", "matrix_free", "mf_elements_per_block"):
            gp.set_tuning(key, 0, B.problem(i).get_tuning(key))
        gp.set_state(U[:, :3], U[:, 3:], En, 0.0)
        gp.newton_system(depths[i])
        _, st = gp.solve(want_x=False)
        gp.newton_update()
        ref.append((_state(gp), st.iterations))
        gp.close()
    for replay in range(2):
        say(f"[batch mixed kinds {precision}] replay {replay}")
        for i, (U, En) in enumerate(states):
            B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
        B.newton_system(depths)
        stats = B.solve()
        B.newton_update()
        for i in range(len(probs)):
            assert stats[i].converged and stats[i].iterations == ref[i][1], (i, stats[i].iterations, ref[i][1])
            assert np.array_equal(_state(B.problem(i)), ref[i][0]), i
    B.close()


@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_batch_bitwise_cycles_beyond_the_register_kernels(precision):
    """A Krylov space of 64 and a weak smoother: the Arnoldi steps pass the 32
    basis vectors up to which the Gram-Schmidt kernels keep a row's entries in
    registers (single solves and batches alike), so updates and projections
    go through the separate kernels, grouped by eight vectors.  The batch is
    bitwise the single solves, whose residuals are the true FP64 ones."""
    from paper_2011_08802_amd import mvpf
    probs = small_batch()[:3]
    states = [seeded_state(p, 1e-3) for p in probs]
    opts = dict(nu_pre=1, nu_post=1, omega=0.3, rtol=1e-11, restart=64)
    ref = []
    for p, (U, En) in zip(probs, states):
        gp = mvpf.Problem(p, precision, **opts)
        gp.set_state(U[:, :3], U[:, 3:], En, 0.0)
        gp.newton_system(p.depth_increment)
        _, st = gp.solve(want_x=False)
        assert st.converged and st.rel_residual <= 1e-11 and st.iterations > 33, st.iterations
        gp.newton_update()
        ref.append((_state(gp), st.iterations))
        gp.close()
    B = mvpf.Batch(probs, precision, **opts)
    for i, (U, En) in enumerate(states):
        B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
    B.newton_system([p.depth_increment for p in probs])
    stats = B.solve()
    B.newton_update()
    for i in range(len(probs)):
        assert stats[i].converged and stats[i].iterations == ref[i][1], (i, stats[i].iterations, ref[i][1])
        assert np.array_equal(_state(B.problem(i)), ref[i][0]), i
    B.close()
