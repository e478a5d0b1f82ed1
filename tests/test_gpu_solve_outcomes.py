"""Adaptive refinement budget (refine_budget = -1) beside a captured graph: the
outcomes of eager solves and of replays reach the next solve, whichever came
last.

eta_target = 0 makes a solve with a zero right-hand side meet the target after
the direct solve, and one with any other miss it after its whole budget, so the
iterations of a solve show the budget it was given: 2 r + 2 after a solve of r
iterations, the full one after a miss.
"""
import numpy as np
import pytest

from paper_2306_14337_amd import binding, kktgen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FULL = 6


@pytest.fixture
def setup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pat, seq = kktgen.make_sequence(60, 91, 2)
    s = binding.KKTSolver(eta_target=0.0, refine_budget=-1, fgmres_max_iters=FULL)
    s.analyze(pat.n, pat.rowptr, pat.colind, seq[0][0])
    vals = torch.from_numpy(seq[1][0]).to("cuda:0")
    b = torch.from_numpy(seq[1][1]).to("cuda:0")
    zero = torch.zeros_like(b)
    gb, gx = torch.zeros_like(b), torch.zeros_like(b)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    s.graph_capture(vals, gb, gx, stream)

    def solve(rhs):
        s.solve(rhs)
        return s.report().iters  # synchronises: the outcome is on the host

    def replay(rhs):
        gb.copy_(rhs)
        torch.cuda.synchronize()
        s.graph_launch(stream)
        return s.report().iters

    s.refactor(vals)
    yield solve, replay, b, zero
    s.close()


def test_replay_does_not_hide_a_missed_target(setup):
    solve, replay, b, zero = setup
    assert solve(b) == 2            # nothing known: 2 * 0 + 2, missed
    assert replay(zero) == 0        # a replay that met the target comes last
    assert solve(b) == FULL
    assert solve(b) == FULL         # and so after its own miss


def test_every_replay_is_seen(setup):
    solve, replay, b, zero = setup
    assert replay(zero) == 0
    assert solve(zero) == 0
    assert replay(b) == FULL        # the same graph again: missed
    assert solve(b) == FULL
    assert solve(zero) == 0
    assert solve(zero) == 0
    assert solve(b) == 2            # met twice since: 2 * 0 + 2


def test_iterations_of_the_last_solve_set_the_budget(setup):
    solve, replay, b, zero = setup
    assert solve(zero) == 0
    assert replay(zero) == 0
    assert replay(zero) == 0
    assert solve(b) == 2
