"""The separate launches of a step with two rows a thread (grid pass, aux, post or
their joint launch; what every larger grid runs) on the small problems that run as
one launch by default: naming a tile height selects them.  Against the one-launch
step bit for bit, and against the FP64 oracle at the bars of the other parity tests
(fields and objective 1e-5, gradient 1e-3)."""
import numpy as np
import pytest

from paper_2305_00234_amd import inputs as I
from tests.gpu_util import (field_errors, gpu_fields_after_steps, gpu_gradient, oracle_fields_after_steps, oracle_gradient,
                            rel_l2, require_gpu, say)
from tests.test_random_configs_gpu import PW_SEEDS, random_case, random_planewave_case
from tests.test_whole_step_gpu import CASES, _case

pytestmark = pytest.mark.gpu


def _flat(g):
    return np.concatenate([np.ravel(x) for x in g]) if isinstance(g, tuple) else np.ravel(g)


def _solve(w, planes=None, checkpoint=None, resident=None):
    from paper_2305_00234_amd.solver import configure
    s = configure(w)
    if planes:
        s.set_tile_planes(planes)
    if checkpoint:
        s.set_checkpointing(checkpoint)
    if resident:
        s.set_resident_segments(resident)
    s.bind_torch(w.steps)
    F = s.forward(w.steps)
    fwd = np.stack([s.field(c) for c in range(6)])
    s.adjoint()
    adj = np.stack([s.field(c) for c in range(6)])
    g, one = _flat(s.gradient()), s.info()["one_launch"]
    s.close()
    return F, fwd, adj, g, one


@pytest.mark.parametrize("planes", [3, 16])
@pytest.mark.parametrize("name", sorted(CASES))
def test_two_row_launches_are_bitwise_the_one_launch_step(name, planes):
    require_gpu()
    w = CASES[name]
    a, b = _solve(w), _solve(w, planes)
    say("two-row launches", name, planes, "F", a[0], b[0])
    assert a[4] == 1 and b[4] == 0
    assert a[0] == b[0] and a[0] > 0
    for x, y in zip(a[1:4], b[1:4]):
        assert np.abs(x).max() > 0 and np.array_equal(x, y)


@pytest.mark.parametrize("seed", range(8))
def test_two_row_launches_match_oracle(seed):
    require_gpu()
    w = random_case(seed + 400)
    F, g, _, _, info = gpu_gradient(w, tile_planes=4)
    Fo, go, _, _ = oracle_gradient(w)
    err = rel_l2(_flat(g), _flat(go))
    say("two-row launches", seed, w.shape, "npml", w.npml, w.objective, "F", F, Fo, "grad", err)
    assert info["one_launch"] == 0
    assert Fo > 0 and abs(F - Fo) <= 1e-5 * abs(Fo)
    assert err <= 1e-3


@pytest.mark.parametrize("seed", PW_SEEDS[:4])
def test_two_row_launches_match_oracle_planewave(seed):
    require_gpu()
    w = random_planewave_case(seed)
    F, g, _, _, info = gpu_gradient(w, tile_planes=6)
    Fo, go, _, _ = oracle_gradient(w)
    err = rel_l2(_flat(g), _flat(go))
    say("two-row launches, plane wave", seed, w.shape, w.gradient, "F", F, Fo, "grad", err)
    assert info["one_launch"] == 0
    assert Fo > 0 and abs(F - Fo) <= 1e-5 * abs(Fo)
    assert err <= 1e-3


def test_two_row_launches_kappa_fields_match_oracle():
    """kappa-graded layers: the y / z layers of the grid kernel, the x layers of the
    launches before and after it."""
    require_gpu()
    w = I.drude_dipole_32(steps=150)
    w.shape, w.npml, w.pml_kappa_max = (70, 37, 35), 6, 5.0
    w.design_lo, w.rho = (20, 14, 13), np.random.default_rng(3).random((7, 6, 9)).astype(np.float32)
    w.dipole_cell, w.gap_lo, w.gap_dims = (15, 17, 16), (22, 16, 15), (2, 2, 2)
    g = gpu_fields_after_steps(w, 150, tile_planes=5)
    st, eE, eH = field_errors(g, oracle_fields_after_steps(w, 150))
    say("two-row launches, kappa", w.shape, "rel L2 state", st, "E", eE, "H", eH)
    assert st <= 1e-5


@pytest.mark.parametrize("seed", range(3))
def test_two_row_launches_segmented(seed):
    """Checkpoint and recompute: objective and gradient bit for bit those of the
    whole history and of the one-launch step."""
    require_gpu()
    w = random_case(seed + 500)
    w.objective, w.window = "time", (5, -1)
    ref = _solve(w)
    got = _solve(w, 5, checkpoint=w.steps // 4, resident=1)
    say("two-row launches, segments", seed, w.shape, "F", ref[0], got[0])
    assert (ref[4], got[4]) == (1, 0)
    assert ref[0] == got[0] and np.array_equal(ref[3], got[3])


def test_named_tile_height_in_a_served_batch():
    """Served together: one-launch solves and one whose tile height is named (same
    padded width) give bitwise their results alone."""
    require_gpu()
    from paper_2305_00234_amd.lib import JOB_DONE, Engine
    from paper_2305_00234_amd.solver import configure
    names = ("full waves", "one wave per row, ragged rows", "gap outside the design")
    alone = [_solve(CASES[n]) for n in names]
    solvers = [configure(CASES[n]) for n in names]
    solvers[1].set_tile_planes(5)
    eng = Engine(1 << 30, max_active=3, chunk_steps=8)
    tickets = [eng.submit(s, CASES[n].steps) for s, n in zip(solvers, names)]
    for t, a in zip(tickets, alone):
        assert eng.wait(t) == JOB_DONE
        F, g, _ = eng.result(t)
        assert F == a[0] and np.array_equal(_flat(g), a[3])
        eng.release(t)
    eng.close()
    for s in solvers:
        s.close()


def test_served_solves_on_both_sides_of_the_batching_line():
    """0.2 M padded cells: rows too wide for the one-launch step batched as grid, aux and
    post launches (three of one width), small one-launch solves batched, and solves just
    above the line on streams of their own; bitwise their results alone."""
    require_gpu()
    from paper_2305_00234_amd.lib import JOB_DONE, Engine
    from paper_2305_00234_amd.solver import configure
    ws = [_case((270, 25, 24), steps=20), _case((290, 24, 25), steps=24), _case((264, 20, 30), npml=4, steps=22),
          _case((300, 26, 25), steps=18), _case((60, 55, 56), steps=26), _case((60, 56, 56), steps=20),
          _case((62, 57, 56), mats=2, steps=20), _case((64, 64, 64), npml=0, steps=20)]
    alone = [_solve(w) for w in ws]
    assert [a[4] for a in alone] == [0, 0, 0, 0, 1, 1, 1, 1]
    solvers = [configure(w) for w in ws]
    eng = Engine(2 << 30, max_active=8, chunk_steps=8)
    tickets = [eng.submit(s, w.steps) for s, w in zip(solvers, ws)]
    for t, a in zip(tickets, alone):
        assert eng.wait(t) == JOB_DONE
        F, g, _ = eng.result(t)
        assert F == a[0] and np.array_equal(_flat(g), a[3])
        eng.release(t)
    eng.close()
    for s in solvers:
        s.close()
