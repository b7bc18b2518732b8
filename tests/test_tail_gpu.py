"""The joint launch of the design cells' update and the x layers' (ccpr_tail_kernel,
which separate-launch steps take where the two touch different words) at the
edges of its rule: bitwise the one-launch step, whose cells do not depend on it."""
import numpy as np
import pytest

from tests.gpu_util import require_gpu, say
from tests.test_whole_step_gpu import _case, _solve

pytestmark = pytest.mark.gpu


def _boxed(w, lo, hi):
    w.tfsf_lo, w.tfsf_hi = (lo,) * 3, (hi,) * 3
    return w


CASES = {
    "one column past the low layer, up to the high one": _case((37, 33, 35), lo=(6, 10, 10), design=(26, 6, 7)),
    "next to both layers": _case((37, 33, 35), lo=(5, 10, 10), design=(27, 6, 7)),
    "one cell inside the faces": _boxed(_case((37, 33, 35), source="planewave", lo=(9, 9, 9), design=(15, 15, 15)), 8, 24),
    "beside the box": _boxed(_case((40, 33, 35), source="planewave", axis=1, lo=(7, 9, 9), design=(6, 8, 8),
                                   gap_at=(20, 16, 16)), 14, 26),
    "per edge, DFT": _case((37, 33, 35), edges=True, gradient="dft", mats=2, lo=(6, 10, 10), design=(25, 6, 7)),
    "no layers": _case((30, 27, 33), npml=0, lo=(1, 9, 9), design=(20, 6, 7)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_joint_launch_is_bitwise_the_one_launch_step(name):
    require_gpu()
    w = CASES[name]
    a, b = _solve(w, 2), _solve(w, 4)
    say("joint launch", name, "F", a[0], "|grad|", float(np.abs(a[3]).max()))
    assert a[0] == b[0]
    for x, y in zip(a[1:], b[1:]):
        assert np.isfinite(x).all()
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [(130, 139, 130), (70, 201, 170)])
def test_chunk_rule_does_not_change_the_fields(n):
    """Grids whose z-chunks the rule makes fewer (three and two waves a row),
    against chunks of the nominal height."""
    require_gpu()
    from tests.gpu_util import gpu_fields_after_steps
    w = _case(n, npml=8, steps=12)
    for x, y in zip(gpu_fields_after_steps(w, 12), gpu_fields_after_steps(w, 12, tile_planes=5)):
        assert np.abs(x).max() > 0 and np.array_equal(x, y)


def test_batched_solves_by_size_and_width():
    """Served together: rows too wide for the one-launch step (batched grid, aux
    and post launches), small ones, and one above the batching limit."""
    require_gpu()
    from paper_2305_00234_amd.lib import JOB_DONE, Engine
    from paper_2305_00234_amd.solver import configure
    ws = [_case((270, 25, 24), steps=20), _case((300, 26, 25), steps=24), _case((37, 33, 35), steps=20),
          _case((130, 139, 130), npml=8, steps=8)]
    alone = [_solve(w, 2) for w in ws]
    solvers = [configure(w) for w in ws]
    eng = Engine(1 << 31, max_active=4, chunk_steps=4)
    tickets = [eng.submit(s, w.steps) for s, w in zip(solvers, ws)]
    for t, a in zip(tickets, alone):
        assert eng.wait(t) == JOB_DONE
        F, g, _ = eng.result(t)
        assert F == a[0] and np.array_equal(g, a[3])
        eng.release(t)
    eng.close()
    for s in solvers:
        s.close()


@pytest.mark.parametrize("edges", [False, True])
def test_designs_without_layers(edges):
    """No CPML: the joint launch per voxel, aux and post launches per edge."""
    require_gpu()
    w = _case((30, 27, 33), npml=0, edges=edges, lo=(1, 9, 9), design=(20, 6, 7), steps=40)
    a, b = _solve(w, 2), _solve(w, 4)
    say("no layers, edges", edges, "F", a[0])
    assert a[0] == b[0]
    for x, y in zip(a[1:], b[1:]):
        assert np.array_equal(x, y)
