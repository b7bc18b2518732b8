"""The plane wave's auxiliary line where the box is longer than the cells one wave of
its kernel owns (192 at 4 cells a lane, 448 at 8): the field inside the box in vacuum
against the same line in FP64 numpy, after the front has crossed part of the box, most
of it and all of it.

A plane wave along a grid axis is the 1-D line itself, so the box holds the line's
values up to the FP32 rounding of the 3-D fields: the repository's 1e-5 on the peak."""
import numpy as np
import pytest

from paper_2305_00234_amd import inputs as I
from tests.gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

BOX = (6, 512)  # along the propagation axis
MARKS = (380, 820, 1080)


def _line(wave, steps, courant, cells):
    E, H = np.zeros(cells + 1), np.zeros(cells + 1)
    E[0] = wave[0]
    out = []
    for n in range(steps):
        H[:-1] += courant * (E[1:] - E[:-1])
        E[1:] += courant * (H[1:] - H[:-1])
        E[0] = wave[n + 1]
        if n + 1 in MARKS:
            out.append(E.copy())
    return out


# waveform length: the line has length / 2 cells more than the box
@pytest.mark.parametrize("length", [1100, 5400, 14400])  # 4 cells a lane, 8, in memory
@pytest.mark.parametrize("axis,sign", [(2, 1), (2, -1), (0, -1)])
def test_box_longer_than_a_wave_of_the_line(axis, sign, length):
    require_gpu()
    from paper_2305_00234_amd.solver import configure
    w = I.drude_dipole_32(steps=10)
    n, lo, hi = [24, 24, 24], [6, 6, 6], [17, 17, 17]
    n[axis], lo[axis], hi[axis] = 520, BOX[0], BOX[1]
    w.shape, w.npml = tuple(n), 4
    w.mat1 = w.mat2 = (I.VACUUM,) * 3
    w.gamma = 0.0
    w.design_lo, w.rho, w.gap_lo, w.gap_dims = (9, 9, 9), np.full((3, 3, 3), 0.5, np.float32), (10, 10, 10), (1, 1, 1)
    w.source, w.pw_prop_axis, w.pw_sign, w.pw_pol_axis = "planewave", axis, sign, (axis + 1) % 3
    w.tfsf_lo, w.tfsf_hi = tuple(lo), tuple(hi)
    t = np.arange(length, dtype=np.float64)
    w.wave = np.where(t <= MARKS[-1], np.sin(0.21 * t) * np.minimum(1.0, t / 60.0), 0.0)
    # cell u of the line lies 2 cells before the box at u = 0
    z = np.arange(BOX[0] + 1, BOX[1])
    u = z - BOX[0] + 2 if sign > 0 else BOX[1] + 2 - z
    # (beyond the last mark the line carries on: 700 cells hold everything that reaches the box)
    want = _line(w.wave, MARKS[-1], w.courant, 700)
    s = configure(w)
    s.bind_torch(0)
    s.reset()
    done, errs = 0, []
    for mark, ref in zip(MARKS, want):
        s.step(mark - done)
        done = mark
        f = s.field(w.pw_pol_axis)  # [z][y][x]
        at = [11, 11, 11]
        at[2 - axis] = z
        got = np.asarray(f, np.float64)[tuple(at)]
        errs.append(float(np.abs(got - ref[u]).max()))
        assert np.abs(ref[u]).max() > 0.9
    s.close()
    say("line", "axis", axis, "sign", sign, "length", length, "largest error", errs)
    assert max(errs) <= 1e-5
