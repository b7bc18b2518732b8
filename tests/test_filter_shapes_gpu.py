"""The filter's two kernels (one output a thread in 16 x 16 tiles, 4 or 8 in 32 x 32
ones) on both sides of the rule that chooses between them, against the FP64 oracle:
long thin grids, half-empty tiles, the smallest spheres, full tiles.

Tolerance as for the tiles' edges: sums of at most some thousand positive FP32
products lose below 1e-5 of the result (random walk of n roundings of 2^-24: 3e-6 at
n = 3000); the chain rule sums in FP64 from FP32 weights and filtered values."""
import numpy as np
import pytest

from oracle import filters as OF
from tests.gpu_util import rel_l2, require_gpu, say

pytestmark = pytest.mark.gpu

TOL = 1e-5


# [nz][ny][nx], radius; the kernel of the forward filter and of the chain rule
@pytest.mark.parametrize("shape,R", [
    ((90, 129, 130), 3.2),   # 32 x 32 both, tiles inside the box along x
    ((300, 40, 40), 9.0),    # 32 x 32 both, large sphere in a small box
    ((1100, 33, 17), 2.5),   # 32 x 32 both (two of three 16-row tiles filled)
    ((110, 35, 101), 1.5),   # 16 x 16 forward, 32 x 32 chain rule (4 outputs a thread)
    ((800, 34, 33), 1.8),    # 16 x 16 both: small sphere, half-empty tiles
    ((1100, 10, 9), 4.2),    # 16 x 16 both: empty tiles
    ((2000, 20, 20), 1.2),   # 16 x 16 forward: smallest sphere
])
def test_voxel_shapes_match_oracle(shape, R):
    torch = require_gpu()
    from paper_2305_00234_amd.lib import filter_project, filter_project_grad
    rng = np.random.default_rng(15)
    rho, g_b, beta, eta = rng.random(shape).astype(np.float32), rng.standard_normal(shape), 8.0, 0.45
    rt, rb, ws = filter_project(torch.tensor(rho, device="cuda"), R, beta, eta)
    g = filter_project_grad(torch.tensor(g_b, device="cuda"), rt, ws, R, beta, eta).cpu().numpy()
    rt, rb, ws = rt.cpu().numpy(), rb.cpu().numpy(), ws.cpu().numpy()
    errs = (rel_l2(rt, OF.cone_filter(rho.astype(np.float64), R)),
            rel_l2(rb, OF.project(rt.astype(np.float64), beta, eta)), rel_l2(ws, OF.weight_sums(shape, R)),
            rel_l2(g, OF.filter_project_grad(g_b, rho.astype(np.float64), R, beta, eta)))
    say("voxel shapes", shape, R, errs)
    assert max(errs) <= TOL


# (x, y, z) cells
@pytest.mark.parametrize("dims,R", [
    ((70, 40, 100), 2.2),   # 32 x 32 both, two planes a workgroup in the chain rule
    ((8, 8, 450), 1.3),     # 16 x 16 both: empty tiles
    ((4, 3, 900), 6.0),     # 16 x 16 both, sphere wider than the box
    ((14, 100, 140), 1.5),  # 16 x 16 both: small sphere, half-empty tiles
    ((14, 100, 90), 2.1),   # 16 x 16 forward, 32 x 32 chain rule
    ((16, 40, 300), 1.6),   # 32 x 32 both, one column past a tile of 16
])
def test_edge_shapes_match_oracle(dims, R):
    torch = require_gpu()
    from paper_2305_00234_amd.lib import filter_project_edges, filter_project_grad_edges
    rng = np.random.default_rng(16)
    sh = [OF.edge_shape(dims, c) for c in range(3)]
    rho = [rng.random(s).astype(np.float32) for s in sh]
    g_b = [rng.standard_normal(s) for s in sh]
    beta, eta = 8.0, 0.45

    def flat(parts):
        return np.concatenate([p.ravel() for p in parts])

    rt, rb, ws = filter_project_edges(torch.tensor(flat(rho), device="cuda"), dims, R, beta, eta)
    g = filter_project_grad_edges(torch.tensor(flat(g_b), device="cuda"), rt, ws, dims, R, beta, eta).cpu().numpy()
    rt, rb, ws = rt.cpu().numpy(), rb.cpu().numpy(), ws.cpu().numpy()
    r64 = [r.astype(np.float64) for r in rho]
    errs = (rel_l2(rt, flat(OF.cone_filter_edges(r64, dims, R))),
            rel_l2(rb, OF.project(rt.astype(np.float64), beta, eta)),
            rel_l2(ws, flat(OF.edge_weight_sums(dims, R))),
            rel_l2(g, flat(OF.filter_project_grad_edges(g_b, r64, dims, R, beta, eta))))
    say("edge shapes", dims, R, errs)
    assert max(errs) <= TOL
