"""Kernels at the sizes where their tiles, ranges and remainders change, against
plain FP64 products."""
from __future__ import annotations

import ctypes

import pytest
import torch

import paper_2211_07894_amd as L
from paper_2211_07894_amd import lrdm as B

pytestmark = pytest.mark.gpu


def _grid(n):
    return L.Grid(n, tuple(0.43 * x for x in n))


def _rand(gen, *shape, dtype=torch.float64):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def _gen(seed):
    g = torch.Generator("cuda")
    g.manual_seed(seed)
    return g


def _rel(a, b):
    return float((a - b).norm() / b.norm())


# an FP64 sum of M products is off by at most M u of its terms' absolute sum; for
# random terms that sum is about sqrt(M) times the result, so M^1.5 u bounds it
@pytest.mark.parametrize("n,N,nspin,r", [
    ((16, 16, 16), 16, 1, 1), ((5, 7, 9), 31, 2, 1), ((24, 24, 24), 32, 1, 4),
    ((9, 11, 13), 33, 1, 2), ((8, 8, 3), 64, 1, 1), ((27, 33, 35), 65, 2, 1),
    ((20, 21, 22), 384, 1, 1), ((20, 21, 22), 385, 1, 1), ((30, 30, 31), 130, 1, 3),
    ((48, 48, 16), 256, 1, 9),
])
def test_projection_fp64(n, N, nspin, r):
    grid, gen = _grid(n), _gen(N + r)
    P = _rand(gen, nspin, N, grid.M)
    dV = _rand(gen, r, nspin, grid.M)
    H = L.projected_perturbation(grid, P, dV, nspin, "fp64")
    bound = grid.M ** 1.5 * 2.0 ** -53
    for k in range(r):
        for c in range(nspin):
            ref = (P[c] * dV[k, c]) @ P[c].t()
            assert _rel(H[k, c], ref) < bound
            assert torch.equal(H[k, c], H[k, c].t())


def test_projection_under_a_workspace_limit():
    """A context too small for the preferred partial sums still takes the call."""
    n, N, r = (24, 24, 24), 90, 2
    grid, gen = _grid(n), _gen(5)
    P, dV = _rand(gen, 1, N, grid.M), _rand(gen, r, 1, grid.M)
    free = L.projected_perturbation(grid, P, dV, 1, "fp64")
    tile = 128 * 128 * 8                       # 2 directions, at most 6 ranges of one tile
    ctx = B.Context(0, torch.cuda.current_stream().cuda_stream, 2 * 6 * tile + (1 << 20))
    H = torch.empty_like(free)
    g = grid.c()
    ctx.check(ctx.lib.lrdm_projected_perturbation(
        ctx.ptr, ctypes.byref(g), ctypes.c_void_p(P.data_ptr()), N, 1,
        ctypes.c_void_p(dV.data_ptr()), r, 0, ctypes.c_void_p(H.data_ptr())))
    torch.cuda.synchronize()
    assert ctx.workspace_bytes <= 2 * 6 * tile + (1 << 20)
    assert _rel(H, free) < grid.M ** 1.5 * 2.0 ** -53
    ctx.close()
