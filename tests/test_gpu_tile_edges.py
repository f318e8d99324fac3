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


# ranges and parts of ranges at both sides of their lines; a sum of 128 (BF16X3, pieces
# of 2^-24) or 32 products in FP32 under a FP64 sum is off by at most that many roundings
# of its terms' absolute sum, again about sqrt(M) times the result
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("n,N,nspin,r", [
    ((8, 8, 8), 16, 1, 1), ((16, 16, 16), 64, 2, 1), ((24, 24, 24), 32, 1, 4),
    ((25, 24, 23), 65, 1, 2), ((27, 33, 35), 90, 2, 1), ((48, 48, 16), 256, 1, 9),
    ((40, 40, 40), 129, 1, 1),
])
def test_projection_fp32(prec, n, N, nspin, r):
    grid, gen = _grid(n), _gen(N + r)
    P = _rand(gen, nspin, N, grid.M, dtype=torch.float32)
    dV = _rand(gen, r, nspin, grid.M)
    H = L.projected_perturbation(grid, P, dV, nspin, prec)
    bound = (32 if prec == "fp32" else 128) * grid.M ** 0.5 * 2.0 ** -24
    for k in range(r):
        for c in range(nspin):
            ref = (P[c].double() * dV[k, c]) @ P[c].double().t()
            assert _rel(H[k, c], ref) < bound
            assert torch.equal(H[k, c], H[k, c].t())


# both sides of every line of the back-projection's rule, short strips and points.  H' is
# off by M^1.5 u as above, and so is the density its entries add up to; the sums over the
# N^2 pairs add N^2 u at most
@pytest.mark.parametrize("n,N,nspin,r", [
    ((9, 7, 5), 16, 1, 1), ((9, 7, 5), 17, 2, 3), ((16, 16, 16), 32, 1, 2),
    ((16, 16, 16), 33, 2, 5), ((13, 12, 11), 160, 1, 2), ((13, 12, 11), 161, 2, 1),
    ((11, 10, 12), 256, 1, 3), ((11, 10, 12), 257, 1, 1), ((12, 12, 12), 512, 1, 2),
    ((12, 12, 12), 513, 1, 1), ((40, 40, 40), 40, 1, 6),
])
def test_response_fp64(n, N, nspin, r):
    grid, gen = _grid(n), _gen(N + r)
    P = _rand(gen, nspin, N, grid.M)
    dV = _rand(gen, r, nspin, grid.M)
    eps = torch.linspace(-1.0, 0.5, N, device="cuda", dtype=torch.float64)
    eps = torch.stack([eps + 0.01 * c for c in range(nspin)]).contiguous()
    kT = 0.05
    occ = L.Occupation(nspin, kT, float(N if nspin == 1 else N // 2))
    out, mu, dmu = L.density_response(grid, P, eps, occ, dV, "fp64")
    dv = 1.0
    for length, points in zip(grid.L, grid.n):
        dv *= length / points
    s = 2.0 if nspin == 1 else 1.0
    out = out.reshape(r, nspin, grid.M)
    ref = torch.empty_like(out)
    for c in range(nspin):
        y = (eps[c] - mu) / kT
        f, g = torch.sigmoid(-y), torch.sigmoid(y)
        z = -(y[:, None] - y[None, :]).abs()
        phi = torch.where(z == 0, torch.ones_like(z), torch.expm1(z) / z)
        low = (y[:, None] <= y[None, :])
        F = -torch.where(low, f[:, None] * g[None, :], f[None, :] * g[:, None]) * phi / kT
        for k in range(r):
            G = F * ((P[c] * dV[k, c]) @ P[c].t()) + dmu[k] * torch.diag(f * g / kT)
            ref[k, c] = s / dv * ((G @ P[c]) * P[c]).sum(0)
    assert _rel(out, ref) < (4 * grid.M ** 1.5 + N * N) * 2.0 ** -53


def _chebyshev(grid, V, X, degree, a, b, a0):
    """The scaled recurrence in FP64 by shifts."""
    h = [grid.L[d] / grid.n[d] for d in range(3)]
    e, c0 = (b - a) / 2, (b + a) / 2
    s1 = s = e / (a0 - c0)

    def shifted(y):
        out = (V - c0) * y
        for hd, ax in zip(h, (-1, -2, -3)):
            out = out - 0.5 * (torch.roll(y, 1, ax) + torch.roll(y, -1, ax) - 2 * y) / hd ** 2
        return out

    y0, y1 = X, (s1 / e) * shifted(X)
    for _ in range(2, degree + 1):
        sn = 1.0 / (2.0 / s1 - s)
        y0, y1 = y1, (2 * sn / e) * shifted(y1) - s * sn * y0
        s = sn
    return y1


# Gram and Rayleigh products of FP32 blocks on tiles of 32, 64 and 128 rows, at their
# remainders: the basis is orthonormal to its FP32 rounding and the Ritz values are those
# of the block's span.  B = L Q with |entries| random: cond(B) is a few, so that N
# roundings of 2^-24 bound both, relative to the Hamiltonian's largest value
@pytest.mark.parametrize("n,N", [((8, 8, 8), 16), ((9, 11, 13), 33), ((16, 16, 16), 65),
                                 ((32, 32, 32), 129), ((64, 64, 32), 300), ((24, 25, 26), 513)])
def test_ritz_fp32(n, N):
    grid, gen = _grid(n), _gen(N)
    V = _rand(gen, *grid.shape)
    X = _rand(gen, N, grid.M, dtype=torch.float32)
    Q = torch.linalg.qr(X.double().t())[0].t().contiguous()
    HQ = _chebyshev(grid, V, Q.reshape(N, *grid.shape), 1, -1.0, 1.0, 1.0).reshape(N, -1)
    ref = torch.linalg.eigvalsh(HQ @ Q.t())
    eps = L.subspace_rayleigh_ritz(grid, V, X, prec="fp32")
    h2 = sum((points / length) ** 2 for points, length in zip(grid.n, grid.L))
    top = 2 * h2 + float(V.abs().max())
    assert float((eps.flatten() - ref).abs().max()) < N * 2.0 ** -24 * top
    S = X.double() @ X.double().t() * float(torch.tensor(grid.L).prod() / grid.M)
    S = S / S.diagonal().mean()
    assert float((S - torch.eye(N, device="cuda", dtype=S.dtype)).abs().max()) < N * 2.0 ** -24


# whole states in LDS (24^3 FP64 and 32^3 are the largest of their kind; 64 steps are the
# most of one launch), sweeps of every remainder and with z runs, one and two groups per
# thread, single steps where nx is not a multiple of the 16-byte group
@pytest.mark.parametrize("prec,n,N,degree", [
    ("fp64", (24, 24, 24), 3, 20), ("fp64", (8, 8, 8), 5, 64), ("fp64", (8, 8, 8), 5, 65),
    ("fp32", (32, 32, 32), 2, 7), ("fp64", (20, 18, 13), 3, 11), ("fp64", (32, 32, 32), 40, 1),
    ("fp64", (32, 32, 24), 300, 9), ("fp32", (40, 36, 44), 70, 13), ("fp64", (48, 48, 16), 9, 8),
    ("fp64", (64, 64, 12), 20, 5), ("fp32", (64, 64, 64), 300, 10), ("fp32", (30, 22, 26), 4, 6),
])
def test_filter_forms(prec, n, N, degree):
    grid, gen = _grid(n), _gen(degree)
    dt = torch.float64 if prec == "fp64" else torch.float32
    V, X = _rand(gen, *grid.shape), _rand(gen, N, *grid.shape, dtype=dt)
    Y = L.chfsi_filter(grid, V, X, degree, 3.0, 34.0, -2.0, prec=prec)
    pick = sorted({0, N // 2, N - 1})
    ref = _chebyshev(grid, V, X[pick].double(), degree, 3.0, 34.0, -2.0)
    # the scaled recurrence does not amplify: a few roundings a step
    assert _rel(Y[pick].double(), ref) < 8 * degree * (2.0 ** -53 if prec == "fp64" else 2.0 ** -24)


@pytest.mark.parametrize("N", [2, 7, 300])
def test_filter_under_a_workspace_limit(N):
    """With room for the block of the single steps only, the sweeps take smaller batches
    (or the single steps)."""
    grid, gen = _grid((48, 40, 36)), _gen(N)
    V, X = _rand(gen, *grid.shape), _rand(gen, N, *grid.shape, dtype=torch.float32)
    Y = L.chfsi_filter(grid, V, X, 12, 3.0, 34.0, -2.0, prec="fp32")
    limit = N * grid.M * 4 + grid.M * 4 + (1 << 20) + 512
    ctx = B.Context(0, torch.cuda.current_stream().cuda_stream, limit)
    Z, g = torch.empty_like(Y), grid.c()
    ctx.check(ctx.lib.chfsi_filter(ctx.ptr, ctypes.byref(g), *(ctypes.c_void_p(t.data_ptr())
                                                               for t in (V, X, Z)),
                                   N, 1, 12, 3.0, 34.0, -2.0))
    torch.cuda.synchronize()
    assert ctx.workspace_bytes <= limit
    assert _rel(Z, Y) < 8 * 12 * 2.0 ** -24
    ctx.close()


# planes and columns of every padding, runs of 16 and of 64 columns, an axis past the LDS
# form; -Lap dV = 4 pi (u - mean): the symbol's largest value is 12 / h^2, its smallest
# non-zero one (2 pi / L)^2, so that a rounding of dV shows (12 / h^2) (L / 2 pi)^2-fold,
# and each of the six passes adds n of them at most
@pytest.mark.parametrize("n,r", [
    ((5, 7, 9), 2), ((16, 17, 3), 1), ((33, 4, 20), 1), ((64, 5, 18), 2), ((4, 6, 64), 1),
    ((65, 4, 5), 1), ((20, 20, 20), 40), ((64, 64, 64), 4), ((48, 49, 31), 1),
])
def test_hartree_forms(n, r):
    grid, gen = _grid(n), _gen(sum(n))
    u = _rand(gen, r, *grid.shape)
    v = L.hartree_kernel(grid, u).reshape(u.shape)
    lap, most = torch.zeros_like(v), max(n)
    for points, length, ax in zip(grid.n, grid.L, (-1, -2, -3)):
        h = length / points
        lap += (torch.roll(v, 1, ax) + torch.roll(v, -1, ax) - 2 * v) / h ** 2
    ref = 4 * torch.pi * (u - u.mean((-3, -2, -1), keepdim=True))
    assert _rel(-lap, ref) < 6 * most * 12 * (most / 6.28) ** 2 * 2.0 ** -53


# one wave a midpoint and four of them, at counts around their passes of 64 and 256
@pytest.mark.parametrize("count,nspin", [(1, 1), (3, 2), (63, 1), (64, 1), (65, 1), (128, 2),
                                         (257, 1), (1024, 2)])
def test_fermi_level(count, nspin):
    gen = _gen(count)
    eps = torch.rand((nspin, count), generator=gen, device="cuda", dtype=torch.float64)
    kT, s = 0.02, 2.0 if nspin == 1 else 1.0
    ne = 0.4 * s * nspin * count
    mu = L.fermi_occupations(eps, L.Occupation(nspin, kT, ne))[0]
    # mu within 2 ulp of where the computed count crosses ne; the count's own rounding is
    # at most the number of states times 2^-53 of it, the exponent's 50 more
    got = s * torch.sigmoid((mu - eps) / kT).sum()
    assert abs(float(got) - ne) < (nspin * count + 200) * 2.0 ** -52 * ne
