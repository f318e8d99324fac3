"""The workspace's growth, on the CPU build of the library, whose device memory a test
can make refuse allocations from a size on."""
import ctypes
import os

import numpy as np
import pytest

from paper_2211_07894_amd import lrdm as B
from tests.cpu_emu import build_emu

ANY = ctypes.c_size_t(-1).value


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(build_emu.CLANG):
        pytest.skip("needs the host clang of ROCm")
    lib = ctypes.CDLL(build_emu.build("", shared=True))
    vp, i32 = ctypes.c_void_p, ctypes.c_int32
    lib.lrdm_create.argtypes = [ctypes.POINTER(vp), ctypes.c_int, vp, ctypes.c_size_t]
    lib.lrdm_destroy.argtypes = [vp]
    lib.lrdm_projected_perturbation.argtypes = [vp, ctypes.POINTER(B.c_grid), vp, i32, i32, vp,
                                                i32, ctypes.c_int, vp]
    lib.density_response_batched.argtypes = [vp, ctypes.POINTER(B.c_system), i32, ctypes.c_int]
    lib.lrdm_workspace_bytes.argtypes = lib.lrdm_last_error.argtypes = [vp]
    lib.lrdm_workspace_bytes.restype = ctypes.c_size_t
    lib.lrdm_last_error.restype = ctypes.c_char_p
    lib.lrdm_emu_device.argtypes = [ctypes.c_size_t, ctypes.c_int]
    lib.lrdm_emu_mallocs.restype = lib.lrdm_emu_frees.restype = ctypes.c_long
    yield lib
    lib.lrdm_emu_device(ANY, 0)


class Calls:
    """Projections of one context: the preferred partial sums grow with the points, the
    least ones much less."""

    def __init__(self, lib, stream=0, limit=0):
        self.lib, self.ctx = lib, ctypes.c_void_p()
        lib.lrdm_emu_device(ANY, 0)
        assert lib.lrdm_create(ctypes.byref(self.ctx), 0, stream, limit) == 0

    def __enter__(self):
        return self

    def __exit__(self, *_):
        self.lib.lrdm_emu_device(ANY, 0)
        self.lib.lrdm_destroy(self.ctx)

    def device(self, refuse_from=ANY, capturing=0):
        self.lib.lrdm_emu_device(refuse_from, capturing)

    @property
    def bytes(self):
        return self.lib.lrdm_workspace_bytes(self.ctx)

    def moves(self):
        return self.lib.lrdm_emu_mallocs(), self.lib.lrdm_emu_frees()

    def project(self, n, N=40, r=1, prec="fp64"):
        rng = np.random.default_rng(n[0] + N)
        M = n[0] * n[1] * n[2]
        P, dV = rng.standard_normal((N, M)), rng.standard_normal((r, M))
        P = P.astype(np.float64 if prec == "fp64" else np.float32)
        H = np.zeros((r, N, N))
        g = B.c_grid()
        for d in range(3):
            g.n[d], g.L[d] = n[d], 0.4 * n[d]
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
        st = self.lib.lrdm_projected_perturbation(self.ctx, ctypes.byref(g), p(P), N, 1, p(dV), r,
                                                  B.PREC[prec], p(H))
        assert st == 0, self.lib.lrdm_last_error(self.ctx)
        ref = (P[None].astype(np.float64) * dV[:, None]) @ P.astype(np.float64).T
        # a sum of M terms in FP64 (of K-tiles of 32 in FP32): M u (32 u) of their absolute
        # sum, about sqrt(M) times the result
        bound = M * 2.0 ** -53 if prec == "fp64" else 32 * 2.0 ** -24
        assert np.abs(H - ref).max() < M ** 0.5 * bound * np.abs(ref).max()

    def batch(self, count, n=(16, 16, 16), N=6, prec="fp64"):
        """`count` systems of one size, which differ in their fields."""
        rng = np.random.default_rng(count)
        M = n[0] * n[1] * n[2]
        sy, keep = (B.c_system * count)(), []
        g = B.c_grid()
        for d in range(3):
            g.n[d], g.L[d] = n[d], 0.4 * n[d]
        P = np.linalg.qr(rng.standard_normal((M, N)))[0].T
        P = np.ascontiguousarray(P, dtype=np.float64 if prec == "fp64" else np.float32)
        eps = np.linspace(-1.0, 0.5, N)
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
        occ = B.c_occ(1, 0.05, float(N))
        for k in range(count):
            dV, drho, mu, dmu = rng.standard_normal((1, M)), np.zeros((1, M)), np.zeros(1), np.zeros(1)
            keep.append((dV, drho))
            sy[k] = B.c_system(g, p(P), p(eps), N, occ, p(dV), 1, p(drho), p(mu), p(dmu))
            keep.append((mu, dmu))
        st = self.lib.density_response_batched(self.ctx, sy, count, B.PREC[prec])
        assert st == 0, self.lib.lrdm_last_error(self.ctx)
        # each system against itself alone: to the bit
        for k in range(count):
            dV, drho = keep[2 * k]
            got = drho.copy()
            drho[:] = np.nan
            one = (B.c_system * 1)(sy[k])
            assert self.lib.density_response_batched(self.ctx, one, 1, B.PREC[prec]) == 0
            assert np.array_equal(got, drho)


def preferred(lib, n, **kw):
    with Calls(lib) as c:
        c.project(n, **kw)
        return c.bytes


def test_a_refused_preferred_size_costs_one_attempt(lib):
    """Equal calls on a device that holds the least workspace but not the preferred one:
    all succeed, and only the first allocates."""
    n = (24, 24, 24)
    with Calls(lib) as c:
        c.device(refuse_from=preferred(lib, n))
        c.project(n)
        held, moves = c.bytes, c.moves()
        for _ in range(3):
            c.project(n)
            assert (c.bytes, c.moves()) == (held, moves)
        # a call that needs more asks for what it prefers again
        c.device()
        c.project((32, 32, 32), r=10)
        assert c.bytes == preferred(lib, (32, 32, 32), r=10)


def test_growth_for_a_preferred_size_keeps_the_workspace_until_it_succeeds(lib):
    """A workspace that already covers the least size is not given up for one the device
    cannot give."""
    small, large = (12, 12, 12), (24, 24, 24)
    most = preferred(lib, large)
    with Calls(lib) as c:
        c.project(small, r=4)
        held, moves = c.bytes, c.moves()
        assert held < most
        c.device(refuse_from=held + 1)
        c.project(large)
        assert (c.bytes, c.moves()) == (held, moves)


def test_a_captured_workspace_is_kept(lib):
    """A call captured into a graph holds the workspace's address: calls that could run
    within it do not move it afterwards, whatever size they prefer."""
    small, large = (12, 12, 12), (24, 24, 24)
    most = preferred(lib, large)
    with Calls(lib, stream=1) as c:
        c.project(small, r=4)
        held, moves = c.bytes, c.moves()
        assert held < most
        c.device(capturing=1)
        c.project(small, r=4)
        c.device()
        c.project(large)
        assert (c.bytes, c.moves()) == (held, moves)
    with Calls(lib, stream=1) as c:    # nothing captured: it grows
        c.project(small, r=4)
        c.project(large)
        assert c.bytes == most


def test_fp32_projection_holds_its_own_partial_sums_only(lib):
    """128 x 128 tiles of ranges of 512 points and more; the 64-row tiles of the FP64 form
    would take twice that here."""
    n, N = (24, 24, 24), 200
    ranges, tiles = 24 ** 3 // 512, 3
    most = ranges * tiles * 128 * 128 * 8 + (1 << 20) + 256
    assert preferred(lib, n, N=N, prec="fp32") <= most


def test_batch_workspace_is_bounded(lib):
    """Systems that run one after another on a stream share its region, and the fused form's
    partial sums (1 MiB a system here) are those of one launch of 16."""
    held = {}
    for prec in ("fp64", "fp32"):
        for count in (4, 18, 34):
            with Calls(lib) as c:
                c.batch(count, prec=prec)
                held[prec, count] = c.bytes
    assert held["fp64", 34] == held["fp64", 4]
    copies = 4096 * 32 * 4 + (1 << 16)          # Psi transposed, Gamma and the N x N matrices
    assert held["fp32", 34] - held["fp32", 18] <= 16 * copies


@pytest.mark.parametrize("M", [27 * 33 * 35, 45 ** 3, 63 * 61 * 63])
@pytest.mark.parametrize("N,batch", [(40, 1), (90, 2), (129, 60), (257, 1), (400, 8), (800, 2)])
def test_staged_ranges_fill_the_rounds(lib, M, N, batch):
    """The count of a projection staged through registers, one workgroup per tile and CU: no
    more rounds of workgroups, times K-tiles and a fixed cost of 6, than the longest ranges
    take (groups of tiles that divide among the eight dies stay on one each)."""
    splits = lib._ZN4lrdm17tn_default_splitsEiliii
    cap = lib._ZN4lrdm12tn_range_capEiliii
    for f in (splits, cap):
        f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    tiles = -(-N // 128) * (-(-N // 128) + 1) // 2

    def cost(s):
        whole = s * batch % 8 == 0
        rounds = -(-(s * batch // 8 * tiles) // 32) if whole else -(-s * batch * tiles // 256)
        return rounds * (-(-M // (32 * s)) + 6)

    long_ranges, staged = 0, 4
    got = splits(N, M, batch, staged, 0)
    assert 1 <= got <= cap(N, M, batch, staged, 0)
    assert cost(got) <= cost(splits(N, M, batch, long_ranges, 0)) / 0.95


def test_fp64_tiles_of_rows_megabytes_apart(lib):
    """Tiles of 64 rows up to 384 states, but not for the last 16 where rows lie 2 MB apart
    and 128-row tiles fill the chip."""
    direct = lib._ZN4lrdm12tn_direct_okEili
    direct.argtypes, direct.restype = [ctypes.c_int, ctypes.c_int64, ctypes.c_int], ctypes.c_bool
    for N, M, batch, want in [(384, 64 ** 3, 8, False), (384, 60 ** 3, 8, True),
                              (368, 64 ** 3, 8, True), (384, 64 ** 3, 1, True),
                              (385, 60 ** 3, 8, False), (1024, 24 ** 3, 1, True)]:
        assert direct(N, M, batch) == want, (N, M, batch)
