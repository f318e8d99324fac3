"""Which form of a kernel a call takes, and what does not depend on it."""
from __future__ import annotations

import pytest
import torch

import paper_2211_07894_amd as L
from paper_2211_07894_amd import lrdm as B

pytestmark = pytest.mark.gpu


def _grid(n):
    return L.Grid(n, tuple(0.43 * x for x in n))


def _gen(seed):
    g = torch.Generator("cuda")
    g.manual_seed(seed)
    return g


def _rand(gen, *shape, dtype=torch.float64):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def _system(n, N, nspin, r, seed):
    """A system whose states fall off by 2^26 along the box: the partial sums of its
    projection lie up to 52 binary orders apart, and so round in every order of adding."""
    grid, gen = _grid(n), _gen(seed)
    fall = torch.exp2(-26.0 * torch.arange(grid.M, device="cuda") / grid.M)
    P = (_rand(gen, nspin, N, grid.M) * fall).float()
    eps = torch.linspace(-1.0, 0.5, N, device="cuda", dtype=torch.float64).repeat(nspin, 1)
    return dict(grid=grid, Psi=P, eps=eps.contiguous(), occ=L.Occupation(nspin, 0.05, 0.8 * N),
                dV=_rand(gen, r, nspin, grid.M))


# a system's sums are those of a call of its own, whichever systems share the batch
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_batch_sums_as_single_calls(prec):
    small = [_system((32, 32, 32), 98, 2, 4, 1), _system((24, 24, 24), 32, 1, 4, 2),
             _system((15, 14, 13), 40, 1, 2, 3)]
    large = [_system((40, 40, 40), 300, 2, 8, 4), _system((48, 48, 48), 256, 1, 8, 5)]
    for systems in (small, small + large):
        out = L.density_response_batched(systems, prec=prec)
        for (drho, mu, dmu), s in zip(out, systems):
            ref = L.density_response(s["grid"], s["Psi"], s["eps"], s["occ"], s["dV"], prec=prec)
            for got, want in zip((drho, mu, dmu), ref):
                assert torch.equal(got, want)


def _time(f, reps=10):
    f()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(reps):
        f()
    b.record()
    b.synchronize()
    return a.elapsed_time(b) / reps


# rows that cannot be copied in 16-byte chunks: the tuner tries the count an untuned call
# takes, 60 ranges here (80 us; counts up to 8 take 460 us and more)
@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
def test_autotune_keeps_the_untuned_count_in_reach(prec):
    n, N = (27, 33, 35), 90
    grid, gen = _grid(n), _gen(1)
    P, dV = _rand(gen, 2, N, grid.M, dtype=torch.float32), _rand(gen, 1, 2, grid.M)
    call = lambda: L.projected_perturbation(grid, P, dV, 2, prec)  # noqa: E731
    B.release_contexts()
    untuned = _time(call)
    L.autotune(grid, N, 2, 1, prec)
    assert _time(call) < 2 * untuned
    B.release_contexts()
