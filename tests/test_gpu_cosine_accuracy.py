"""The sums of 9 to 16 replicas come from other kernels than those of up to 8 (two wavefronts, which begin a new chain of additions
every 16 parameters of a lane) and must be no further from the exact ones.

Exact: the fp64 products of fp32 differences are exact; they are folded in halves with the error of every addition kept
(two-sum), which leaves about 1e-30.  Measure: root mean square of the relative error of the diagonal entries, over seeds.  The
same entries from a call with the first 8 replicas alone are the yardstick, but no less than what any tree of additions leaves:
a rounding to nearest errs by u / sqrt(3) of the binade, u = 2^-53, 0.43 u of the value on average over mantissas, and the
levels of a tree, 2^k operands of 2^-k of the size, add up to 0.43 u * sqrt(1 + 1/2 + 1/4 + ...) = 0.6 u.  The entries of a seed
share g, so a ratio of two measures scatters by a fifth: the bound is 1.6.  Diagonal entries in one chain of a lane's 800 parameters
are at twice the yardstick for 52.9 M parameters with outliers."""
import pytest
import torch

import paper_2501_18512_amd as sdl

pytestmark = pytest.mark.gpu


def _exact(p):
    """The sum of p as a pair of fp64 numbers."""
    hi, lo = p, torch.zeros_like(p)
    while hi.numel() > 1:
        n, h = hi.numel(), (hi.numel() + 1) // 2
        a, b = hi[:h], torch.nn.functional.pad(hi[h:], (0, 2 * h - n))
        s = a + b
        v = s - a
        lo = lo[:h] + torch.nn.functional.pad(lo[h:], (0, 2 * h - n)) + ((a - (s - v)) + (b - v))
        hi = s
    return float(hi), float(lo)


def _inputs(recipe, n, M, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    g = torch.randn(n, device="cuda", generator=gen) * 0.02
    w = []
    for _ in range(M):
        z = torch.randn(n, device="cuda", generator=gen) * 1e-3
        if recipe == "outliers":
            u = torch.rand(n, device="cuda", generator=gen)
            z = torch.where(u < 1e-3, torch.where(u < 5e-4, 0.1, -0.1), z)
        w.append((z if recipe == "full" else g - z).to(torch.bfloat16))     # full: differences with all 24 bits
    return g, w


def _rms_error(g, w, M, entries, exact):
    result, workspace = sdl.alloc_cosine(M)
    sdl.sdl_outer_grad_cosine(g, w[:M], g.numel(), result[0], workspace)
    G = sdl.split_cosine_result(result[0], M)[0].cpu()
    return [((float(G[m, m]) - exact[m][0]) - exact[m][1]) / exact[m][0] for m in entries]


@pytest.mark.parametrize("n,seeds", [((1 << 18), 8), ((1 << 23) + 333, 4), (52_900_001, 1)])
@pytest.mark.parametrize("recipe", ["outliers", "full"])
def test_wide_sums_are_as_exact_as_those_of_8_replicas(recipe, n, seeds):
    errors = {M: [] for M in (8, 9, 12, 13, 16)}
    for seed in range(seeds):
        g, w = _inputs(recipe, n, 16, seed)
        exact = [_exact((g - x.float()).double().square_()) for x in w[:8]]
        for M in errors:
            errors[M] += _rms_error(g, w, M, range(8), exact)
    rms = {M: (sum(e * e for e in x) / len(x)) ** 0.5 for M, x in errors.items()}
    print(f"{recipe} n={n}: " + ", ".join(f"M={M} {x:.2e}" for M, x in rms.items()), flush=True)
    for M in errors:
        assert rms[M] <= 1.6 * max(rms[8], 0.6 * 2.0 ** -53), f"M={M}: {rms}"


def _agreeing(recipe, rho, n, M, seed):
    """Replicas whose outer gradients share a part: correlated by rho, outliers in the same places."""
    gen = torch.Generator("cuda").manual_seed(seed)
    draw = lambda: torch.randn(n, device="cuda", generator=gen) * 1e-3
    g, common, u = draw() * 20, draw(), torch.rand(n, device="cuda", generator=gen)
    w = []
    for _ in range(M):
        z = common * rho ** 0.5 + draw() * (1 - rho) ** 0.5
        if recipe == "outliers":
            z = torch.where(u < 1e-3, torch.where(u < 5e-4, 0.1, -0.1), z)
        w.append((g - z).to(torch.bfloat16))
    return g, w


@pytest.mark.parametrize("rho", [0.5, 0.9])
@pytest.mark.parametrize("recipe", ["normal", "outliers"])
def test_products_of_replicas_that_agree_are_as_exact_as_those_of_8(recipe, rho):
    """The entries a != b, their error in units of sqrt(G[a][a] G[b][b]): products of replicas that point the same way are biased like
    squares, and what holds for the diagonal has to hold for them.  Same yardstick and bound.  (One chain of additions for all of
    a lane's parameters: 2 to 8 times the yardstick.)"""
    n, seeds, pick = 52_900_001, 2, [0, 1, 3, 6, 8, 11, 12, 15]
    errors = {M: [] for M in (8, 9, 12, 13, 16)}
    for seed in range(seeds):
        g, w = _agreeing(recipe, rho, n, 16, seed)
        d = {a: (g - w[a].float()).double() for a in pick}
        norm = {a: _exact(d[a].square())[0] ** 0.5 for a in pick}
        exact = {(a, b): _exact(d[a] * d[b]) for a in pick for b in pick if a < b}
        del d
        for M in errors:
            result, workspace = sdl.alloc_cosine(M)
            sdl.sdl_outer_grad_cosine(g, w[:M], n, result[0], workspace)
            G = sdl.split_cosine_result(result[0], M)[0].cpu()
            errors[M] += [((float(G[a, b]) - hi) - lo) / (norm[a] * norm[b]) for (a, b), (hi, lo) in exact.items() if b < M]
    rms = {M: (sum(e * e for e in x) / len(x)) ** 0.5 for M, x in errors.items()}
    print(f"{recipe} rho={rho}: " + ", ".join(f"M={M} {x:.2e}" for M, x in rms.items()), flush=True)
    for M in errors:
        assert rms[M] <= 1.6 * max(rms[8], 0.6 * 2.0 ** -53), f"M={M}: {rms}"


@pytest.mark.parametrize("n", [700, (1 << 18), (1 << 23) + 333, 52_900_001])
@pytest.mark.parametrize("M", range(8, 17))
def test_equal_replicas_have_equal_entries(M, n):
    """Every entry is the same sum in the same order, so that norms and products are the same number and cos is 1 (one rounding for
    each of two square roots, their product and the quotient: 4 units in the last place)."""
    g, w = _agreeing("outliers", 1.0, n, 1, M)
    result, workspace = sdl.alloc_cosine(M)
    sdl.sdl_outer_grad_cosine(g, w * M, n, result[0], workspace)
    G, cos, _ = sdl.split_cosine_result(result[0], M)
    assert (G == G[0, 0]).all(), (G / G[0, 0] - 1).abs().max().item()
    assert (cos - 1).abs().max().item() <= 4 * 2.0 ** -52


@pytest.mark.parametrize("n", [8_000_000, 20_000_000])
def test_digits_are_as_exact_as_fmas(n):
    """13 and 16 replicas in a large call against 12, whose sums are plain FMAs: the same diagonal entries, 12 seeds.  (The same inputs give the
    same bits, so there is no scatter to allow for.)"""
    errors = {M: [] for M in (12, 13, 16)}
    for seed in range(12):
        g, w = _inputs("normal", n, 16, seed)
        exact = [_exact((g - x.float()).double().square_()) for x in w[:12]]
        for M in errors:
            errors[M] += _rms_error(g, w, M, range(12), exact)
    rms = {M: (sum(e * e for e in x) / len(x)) ** 0.5 for M, x in errors.items()}
    print(f"n={n}: " + ", ".join(f"M={M} {x:.2e}" for M, x in rms.items()), flush=True)
    assert max(rms[13], rms[16]) <= rms[12]
