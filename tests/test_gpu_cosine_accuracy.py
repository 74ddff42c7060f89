"""The sums of 9 to 16 replicas come from other kernels than those of up to 8 (two wavefronts; matrix cores, which round towards
zero) and must be no further from the exact ones.

Exact: the fp64 products of fp32 differences are exact; they are folded in halves with the error of every addition kept
(two-sum), which leaves about 1e-30.  Measure: root mean square of the relative error of the diagonal entries, over seeds.  The
same entries from a call with the first 8 replicas alone are the yardstick, but no less than what any tree of additions leaves:
a rounding to nearest errs by u / sqrt(3) of the binade, u = 2^-53, 0.43 u of the value on average over mantissas, and the
levels of a tree, 2^k operands of 2^-k of the size, add up to 0.43 u * sqrt(1 + 1/2 + 1/4 + ...) = 0.6 u.  The entries of a seed
share g, so a ratio of two measures scatters by a fifth: the bound is 1.6.  Sums of the matrix cores in chains of 64
parameters are at 1.5 to 3 times the yardstick, those of two wavefronts with half as many workgroups at twice of it for
52.9 M parameters."""
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
