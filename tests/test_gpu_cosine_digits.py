"""15 and 16 replicas and 2^21 parameters in a launch or more, 13 and 14 and 10 * 2^19: the differences as six digits of a multiple of 2^-22 of a
scale of their replica's, with products that the matrix cores add up in whole numbers, and 64 parameters at a time in fp64 where a difference
is no such multiple.  Sizes at the edges of the tiles (512 parameters, the wavefronts 64 at a time) and of the range, arrays at any element,
and differences that the scale does not suit: growing by 2^60 along the array, none at all, below 2^-98, near the largest fp32 number, all
alike with a few that are 2^10 to 2^28 times as large, not finite.

Reference: exact sums (fp64 products of fp32 differences are exact; folded in halves with the error of every addition kept).  What may
differ are roundings of fp64 additions: at most 64 in a row where 64 parameters are added up in fp64, 13 for the sums of digits, 4 for the
two wavefronts and the transpose, and 25 for the partial matrices (8 and 3 in each of two levels, 3 more for a fragment): fewer than 128, each 2^-53
of at most sqrt(G[a][a] G[b][b]), and so 2^-46 of that."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl
from gpu_util import exact_gram
from paper_2501_18512_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LINE = {13: 10 << 19, 14: 10 << 19, 15: 1 << 21, 16: 1 << 21}


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_the_digit_kernel_uses_no_scratch(tmp_path):
    src = next(s for s in build.SOURCES if s.endswith("sdl_cosine.hip"))
    flags = [f for f in build.FLAGS if f != "-shared"]
    out = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o",
                          str(tmp_path / "cosine.o")], check=True, capture_output=True, text=True).stderr
    scratch = dict(re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", out, re.S))
    assert sorted(int(x) for k, x in scratch.items() if "sdl_digit_sums" in k) == [0, 0]


def _inputs(kind, n, M, shift):
    gen = torch.Generator("cuda").manual_seed(n + M)
    draw = lambda: torch.randn(n + shift, device="cuda", generator=gen)
    scale = 1.0
    if kind == "growing":
        scale = torch.exp2(torch.arange(n + shift, device="cuda") * (60.0 / n) - 40.0)
    g = draw() * 0.02 * scale
    w = [(g - draw() * 1e-3 * scale).to(torch.bfloat16) for _ in range(M)]
    if kind == "t3":
        w = [(g - draw() * 1e-3 / (sum(draw().square() for _ in range(3)) / 3).sqrt()).to(torch.bfloat16) for _ in range(M)]
    if kind == "outliers":
        for x in w:
            x[torch.randint(n, (n // 1000,), device="cuda", generator=gen)] += 0.1
    if kind in ("tiny", "huge"):
        power = 2.0 ** (-110 if kind == "tiny" else 120)
        g, w = g * power, [x * power for x in w]
    if kind == "ladder":                 # each replica's differences half of those of the one before, large ones in all of them at the end
        w = [(g - draw() * 2.0 ** (-9 - m)).to(torch.bfloat16) for m in range(M)]
        for x in w:
            x[n - 5000::500] += 1
    if kind == "zeros":                  # no difference for a third of the replicas, and what the digits lack bits for beside it or elsewhere
        g[::7] = g[::7].to(torch.bfloat16).float()
        g[5::999] *= 2.0 ** -60
        for m, x in enumerate(w):
            x[::7] = g[::7].to(torch.bfloat16) if m % 3 == 0 else x[::7]
            x[5::999] = 0
    if kind == "uneven":                 # no difference, differences below 2^-98, a scale of their own
        g = g.to(torch.bfloat16).float()
        w[1] = g.to(torch.bfloat16)
        w[4] = w[1].clone()
        w[4][::3] = 0
        g[::3] *= 2.0 ** -100
        w[7] = w[7] * 2.0 ** 60
    return g[shift:], [x[shift:] for x in w]


def _check(got, exact, M):
    G, cos, mean = (x.cpu().numpy() for x in sdl.split_cosine_result(got, M))
    want, rest = exact
    norm = np.sqrt(np.diag(want))
    outer = np.outer(norm, norm)
    assert (np.abs((G - want) - rest) <= 2.0 ** -46 * outer).all(), np.nanmax(np.abs((G - want) - rest) / outer)
    want_cos = np.divide(want, outer, out=np.zeros_like(want), where=outer > 0)
    np.testing.assert_allclose(cos, want_cos, atol=2.0 ** -45, rtol=0)
    np.testing.assert_allclose(mean, want_cos[np.triu_indices(M, 1)].mean(), atol=2.0 ** -45, rtol=0)


def _exact(g, w):
    return tuple(x.cpu().numpy() for x in exact_gram(g, w))


@pytest.mark.gpu
@pytest.mark.parametrize("M,shift", [(13, 0), (14, 1), (15, 0), (16, 1), (16, 0)])
@pytest.mark.parametrize("kind,extra", [("normal", -1), ("normal", 0), ("normal", 1), ("outliers", 511), ("growing", 513), ("tiny", 65),
                                        ("huge", 700), ("uneven", 0), ("ladder", 190), ("zeros", 77)])
def test_sums_of_digits(kind, extra, M, shift):
    n = LINE[M] + extra
    g, w = _inputs(kind, n, M, shift)
    result, workspace = sdl.alloc_cosine(M)
    sdl.sdl_outer_grad_cosine(g, w, n, result[0], workspace)
    _check(result[0], _exact(g, w), M)


@pytest.mark.gpu
@pytest.mark.parametrize("M", [13, 16])
@pytest.mark.parametrize("every", [704, 17_226])
@pytest.mark.parametrize("power", [10, 12, 14, 16, 18, 20, 24, 28])
def test_equal_differences_and_a_few_large_ones(power, every, M):
    """What one of them loses all of them lose, with one sign."""
    n = LINE[M] + 700
    g = torch.full((n,), 0.1 * (1 + 2.0 ** -9 + 2.0 ** -17 + 2.0 ** -23), device="cuda") * 2.0 ** -power
    w = [torch.zeros(n, dtype=torch.bfloat16, device="cuda") for _ in range(M)]
    for m in range(0, M, 2):
        w[m][37 * m::every] = -0.1
    result, workspace = sdl.alloc_cosine(M)
    sdl.sdl_outer_grad_cosine(g, w, n, result[0], workspace)
    _check(result[0], _exact(g, w), M)


@pytest.mark.gpu
@pytest.mark.parametrize("M", [13, 16])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_non_finite_replica_stays_in_its_row(M, bad):
    n = LINE[M] + 17
    g, w = _inputs("normal", n, M, 0)
    clean, rest = _exact(g, w)
    for m, at in ((0, 0), (M // 2, 70_003), (M - 1, n - 1)):
        v = list(w)
        v[m] = w[m].clone()
        v[m][at] = bad
        result, workspace = sdl.alloc_cosine(M)
        sdl.sdl_outer_grad_cosine(g, v, n, result[0], workspace)
        G = sdl.split_cosine_result(result[0], M)[0].cpu().numpy()
        keep = np.arange(M) != m
        assert (np.abs((G - clean) - rest)[np.ix_(keep, keep)] <= 2.0 ** -46 * clean.max()).all()
        want = (g - v[m].float()).double() @ torch.stack([(g - x.float()).double() for x in v]).T
        np.testing.assert_array_equal(np.sign(G[m]), np.sign(want.cpu().numpy()))     # inf, -inf or NaN alike
        assert not np.isfinite(G[m]).any()


@pytest.mark.gpu
@pytest.mark.parametrize("M", [13, 16])
@pytest.mark.parametrize("nan,inf", [([2], []), ([0, 5], []), ([2], [2, 7]), (range(13), [])])
def test_replicas_without_numbers(M, nan, inf):
    """Whole replicas NaN, in the first span alone and in the steps of infinities."""
    sizes = [LINE[M] + 333, 5000, 12_345]
    plan = sdl.sdl_fragment_plan(sizes, [0] * 3, 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    g, w = _inputs("normal", sum(sizes), M, 0)
    for m in inf:
        w[m][700:LINE[M]:1000] = float("inf")
    for m in nan:
        w[m][:LINE[M] if m else sizes[0]] = float("nan")
    results, workspace = sdl.alloc_cosine(M, 3)
    fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
    sdl.sdl_outer_grad_cosine_plan(plan, 0, g, w, results, fragment, workspace)
    finite = np.array([m not in nan and m not in inf for m in range(M)])
    keep = np.ix_(finite, finite)
    clean = [g.clone() if not ok else x for x, ok in zip(w, finite)]          # (a difference of 0)
    total = np.zeros((M, M))
    for (o, n, _), got in zip(sdl.sdl_plan_fragment_spans(plan, 0), results):
        G = sdl.split_cosine_result(got, M)[0].cpu().numpy()
        want, rest = _exact(g[o:o + n], [x[o:o + n] for x in (clean if o == 0 else w)])
        total += want
        ok = keep if o == 0 else np.ix_(range(M), range(M))
        assert (np.abs((G - want) - rest)[ok] <= 2.0 ** -46 * want.max()).all()
        if o == 0:
            assert np.isnan(G[list(nan)]).all() and np.isnan(G[:, list(nan)]).all()
            assert not np.isfinite(G[inf]).any() and all(G[m, m] == np.inf for m in inf if m not in nan)
    G = sdl.split_cosine_result(fragment, M)[0].cpu().numpy()
    assert (np.abs(G - total)[keep] <= 2.0 ** -45 * total.max()).all() if finite.any() else True
    assert np.isnan(G[list(nan)]).all()


def _time_of(n, first, second):
    """us of a call on either list of replicas: the two in turn, the median of each."""
    M = len(first[1])
    result, workspace = sdl.alloc_cosine(M)
    times = [], []
    for turn in range(24):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        g, w = (first, second)[turn % 2]
        start.record()
        for _ in range(5):
            sdl.sdl_outer_grad_cosine(g, w, n, result[0], workspace)
        end.record()
        end.synchronize()
        times[turn % 2].append(start.elapsed_time(end) * 200)
    out = [sorted(x[2:])[5] for x in times]
    print("{:.1f} us, {:.1f} us".format(*out), flush=True)
    return out


@pytest.mark.gpu
def test_a_replica_without_numbers_takes_no_longer():
    """One replica all NaN: the others' sums stay on the matrix cores (1.2 times a call without it; 1.8 with every step in fp64, 7.5 lane by
    lane)."""
    n = 20_000_000
    g, w = _inputs("normal", n, 16, 0)
    bad = [torch.full_like(x, float("nan")) if m == 3 else x for m, x in enumerate(w)]
    usual, nan = _time_of(n, (g, w), (g, bad))
    assert nan <= 1.5 * usual


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["outliers", "t3"])
def test_large_differences_here_and_there_take_no_longer(kind):
    """Replicas whose largest differences grow one after the other make room for them at once (1.03 times a call on normal differences; 1.3 with a
    new scale for each)."""
    n = 4_000_000
    usual, other = _time_of(n, _inputs("normal", n, 16, 0), _inputs(kind, n, 16, 0))
    assert other <= 1.15 * usual


@pytest.mark.gpu
@pytest.mark.parametrize("M", [13, 16])
@pytest.mark.parametrize("n_spans", [3, 48, 49])
def test_spans_that_share_workgroups(M, n_spans):
    rng = np.random.default_rng(n_spans)
    numel = [int(x) for x in rng.integers(1, 3000, n_spans)]
    numel[1] = LINE[M]
    plan = sdl.sdl_fragment_plan(numel, [0] * n_spans, 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    g, w = _inputs("normal", plan.total_numel, M, 0)
    spans = sdl.sdl_plan_fragment_spans(plan, 0)
    results, workspace = sdl.alloc_cosine(M, len(spans))
    fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
    sdl.sdl_outer_grad_cosine_plan(plan, 0, g, w, results, fragment, workspace)
    parts = [_exact(g[o:o + n], [x[o:o + n] for x in w]) for o, n, _ in spans]
    for k, exact in enumerate(parts):
        _check(results[k], exact, M)
    _check(fragment, (sum(want for want, _ in parts), sum(rest for _, rest in parts)), M)
