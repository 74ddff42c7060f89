"""More than 8 replicas: two wavefronts with half of the matrix each, by kernels for 9 and 10, 11 and 12, 13 and 14, 15 and 16 (8
replicas, whose tiles have 512 parameters, beside them).  Sizes at the edges of the tiles (256 parameters, 64 of them at a
time), arrays at any element, a set that several workgroups share, sets and their fragment out of one launch and of two, and a
NaN and an infinity in one replica, which must stay in that replica's row and column."""
import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl
import workloads

pytestmark = pytest.mark.gpu


def _reference(g, w):
    d = torch.stack([(g - x.float()).double() for x in w])
    return (d @ d.T).cpu().numpy()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("M", range(8, 17))
def test_wide_gram(M, shift):
    for n in (1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1024 + 31, 4096 * 512 + 700):
        g0, _, w0, _ = workloads.make_span(n + shift, M, tau=0, delta="shared10", base_seed=n, device="cuda")
        g, w = g0[shift:], [x[shift:] for x in w0]
        result, workspace = sdl.alloc_cosine(M)
        sdl.sdl_outer_grad_cosine(g, w, n, result[0], workspace)
        G, cos, mean = (x.cpu().numpy() for x in sdl.split_cosine_result(result[0], M))
        want = _reference(g, w)
        # the same exact products in another order: rounding of fp64 sums only
        norm = np.sqrt(np.diag(want))
        assert np.abs(G - want).max(initial=0) <= 1e-11 * np.outer(norm, norm).max(), n
        np.testing.assert_allclose(cos, want / np.outer(norm, norm), atol=1e-11, rtol=0)
        np.testing.assert_allclose(mean, (want / np.outer(norm, norm))[np.triu_indices(M, 1)].mean(), atol=1e-11, rtol=0)


@pytest.mark.parametrize("M", [9, 12, 13, 16])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_replica_stays_in_its_row(M, bad):
    n = 3 * 512 + 17
    g, _, w, _ = workloads.make_span(n, M, tau=0, delta="normal", base_seed=M, device="cuda")
    clean = _reference(g, w)
    for m in (0, M // 2, M - 1):
        v = [x.clone() for x in w]
        v[m][700] = bad
        result, workspace = sdl.alloc_cosine(M)
        sdl.sdl_outer_grad_cosine(g, v, n, result[0], workspace)
        G = sdl.split_cosine_result(result[0], M)[0].cpu().numpy()
        keep = np.arange(M) != m
        np.testing.assert_allclose(G[np.ix_(keep, keep)], clean[np.ix_(keep, keep)], rtol=0, atol=1e-11 * clean.max())
        assert not np.isfinite(G[m]).any() and not np.isfinite(G[:, m]).any()


@pytest.mark.parametrize("M", [9, 12, 13, 16])
@pytest.mark.parametrize("n_spans,large", [(3, 0), (48, 0), (48, 1_500_001), (49, 0), (49, 1_500_001)])
def test_spans_and_their_fragment(M, n_spans, large):
    """Up to 48 spans are one launch, which gives the fragment's result as well, added in one level (a few workgroups) or two (a
    large span); more are two launches and a sum of the spans' matrices."""
    rng = np.random.default_rng(n_spans)
    numel = [int(x) for x in rng.integers(20, 2000, n_spans)]
    if large:
        numel[n_spans // 2] = large
    plan = sdl.sdl_fragment_plan(numel, [0] * n_spans, 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    g, _, w, _ = workloads.make_span(plan.total_numel, M, tau=0, delta="shared10", base_seed=M, device="cuda")
    spans = sdl.sdl_plan_fragment_spans(plan, 0)
    results, workspace = sdl.alloc_cosine(M, len(spans))
    fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
    sdl.sdl_outer_grad_cosine_plan(plan, 0, g, w, results, fragment, workspace)
    parts = [(results[k], _reference(g[o:o + n], [x[o:o + n] for x in w])) for k, (o, n, _) in enumerate(spans)]
    for got, want in parts + [(fragment, sum(x for _, x in parts))]:
        G, cos, mean = (x.cpu().numpy() for x in sdl.split_cosine_result(got, M))
        norm = np.sqrt(np.diag(want))
        # the same exact products in another order: rounding of fp64 sums only
        assert np.abs(G - want).max() <= 1e-11 * np.outer(norm, norm).max()
        np.testing.assert_allclose(cos, want / np.outer(norm, norm), atol=1e-11, rtol=0)
        np.testing.assert_allclose(mean, (want / np.outer(norm, norm))[np.triu_indices(M, 1)].mean(), atol=1e-11, rtol=0)
