"""Up to 8 replicas: a workgroup finds its piece (a set, or a window of a large one) among up to 96, and its lanes share the sums
out as they add them up, 1 to 36 of them.  Numbers of sets at the edges of the groups of 16, large sets among small ones, empty sets."""
import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", range(1, 9))
@pytest.mark.parametrize("n_sets", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49])
def test_every_set_and_the_fragment(M, n_sets):
    rng = np.random.default_rng(100 * M + n_sets)
    numel = [int(x) for x in rng.integers(0, 3000, n_sets)]
    numel[n_sets // 2] = 900_001          # several windows
    if n_sets > 2:
        numel[1] = 0
    plan = sdl.sdl_fragment_plan(numel, [0] * n_sets, 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    g, _, w, _ = workloads.make_span(plan.total_numel, M, tau=0, delta="shared10", base_seed=M, device="cuda")
    spans = sdl.sdl_plan_fragment_spans(plan, 0)
    results, workspace = sdl.alloc_cosine(M, len(spans))
    workspace.fill_(0xff)                  # NaN: nothing may come from a matrix that nobody wrote
    fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
    sdl.sdl_outer_grad_cosine_plan(plan, 0, g, w, results, fragment, workspace)
    d = torch.stack([(g - x.float()).double() for x in w])
    want = [(d[:, o:o + n] @ d[:, o:o + n].T).cpu().numpy() for o, n, _ in spans]
    for got, ref in [(results[k], x) for k, x in enumerate(want)] + [(fragment, sum(want))]:
        G, cos, mean = (x.cpu().numpy() for x in sdl.split_cosine_result(got, M))
        norm = np.sqrt(np.diag(ref))
        # the same exact products in another order: rounding of fp64 sums only
        assert np.abs(G - ref).max() <= 1e-11 * np.outer(norm, norm).max()
        c = np.divide(ref, np.outer(norm, norm), out=np.zeros_like(ref), where=np.outer(norm, norm) > 0)
        np.testing.assert_allclose(cos, c, atol=1e-11, rtol=0)
        np.testing.assert_allclose(mean, c[np.triu_indices(M, 1)].mean() if M > 1 else 0.0, atol=1e-11, rtol=0)
