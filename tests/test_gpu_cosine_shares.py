"""9 to 16 replicas: the sets' tiles of 256 parameters lie one behind the other and are shared out among the workgroups in three
shares, whatever sets they belong to.  Sets that end where a workgroup's part ends and sets that do not, sets within one workgroup
and sets over all of them, sets without parameters, fewer tiles than workgroups, and chains of 4 tiles with and without a rest."""
import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl
import workloads

pytestmark = pytest.mark.gpu

T = 256
SETS = {
    "one_tile_each": [T] * 48,
    "equal_parts": [T * 64] * 48,                       # 3072 tiles
    "rests": [T * 64 + k for k in range(48)],
    "one_set_of_all_workgroups": [T * (4 * 1536 + 7) + 3],
    "around_the_shares": [T * 8500, T * 1050, T * 450, 5, T * 17],
    "none_in_between": [0, T * 5, 0, 0, 300, T * 2000 + 1, 0],
    "nothing": [0, 0],
}


@pytest.mark.parametrize("M", [9, 10, 11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("name", SETS)
def test_sets_and_their_fragment(M, name):
    numel = SETS[name]
    plan = sdl.sdl_fragment_plan(numel, [0] * len(numel), 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    total = max(plan.total_numel, 1)
    g, _, w, _ = workloads.make_span(total, M, tau=0, delta="shared10", base_seed=M, device="cuda")
    spans = sdl.sdl_plan_fragment_spans(plan, 0)
    results, workspace = sdl.alloc_cosine(M, max(len(spans), 1))
    workspace.fill_(float("nan") if workspace.is_floating_point() else 0xff)      # nothing may come from a matrix that nobody wrote
    fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
    sdl.sdl_outer_grad_cosine_plan(plan, 0, g, w, results, fragment, workspace)
    d = torch.stack([(g - x.float()).double() for x in w])
    want = [(d[:, o:o + n] @ d[:, o:o + n].T).cpu().numpy() for o, n, _ in spans]
    parts = [(results[k], x) for k, x in enumerate(want)] + [(fragment, sum(want) if want else np.zeros((M, M)))]
    for got, ref in parts:
        G, cos, mean = (x.cpu().numpy() for x in sdl.split_cosine_result(got, M))
        norm = np.sqrt(np.diag(ref))
        # the same exact products in another order: rounding of fp64 sums only
        assert np.abs(G - ref).max() <= 1e-11 * np.outer(norm, norm).max()
        c = np.divide(ref, np.outer(norm, norm), out=np.zeros_like(ref), where=np.outer(norm, norm) > 0)
        np.testing.assert_allclose(cos, c, atol=1e-11, rtol=0)
        np.testing.assert_allclose(mean, c[np.triu_indices(M, 1)].mean(), atol=1e-11, rtol=0)


@pytest.mark.parametrize("M", [9, 12, 13, 16])
def test_each_set_by_its_own_alignment(M):
    """Sets on 16 bytes in every array, on 16 bytes of fp32 and 8 of bf16, and at odd elements, one behind the other in one launch:
    the first and the last of 48 sets aligned, and neither."""
    for shift in (0, 4):
        numel = [8 * T] + [[3 * T + 1, 2 * T + 7, T + 4, 5 * T + 4][k % 4] for k in range(46)] + [4 * T + 3]
        plan = sdl.sdl_fragment_plan(numel, [0] * 48, 1, 1, sdl.PATTERN_STRIDED, 10, 0)
        g0, _, w0, _ = workloads.make_span(plan.total_numel + shift, M, tau=0, delta="shared10", base_seed=M, device="cuda")
        g, w = g0[shift:], [x[shift:] for x in w0]
        spans = sdl.sdl_plan_fragment_spans(plan, 0)
        assert {(o + shift) % 8 for o, _, _ in spans} == {0, 4, 1 + shift}
        results, workspace = sdl.alloc_cosine(M, 48)
        fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
        sdl.sdl_outer_grad_cosine_plan(plan, 0, g, w, results, fragment, workspace)
        d = torch.stack([(g - x.float()).double() for x in w])
        want = [(d[:, o:o + n] @ d[:, o:o + n].T).cpu().numpy() for o, n, _ in spans]
        for got, ref in [(results[k], x) for k, x in enumerate(want)] + [(fragment, sum(want))]:
            G = sdl.split_cosine_result(got, M)[0].cpu().numpy()
            norm = np.sqrt(np.diag(ref))
            # the same exact products in another order: rounding of fp64 sums only
            assert np.abs(G - ref).max() <= 1e-11 * np.outer(norm, norm).max()
