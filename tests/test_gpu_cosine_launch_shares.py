"""More than 8 replicas: the tiles of a launch are dealt out in one share up to 6 * 2^20 parameters, in two up to 24 * 2^20 and in three beyond.  Numbers
of parameters at those edges, as one set and as several that share workgroups.

Reference: exact sums.  An entry's products go through fewer than 256 fp64 additions one after the other: 64 in a step that has no digits, 16 and 25 in a chain of
FMAs and the chains of a lane, 13 for the sums of digits, 6 over the lanes, up to 46 for the partial matrices."""
import pytest
import torch

import paper_2501_18512_amd as sdl
from gpu_util import exact_gram, gram_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [9, 12, 14, 16])
@pytest.mark.parametrize("edge", [6 << 20, 24 << 20])
@pytest.mark.parametrize("extra", [0, 1])
def test_both_sides_of_an_edge(M, edge, extra):
    gen = torch.Generator("cuda").manual_seed(M)
    n = edge + extra
    g = torch.randn(n, device="cuda", generator=gen)
    w = [(g - torch.randn(n, device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(M)]
    for sizes in ([n], [700, n // 3, 5, n - n // 3 - 705 - 513, 513]):
        plan = sdl.sdl_fragment_plan(sizes, [0] * len(sizes), 1, 1, sdl.PATTERN_STRIDED, 10, 0)
        results, workspace = sdl.alloc_cosine(M, len(sizes))
        workspace.fill_(0xff)              # NaN: nothing may come from a matrix that nobody wrote
        fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
        sdl.sdl_outer_grad_cosine_plan(plan, 0, g, w, results, fragment, workspace)
        exact, at = [], 0
        for s in sizes:
            exact.append(exact_gram(g[at:at + s], [x[at:at + s] for x in w]))
            at += s
        exact.append(tuple(sum(x) for x in zip(*exact)))
        for r, (want, rest) in zip([*results, fragment], exact):
            assert gram_error(sdl.split_cosine_result(r, M)[0], want, rest) <= 256
