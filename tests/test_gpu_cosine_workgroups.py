"""Up to 8 replicas: a launch is at most 2048 workgroups of four wavefronts, 2560 beyond 64 * 2^20 parameters, or 8192 of one: for 8 replicas in more
than 48 sets.  Both sides of these edges, numbers of tiles that leave wavefronts of a workgroup without one, and sets at odd elements.

Reference: exact sums.  An entry's products go through fewer than 256 fp64 additions one after the other: 8 for each of up to 17 tiles of a wavefront, 6 over
its lanes and 2 over the wavefronts, up to 46 for the partial matrices.

The order of the sums is fixed by the sizes and, with digits, the values: the same numbers at other addresses give the same bits."""
import pytest
import torch

import paper_2501_18512_amd as sdl
from gpu_util import exact_gram, gram_error

pytestmark = pytest.mark.gpu

FOUR = 64 << 20
CASES = [[FOUR], [FOUR + 1], [700, FOUR // 3, 5, FOUR - FOUR // 3 - 705 - 513, 513],
         [1], [511], [512], [513], [1536], [2047], [2049], [512 * 8192 - 1], [512 * 8192 + 513],
         [1 + 37 * i for i in range(48)], [1 + 211 * i for i in range(49)], [5000 + i for i in range(224)],
         [8, (1 << 20) - 8], [3, (1 << 20) - 3], [3, (1 << 20) - 2], [8, (2 << 20) - 8], [5, (2 << 20) + 1]]


@pytest.mark.parametrize("M", [1, 2, 3, 4, 6, 7, 8])
@pytest.mark.parametrize("sizes", CASES, ids=lambda s: f"{len(s)}x{s[0]}")
def test_both_sides_of_an_edge(M, sizes):
    gen = torch.Generator("cuda").manual_seed(M)
    n = sum(sizes)
    g = torch.randn(n, device="cuda", generator=gen)
    w = [(g - torch.randn(n, device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(M)]
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


@pytest.mark.parametrize("M", [1, 3, 5, 6, 7, 8, 9, 12, 13, 16])
@pytest.mark.parametrize("sizes", [[3_000_017], [9_000_001], [1 + 20 * i for i in range(60)], [700, 4_000_000, 5, 513]], ids=lambda s: f"{len(s)}x{s[0]}")
def test_same_bits_at_any_address(M, sizes):
    gen = torch.Generator("cuda").manual_seed(M)
    n = sum(sizes)
    g = torch.randn(n, device="cuda", generator=gen)
    w = [(g - torch.randn(n, device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(M)]
    plan = sdl.sdl_fragment_plan(sizes, [0] * len(sizes), 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    out = []
    for shift in (0, 1, 3):
        at = lambda x, k: torch.cat([x[:k], x])[k:]                    # the same numbers, k elements further on
        results, workspace = sdl.alloc_cosine(M, len(sizes))
        fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
        sdl.sdl_outer_grad_cosine_plan(plan, 0, at(g, shift), [at(x, shift + m % 2 * (shift > 0)) for m, x in enumerate(w)], results, fragment, workspace)
        out.append(torch.cat([results.flatten(), fragment]).view(torch.int64))
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
