"""More than 8 replicas: the tiles of a launch are dealt out in one share up to 6 * 2^20 parameters, in two up to 24 * 2^20 and in three beyond.  Numbers
of parameters at those edges, as one set and as several that share workgroups."""
import pytest
import torch

import paper_2501_18512_amd as sdl

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
        want, at = [], 0
        for s in sizes:
            total = torch.zeros(M, M, dtype=torch.float64, device="cuda")
            for lo in range(at, at + s, 1 << 19):
                hi = min(lo + (1 << 19), at + s)
                d = torch.stack([(g[lo:hi] - x[lo:hi].float()).double() for x in w])
                total += d @ d.T
            want.append(total)
            at += s
        got = [sdl.split_cosine_result(r, M)[0] for r in [*results, fragment]]
        for a, b in zip(got, want + [sum(want)]):
            norm = torch.diagonal(b).sqrt()
            # the same exact products in another order: 2^19 of them one after the other, more than either side adds, err by 2^-34 at most
            assert ((a - b).abs() <= 2.0 ** -34 * norm[:, None] * norm[None, :]).all()
