"""Many parameter sets: a launch takes up to 224 of them, more than 48 only while they have no more than 2^23 parameters, up to 528 are finished
together, and the fragment's result comes out of the same launch or, with more, from the sets' results.  Numbers of sets at those edges, launches cut
by the number of parameters, sets without any, and sets that start behind element 2^32.

Reference: exact sums.  An entry's products go through fewer than 256 fp64 additions one after the other: up to 152 in a lane (FMAs; with digits 77), 8 over lanes and
wavefronts, up to 46 for the partial matrices."""
import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl
from gpu_util import gram_error, gram_of

pytestmark = pytest.mark.gpu
SMALL = 1200


def _run(plan, p, M, g, w):
    spans = sdl.sdl_plan_fragment_spans(plan, p)
    results, workspace = sdl.alloc_cosine(M, len(spans))
    workspace.fill_(0xff)                  # NaN: nothing may come from a matrix that nobody wrote
    fragment = torch.empty(sdl.cosine_result_doubles(M), dtype=torch.float64, device="cuda")
    sdl.sdl_outer_grad_cosine_plan(plan, p, g, w, results, fragment, workspace)
    return spans, results, fragment


def _check(spans, results, fragment, M, d, base=0):
    starts = [o - base for o, _, _ in spans]
    want, rest = (torch.zeros(len(spans) + 1, M, M, dtype=torch.float64, device="cuda") for _ in range(2))
    small = [k for k, (_, n, _) in enumerate(spans) if n <= SMALL]                  # these all at once, with zeros behind their ends
    at = torch.arange(SMALL, device="cuda")
    first = torch.tensor([starts[k] for k in small], device="cuda")
    there = at < torch.tensor([spans[k][1] for k in small], device="cuda")[:, None]
    padded = d[:, (first[:, None] + at).clamp(max=d.shape[1] - 1)] * there
    want[small], rest[small] = gram_of(padded.transpose(0, 1).contiguous())
    for k, (_, n, _) in enumerate(spans):
        if n > SMALL:
            want[k], rest[k] = gram_of(d[:, starts[k]:starts[k] + n])
    want[-1], rest[-1] = want[:-1].sum(0), rest[:-1].sum(0)
    got = torch.cat([results[:len(spans), :M * M], fragment[None, :M * M]]).view(-1, M, M)
    norm = torch.diagonal(want, dim1=1, dim2=2).sqrt()
    assert gram_error(got[:-1], want[:-1], rest[:-1]) <= 256
    # the fragment's: as many more as there are sets, on both sides, and what the sum of the sets' exact results rounds
    assert gram_error(got[-1], want[-1], rest[-1]) <= 256 + 2 * len(spans)
    cos = torch.cat([results[:len(spans), M * M:2 * M * M], fragment[None, M * M:2 * M * M]]).view(-1, M, M)
    assert (torch.diagonal(cos, dim1=1, dim2=2)[norm > 0] - 1).abs().max() <= 2.0 ** -50


@pytest.mark.parametrize("M", [1, 2, 5, 8, 9, 12, 16])
@pytest.mark.parametrize("n_sets,large", [(49, {}), (97, {}), (112, {}), (223, {}), (224, {}), (225, {}), (272, {3: 300_000}), (527, {}), (528, {}), (529, {}), (1057, {}),
                                          (100, {60: 8_500_000}), (100, {0: 8_500_000, 99: 2_000_001}), (230, {k: 100_000 + k for k in range(0, 230, 2)})])
def test_sets_over_launches(M, n_sets, large):
    rng = np.random.default_rng(n_sets)
    numel = [int(x) for x in rng.integers(0, 1200, n_sets)]
    numel[1] = numel[n_sets - 2] = 0
    for k, n in large.items():
        numel[k] = n
    plan = sdl.sdl_fragment_plan(numel, [0] * n_sets, 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    gen = torch.Generator("cuda").manual_seed(M)
    g = torch.randn(plan.total_numel, device="cuda", generator=gen)
    w = [(g - torch.randn(g.numel(), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(M)]
    d = torch.stack([(g - x.float()).double() for x in w])
    _check(*_run(plan, 0, M, g, w), M, d)


@pytest.mark.parametrize("M", [2, 9, 13, 16])
def test_sets_behind_element_2_to_the_32(M):
    first = (1 << 32) + 8
    sizes = [first, 1000, 513, 3_700_000, 70_001]
    plan = sdl.sdl_fragment_plan(sizes, [0, 1, 1, 1, 1], 2, 2, sdl.PATTERN_STRIDED, 10, 0)
    rest = sum(sizes[1:])
    g = torch.empty(first + rest, device="cuda")
    w = torch.empty(first + rest, device="cuda", dtype=torch.bfloat16)
    gen = torch.Generator("cuda").manual_seed(M)
    g[first:] = torch.randn(rest, device="cuda", generator=gen)
    w[first:] = g[first:] - torch.randn(rest, device="cuda", generator=gen)
    d = (g[first:] - w[first:].float()).double()[None].expand(M, -1).contiguous()
    _check(*_run(plan, 1, M, g, [w] * M), M, d, first)
