"""The absolute-maximum pre-pass of the whole-span scale: numbers of wavefronts at the edges of its rules (one for 16 tiles of
512 parameters, 1024 to 8192 of them; up to 64 spans a launch, found by their first workgroups), the maximum in the first and
the last element of every span, scale words that hold something else before the call, model arrays at any element."""
import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_spans,numel", [(1, 1), (3, 511), (1, 512 * 1024 + 1), (2, 512 * 16 * 1024 + 512 + 7), (33, 4099),
                                           (64, 513), (65, 513), (130, 100), (1, 512 * 16 * 8192 + 33)])
@pytest.mark.parametrize("M", [1, 3, 9])
def test_scale_words_are_the_spans_maxima(n_spans, numel, M):
    if n_spans * numel > 1 << 26 and M > 1:
        pytest.skip("the largest size once")
    sizes = [numel + k % 3 for k in range(n_spans)]            # spans at any element
    plan = sdl.sdl_fragment_plan(sizes, [0] * n_spans, 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    total = plan.total_numel
    gen = torch.Generator("cuda").manual_seed(n_spans)
    g = torch.randn(total, device="cuda", generator=gen) * 1e-3
    w = [torch.zeros(total, dtype=torch.bfloat16, device="cuda") for _ in range(M)]
    spans = sdl.sdl_plan_fragment_spans(plan, 0)
    for k, (o, n, _) in enumerate(spans):
        for m in range(M):
            w[m][o if (k + m) % 2 else o + n - 1] = -1.0 - k - m
    cb, sb = sdl.sdl_plan_message_bytes(plan, 0, sdl.FMT_E3M0_SPAN)
    codes = [torch.zeros(max(cb, 16), dtype=torch.uint8, device="cuda") for _ in range(M)]
    scales = [torch.full((sb,), 0x7f, dtype=torch.uint8, device="cuda") for _ in range(M)]
    sdl.sdl_quantize_outer_grad_plan(plan, 0, g, w, sdl.FMT_E3M0_SPAN, codes, scales)
    for m in range(M):
        want = np.array([float((g[o:o + n] - w[m][o:o + n].float()).abs().max()) for o, n, _ in spans], np.float32)
        assert np.array_equal(scales[m].cpu().numpy().view(np.float32), want), f"replica {m}"
