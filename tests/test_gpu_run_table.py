"""Where a run starts and ends decides how its tiles reach memory.  Runs on multiples of four elements in 16-byte aligned arrays,
their ragged last tiles too, take the buffer path under a range check as long as what is left; the same model one element
further takes the path for any alignment, and both must give the same bits: every call, every kind of format, replica counts with
and without a variant of their own.  Lengths at the edges of a lane, a scale block, a row and a tile.

A launch takes up to 272 runs (160 with a whole-span scale); counts at the edges of that, against the same path."""
import pytest
import torch

import paper_2501_18512_amd as sdl
import workloads

pytestmark = pytest.mark.gpu

LR, MU, ALPHA = 0.7, 0.9, 0.5
EDGES = [4, 8, 28, 32, 36, 60, 68, 124, 132, 252, 256, 260, 508, 512, 516, 764, 772, 1020, 1028, 2052, 4 * 1031]


def _plan(numel):
    return sdl.sdl_fragment_plan(numel, [0] * len(numel), 1, 1, sdl.PATTERN_STRIDED, 10, 1)


def _model(total, M, shift, seed):
    g0, _, s0, n0 = workloads.make_span(total, M, tau=1, delta="student_t3", base_seed=seed, device="cuda")
    gen = torch.Generator("cuda").manual_seed(seed)
    mom0 = torch.randn(total, device="cuda", generator=gen) * 1e-3

    def at(x):
        y = torch.zeros(total + shift + 64, dtype=x.dtype, device="cuda")[shift:shift + total]
        return y.copy_(x)

    return at(g0), at(mom0), [at(x) for x in s0], [at(x) for x in n0]


def _messages(plan, fmt, M):
    cb, sb = sdl.sdl_plan_message_bytes(plan, 0, fmt)
    return ([torch.full((max(cb, 16),), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(M)],
            [torch.full((max(sb, 16),), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(M)])


def _all_calls(numel, fmt, M, shift):
    """Everything that the calls write, for a model whose arrays start `shift` elements behind an aligned address."""
    plan, out = _plan(numel), []
    total = plan.total_numel
    g, mom, ws, wn = _model(total, M, shift, M)
    codes, scales = _messages(plan, fmt, M)
    sdl.sdl_quantize_outer_grad_plan(plan, 0, g, ws, fmt, codes, scales)
    out += codes + scales
    g2, mom2, wn2 = g.clone(), mom.clone(), [w.clone() for w in wn]
    if shift:                                         # clones are aligned
        g2, mom2, _, wn2 = _model(total, M, shift, M)
    sdl.sdl_receive_outer_step_plan(plan, 0, g2, mom2, codes, scales, wn2, fmt, LR, MU, ALPHA)
    out += [g2, mom2] + wn2
    g3, mom3, _, wn3 = _model(total, M, shift, M)
    sdl.sdl_dequant_reduce_nesterov_plan(plan, 0, g3, mom3, codes, scales, fmt, LR, MU)
    sdl.sdl_merge_overlap_plan(plan, 0, g3, wn3, ALPHA)
    out += [g3, mom3] + wn3
    g4, mom4, ws4, wn4 = _model(total, M, shift, M)
    codes4, scales4 = _messages(plan, fmt, M)
    sdl.sdl_fragment_outer_step_plan_ex(plan, 0, g4, mom4, ws4, wn4, fmt, LR, MU, ALPHA, codes4, scales4)
    out += codes4 + scales4 + [g4, mom4] + wn4
    sdl.sdl_fragment_outer_step_plan_static(plan, 0, g, mom, ws, wn, fmt, LR, MU, ALPHA)
    out += [g, mom] + wn
    g5, mom5, ws5, _ = _model(total, M, shift, M)
    sdl.sdl_fragment_outer_step_plan_static(plan, 0, g5, mom5, ws5, ws5, fmt, LR, MU, ALPHA)
    return out + [g5, mom5] + ws5


def _same(a, b):
    assert len(a) == len(b)
    for k, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x.contiguous().view(torch.uint8), y.contiguous().view(torch.uint8)), f"output {k}"


@pytest.mark.parametrize("M", [1, 2, 3, 4, 6, 8, 16])
@pytest.mark.parametrize("fmt", ["e3m0", "e3m0_b128", "e3m0_span", "e4m3", "bf16", "fp32"])
def test_aligned_runs_and_tails_give_what_any_alignment_gives(fmt, M):
    _same(_all_calls(EDGES, sdl.FORMATS[fmt], M, 0), _all_calls(EDGES, sdl.FORMATS[fmt], M, 1))


@pytest.mark.parametrize("n_runs", [159, 160, 161, 271, 272, 273, 321, 545])
@pytest.mark.parametrize("fmt", ["e3m0", "e3m0_span"])
def test_more_runs_than_a_launch_takes(fmt, n_runs):
    numel = [EDGES[i % 17] + 4 * (i % 3) * 67 + 4 for i in range(n_runs)]
    plan = _plan(numel)
    F, M = sdl.FORMATS[fmt], 2
    assert len(sdl.sdl_plan_fragment_runs(plan, 0)) > 0.9 * n_runs     # (a few join their neighbours)
    whole = _all_calls(numel, F, M, 0)
    _same(whole, _all_calls(numel, F, M, 1))
    # run by run through the calls for one span
    g, mom, ws, wn = _model(plan.total_numel, M, 0, M)
    for o, n, _ in (sdl.sdl_plan_fragment_spans(plan, 0) if fmt == "e3m0_span" else sdl.sdl_plan_fragment_runs(plan, 0)):
        codes, scales = sdl.alloc_exchange(F, n, M, device="cuda")
        sdl.sdl_fragment_outer_step(g[o:o + n], mom[o:o + n], [w[o:o + n] for w in ws], [w[o:o + n] for w in wn], n, F, LR, MU, ALPHA,
                                    codes, scales)
    fused = whole[-2 * (2 + M):-(2 + M)]
    _same(fused, [g, mom] + wn)


@pytest.mark.parametrize("M", [1, 2, 3, 4, 8])
@pytest.mark.parametrize("fmt", ["e3m0", "e3m0_span", "e4m3", "bf16"])
def test_long_runs_off_16_bytes_give_what_any_alignment_gives(fmt, M):
    """From 65536 parameters a run that starts on a multiple of four elements and not of eight takes the path for any alignment in
    every call but the send: lengths around that, each off 16 bytes and on them, against the same model one element further."""
    numel = [4, 65532, 65532, 65540, 65548, 131076, 4, 65536]
    assert {sum(numel[:k]) % 8 for k in (1, 3, 5, 7)} == {4} and {sum(numel[:k]) % 8 for k in (2, 4)} == {0}
    _same(_all_calls(numel, sdl.FORMATS[fmt], M, 0), _all_calls(numel, sdl.FORMATS[fmt], M, 1))
