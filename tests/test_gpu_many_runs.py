"""Fragments of many runs: a launch takes up to 272 of them (160 with a whole-span scale), found in groups of 16 by their first
workgroups, and the next launch starts where it ends, in the messages and in staged state too.  Run counts at the edges of a
group and of a launch, against the oracle run by run: the fused step without messages at all of them, the calls that read or write
messages behind the end of a launch.  Runs of odd lengths, whose last tiles take range-checked accesses of single elements, and of
multiples of four, whose last tiles take the wide ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_18512_amd as sdl
import workloads
from gpu_util import HostCopy, assert_bf16_within_ulp, assert_bytes_equal, assert_f32_close, host_bits, host_f32

pytestmark = pytest.mark.gpu


def _lengths(rng, n, odd):
    """Lengths that never join (odd ones, or multiples of 4 and not of 128); some runs take several tiles, so that first workgroups
    are not run numbers."""
    return [int(x) * 2 + 1 if odd else int(x) // 31 * 128 + int(x) % 31 * 4 + 4 for x in rng.integers(0, 700 if odd else 340, n)]


@pytest.mark.parametrize("odd", [True, False])
@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("n_runs", [1, 15, 16, 17, 33, 111, 112, 113, 128, 225, 271, 272, 273, 545])
def test_fused_step_over_many_runs(n_runs, staged, odd):
    rng = np.random.default_rng(n_runs)
    numel = _lengths(rng, n_runs, odd)
    plan = sdl.sdl_fragment_plan(numel, [0] * n_runs, 1, 1, sdl.PATTERN_STRIDED, 10, 1)
    runs = sdl.sdl_plan_fragment_runs(plan, 0)
    assert len(runs) == n_runs
    total, M, fmt = plan.total_numel, 2, sdl.FMT_E3M0
    g, mom, w_send, w_now = workloads.make_span(total, M, tau=1, delta="student_t3", base_seed=n_runs, device="cuda")
    host = HostCopy(g, mom, w_send, w_now)
    if staged:
        pad = [-(-n // 512) * 512 for _, n, _ in runs]
        start = np.concatenate([[0], np.cumsum(pad)])
        assert sdl.sdl_plan_staged_numel(plan, 0) == start[-1]
        gf, mf = torch.zeros(int(start[-1]), device="cuda"), torch.zeros(int(start[-1]), device="cuda")
        for (o, n, _), s in zip(runs, start):
            gf[s:s + n], mf[s:s + n] = g[o:o + n], mom[o:o + n]
        sdl.sdl_fragment_outer_step_staged(plan, 0, gf, mf, w_send, w_now, fmt, 0.7, 0.9, 0.5)
        for (o, n, _), s in zip(runs, start):
            g[o:o + n], mom[o:o + n] = gf[s:s + n], mf[s:s + n]
    else:
        sdl.sdl_fragment_outer_step_plan(plan, 0, g, mom, w_send, w_now, fmt, 0.7, 0.9, 0.5)
    torch.cuda.synchronize()
    for o, n, _ in runs:
        sl = slice(o, o + n)
        oracle.fragment_outer_step(host.g[sl], host.mom[sl], [w[sl] for w in host.w_send], [w[sl] for w in host.w_now],
                                   fmt, 0.7, 0.9, 0.5)
    assert_f32_close(host_f32(g), host.g, "g")
    assert_f32_close(host_f32(mom), host.mom, "mom")
    for m in range(M):
        assert_bf16_within_ulp(host_bits(w_now[m]), host.w_now[m], f"w_now[{m}]")


LR, MU, ALPHA = 0.7, 0.9, 0.5


def _ok(status):
    assert status == 0


def _send(staged, plan, g, w_send, fmt, codes, scales):
    if not staged:
        return sdl.sdl_quantize_outer_grad_plan(plan, 1, g, w_send, fmt, codes, scales)
    _ok(sdl._lib.sdl_quantize_outer_grad_staged(plan._h, 1, g.data_ptr(), sdl._ptr_array(w_send), len(w_send), fmt,
                                                sdl._ptr_array(codes), sdl._ptr_array(scales), sdl._stream(None)))


def _reduce_and_merge(staged, plan, g, mom, codes, scales, w_now, fmt):
    if not staged:
        sdl.sdl_dequant_reduce_nesterov_plan(plan, 1, g, mom, codes, scales, fmt, LR, MU)
        return sdl.sdl_merge_overlap_plan(plan, 1, g, w_now, ALPHA)
    _ok(sdl._lib.sdl_dequant_reduce_nesterov_staged(plan._h, 1, g.data_ptr(), mom.data_ptr(), sdl._ptr_array(codes),
                                                    sdl._ptr_array(scales), len(codes), fmt, LR, MU, sdl._stream(None)))
    _ok(sdl._lib.sdl_merge_overlap_staged(plan._h, 1, g.data_ptr(), sdl._ptr_array(w_now), len(w_now), ALPHA,
                                          sdl._stream(None)))


def _receive(staged, plan, g, mom, codes, scales, w_now, fmt):
    if not staged:
        return sdl.sdl_receive_outer_step_plan(plan, 1, g, mom, codes, scales, w_now, fmt, LR, MU, ALPHA)
    _ok(sdl._lib.sdl_receive_outer_step_staged(plan._h, 1, g.data_ptr(), mom.data_ptr(), sdl._ptr_array(codes),
                                               sdl._ptr_array(scales), sdl._ptr_array(w_now), len(w_now), fmt, LR, MU, ALPHA,
                                               sdl._stream(None)))


@pytest.mark.parametrize("odd", [True, False])
@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("M", [2, 3])                      # tiles of one row and of two
@pytest.mark.parametrize("fmt,n_runs", [(sdl.FMT_E3M0_B128, 273), (sdl.FMT_E3M0_B128, 545), (sdl.FMT_E3M0_SPAN, 161),
                                        (sdl.FMT_E3M0_SPAN, 321), (sdl.FMT_BF16, 272), (sdl.FMT_BF16, 273)])
def test_messages_over_several_launches(n_runs, fmt, M, staged, odd):
    rng = np.random.default_rng(n_runs + M)
    # every second group is the other fragment's: the runs lie apart, the first not at the start
    numel = _lengths(rng, 2 * n_runs, odd)
    plan = sdl.sdl_fragment_plan(numel, [k % 2 for k in range(2 * n_runs)], 2, 2, sdl.PATTERN_STRIDED, 10, 1)
    runs = sdl.sdl_plan_fragment_runs(plan, 1)
    assert len(runs) == n_runs
    g, mom, w_send, w_now = workloads.make_span(plan.total_numel, M, tau=1, delta="student_t3", base_seed=n_runs, device="cuda")
    host = HostCopy(g, mom, w_send, w_now)
    start = np.concatenate([[0], np.cumsum([-(-n // 512) * 512 for _, n, _ in runs])])     # in messages and staged state
    cb, sb = sdl.sdl_plan_message_bytes(plan, 1, fmt)

    def messages():
        return ([torch.zeros(cb, dtype=torch.uint8, device="cuda") for _ in range(M)],
                [torch.zeros(max(sb, 16), dtype=torch.uint8, device="cuda") for _ in range(M)])

    def state():
        if not staged:
            return g.clone(), mom.clone()
        gf, mf = torch.zeros(int(start[-1]), device="cuda"), torch.zeros(int(start[-1]), device="cuda")
        for (o, n, _), s in zip(runs, start):
            gf[s:s + n], mf[s:s + n] = g[o:o + n], mom[o:o + n]
        return gf, mf

    sent, sent_scales = messages()
    g1, m1 = state()
    _send(staged, plan, g1, w_send, fmt, sent, sent_scales)
    g2, m2 = state()
    w2 = [w.clone() for w in w_now]
    _reduce_and_merge(staged, plan, g2, m2, sent, sent_scales, w2, fmt)
    g3, m3 = state()
    w3 = [w.clone() for w in w_now]
    _receive(staged, plan, g3, m3, sent, sent_scales, w3, fmt)
    written, written_scales = messages()
    g4, m4 = state()
    w4 = [w.clone() for w in w_now]
    call = sdl.sdl_fragment_outer_step_staged_ex if staged else sdl.sdl_fragment_outer_step_plan_ex
    call(plan, 1, g4, m4, w_send, w4, fmt, LR, MU, ALPHA, written, written_scales)
    torch.cuda.synchronize()

    want_codes = [np.zeros(cb, np.uint8) for _ in range(M)]
    want_scales = [np.zeros(max(sb, 16), np.uint8) for _ in range(M)]
    for k, (o, n, _) in enumerate(runs):
        sl = slice(o, o + n)
        rc, rs = oracle.fragment_outer_step(host.g[sl], host.mom[sl], [w[sl] for w in host.w_send], [w[sl] for w in host.w_now],
                                            fmt, LR, MU, ALPHA, want_codes=True)
        at, scale_at = sdl.sdl_exchange_bytes(fmt, int(start[k]))
        if fmt == sdl.FMT_E3M0_SPAN:
            scale_at = 4 * k
        for m in range(M):
            want_codes[m][at:at + rc[m].size] = rc[m]
            want_scales[m][scale_at:scale_at + rs[m].size] = rs[m]
    for m in range(M):
        for what, codes, scales in (("send", sent, sent_scales), ("fused", written, written_scales)):
            assert_bytes_equal(codes[m].cpu().numpy(), want_codes[m], f"{what} codes[{m}]")
            assert_bytes_equal(scales[m].cpu().numpy(), want_scales[m], f"{what} scales[{m}]")
    for what, gs, ms, ws in (("reduce, merge", g2, m2, w2), ("receive", g3, m3, w3), ("fused", g4, m4, w4)):
        gs, ms = host_f32(gs), host_f32(ms)
        if staged:
            flat_g, flat_m = host.g.copy(), host.mom.copy()
            for (o, n, _), s in zip(runs, start):
                flat_g[o:o + n], flat_m[o:o + n] = gs[s:s + n], ms[s:s + n]
            gs, ms = flat_g, flat_m
        assert_f32_close(gs, host.g, f"{what} g")
        assert_f32_close(ms, host.mom, f"{what} mom")
        for m in range(M):
            assert_bf16_within_ulp(host_bits(ws[m]), host.w_now[m], f"{what} w_now[{m}]")
