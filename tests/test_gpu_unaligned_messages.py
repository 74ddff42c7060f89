"""Message arrays at any byte (4- and 8-bit codes) or element (bf16, fp32): messages packed back to back.  Whole tiles go
through element-aligned vectors, the ragged last one through range-checked accesses; sizes at the edges of rows and tiles."""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_18512_amd as sdl
import workloads
from gpu_util import HostCopy, assert_bf16_within_ulp, assert_bytes_equal, assert_f32_close, host_bits, host_f32

pytestmark = pytest.mark.gpu
FMTS = [sdl.FMT_E3M0, sdl.FMT_E4M3, sdl.FMT_BF16, sdl.FMT_FP32, sdl.FMT_E3M0_B128, sdl.FMT_E3M0_SPAN]


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("M", [1, 3, 4])
@pytest.mark.parametrize("shift", [1, 7])
def test_packed_messages(fmt, M, shift):
    width = {sdl.FMT_BF16: 2, sdl.FMT_FP32: 4}.get(fmt, 1)
    for n in (1, 3, 254, 255, 256, 257, 511, 512, 513, 769, 1025, 5 * 512 + 31):
        cb, sb = sdl.sdl_exchange_bytes(fmt, n)
        g, mom, w_send, w_now = workloads.make_span(n, M, tau=1, delta="student_t3", base_seed=n, device="cuda")
        ref = HostCopy(g, mom, w_send, w_now)
        # every code array starts `shift` elements behind the last one's end; 0xa5 must survive in between
        step = cb + shift * width
        wire = torch.full((M * step + 16,), 0xa5, dtype=torch.uint8, device="cuda")
        codes = [wire[shift * width + m * step:][:cb] for m in range(M)]
        scales = [torch.zeros(max(sb, 4), dtype=torch.uint8, device="cuda") for _ in range(M)]
        sdl.sdl_quantize_outer_grad(g, w_send, n, fmt, codes, scales)
        rc, rs = oracle.quantize_outer_grad(ref.g, ref.w_send, fmt)
        got = wire.cpu().numpy()
        want = np.full_like(got, 0xa5)
        for m in range(M):
            want[shift * width + m * step:][:cb] = rc[m]
            if sb:
                assert_bytes_equal(scales[m][:sb].cpu().numpy(), rs[m], f"n={n} scales[{m}]")
        assert_bytes_equal(got, want, f"n={n} packed codes")
        sdl.sdl_receive_outer_step(g, mom, codes, scales, w_now, n, fmt, 0.7, 0.9, 0.5)
        torch.cuda.synchronize()
        oracle.dequant_reduce_nesterov(ref.g, ref.mom, rc, rs, fmt, 0.7, 0.9)
        oracle.merge_overlap(ref.g, ref.w_now, 0.5)
        assert_f32_close(host_f32(g), ref.g, f"n={n} g")
        assert_f32_close(host_f32(mom), ref.mom, f"n={n} mom")
        for m in range(M):
            assert_bf16_within_ulp(host_bits(w_now[m]), ref.w_now[m], f"n={n} w_now[{m}]")


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("M", [1, 2, 4, 8])
@pytest.mark.parametrize("shift", [1, 7])
def test_packed_messages_of_the_other_calls(fmt, M, shift):
    """The receive side without the merge (tiles of one row), and the fused step that writes the messages."""
    width = {sdl.FMT_BF16: 2, sdl.FMT_FP32: 4}.get(fmt, 1)
    for n in (3, 255, 256, 257, 511, 512, 513, 3 * 512 + 31):
        cb, sb = sdl.sdl_exchange_bytes(fmt, n)
        g, mom, w_send, w_now = workloads.make_span(n, M, tau=1, delta="student_t3", base_seed=n, device="cuda")
        ref = HostCopy(g, mom, w_send, w_now)
        step = cb + shift * width
        wire = torch.full((M * step + 16,), 0xa5, dtype=torch.uint8, device="cuda")
        codes = [wire[shift * width + m * step:][:cb] for m in range(M)]
        scales = [torch.zeros(max(sb, 4), dtype=torch.uint8, device="cuda") for _ in range(M)]
        g2, mom2, w2 = g.clone(), mom.clone(), [w.clone() for w in w_now]
        sdl.sdl_fragment_outer_step(g2, mom2, w_send, w2, n, fmt, 0.7, 0.9, 0.5, codes, scales)
        sdl.sdl_dequant_reduce_nesterov(g, mom, codes, scales, n, fmt, 0.7, 0.9)
        sdl.sdl_merge_overlap(g, w_now, n, 0.5)
        torch.cuda.synchronize()
        rc, rs = oracle.fragment_outer_step(ref.g, ref.mom, ref.w_send, ref.w_now, fmt, 0.7, 0.9, 0.5, want_codes=True)
        got = wire.cpu().numpy()
        want = np.full_like(got, 0xa5)
        for m in range(M):
            want[shift * width + m * step:][:cb] = rc[m]
            if sb:
                assert_bytes_equal(scales[m][:sb].cpu().numpy(), rs[m], f"n={n} scales[{m}]")
        assert_bytes_equal(got, want, f"n={n} packed codes")
        for what, gs, ms, ws in (("reduce, merge", g, mom, w_now), ("fused", g2, mom2, w2)):
            assert_f32_close(host_f32(gs), ref.g, f"{what} n={n} g")
            assert_f32_close(host_f32(ms), ref.mom, f"{what} n={n} mom")
            for m in range(M):
                assert_bf16_within_ulp(host_bits(ws[m]), ref.w_now[m], f"{what} n={n} w_now[{m}]")
