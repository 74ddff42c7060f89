"""Model arrays at any element: workgroups take their tiles in chunks of 2048 parameters per XCD, in groups of 64 (tiles of one
row) or 32 workgroups (tiles of two), and one by one behind the last whole group.  Numbers of tiles around those groups,
against the oracle; the messages of the send side and the merge walk the same order."""
import pytest
import torch

import oracle
import paper_2501_18512_amd as sdl
import workloads
from gpu_util import (HostCopy, assert_bf16_within_ulp, assert_bytes_equal, check_fused_against_oracle, host_bits)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,row", [(2, 256), (3, 512)])
@pytest.mark.parametrize("tiles", [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191])
def test_chunks_of_tiles(tiles, M, row):
    for n in (tiles * row, tiles * row - 1, tiles * row - row + 1):
        g, mom, w_send, w_now = workloads.make_span(n + 1, M, tau=1, delta="student_t3", base_seed=n, device="cuda")
        g, mom, w_send, w_now = g[1:], mom[1:], [w[1:] for w in w_send], [w[1:] for w in w_now]
        codes, scales = sdl.alloc_exchange(sdl.FMT_E3M0, n, M)
        sdl.sdl_quantize_outer_grad(g, w_send, n, sdl.FMT_E3M0, codes, scales)
        merged = [torch.cat([w[:1], w])[1:] for w in w_now]            # at an odd element again
        sdl.sdl_merge_overlap(g, merged, n, 0.5)
        torch.cuda.synchronize()
        ref = HostCopy(g, mom, w_send, w_now)
        rc, rs = oracle.quantize_outer_grad(ref.g, ref.w_send, sdl.FMT_E3M0)
        oracle.merge_overlap(ref.g, ref.w_now, 0.5)
        for m in range(M):
            assert_bytes_equal(codes[m][:rc[m].size].cpu().numpy(), rc[m], f"n={n} codes[{m}]")
            assert_bytes_equal(scales[m][:rs[m].size].cpu().numpy(), rs[m], f"n={n} scales[{m}]")
            assert_bf16_within_ulp(host_bits(merged[m]), ref.w_now[m], f"n={n} merged[{m}]")
        check_fused_against_oracle(g, mom, w_send, w_now, sdl.FMT_E3M0, 0.7, 0.9, 0.5, emit=False, what=f"n={n}")
