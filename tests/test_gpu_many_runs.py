"""Fragments of many runs: a launch takes up to 112 of them, found in groups of 16 by their first workgroups, and the next
launch starts where it ends.  Run counts at the edges of a group and of a launch, against the oracle run by run."""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_18512_amd as sdl
import workloads
from gpu_util import HostCopy, assert_bf16_within_ulp, assert_f32_close, host_bits, host_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("n_runs", [1, 15, 16, 17, 33, 111, 112, 113, 128, 225])
def test_fused_step_over_many_runs(n_runs, staged):
    rng = np.random.default_rng(n_runs)
    # odd sizes never join, and some runs take several tiles, so that first workgroups are not run numbers
    numel = [int(n) * 2 + 1 for n in rng.integers(0, 700, n_runs)]
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
