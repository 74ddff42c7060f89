"""Helpers of the GPU parity tests: host copies for the oracle and the comparison bars.

Bars (from the benchmark spec of this repository): codes, scale bytes and schedule
bit-exact; fp32 global parameters and momentum rtol 1e-6 / atol 1e-7; bf16 replicas
within one bf16 ulp.
"""
import numpy as np
import torch

import oracle
import paper_2501_18512_amd as sdl
import workloads

RTOL, ATOL = 1e-6, 1e-7
FMT_NAMES = {0: "fp32", 1: "bf16", 2: "e4m3", 3: "e3m0", 4: "e3m0_b64", 5: "e3m0_b128", 6: "e3m0_span", 7: "e3m0_rn"}


def host_f32(t):
    return t.detach().cpu().numpy().copy()


def host_bits(t):
    return workloads.bf16_bits(t)


def assert_f32_close(got, want, what):
    got, want = np.asarray(got), np.asarray(want)
    assert got.shape == want.shape, (what, got.shape, want.shape)
    nan_g, nan_w = np.isnan(got), np.isnan(want)
    assert np.array_equal(nan_g, nan_w), f"{what}: NaN positions differ"
    ok = np.isclose(got, want, rtol=RTOL, atol=ATOL, equal_nan=True)
    if not ok.all():
        i = int(np.argmin(ok))
        raise AssertionError(f"{what}: {int((~ok).sum())} of {ok.size} out of tolerance, first at {i}: "
                             f"got {got[i]!r} want {want[i]!r}")


def _bf16_key(bits):
    """Monotonic integer key of bf16 bit patterns (so that neighbours differ by 1)."""
    b = bits.astype(np.int32)
    return np.where(b & 0x8000, -(b & 0x7fff), b & 0x7fff)


def assert_bf16_within_ulp(got_bits, want_bits, what):
    nan_g = (got_bits & 0x7fff) > 0x7f80
    nan_w = (want_bits & 0x7fff) > 0x7f80
    assert np.array_equal(nan_g, nan_w), f"{what}: NaN positions differ"
    d = np.abs(_bf16_key(got_bits) - _bf16_key(want_bits))
    d[nan_g] = 0
    if d.max(initial=0) > 1:
        i = int(np.argmax(d))
        raise AssertionError(f"{what}: {int((d > 1).sum())} elements differ by more than one bf16 ulp, "
                             f"first at {i}: got {got_bits[i]:#06x} want {want_bits[i]:#06x}")
    return int((d != 0).sum())


def assert_bytes_equal(got, want, what):
    got, want = np.asarray(got), np.asarray(want)
    assert got.shape == want.shape, (what, got.shape, want.shape)
    if not np.array_equal(got, want):
        bad = np.nonzero(got != want)[0]
        i = int(bad[0])
        raise AssertionError(f"{what}: {bad.size} of {got.size} bytes differ, first at {i}: "
                             f"got {got[i]:#04x} want {want[i]:#04x}")


class HostCopy:
    """Host snapshot of one span's state, in the oracle's array types."""

    def __init__(self, g, mom, w_send, w_now):
        self.g, self.mom = host_f32(g), host_f32(mom)
        self.w_send = [host_bits(w) for w in w_send]
        aliased = all(a is b or a.data_ptr() == b.data_ptr() for a, b in zip(w_send, w_now))
        self.w_now = self.w_send if aliased else [host_bits(w) for w in w_now]


def check_fused_against_oracle(g, mom, w_send, w_now, fmt, lr, mu, alpha, *, emit=True, threads=8,
                               what=""):
    """Run the fused GPU step in place on device tensors and the oracle on a host copy of the
    same bits; compare everything.  Returns the host copy after the step."""
    n = g.numel()
    ref = HostCopy(g, mom, w_send, w_now)
    codes = scales = None
    if emit:
        codes, scales = sdl.alloc_exchange(fmt, n, len(w_send), device=g.device)
    elif fmt == sdl.FMT_E3M0_SPAN:
        scales = sdl.alloc_exchange(fmt, n, len(w_send), device=g.device)[1]   # workspace for the span maximum
    sdl.sdl_fragment_outer_step(g, mom, w_send, w_now, n, fmt, lr, mu, alpha, codes, scales)
    torch.cuda.synchronize()
    if emit:
        rc, rs = oracle.fragment_outer_step(ref.g, ref.mom, ref.w_send, ref.w_now, fmt, lr, mu, alpha,
                                            want_codes=True)
        cb, sb = sdl.sdl_exchange_bytes(fmt, n)
        for m in range(len(w_send)):
            assert_bytes_equal(codes[m][:cb].cpu().numpy(), rc[m], f"{what} codes[{m}]")
            if sb:
                assert_bytes_equal(scales[m][:sb].cpu().numpy(), rs[m], f"{what} scales[{m}]")
    else:
        oracle.fragment_outer_step_chunked(ref.g, ref.mom, ref.w_send, ref.w_now, fmt, lr, mu, alpha,
                                           threads=threads)
    assert_f32_close(host_f32(g), ref.g, f"{what} g")
    assert_f32_close(host_f32(mom), ref.mom, f"{what} mom")
    for m in range(len(w_now)):
        assert_bf16_within_ulp(host_bits(w_now[m]), ref.w_now[m], f"{what} w_now[{m}]")
    return ref


# ------------------------------------------------------------------ whole-model state

class FlatModel:
    """The M replicas, global parameters and momentum of a decoder-shaped model as flat device
    arrays (the layout sdl_fragment_outer_step_plan works on)."""

    def __init__(self, wl: "workloads.Workload", device="cuda", fill_fragments=None):
        shape = workloads.SHAPES[wl.shape]
        self.wl = wl
        self.numel, self.block, self.names = shape.units()
        self.L = shape.n_layers
        self.plan = sdl.sdl_fragment_plan(self.numel, self.block, self.L, wl.P, sdl.PATTERN_STRIDED,
                                          wl.H, wl.tau)
        total = self.plan.total_numel
        # one allocation, carved as the library recommends: the layout bench.py times
        self.g, self.mom, self.w_send, self.w_now, self.pool = sdl.alloc_flat_model(total, wl.M, wl.tau > 0,
                                                                                    device=device)
        frags = range(wl.P) if fill_fragments is None else fill_fragments
        for p in frags:
            self.fill_fragment(p)

    def fill_fragment(self, p):
        for off, n, unit in sdl.sdl_plan_fragment_spans(self.plan, p):
            sl = slice(off, off + n)
            workloads.fill_span(self.g[sl], self.mom[sl], [w[sl] for w in self.w_send],
                                [w[sl] for w in self.w_now], unit=unit, tau=self.wl.tau,
                                delta=self.wl.delta, base_seed=self.wl.seed)

    def step(self, p, fmt=None, alpha=None):
        wl = self.wl
        sdl.sdl_fragment_outer_step_plan(self.plan, p, self.g, self.mom, self.w_send, self.w_now,
                                         sdl.FORMATS[wl.fmt] if fmt is None else fmt, wl.lr, wl.mu,
                                         wl.alpha if alpha is None else alpha)

    def windows(self, p, n_random=16, width=1 << 16, seed=0):
        """Block-aligned sample windows inside fragment p: the first and last `width` elements of
        every span plus n_random random ones.  (offset, length) in flat-model elements."""
        rng = np.random.default_rng(seed)
        spans = sdl.sdl_plan_fragment_spans(self.plan, p)
        out = []
        for off, n, _ in spans:
            w = min(width, n)
            out.append((off, w))
            if n > w:
                tail = (n - w) // 32 * 32            # keep windows on the span's 32-element grid
                out.append((off + tail, n - tail))
        big = [(off, n) for off, n, _ in spans if n > 4 * width]
        for _ in range(n_random if big else 0):
            off, n = big[int(rng.integers(len(big)))]
            start = int(rng.integers(0, (n - width) // 32)) * 32
            out.append((off + start, width))
        return out

    def snapshot(self, windows):
        return [HostCopy(self.g[o:o + n], self.mom[o:o + n], [w[o:o + n] for w in self.w_send],
                         [w[o:o + n] for w in self.w_now]) for o, n in windows]

    def verify(self, windows, snaps, fmt=None, alpha=None, what=""):
        """Advance each snapshot with the oracle and compare with the device state."""
        wl = self.wl
        fmt = sdl.FORMATS[wl.fmt] if fmt is None else fmt
        alpha = wl.alpha if alpha is None else alpha
        changed = 0
        for (o, n), ref in zip(windows, snaps):
            oracle.fragment_outer_step_chunked(ref.g, ref.mom, ref.w_send, ref.w_now, fmt, wl.lr, wl.mu,
                                               alpha, threads=8)
            tag = f"{what} window@{o}+{n}"
            assert_f32_close(host_f32(self.g[o:o + n]), ref.g, tag + " g")
            assert_f32_close(host_f32(self.mom[o:o + n]), ref.mom, tag + " mom")
            for m in range(wl.M):
                changed += assert_bf16_within_ulp(host_bits(self.w_now[m][o:o + n]), ref.w_now[m],
                                                  tag + f" w_now[{m}]")
        return changed


# ------------------------------------------------------------- sums of products, exactly

def _two_sum(a, b):
    s = a + b
    v = s - a
    return s, (a - (s - v)) + (b - v)


def gram_of(d):
    """Gram matrices of d [..., M, n], fp32 numbers held as fp64, each as a pair of fp64 matrices: products of two fp32 numbers are exact in fp64, and
    they are folded in halves with the error of every addition kept, which leaves about 1e-30."""
    M = d.shape[-2]
    want, rest = (torch.zeros(*d.shape[:-1], M, dtype=torch.float64, device=d.device) for _ in range(2))
    if d.shape[-1] == 0:
        return want, rest
    pad = torch.nn.functional.pad
    for a in range(M):
        hi = d[..., a:a + 1, :] * d[..., a:, :]
        lo = torch.zeros_like(hi)
        while hi.shape[-1] > 1:
            n, h = hi.shape[-1], (hi.shape[-1] + 1) // 2
            hi, err = _two_sum(hi[..., :h], pad(hi[..., h:], (0, 2 * h - n)))
            lo = lo[..., :h] + pad(lo[..., h:], (0, 2 * h - n)) + err
        for out, x in ((want, hi), (rest, lo)):
            out[..., a, a:] = x[..., 0]
            out[..., a:, a] = x[..., 0]
    return want, rest


def exact_gram(g, w, chunk=1 << 22):
    """The Gram matrix of the outer gradients g - w[m], as a pair of fp64 matrices."""
    want, rest = gram_of(torch.zeros(len(w), 0, dtype=torch.float64, device=g.device))
    for lo in range(0, g.numel(), chunk):
        part, part_rest = gram_of(torch.stack([(g[lo:lo + chunk] - x[lo:lo + chunk].float()).double() for x in w]))
        want, err = _two_sum(want, part)
        rest = rest + part_rest + err
    return want, rest


def gram_error(got, want, rest):
    """Largest error in units of 2^-53 sqrt(G[a][a] G[b][b]): at most the number of fp64 additions that an entry's products go through one after
    the other, as each rounds a sum of at most that size to 2^-53 of it."""
    norm = torch.diagonal(want, dim1=-2, dim2=-1).sqrt()
    unit = 2.0 ** -53 * norm[..., :, None] * norm[..., None, :]
    error = ((got - want) - rest).abs()
    assert (error[unit == 0] == 0).all()
    return float((error / unit)[unit > 0].max()) if (unit > 0).any() else 0.0
