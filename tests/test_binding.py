"""The extension module that converts the arguments of the device calls (CPU only): with functions in the library's place that note what
they are called with, every argument arrives where the C interface has it, as ctypes would convert it; and what the
binding refuses is refused before the library is called."""
import ctypes
import decimal
import fractions
import inspect
import os
import struct
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl

NAMES = sorted(n for n in dir(sdl._binding) if n.startswith("sdl_"))
LISTS = {"w_send", "w_now", "w_send_base", "w_now_base", "codes", "scales"}
SCALARS = {"n": 123_456_789_012, "fmt": 3, "p": 7, "lr": 0.7, "mu": 0.9, "alpha": 0.25, "stream": 0x5700}


class Tensor:
    def __init__(self, at, on_device=True, contiguous=True):
        self.at, self.is_cuda, self.contiguous = at, on_device, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.at


class Owner:
    _h = ctypes.c_void_p(0x7777000011)


def _real():
    return {n: ctypes.cast(getattr(sdl._lib, n), ctypes.c_void_p).value for n in NAMES}


@pytest.fixture
def calls():
    """What the library's functions are called with: name -> argument tuples, arrays of addresses as lists of 16."""
    seen, kept, table = {}, [], {}
    for name in NAMES:
        types = getattr(sdl._lib, name).argtypes

        def note(*args, name=name):
            seen.setdefault(name, []).append(args)
            return 0
        f = ctypes.CFUNCTYPE(ctypes.c_int, *types)(note)
        kept.append(f)
        table[name] = ctypes.cast(f, ctypes.c_void_p).value
    hooks = (sdl._stream, torch.cuda.is_initialized, sdl._get_device, sdl._raw_stream)
    sdl._binding.setup(table, *hooks)
    yield seen
    sdl._binding.setup(_real(), *hooks)


def _arguments(name, M):
    """Arguments of the binding's function, and what the C function of that name is to get (lists: M addresses)."""
    given, at = {}, 0x100000000
    for k in inspect.signature(getattr(sdl, name)).parameters:
        if k == "plan":
            given[k] = Owner()
        elif k in LISTS:
            given[k] = [Tensor(at + 64 * i) for i in range(M)]
        elif k in SCALARS:
            given[k] = SCALARS[k]
        else:
            given[k] = Tensor(at)
        at += 0x10000
    return given


def _as_c(given):
    """The arguments in the order of the C interface: the plan first, M behind the last list of replicas (or the codes), the lists of
    messages where that interface has them."""
    out = []
    for k, v in given.items():
        if k == "plan":
            out.append(("plan", Owner._h.value))
        elif k in LISTS:
            out.append((k, [t.at for t in v]))
        elif k in SCALARS:
            out.append((k, v))
        else:
            out.append((k, v.at))
    return dict(out)


C_ORDER = {
    "sdl_quantize_outer_grad": "g w_send M n fmt codes scales stream",
    "sdl_dequant_reduce_nesterov": "g mom codes scales M n fmt lr mu stream",
    "sdl_merge_overlap": "g_new w_now M n alpha stream",
    "sdl_receive_outer_step": "g mom codes scales w_now M n fmt lr mu alpha stream",
    "sdl_fragment_outer_step": "g mom w_send w_now M n fmt lr mu alpha codes scales stream",
    "sdl_quantize_outer_grad_plan": "plan p g_base w_send_base M fmt codes scales stream",
    "sdl_dequant_reduce_nesterov_plan": "plan p g_base mom_base codes scales M fmt lr mu stream",
    "sdl_merge_overlap_plan": "plan p g_new_base w_now_base M alpha stream",
    "sdl_receive_outer_step_plan": "plan p g_base mom_base codes scales w_now_base M fmt lr mu alpha stream",
    "sdl_fragment_outer_step_plan": "plan p g_base mom_base w_send_base w_now_base M fmt lr mu alpha stream",
    "sdl_fragment_outer_step_plan_static": "plan p g_base mom_base w_send_base w_now_base M fmt lr mu alpha stream",
    "sdl_fragment_outer_step_plan_ex": "plan p g_base mom_base w_send_base w_now_base M fmt lr mu alpha codes scales stream",
    "sdl_fragment_outer_step_staged_ex": "plan p g_frag mom_frag w_send_base w_now_base M fmt lr mu alpha codes scales stream",
}


def test_every_function_is_checked():
    assert sorted(C_ORDER) == NAMES


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("M", [1, 3, 16])
def test_arguments_arrive(calls, name, M):
    given = _arguments(name, M)
    want = dict(_as_c(given), M=M)
    arrays = {}

    def look(*args):
        for k, v in zip(C_ORDER[name].split(), args):
            if k in LISTS:
                arrays[k] = list((ctypes.c_uint64 * M).from_address(v))
        return 0
    f = ctypes.CFUNCTYPE(ctypes.c_int, *getattr(sdl._lib, name).argtypes)(look)
    getattr(sdl, name)(*given.values())
    (got,) = calls[name]
    assert len(got) == len(C_ORDER[name].split())
    for k, v in zip(C_ORDER[name].split(), got):
        if k in ("lr", "mu", "alpha"):
            assert v == float(np.float32(want[k])), k
        elif k not in LISTS:
            assert v == want[k], k
    table = dict(_real(), **{name: ctypes.cast(f, ctypes.c_void_p).value})
    sdl._binding.setup(table, sdl._stream, torch.cuda.is_initialized, sdl._get_device, sdl._raw_stream)
    getattr(sdl, name)(*given.values())           # arrays are looked at while the call lasts
    assert arrays == {k: want[k] for k in C_ORDER[name].split() if k in LISTS}


@pytest.mark.parametrize("name", NAMES)
def test_what_is_refused(calls, name):
    given = _arguments(name, 2)
    call = getattr(sdl, name)
    tensors = [k for k in given if k not in SCALARS and k != "plan"]
    for k in tensors:
        for bad in (Tensor(64, on_device=False), Tensor(64, contiguous=False), torch.zeros(4)):
            with pytest.raises(ValueError):
                call(*dict(given, **{k: [given[k][0], bad] if k in LISTS else bad}).values())
        with pytest.raises(AttributeError):
            call(*dict(given, **{k: ["x", "y"] if k in LISTS else object()}).values())
    counted = [k for k in tensors if k in ("w_send", "w_now", "w_send_base", "w_now_base")] or ["codes"]
    if name == "sdl_fragment_outer_step_staged_ex":
        counted = counted[:1]                    # the replicas are as many as in w_send
    with pytest.raises(TypeError):
        call(*dict(given, **{counted[-1]: None}).values())
    with pytest.raises(TypeError):
        call(*dict(given, **{counted[-1]: (t for t in given[counted[-1]])}).values())
    if len(counted) == 2:
        with pytest.raises(sdl.SdlError):
            call(*dict(given, **{counted[0]: given[counted[0]][:1]}).values())
    for k in ("n", "fmt", "p"):
        if k in given:
            with pytest.raises(TypeError):
                call(*dict(given, **{k: 1.0}).values())
    assert not calls
    # accepted as ever: addresses, missing messages, integers and numbers of other kinds, more replicas than the library takes (for it to refuse)
    plain = {k: [x.at for x in v] if k in LISTS else v.at if isinstance(v, Tensor) else v for k, v in given.items()}
    plain.update({k: None for k in ("scales",) if k in given}, **{k: np.int64(v) for k, v in given.items() if k in ("n", "fmt", "p")},
                 **{k: np.float32(v) for k, v in given.items() if k in ("lr", "mu", "alpha")})
    call(*plain.values())
    call(*{k: v * 20 if k in LISTS else v for k, v in given.items()}.values())
    assert calls[name][0][C_ORDER[name].split().index("M")] == 2 and calls[name][1][C_ORDER[name].split().index("M")] == 40


def test_too_many_replicas_are_refused_by_the_library():
    given = _arguments("sdl_quantize_outer_grad", 17)
    with pytest.raises(sdl.SdlError):
        sdl.sdl_quantize_outer_grad(*given.values())


def test_a_plan_that_has_been_given_back():
    given = _arguments("sdl_merge_overlap_plan", 2)
    given["plan"]._h = None
    with pytest.raises(sdl.SdlError):
        sdl.sdl_merge_overlap_plan(*given.values())


CHANGES_ITS_LIST = r"""
import sys
import paper_2501_18512_amd as sdl

class Tensor:
    is_cuda = True
    def __init__(self, at): self.at = at
    def is_contiguous(self): return True
    def data_ptr(self): return self.at

class Clears(Tensor):
    def is_contiguous(self):
        tensors.clear()
        junk.extend(Tensor(7) for _ in range(1000))      # what was freed is used again
        return True

junk = []
tensors = [Clears(0)] + [Tensor(0) for _ in range(11)]   # null addresses: the library refuses them
try:
    sdl.sdl_merge_overlap(Tensor(64), tensors, 1, 0.5, stream=0)
except sdl.SdlError as e:
    print("refused", e.status, len(tensors))
"""


def test_a_list_that_changes_while_it_is_looked_at():
    """In a process of its own: what reads the list's items after they have gone ends it."""
    res = subprocess.run([sys.executable, "-c", CHANGES_ITS_LIST], capture_output=True, text=True, timeout=300,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert res.returncode == 0 and res.stdout.split() == ["refused", "-1", "0"], (res.returncode, res.stdout, res.stderr[-2000:])


def test_replicas_are_as_many_as_were_looked_at(calls):
    class Growing(list):
        def __iter__(self):
            return iter(list.copy(self)[:2])
    given = _arguments("sdl_merge_overlap", 5)
    given["w_now"] = Growing(given["w_now"])
    sdl.sdl_merge_overlap(*given.values())
    assert calls["sdl_merge_overlap"][0][2] == 2


class _As:
    def __init__(self, value):
        self._as_parameter_ = value


class _Index:
    def __index__(self):
        return 5


VALUES = [5, -1, True, (1 << 33) + 5, (1 << 70) + 5, 10 ** 400, 0.25, 1e300, np.int64(5), np.uint8(5), np.float32(0.25), np.float64(0.3), np.array(0.3), _Index(),
          None, "x", b"x", object(), fractions.Fraction(5), decimal.Decimal(5), torch.tensor(5), torch.tensor(0.5),
          *(t(5) for t in (ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int, ctypes.c_longlong, ctypes.c_void_p, ctypes.c_float, ctypes.c_double)),
          *(_As(t(5)) for t in (int, float, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int, ctypes.c_float))]


@pytest.mark.parametrize("name", NAMES)
def test_numbers_are_what_ctypes_makes_of_them(calls, name):
    """A value of any type reaches the library as a call through ctypes passes it on, or is refused as ctypes refuses it."""
    given = _arguments(name, 2)
    order = C_ORDER[name].split()
    for k in [k for k in given if k in SCALARS and k != "stream"]:
        at = order.index(k)
        ctype = getattr(sdl._lib, name).argtypes[at]
        by_ctypes = ctypes.CFUNCTYPE(ctype, ctype)(lambda x: x)
        for value in VALUES:
            calls.clear()
            try:
                want = by_ctypes(value)
            except ctypes.ArgumentError:
                with pytest.raises(ctypes.ArgumentError):
                    getattr(sdl, name)(*dict(given, **{k: value}).values())
                assert not calls
                continue
            getattr(sdl, name)(*dict(given, **{k: value}).values())
            assert calls[name][0][at] == want or (want != want and calls[name][0][at] != calls[name][0][at]), (k, value)


def test_addresses_streams_and_handles_of_other_types(calls):
    given = _arguments("sdl_merge_overlap_plan", 2)
    call = lambda **x: (sdl.sdl_merge_overlap_plan(*dict(given, **x).values()), calls.pop("sdl_merge_overlap_plan")[0])[1]
    for value, want in ((None, None), (64, 64), (-64, 2 ** 64 - 64), (2 ** 70 + 64, 64), (Tensor(-64), 2 ** 64 - 64), (Tensor(ctypes.c_void_p(64)), 64),
                        (Tensor(None), None), (Tensor(_As(64)), 64)):
        assert call(g_new_base=value)[2] == want
    for value in (Tensor(np.int64(64)), Tensor(64.0)):
        with pytest.raises(ctypes.ArgumentError):
            call(g_new_base=value)
    for value in (np.int64(64), _Index(), 64):                    # in a list: as struct packs an address
        call(w_now_base=[Tensor(64), Tensor(value)])
    for value in (64.0, None, 2 ** 70):
        with pytest.raises(struct.error):
            call(w_now_base=[Tensor(64), Tensor(value)])
    stream = lambda value: type("Stream", (), {"cuda_stream": value})()
    for value, want in ((0, None), (5, 5), (2 ** 70 + 5, 5), (stream(5), 5), (stream(None), None), (stream(ctypes.c_void_p(5)), 5)):
        assert call(stream=value)[6] == want
    with pytest.raises(ctypes.ArgumentError):
        call(stream=stream(np.int64(5)))
    plan = lambda value: type("Owner", (), {"_h": value})()
    for value, want in ((5, 5), (None, None), (ctypes.c_void_p(5), 5), (ctypes.c_void_p(None), None), (_As(5), 5)):
        assert call(plan=plan(value))[0] == want
    for value in (1.5, ctypes.c_uint64(5)):
        with pytest.raises(ctypes.ArgumentError):
            call(plan=plan(value))
    assert not calls


def test_the_staged_step_takes_more_replicas_to_write_than_to_read(calls):
    name = "sdl_fragment_outer_step_staged_ex"
    given = _arguments(name, 3)
    for w_now in (given["w_now_base"], (t for t in given["w_now_base"]), None):
        sdl.sdl_fragment_outer_step_staged_ex(*dict(given, w_send_base=given["w_send_base"][:2], w_now_base=w_now).values())
    at = {k: i for i, k in enumerate(C_ORDER[name].split())}
    assert [c[at["M"]] for c in calls[name]] == [2, 2, 2] and [bool(c[at["w_now_base"]]) for c in calls[name]] == [True, True, False]


@pytest.mark.parametrize("w_now", [[64], None])
def test_the_staged_step_without_a_replica_to_write_is_refused_by_the_library(w_now):
    """(On a plan of one span, with addresses that are not read on the way to the refusal.)"""
    plan = sdl.sdl_fragment_plan([512], [0], 1, 1, sdl.PATTERN_STRIDED, 10, 0)
    with pytest.raises(sdl.SdlError) as e:
        sdl.sdl_fragment_outer_step_staged_ex(plan, 0, 64, 64, [64, 64], w_now, sdl.FMT_FP32, 0.7, 0.9, 0.5, None, None, 0)
    assert e.value.status == -1
