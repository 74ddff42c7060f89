"""Random calls of the extension module of csrc/sdl_binding.c: binding_fuzz.py <extension> <library of stand-ins>."""
import ctypes, importlib.util, itertools, random, struct, sys
spec = importlib.util.spec_from_file_location("_binding", sys.argv[1])
b = importlib.util.module_from_spec(spec)
spec.loader.exec_module(b)
lib = ctypes.CDLL(sys.argv[2])
names = [n for n in dir(b) if n.startswith("sdl_")]
same = lambda t: ctypes.CFUNCTYPE(t, t)(lambda x: x)
b.converters(ctypes.c_void_p, *map(same, (ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int, ctypes.c_float, ctypes.c_void_p)),
             lambda x: struct.unpack("P", struct.pack("P", x))[0])
b.setup({n: ctypes.cast(getattr(lib, n), ctypes.c_void_p).value for n in names}, lambda s: s, lambda: False, lambda: 0, None)

class Tensor:
    is_cuda = True
    def __init__(self, at, act=None): self.at, self.act = at, act
    def is_contiguous(self):
        if self.act: self.act()
        return True
    def data_ptr(self): return self.at

class Owner:
    def __init__(self, h): self._h = h

rng = random.Random(1)
kept, calls, refused = [], 0, 0

def tensors():
    out = []
    n = rng.choice([0, 1, 2, 2, 3, 8, 15, 16, 17, 40])
    def act():
        rng.choice([out.clear, lambda: out.extend(Tensor(9) for _ in range(100)), lambda: out.__delitem__(slice(0, 2)), lambda: None])()
        kept.extend(bytearray(64) for _ in range(20))
        del kept[:-100]
    odd = rng.random() < 0.3
    for i in range(n):
        out.append(rng.choice([lambda: Tensor(64 * i), lambda: Tensor(64 * i), lambda: Tensor(64 * i, act), lambda: None, lambda: 64, lambda: object(),
                               lambda: Tensor("x"), lambda: Tensor(ctypes.c_void_p(64)), lambda: 2 ** 70])() if odd and rng.random() < 0.3 else Tensor(64 * i))
    return rng.choice([lambda: out, lambda: out, lambda: tuple(out), lambda: iter(list(out)), lambda: None, lambda: 5, lambda: "ab"])() if rng.random() < 0.1 else out

number = lambda: rng.choice([5, 5, 5, 0.5, 0.5, 0.5, -1, 2 ** 70, None, "x", ctypes.c_uint64(5), ctypes.c_float(0.5), 10 ** 400])
pointer = lambda: rng.choice([64, None, Tensor(64), Tensor(64), Tensor(None), object(), -1, 2 ** 70])
owner = lambda: Owner(rng.choice([5, None, ctypes.c_void_p(5), ctypes.c_void_p(None), "x", 1.5]))
# what each argument is: P plan, A address, L list, I whole number, F number, S stream
SHAPES = {"sdl_quantize_outer_grad": "ALIILLS", "sdl_dequant_reduce_nesterov": "AALLIIFFS", "sdl_merge_overlap": "ALIFS",
          "sdl_receive_outer_step": "AALLLIIFFFS", "sdl_fragment_outer_step": "AALLIIFFFLLS", "sdl_quantize_outer_grad_plan": "PIALILLS",
          "sdl_dequant_reduce_nesterov_plan": "PIAALLIFFS", "sdl_merge_overlap_plan": "PIALFS", "sdl_receive_outer_step_plan": "PIAALLLIFFFS",
          "sdl_fragment_outer_step_plan": "PIAALLIFFFS", "sdl_fragment_outer_step_plan_static": "PIAALLIFFFS",
          "sdl_fragment_outer_step_plan_ex": "PIAALLIFFFLLS", "sdl_fragment_outer_step_staged_ex": "PIAALLIFFFLLS"}
assert sorted(SHAPES) == names
for turn in range(3000):
    for name, shape in SHAPES.items():
        easy = turn % 2
        make = {"P": lambda: Owner(ctypes.c_void_p(5)) if easy else owner(), "A": lambda: Tensor(64) if easy else pointer(), "L": tensors,
                "I": lambda: 3 if easy else number(), "F": lambda: 0.5 if easy else number(), "S": lambda: rng.choice([0, 5, None])}
        args = [make[k]() for k in shape]
        if rng.random() < 0.02: args.pop()
        try:
            getattr(b, name)(*args)
            calls += 1
        except (TypeError, AttributeError, ValueError, OverflowError, ctypes.ArgumentError, struct.error):
            refused += 1
print("calls", calls, "refused", refused)
