"""The native argument marshalling against the Python functions that it takes over: what reaches the C entry point is the
same for every kind of argument, given by position, by name or left out, and what is refused is refused alike.  The entry
points are replaced by recorders, so nothing here needs a GPU."""
import copy
import ctypes
import functools
import inspect
import os
import pickle
import random
import weakref

import numpy as np
import pytest
import torch

import paper_2505_20776_amd as sx
from paper_2505_20776_amd import binding

if not (os.path.exists(binding._LIB_PATH) and os.path.exists(binding._MARSHAL_PATH)):
    from paper_2505_20776_amd.build import build_library
    build_library(verbose=False)
sx.load_library()
assert binding._marshal is not None, binding._marshal_error
NAMES = binding._marshal.FUNCTIONS


class _Recorder:
    """A C function of the entry point's signature that notes its arguments and returns `status`."""

    def __init__(self, name):
        real = getattr(sx.load_library(), "specext_" + name)
        types = [ctypes.c_void_p if t is ctypes.POINTER(sx.specext_desc) else t for t in real.argtypes]
        self.calls, self.status = [], 0

        def note(*args):
            self.calls.append(args)
            return self.status

        self.c = ctypes.CFUNCTYPE(ctypes.c_int, *types)(note)

    def address(self):
        return ctypes.cast(self.c, ctypes.c_void_p).value


@pytest.fixture
def recorded():
    real = sx.load_library()
    recorders = {n: _Recorder(n) for n in NAMES}
    fake = type("Fake", (), {"specext_" + n: staticmethod(r.c) for n, r in recorders.items()})()
    fake.specext_strerror = real.specext_strerror
    binding._lib = fake
    for n, r in recorders.items():
        binding._marshal.bind(n, r.address())
    yield recorders
    binding._lib = None
    sx.load_library()


INTS = ("score_row", "k", "n_chunks", "max_idx", "n_layers", "n_kv_heads", "src_len", "dst_cap", "head_dim", "chunk_size",
        "elem_bytes", "src_cap", "n_tree", "max_accept", "prefix_len", "cache_capacity", "n_q_heads", "q_len", "kv_len",
        "dtype", "out_dtype")


def _argument(rng, function, name):
    if name == "desc":
        return sx.make_desc(dtype=1, n_q_heads=4, n_kv_heads=2, head_dim=64, prefix_len=9, n_tree=rng.randrange(1, 9))
    if name == "check":
        return rng.choice([True, False])
    if name == "stream":
        return rng.choice([0, 1234, 2**47 + 16])
    if name == "workspace_nbytes":
        return rng.choice([None, 0, 77, 2**40])
    if name == "softmax_scale":
        return rng.choice([0.0, 0.125, 1e-40, 1])
    if "stride" in name:
        return rng.choice([0, 128, 2**40])
    if name in INTS and not (function == "prefill_attn" and name == "k"):      # there a tensor
        return rng.choice([0, 1, -1, 7, 2**31 - 1, 2**33 + 5, np.int64(12), 3.0])
    tensor = torch.zeros((4, 6), dtype=rng.choice([torch.float32, torch.bfloat16, torch.int32]))[rng.randrange(3):]
    if name == "workspace":
        return tensor
    return rng.choice([tensor, tensor, tensor.t(), torch.nn.Parameter(tensor.float()), None, 0, 4096, 2**47])


@pytest.mark.parametrize("name", NAMES)
def test_same_arguments_reach_the_entry_point(name, recorded):
    call = getattr(sx, name)
    assert inspect.signature(call) == inspect.signature(call.__wrapped__) and call.__name__ == name
    params = inspect.signature(call).parameters
    rng = random.Random(name)
    for _ in range(150):
        args, kwargs, by_name = [], {}, False
        for p in params.values():
            optional = p.default is not inspect.Parameter.empty
            if optional and p.name != "stream" and rng.random() < 0.4:      # the current stream needs a GPU
                by_name = True
                continue
            by_name = by_name or rng.random() < 0.1
            value = _argument(rng, name, p.name)
            if by_name:
                kwargs[p.name] = value
            else:
                args.append(value)
        assert call(*args, **kwargs) == 0
        assert call.__wrapped__(*args, **kwargs) == 0
        native, python = recorded[name].calls
        assert native == python, (args, kwargs)
        recorded[name].calls.clear()


@pytest.mark.parametrize("name", NAMES)
def test_status_and_wrong_calls(name, recorded):
    call = getattr(sx, name)
    params = list(inspect.signature(call).parameters.values())
    rng = random.Random(1)
    kwargs = {p.name: _argument(rng, name, p.name) for p in params}
    recorded[name].status = -2
    for src_cap in (0, 7):                   # the one parameter that may follow `check`
        if "src_cap" in kwargs:
            kwargs["src_cap"] = src_cap
        kwargs["check"] = False
        assert call(**kwargs) == -2
        kwargs["check"] = True
        with pytest.raises(sx.SpecextError, match="specext_" + name) as e:
            call(**kwargs)
        assert e.value.status == -2
    recorded[name].status = 0
    recorded[name].calls.clear()
    first = params[0].name
    for bad in ({**kwargs, "no_such": 1}, {k: v for k, v in kwargs.items() if k != first}, {**kwargs, first: "text"}):
        for f in (call, call.__wrapped__):
            with pytest.raises((TypeError, AttributeError, ctypes.ArgumentError)):
                f(**bad)
    with pytest.raises(TypeError):
        call(*([None] * (len(params) + 1)))
    assert not recorded[name].calls


def test_tensors_without_storage_and_subclasses(recorded):
    class Sub(torch.Tensor):
        pass

    plain = torch.zeros(8)
    for scores in (plain.as_subclass(Sub), plain):
        sx.select_chunks(scores, 8, 2, plain, plain, stream=0)
    assert recorded["select_chunks"].calls[0] == recorded["select_chunks"].calls[1]
    with pytest.raises((RuntimeError, NotImplementedError, ValueError)):
        sx.select_chunks(torch.sparse_coo_tensor(torch.zeros((1, 1), dtype=torch.long), torch.ones(1), (8,)), 8, 2, plain, plain, stream=0)


@pytest.mark.parametrize("name", NAMES)
def test_used_as_a_function_is(name):
    """What a program may do with a module's function beside calling it."""
    f = getattr(sx, name)
    assert pickle.loads(pickle.dumps(f)) is f and copy.copy(f) is f and copy.deepcopy({"f": f})["f"] is f
    assert weakref.ref(f)() is f and len({f, f}) == 1 and f == f
    assert inspect.isroutine(f) and callable(f) and inspect.unwrap(f) is f.__wrapped__ and "def " + name in inspect.getsource(f)
    assert f.__module__ == binding.__name__ and f.__qualname__ == name and f.__globals__ is vars(binding) and repr(f).startswith("<function " + name)
    with pytest.raises(AttributeError, match="no_such"):
        f.no_such
    f.note = 1
    assert f.note == 1 and vars(f) == {"note": 1} and "note" in dir(f)
    del f.note
    assert not hasattr(f, "note") and not vars(f)
    holder = type("Holder", (), {"call": f})()
    assert holder.call.__self__ is holder and holder.call.__func__ is f and type(holder).call is f
    assert functools.wraps(f)(lambda: None).__name__ == name


def test_weak_reference_outlived():
    def plain():
        pass

    f = binding._marshal.wrap(NAMES[0], plain, sx.specext_desc, binding._check)
    gone = []
    ref = weakref.ref(f, gone.append)
    del f
    assert ref() is None and gone == [ref]
