"""CPU tests of the extension module that makes the ordinary calls of the per-layer entry points (csrc/fast_call.cpp): the
words that reach the C function, and what it leaves to the ctypes wrapper."""
import ctypes as C
import pickle
import types as pytypes

import numpy as np
import pytest
import torch

import paper_2605_03375_amd as package
from paper_2605_03375_amd import binding as B
from paper_2605_03375_amd import build

STREAM = 0x5555_0000_1230


@pytest.fixture(scope="module")
def module():
    build.build_fast_call(force=False)
    from paper_2605_03375_amd import _fast_call
    B.product_lib()
    _fast_call.setup((B.tutti_pool, B.tutti_objcfg, B.tutti_ring, B.tutti_filestore), torch.Tensor, lambda: 3,
                     lambda device: STREAM + device, B._check)
    _fast_call.enable(True)
    yield _fast_call
    _fast_call.enable(False)
    B._bind_fast_calls()


def _recorder(name, rc=0):
    """A C function of the entry point's type that records its arguments."""
    got = []
    types = [t if t in (C.c_uint32, C.c_uint64) else C.c_void_p for t in getattr(B.product_lib(), name).argtypes]

    def body(*a):
        got.append(tuple(0 if x is None else x for x in a))
        return rc
    return C.CFUNCTYPE(C.c_int, *types)(body), types, got


def _callable(module, name, rc=0):
    fn, types, got = _recorder(name, rc)
    wrapper = getattr(B, name)
    left = []
    names, defaults = wrapper.__code__.co_varnames[:wrapper.__code__.co_argcount], wrapper.__defaults__
    call = module.wrap(name, lambda *a, **k: left.append((a, k)), names, defaults)
    module.bind(call, C.cast(fn, C.c_void_p).value)
    return call, types, got, left, names, defaults, fn


def _arguments(types, names, name):
    records = {"pool": B.make_pool(None, None, num_blocks=4, block_tokens=16, num_kv_heads=2, head_dim=64, elt_bytes=2),
               "cfg": B.make_cfg(), "ring": B.make_ring(None, None, 4), "store": B.make_filestore(None, 0, 0, 0)}
    given, want = [], []
    for k, (t, n) in enumerate(zip(types, names)):
        if n in records:
            given.append(records[n])
            want.append(C.addressof(records[n]))
        elif n == "stream":
            given.append(77)
            want.append(77)
        elif t is C.c_void_p:
            x = [torch.zeros(4 + k), None, 4096 * (k + 1)][k % 3]
            given.append(x)
            want.append(x.data_ptr() if torch.is_tensor(x) else x or 0)
        else:
            v = (1 << 32) + 1000 + k
            given.append(v)
            want.append(v if t is C.c_uint64 else 1000 + k)
    return given, want


@pytest.mark.parametrize("name", B._FAST_NAMES)
def test_the_words_that_arrive(module, name):
    call, types, got, left, names, defaults, keep = _callable(module, name)
    assert len(names) == len(types) and names[-1] == "stream"
    given, want = _arguments(types, names, name)
    assert call(*given) == 0 and got.pop() == tuple(want)
    half = len(given) // 2
    assert call(*given[:half], **dict(reversed(list(zip(names, given))[half:]))) == 0 and got.pop() == tuple(want)
    n_def = len(defaults)
    assert call(*given[:-n_def]) == 0
    assert got.pop() == tuple(want[:-n_def]) + (0,) * (n_def - 1) + (STREAM + 3,)
    assert call(*given[:-1], stream=None) == 0 and got.pop() == tuple(want[:-1]) + (STREAM + 3,)
    assert not left


def test_what_is_left_to_the_wrapper(module):
    call, types, got, left, names, defaults, keep = _callable(module, "tutti_layer_restore")
    given, want = _arguments(types, names, "tutti_layer_restore")

    def swapped(i, x):
        a = list(given)
        a[i] = x
        return a

    class Own(torch.Tensor):
        pass

    for args, kw in [(swapped(3, np.int64(4)), {}), (swapped(3, True), {}), (swapped(3, 4.0), {}), (swapped(0, None), {}),
                     (swapped(0, given[1]), {}), (swapped(2, np.zeros(4)), {}), (swapped(2, torch.zeros(4).as_subclass(Own)), {}),
                     (swapped(2, torch.nn.Parameter(torch.zeros(4))), {}), (given + [1], {}), (given[:5], {}),
                     (given, {"stream": 1}), (given[:-1], {"other": 1}), (swapped(18, object()), {})]:
        call(*args, **kw)
        a, k = left.pop()
        assert len(a) == len(args) and all(x is y for x, y in zip(a, args)) and k == kw and not got
    module.enable(False)
    call(*given)
    module.enable(True)
    assert left.pop() and not got
    call(*given)
    assert got.pop() == tuple(want)


def test_codes_and_identity(module):
    call, types, got, left, names, defaults, keep = _callable(module, "tutti_complete_io", rc=B.ERANGE)
    given, _ = _arguments(types, names, "tutti_complete_io")
    with pytest.raises(B.TuttiError) as e:
        call(*given)
    assert e.value.code == B.ERANGE and e.value.fn == "tutti_complete_io"
    for name in B._FAST_NAMES:
        f = getattr(B, name)
        assert f.__name__ == name and f.__module__ == B.__name__ and pickle.loads(pickle.dumps(f)) is f
    with pytest.raises(ValueError):
        module.wrap("tutti_complete_io", print, ("a", "b"), (None,))


def _bad_wrap(*a):
    raise ValueError("not an entry point of these arguments")


@pytest.mark.parametrize("found", [{}, {"BUILT_FOR": "[torch 0.1]", "wrap": lambda *a: print},
                                   {"BUILT_FOR": f"[torch {torch.__version__}]", "wrap": _bad_wrap}],
                         ids=["of an older build", "for another torch", "for other arguments"])
def test_a_module_of_another_build_is_left_alone(monkeypatch, found):
    monkeypatch.setattr(package, "_fast_call", pytypes.SimpleNamespace(**found), raising=False)
    monkeypatch.setattr(B, "_fast_call", None)
    before = {name: getattr(B, name) for name in B._FAST_NAMES}
    B._install_fast_calls()
    assert B._fast_call is None and all(getattr(B, name) is f for name, f in before.items())


def test_entry_points_that_changed_are_not_bound(module, monkeypatch):
    """The module's idea of an entry point's arguments is compared with the ctypes declaration."""
    lib = B.product_lib()
    for name in B._FAST_NAMES:
        assert module.form(name) == B._form(getattr(lib, name).argtypes) and "?" not in module.form(name)
    assert module.form("tutti_cu_count") is None
    bound = {}
    monkeypatch.setattr(B, "_fast_call", pytypes.SimpleNamespace(
        setup=lambda *a: None, form=lambda name: module.form(name).replace("il", "li", name == "tutti_issue_io"),
        bind=lambda call, at: bound.__setitem__(call.__name__, at)))
    B._bind_fast_calls()
    assert [name for name, at in bound.items() if at == 0] == ["tutti_issue_io"] and len(bound) == len(B._FAST_NAMES)


@pytest.mark.parametrize("missing", ["torch", "headers", "compiler"])
def test_the_library_is_built_without_what_the_module_needs(monkeypatch, tmp_path, missing):
    ran = []
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **k: ran.append(cmd))
    if missing == "torch":
        monkeypatch.setattr(build.importlib.util, "find_spec", lambda name: None)
    elif missing == "headers":
        monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    else:
        monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    assert build.build_lib(force=True) == build.LIB
    assert [cmd[cmd.index("-o") + 1] for cmd in ran] == [build.LIB]
