"""Argument handling of the entry points' callable objects (host only: every call here is refused by the
library's own checks or before it)."""
import numpy as np
import pytest

import paper_2406_11235_amd as q
from paper_2406_11235_amd import binding


def test_positions_and_keywords_are_the_same_call():
    buf = np.zeros(64, dtype=np.uint32)
    for args, kw in (((buf, buf, 64, 48, 1, 0, buf), {"stream": 0}), ((buf, buf, 64, 48, 1, 0, buf, 0), {}),
                     ((buf, buf), {"out": buf, "side": 0, "batch": 1, "block": 48, "n": 64, "stream": 0}),
                     ((buf.ctypes.data, buf, 64, np.int64(48), True, 0, None), {"stream": 0})):
        with pytest.raises(q.QtipError) as e:
            q.qtip_rht(*args, **kw)
        assert e.value.code == -1


@pytest.mark.parametrize("name", binding._GPU_ENTRIES)
def test_wrong_arguments_raise(name):
    f = getattr(q, name)
    with pytest.raises(TypeError, match="missing required argument"):
        f(stream=0)
    with pytest.raises(TypeError, match="unexpected keyword"):
        f(nonsense=1)
    with pytest.raises(TypeError, match="at most"):
        f(*[None] * 20)
    with pytest.raises(TypeError, match="multiple values"):
        f(None, **{{"qtip_rht": "x", "qtip_rht_f32": "x", "qtip_decode_states": "states", "qtip_quantize_gpu": "W",
                    "qtip_block_ldl": "H", "qtip_quantize_ldlq": "W"}.get(name, "codes"): None})
    with pytest.raises((TypeError, AttributeError)):
        f(*[object()] * 7, stream=0)


@pytest.mark.parametrize("name", binding._GPU_ENTRIES)
def test_entry_points_are_like_functions(name):
    import copy
    import inspect
    import pickle
    import weakref
    f = getattr(q, name)
    assert (f.__name__, f.__qualname__, f.__module__) == (name, name, binding.__name__) and f.__doc__
    assert pickle.loads(pickle.dumps(f)) is f and copy.copy(f) is f and copy.deepcopy(f) is f
    assert weakref.ref(f)() is f
    f.note = "kept"
    assert f.note == "kept" and vars(f)["note"] == "kept"
    del f.note
    assert not hasattr(f, "note")

    class Holder:
        method = f
    held = Holder()
    assert Holder.method is f and held.method.__self__ is held and held.method.__func__ is f
    # the signature is the one the call has: every name is taken, what has no default is needed
    parameters = inspect.signature(f).parameters
    needed = [p.name for p in parameters.values() if p.default is p.empty]
    assert {p.default for p in parameters.values()} <= {inspect.Parameter.empty, None} and "stream" in parameters
    for given in (list(parameters), needed + ["stream"]):
        with pytest.raises(q.QtipError):
            f(**{p: 0 for p in given})
    for p in needed:
        with pytest.raises(TypeError, match=f"missing required argument '{p}'"):
            f(**{o: 0 for o in parameters if o != p})
    with pytest.raises(q.QtipError):
        f(*[0] * len(parameters))


def test_calls_that_name_their_stream_leave_torch_alone():
    """torch's GPU state is not looked at, and not initialized, by calls that say where they go (a child process,
    because the library is connected once)."""
    import subprocess
    import sys
    program = """
import torch
def asked(*args): raise AssertionError("asked")
torch.cuda.init = torch.cuda.is_available = torch.cuda._lazy_init = torch.cuda.current_stream = asked
import paper_2406_11235_amd as q
for stream in (0, 64, type("Stream", (), {"cuda_stream": 0})()):
    assert q.qtip_decode_states(64, 0, 16, 1, 0, None, 64, stream) == 0  # nothing to do: no launch
    try:
        q.qtip_rht(0, 0, 64, 64, 1, 0, 0, stream=stream)
    except q.QtipError:
        continue
    raise SystemExit("not refused")
try:
    q.qtip_decode_states(64, 0, 16, 1, 0, None, 64)
except AssertionError:
    raise SystemExit(0)
raise SystemExit("the current stream came from nowhere")
"""
    subprocess.run([sys.executable, "-c", program], check=True, cwd=build_root())


def test_a_forked_child_asks_torch_again():
    """torch.cuda.current_stream() raises in the forked child of a process that has used the GPU, and so does a call
    without a stream, although the parent has torch's getters at hand."""
    import subprocess
    import sys
    program = """
import os
import torch
import paper_2406_11235_amd as q
from paper_2406_11235_amd import binding
def refused(): raise RuntimeError("forked")
def call(): return q.qtip_decode_states(64, 0, 16, 1, 0, None, 64)  # nothing to do: no launch
q.qtip_decode_states(64, 0, 16, 1, 0, None, 64, 0)
binding._call.hooks(binding._ptr, binding._stream, binding._check, binding._connect, lambda: 0, lambda device: 0)
torch.cuda.current_stream = refused
assert call() == 0
child = os.fork()
if child == 0:
    try:
        call()
    except RuntimeError as e:
        os._exit(0 if str(e) == "forked" else 2)
    os._exit(1)
assert os.waitstatus_to_exitcode(os.waitpid(child, 0)[1]) == 0
assert call() == 0
"""
    subprocess.run([sys.executable, "-c", program], check=True, cwd=build_root())


def test_the_extension_is_this_pythons_own():
    """Built under the interpreter's tag, so that no other one finds it, and nothing untagged beside it."""
    import importlib.machinery
    import os
    import sysconfig
    from paper_2406_11235_amd import build
    tag = sysconfig.get_config_var("EXT_SUFFIX")
    assert binding._load_call().__file__ == build.CALL and build.CALL.endswith(tag) and sysconfig.get_config_var("SOABI") in tag
    found = [f for f in os.listdir(os.path.dirname(build.CALL)) if f.startswith("_call") and f.endswith(".so")]
    assert "_call.so" not in found and tag in importlib.machinery.EXTENSION_SUFFIXES


def build_root():
    import os
    return os.path.dirname(os.path.dirname(os.path.abspath(q.__file__)))
