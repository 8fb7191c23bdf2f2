"""The Python side of the calls (csrc/python_binding.cpp) without a GPU: what it accepts and hands on.  No call here reaches a
device: either the arguments say that there is nothing to do, or they are refused on the host."""
import inspect
import os
import pickle
import subprocess
import sys

import pytest
import torch

from paper_2602_00523_amd import sage

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Stream:
    cuda_stream = 0


def loaded():
    """The native call, after the first use that puts it in place of the module's function."""
    with pytest.raises(sage.SageError, match="sage_advance_kv_len -> INVALID_ARG"):
        sage.sage_advance_kv_len(torch.zeros(1, dtype=torch.int32), None, 10, stream=Stream())
    return sage.sage_advance_kv_len


def test_native_calls_keep_their_names():
    """A call stands in for a function after its first use: named, documented, described and pickled like one."""
    call = loaded()
    assert call.__name__ == call.__qualname__ == "sage_advance_kv_len" and call.__module__ == sage.__name__
    assert call.__doc__ == "sage_advance_kv_len(kv_len, accept_len, kv_capacity, stream=None): see include/sage.h"
    assert pickle.loads(pickle.dumps(call)) is call
    assert str(inspect.signature(call)) == "(kv_len, accept_len, kv_capacity, stream=None)"


def test_first_use_leaves_replaced_functions_alone():
    """What a program has put in place of a call (a wrapper, a mock) stays when the native calls are loaded; the others are
    replaced."""
    program = """
from paper_2602_00523_amd import sage
def counted(*a, **kw): pass
plain, sage.sage_build_tree = sage.sage_commit_path, counted
sage._load_native("sage_commit_path")
assert sage.sage_build_tree is counted and sage.sage_commit_path is not plain
"""
    subprocess.run([sys.executable, "-c", program], check=True, cwd=ROOT)


def test_prepare_of_an_unknown_call():
    with pytest.raises(AttributeError, match="sage_no_such_call"):
        sage.prepare("sage_no_such_call")


class Mimic:
    """An array with the methods of a tensor that the calls read, as another library's arrays have them."""

    def __init__(self, t):
        self.t = t
        self.shape, self.dtype = tuple(t.shape), t.dtype

    def data_ptr(self):
        return self.t.data_ptr()

    def stride(self, i):
        return self.t.stride(i)

    def numel(self):
        return self.t.numel()

    def element_size(self):
        return self.t.element_size()


class Elsewhere(torch.Tensor):
    """A tensor subclass that says itself where its data is."""

    def data_ptr(self):
        return 0


def outcome(make, x):
    out, ws = torch.zeros(2, 1, dtype=torch.int32), torch.zeros(8, dtype=torch.uint8)
    try:
        sage.sage_entropy_topk(make(x), 1, None, make(out), None, None, None, None, make(ws), stream=Stream())
    except Exception as e:
        return type(e), str(e)


@pytest.mark.parametrize("x,why", [
    (torch.zeros(2, 64), "WORKSPACE_TOO_SMALL"),         # read to the end: the eight bytes of the workspace are too few
    (torch.zeros(2, 64, dtype=torch.bfloat16), "WORKSPACE_TOO_SMALL"),
    (torch.zeros(2, 66)[:, :60], "INVALID_ARG"),         # the row stride arrives (rows are not 16-byte aligned)
    (torch.zeros(64, 2).T, "contiguous"),
    (torch.zeros(2, 3, 64), "2 dimensions"),
    (torch.zeros(2, 64, dtype=torch.float64), "float32 or bfloat16")])
def test_arguments_with_the_methods_of_a_tensor(x, why):
    """What has a tensor's methods is read like a tensor, with the same errors."""
    tensor = outcome(lambda t: t, x)
    assert why in tensor[1]
    assert outcome(Mimic, x) == tensor


def test_a_tensor_subclass_is_read_through_its_methods():
    """An overridden data_ptr is the one that counts: a null one is refused, also where there is nothing to do."""
    none = Mimic(torch.zeros(1, dtype=torch.int32))
    none.shape = (0,)                                    # no sequence
    sage.sage_advance_kv_len(none, torch.zeros(1, dtype=torch.int32), 10, stream=Stream())
    with pytest.raises(sage.SageError, match="INVALID_ARG"):
        sage.sage_advance_kv_len(none, torch.zeros(1, dtype=torch.int32).as_subclass(Elsewhere), 10, stream=Stream())


def test_arguments_without_them_are_type_errors():
    for x in (4096, [1.0, 2.0], object()):
        with pytest.raises(TypeError, match="must be a tensor"):
            sage.sage_advance_kv_len(torch.zeros(1, dtype=torch.int32), x, 10, stream=Stream())


def test_closing_calls_take_histories_of_more_dimensions():
    """The window is the second size of `hist` whatever follows: an empty batch goes through, a window over 64 is refused."""
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32)  # noqa: E731
    kt, full = Mimic(torch.zeros(1, 64, 2, 64)), i32(64)
    kt.shape = (0, 64, 2, 64)                            # no sequence

    def close(hist):
        sage.sage_close_step(kt, kt, kt, kt, full, full, 100, 128, 64, i32(1, 9), full, hist, full, full, full, 2.0, 3.0, 3, 8,
                             stream=Stream())
    close(i32(1, 10))
    close(i32(1, 10, 1))
    with pytest.raises(sage.SageError, match="INVALID_ARG"):
        close(i32(1, 65, 1))
    with pytest.raises(ValueError):
        close(i32(10))
