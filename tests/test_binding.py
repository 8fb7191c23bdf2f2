"""The Python side of the calls (csrc/python_binding.cpp) without a GPU: what it accepts and hands on.  No call here reaches a
device: either the arguments say that there is nothing to do, or they are refused on the host."""
import inspect
import pickle

import pytest
import torch

from paper_2602_00523_amd import sage


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
