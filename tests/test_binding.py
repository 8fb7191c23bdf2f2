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
