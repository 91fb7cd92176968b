"""The Python binding's own plumbing (CPU)."""
import ctypes

from paper_2308_11759_amd import pmc


def test_shared_python_api_functions_keep_their_types():
    """The binding declares types on function objects of its own only."""
    shared = ctypes.pythonapi.PyBytes_FromStringAndSize
    assert shared.argtypes is None and shared.restype is ctypes.c_int


def test_new_bytes_are_fresh_and_of_the_size_asked_for():
    a, b = pmc._new_bytes(None, 100), pmc._new_bytes(None, 100)
    assert type(a) is bytes and len(a) == len(b) == 100
    ctypes.memmove(ctypes.cast(ctypes.c_char_p(a), ctypes.c_void_p), bytes(range(100)), 100)
    assert a == bytes(range(100)) and a is not b
    assert len(pmc._new_bytes(None, 1)) == 1
