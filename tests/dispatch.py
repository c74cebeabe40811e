"""The library's own dispatch rules, for tests that have to reach one kernel. They are
plain host functions of the library (C++, hence the mangled names), so a test that
names a path fails when a rule moves it to another.

torch is imported first: the library binds to the HIP runtime that torch brings only if
that one is loaded, and a process with two of them dies at its first GPU call."""
import ctypes

import torch  # noqa: F401
from paper_2311_11390_amd import _lib as L


def streams_dI(B, T, N, TR, gvt=False) -> bool:
    """Whether the detached backward with a float dL/dI streams over time chunks
    (``gvt``: with dL/dV or dL/dtheta); else it is the block kernel."""
    f = getattr(L.load(), "_ZN4alif13bwd_stream_giEiiiib")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int] * 4 + [ctypes.c_bool]
    return f(B, T, N, TR, gvt)


def stream_chunks(B, T, N, TR) -> int:
    """Time chunks a row of the streaming backward is cut into."""
    f = getattr(L.load(), "_ZN4alif17bwd_stream_chunksEiiii")
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int] * 4
    return f(B, T, N, TR)


def stream_bytes(B, N, chunks) -> int:
    """Scratch of that many chunks' sums."""
    f = getattr(L.load(), "_ZN4alif16bwd_stream_bytesEiii")
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_int] * 3
    return f(B, N, chunks)


def forward_chains(B, N, TR, NB, traces=False, carries=False) -> bool:
    """Whether the forward runs the recurrence on a wave of its own (k_fwd_chain); else
    it is the block kernel."""
    f = getattr(L.load(), "_ZN4alif12fwd_chain_okEiiiibb")
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int] * 4 + [ctypes.c_bool] * 2
    return f(B, N, TR, NB, traces, carries)
