"""Which kernels a call launches, from the library's own rules (`attn_rules.hpp`, `loss_rules.hpp`, compiled here with
g++): the tests that claim to reach a kernel say which, and a test without a GPU checks that they still do."""
import ctypes
import os
import subprocess
import tempfile

from paper_2503_07680_amd import build as B

_lib = None


def _load():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as tmp:
            so = os.path.join(tmp, "rules.so")
            subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", B.CSRC,
                            os.path.join(os.path.dirname(os.path.abspath(__file__)), "launch_rules_shim.cpp"), "-o", so], check=True)
            _lib = ctypes.CDLL(so)
    return _lib


def _tiles(lengths, rows):
    return sum(-(-n // rows) for n in lengths)


def forward(lengths, Hq, Hkv, d, records=False, tile_rows=None):
    """"singles", "halves", "pairs", "256-row tiles" or "128-row tiles"; the last three with " queued" behind it when their
    items come from queues.  tile_rows: as the forward prefers by default."""
    rows = tile_rows or (256 if (Hq // Hkv) % 2 else 128)
    out = (ctypes.c_int * 4)()
    _load().fwd_route(d, sum(lengths), len(lengths), Hq, Hkv, _tiles(lengths, rows), rows, int(records), out)
    hp, tp, direct, halves = out
    if halves:
        return "halves"
    name = "pairs" if hp == 2 else "256-row tiles" if tp == 2 else "singles" if (Hq // Hkv) % 2 == 0 else "128-row tiles"
    return name if direct else name + " queued"


def backward(lengths, Hq, Hkv, d, records=False):
    """"one launch", "one launch interleaved", "eight waves" or "four waves" (two launches); query heads and items of dK/dV."""
    tiles, out = _tiles(lengths, 128), (ctypes.c_int * 6)()
    _load().bwd_route(d, sum(lengths), len(lengths), Hq, Hkv, tiles, tiles, int(records), out)
    one, interleaved, eight, heads, items, _ = out
    return ("one launch interleaved" if one and interleaved else "one launch" if one else "eight waves" if eight else "four waves",
            heads, items)


def cross_entropy_per_cu(threads, chunks, hold, with_grad):
    """The most workgroups a compute unit gets."""
    return _load().ce_per_cu(threads, chunks, int(hold), int(with_grad))


def cross_entropy_launched_per_cu(threads, chunks, hold, with_grad, T, n_samples):
    """Workgroups a compute unit that a call launches, as far as the kernel's registers allow for that many."""
    return _load().ce_launched_per_cu(threads, chunks, int(hold), int(with_grad), T, n_samples)


def cross_entropy_plan_lds(T, n_samples):
    """Bytes of LDS that a workgroup plans its rows in."""
    return _load().ce_plan_lds(T, n_samples)


def cross_entropy_own_lds(threads, chunks, hold, with_grad):
    """The most bytes of LDS that the main kernel's own arrays take."""
    return _load().ce_own_lds(threads, chunks, int(hold), int(with_grad))
