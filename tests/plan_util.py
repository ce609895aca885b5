"""The host side of a 16-bit call as the library would do it: csrc/plan.h and csrc/launch_rules.h, built with the host compiler."""
import ctypes as C
import functools
import os
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=None)
def shim():
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    with tempfile.TemporaryDirectory() as tmp:
        lib = os.path.join(tmp, "attn_plan.so")
        subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", os.path.join(HERE, "attn_plan_shim.cpp"), "-o", lib], check=True)
        return C.CDLL(lib)


def _plan(shim, L, S, M, computed, heads, dh, n_cus, most_sums):
    n = len(L)
    new_rows = M is not None
    arr = [np.asarray(a if a is not None else [0] * n, np.int32) for a in (L, S, M)]
    comp = np.asarray([1] * n if computed is None else computed, np.uint8)
    info, msg = np.zeros(10, np.int32), C.create_string_buffer(256)
    rc = shim.plan_check(n, *(a.ctypes.data_as(C.c_void_p) for a in arr), comp.ctypes.data_as(C.c_void_p), int(new_rows), heads, dh, n_cus, most_sums,
                         info.ctypes.data_as(C.c_void_p), msg)
    assert rc == 0, f"L {list(L)} S {S} M {M} computed {computed} heads {heads} d_head {dh} units {n_cus} sums {most_sums}: {msg.value.decode()}"
    return info.tolist()


def check(shim, L, S=None, M=None, computed=None, heads=8, dh=64, n_cus=256, most_sums=8):
    """Plans a call (M None: pre-inference), checks the plan row by row and returns what it says."""
    return dict(zip(("blocks", "nsplit", "gs", "items", "filler"), _plan(shim, L, S, M, computed, heads, dh, n_cus, most_sums)))


def sums_in_flight(L, M=None, S=None, computed=None, heads=8, dh=64):
    """Partial sums of a row that the layer tail of the call has in flight, in all layers but the last and in the last."""
    last, others = _plan(shim(), L, S, M, computed, heads, dh, 256, 8)[5:7]
    return others, last


def tail_rows(d, rows):
    """Rows of a layer-tail workgroup."""
    return shim().tail_rows_of(d, rows)


def shared_pieces(attention, L, S, M, computed=None, heads=8, dh=64):
    """Key tiles of the longest piece of the call's attention, and from how many on two wavefront groups share a piece (None: one group)."""
    silu, softmax, longest = _plan(shim(), L, S, M, [0] * len(L) if computed is None else computed, heads, dh, 256, 8)[7:10]
    least = silu if attention == "silu" else softmax
    return longest, least if least < 1 << 20 else None


def user_pieces(L, S, M, user, attention="silu", heads=8, dh=64, n_cus=256):
    """(first, last key tile, shared by two wavefront groups) of the pieces of a user's first row tile in a ranking of cached users."""
    arr = [np.asarray(a, np.int32) for a in (L, S, M)]
    out = np.zeros(24, np.int32)
    count = shim().user_pieces(len(L), *(a.ctypes.data_as(C.c_void_p) for a in arr), user, int(attention == "softmax"), heads, dh, n_cus, out.ctypes.data_as(C.c_void_p))
    return [tuple(p) for p in out.reshape(8, 3)[:count].tolist()]


def projection_tile(d, rows, nblk=4, n_cus=256):
    """Tile of a projection launch: `nblk` of the four column blocks [u | v | q | k] of `rows` rows."""
    return ("64x64", "64x128", "128x128", "128x128/3", "stationary", "256x128")[shim().f1_tile_of(d, nblk, rows, n_cus)]


def projection_tiles(d, L, S, M):
    """Tiles of a two-layer model: ranking on the cache; pre-inference's first and last layer (K and V alone); full recompute's first and
    last layer (K and V of the prefix again; the new rows there are the cached ranking's launch)."""
    prefix, new = sum((n + 255) // 256 * 256 for n in L), sum(S) + sum(M)
    kv = projection_tile(d, prefix, 2)
    return {"cached": projection_tile(d, new), "prefill": projection_tile(d, prefix), "full": projection_tile(d, prefix + new), "kv": kv}
