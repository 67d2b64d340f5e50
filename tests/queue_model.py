"""The work queues of the attention kernels on the CPU: tests/queue_model.cpp, which compiles the kernels' own queue header
and the host's own rules with g++, behind a few functions.  Tests use it to show that their bags reach the branch they are
about."""
from __future__ import annotations

import atexit
import ctypes as C
import functools
import os
import shutil
import subprocess
import tempfile
from typing import NamedTuple, Sequence

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256                                  # compute units of an MI355X
WORKGROUPS_PER_CU = {"fwd": {64: 3, 128: 2}, "dq": {64: 3, 128: 2}}     # what the kernels' registers allow


class Walk(NamedTuple):
    items: int       # work items
    parts: int       # parts that items were dealt out in
    per: int         # workgroups of a queue
    most: int        # most tickets of a queue
    draws: bool      # some queue has more tickets than workgroups
    wrong: int       # items or parts that were not dealt exactly once


@functools.lru_cache(maxsize=None)
def _lib():
    out = tempfile.mkdtemp(prefix="knap_queue_model_")
    atexit.register(shutil.rmtree, out, ignore_errors=True)
    so = os.path.join(out, "queue_model.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Wno-unknown-pragmas",
                    "-I" + os.path.join(ROOT, "paper_2508_06001_amd", "csrc"),
                    os.path.join(ROOT, "tests", "queue_model.cpp"), "-o", so], check=True)
    lib = C.CDLL(so)
    lib.queue_walk.restype = None
    lib.queue_walk.argtypes = [C.POINTER(C.c_int)] + [C.c_int] * 6 + [C.POINTER(C.c_int)]
    lib.queue_walk_even.restype = None
    lib.queue_walk_even.argtypes = [C.POINTER(C.c_int)] + [C.c_int] * 5 + [C.POINTER(C.c_int)]
    lib.queue_walk_pairs.restype = None
    lib.queue_walk_pairs.argtypes = [C.POINTER(C.c_int)] + [C.c_int] * 4 + [C.POINTER(C.c_int)]
    lib.queue_walk_small.restype = None
    lib.queue_walk_small.argtypes = [C.POINTER(C.c_int)] + [C.c_int] * 3 + [C.POINTER(C.c_int)]
    lib.queue_bwd_small.argtypes = [C.c_longlong] + [C.c_int] * 5
    lib.queue_small_items.restype = None
    lib.queue_small_items.argtypes = [C.POINTER(C.c_int)] + [C.c_int] * 5 + [C.POINTER(C.c_int)]
    lib.queue_bwd_joint.argtypes = [C.c_longlong] + [C.c_int] * 5
    lib.queue_eager_set.restype = None
    lib.queue_eager_set.argtypes = [C.c_ulonglong, C.POINTER(C.c_int)]
    lib.queue_captured_set.argtypes = [C.c_ulonglong]
    lib.queue_dkdv_workgroups_per_cu.argtypes = [C.c_int] * 2
    lib.queue_dkdv_pairs.argtypes = [C.c_longlong] + [C.c_int] * 5
    return lib


def dkdv_pairs(lens: Sequence[int], H: int, d: int, causal: bool, cus: int = CUS) -> int:
    return _lib().queue_dkdv_pairs(sum(lens), len(lens), H, d, int(causal), cus)


def grid(kernel: str, d: int, pairs: int = 0, cus: int = CUS) -> int:
    if kernel == "dkdv":
        return cus * _lib().queue_dkdv_workgroups_per_cu(d, pairs)
    return cus * WORKGROUPS_PER_CU[kernel][d]


def eager_set(call: int) -> tuple:
    """Counter set of an eager forward call, and the first of the sets that the call clears (None: it clears none)."""
    out = (C.c_int * 2)()
    _lib().queue_eager_set(call, out)
    return out[0], None if out[1] < 0 else out[1]


def captured_set(call: int) -> int:
    return int(_lib().queue_captured_set(call))


def _walk_even(lens: Sequence[int], H: int, causal: bool, kinds: int, grid_: int) -> Walk:
    out = (C.c_int * 6)()
    _lib().queue_walk_even((C.c_int * len(lens))(*lens), len(lens), H, int(causal), kinds, grid_, out)
    return Walk(out[0], out[1], out[2], out[3], bool(out[4]), out[5])


def walk(kernel: str, lens: Sequence[int], H: int, d: int, causal: bool, pairs: int = 0, cus: int = CUS) -> Walk:
    """The queues of `kernel` ("fwd", "dq" or "dkdv") for a bag."""
    if kernel == "fwd":
        return _walk_even(lens, H, causal, 1, grid("fwd", d, cus=cus))
    pairs = pairs or dkdv_pairs(lens, H, d, causal, cus)
    tile, split = (64 * pairs, 0) if kernel == "dkdv" else (128, 4 if causal else 2)
    out = (C.c_int * 6)()
    _lib().queue_walk((C.c_int * len(lens))(*lens), len(lens), H, tile, int(causal), split,
                      grid(kernel, d, pairs, cus), out)
    return Walk(out[0], out[1], out[2], out[3], bool(out[4]), out[5])


def walk_pairs(lens: Sequence[int], H: int, d: int, cus: int = CUS) -> Walk:
    """The tickets of the forward without the mask; `items` are the pairs of query tiles, of all queues."""
    out = (C.c_int * 6)()
    _lib().queue_walk_pairs((C.c_int * len(lens))(*lens), len(lens), H, d, grid("fwd", d, cus=cus), out)
    return Walk(out[0], out[1], out[2], out[3], bool(out[4]), out[5])


def bwd_joint(lens: Sequence[int], H: int, d: int, causal: bool, cus: int = CUS) -> bool:
    """Whether the backward of this bag is one launch of both kinds of items."""
    return bool(_lib().queue_bwd_joint(sum(lens), len(lens), H, d, int(causal), cus))


def walk_joint(lens: Sequence[int], H: int, d: int, causal: bool, cus: int = CUS) -> Walk:
    """The queues of that launch; `items` are those of one kind, `parts` those of query tiles."""
    return _walk_even(lens, H, causal, 2, grid("dkdv", d, 2, cus))


def bwd_small(lens: Sequence[int], H: int, d: int, causal: bool, cus: int = CUS) -> bool:
    """Whether that launch is the one that can take tiles of 64 rows (walk_small) in place of 128 (walk_joint); see small_items()."""
    return bool(_lib().queue_bwd_small(sum(lens), len(lens), H, d, int(causal), cus))


class SmallItems(NamedTuple):
    host: int        # 0: the host takes tiles of 128 rows, 1: it leaves it to the device, 2: tiles of 64 rows whatever the lengths are
    pays: bool       # the device's decision


def small_items(lens: Sequence[int], H: int, d: int, causal: bool, cus: int = CUS) -> SmallItems:
    out = (C.c_int * 2)()
    _lib().queue_small_items((C.c_int * len(lens))(*lens), len(lens), H, d, int(causal), cus, out)
    return SmallItems(out[0], bool(out[1]))


def walk_small(lens: Sequence[int], H: int, d: int, cus: int = CUS) -> Walk:
    """The queues of the launch of both kinds of 64-row items; `items` are those of one kind."""
    out = (C.c_int * 6)()
    _lib().queue_walk_small((C.c_int * len(lens))(*lens), len(lens), H, grid("dkdv", d, 2, cus), out)
    return Walk(out[0], out[1], out[2], out[3], bool(out[4]), out[5])


def launched(lens: Sequence[int], H: int, d: int, causal: bool) -> tuple:
    """The kernels with a work queue that a forward and a backward of this bag launch: "fwd", and "joint" or "dq" and "dkdv"."""
    return ("fwd", "joint") if bwd_joint(lens, H, d, causal) else ("fwd", "dq", "dkdv")


def walk_launched(kernel: str, lens: Sequence[int], H: int, d: int, causal: bool) -> Walk:
    """The queues of a kernel that this bag launches."""
    assert kernel in launched(lens, H, d, causal), (kernel, lens, H, d, causal)
    return walk_joint(lens, H, d, causal) if kernel == "joint" else walk(kernel, lens, H, d, causal)


def assert_draws(lens: Sequence[int], H: int, d: int, causal: bool, kernels=None) -> None:
    """The bag has more items than workgroups in some queue of each of these kernels (of all it launches)."""
    for kernel in kernels or launched(lens, H, d, causal):
        w = walk_launched(kernel, lens, H, d, causal)
        assert w.draws and w.most > w.per, (kernel, w)
