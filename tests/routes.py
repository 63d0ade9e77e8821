"""The kernel and tile that a product takes, as the library's own rules give it.

Bound to a function of the library that is no part of its C ABI: the launchers
and this query read the same rules, so a test that asserts a route here runs on
that route.
"""

import collections
import ctypes

from paper_2609_33601_amd import jq

Route = collections.namedtuple("Route", "kernel waves rows cols")

KINDS = {"w4a4": 0, "w158a4": 1, "f6": 2, "group_f6": 3}
KERNELS = ("tiled", "narrow", "wide")


def route(kind, M, K, N, G=0, cus=256):
    """Of an M x K by K x N product: "w4a4" and "w158a4" on the packed engine, "f6" and "group_f6" on the BF6 one."""
    fn = jq.lib().jq_internal_route
    fn.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int,
                   ctypes.POINTER(ctypes.c_int * 4)]
    fn.restype = ctypes.c_int
    out = (ctypes.c_int * 4)()
    assert fn(KINDS[kind], M, N, K, G, cus, ctypes.byref(out)) == 0, kind
    return Route(KERNELS[out[0]], out[1], out[2], out[3])


def few_rows(M, K, G=0):
    """Whether the BF6 quantiser takes the few-row kernel for an M x K input."""
    fn = jq.lib().jq_internal_quantize_few
    fn.argtypes, fn.restype = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int], ctypes.c_int
    return bool(fn(M, K, G))


def few_rows_batch(shapes):
    """Whether the batched BF6 quantiser takes one launch of the few-row kernel for M x K inputs."""
    fn = jq.lib().jq_internal_quantize_few_batch
    n = len(shapes)
    fn.argtypes, fn.restype = [ctypes.c_int] + [ctypes.POINTER(ctypes.c_int64 * n)] * 2, ctypes.c_int
    return bool(fn(n, ctypes.byref((ctypes.c_int64 * n)(*[m for m, _ in shapes])),
                   ctypes.byref((ctypes.c_int64 * n)(*[k for _, k in shapes]))))
