"""The sizes that the library's host side chooses, read from the instrumented
build (the same sources; its debug exports launch nothing)."""
import ctypes as C

from paper_2601_21758_amd.build import LIB_STAMPS

_lib = None


def _debug():
    global _lib
    if _lib is None:
        _lib = C.CDLL(LIB_STAMPS)
    return _lib


def _call(name, args, fields):
    out = (C.c_int64 * len(fields))()
    getattr(_debug(), name)(*args, out)
    return dict(zip(fields, out))


def tactical(n, B):
    """Algorithm 1's sample: the thresholds' rank (0: none taken), every 2^lg_step-th chunk, samples, the places they
    are spread over and the places there is room for; the workspace offset of the rows' member counts (int32) and
    the most members a row may have."""
    return _call("ewsjf_debug_tactical", (C.c_int64(n), C.c_int32(B)),
                 ("rank", "lg_step", "samples", "places", "room", "count_at", "list_cap"))


def plan(op, n, rows, B):
    """The selection plan of an operation (_lib.OP_STEP, OP_SELECT, OP_TRIAL): workgroups per row, bar groups per wave
    (log2), list entries per workgroup, entries a wave keeps at least when its region overflows; of a step under
    several vectors, the filter's rank (0: not filtered) and the survivors it has room for (their number is the
    workspace's first int32, the vectors' thresholds its float32 from byte 256 on)."""
    return _call("ewsjf_debug_plan", (C.c_int(op), C.c_int64(n), C.c_int32(rows), C.c_int32(B)),
                 ("G", "lg", "M", "fit", "filter", "room"))
