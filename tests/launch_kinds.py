"""The kinds of sampling launch (csrc/internal.hpp), and which one a problem takes."""
import ctypes as C

from paper_2202_01753_amd import mcubes as M

PLAIN, TRACED, COPIES, SPLIT, FUSED, STAGED, STAGED_UNIT, PER_AXIS = range(8)


def launch_kind(bp: M.BoundProblem, adjust: bool = True, run: bool = False) -> int:
    fn = M.lib().mcubes_launch_kind
    fn.argtypes, fn.restype = [C.c_void_p, C.c_int32, C.c_int32], C.c_int32
    kind = fn(bp.ref, int(adjust), int(run))
    assert kind >= 0
    return kind
