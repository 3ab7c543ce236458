"""The test-only library that launches count, fill and statistics kernels on arrays of a test's making."""
import ctypes
import os
import subprocess

from paper_2401_08586_amd import build as B

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")
SRC = os.path.join(HERE, "search_harness.hip")
LIB = os.path.join(HERE, "libsearch_harness.so")


def build():
    tmp = LIB + ".tmp"
    subprocess.check_call(["hipcc", *B.FLAGS, "-I", B.CSRC, "-o", tmp, SRC, "-L", B.HERE, "-lnnps",
                           "-Wl,-rpath,$ORIGIN/../../paper_2401_08586_amd"])
    os.replace(tmp, LIB)
    return LIB


_POINTERS = ("pos row_ptr col dist set_room offs cell_offs skey perm cell_start spos rq bstart bset nblk counts counts_s "
             "rsort bdesc branks heavy flags cbits wdense usz uoff ulist unit_off ucell dn dboff dbits "
             "blk_stats dstats stats rpool").split()


class Args(ctypes.Structure):
    """HarnessArgs of search_harness.hip."""
    _fields_ = ([(k, ctypes.c_int32) for k in ("dim", "mode", "n", "half")] +
                [(k, ctypes.c_int64) for k in ("capacity", "dbits_cap")] + [(k, ctypes.c_void_p) for k in _POINTERS] +
                [("radius", ctypes.c_double)] + [(k, ctypes.c_int32) for k in ("t_lo", "t_hi", "t_mid", "nblk_max", "rpool_cap", "sparse")])


def load():
    if not os.path.exists(LIB):
        build()
    lib = ctypes.CDLL(LIB)
    lib.harness_count.argtypes = [ctypes.POINTER(Args)]
    lib.harness_fill.argtypes = lib.harness_stats.argtypes = [ctypes.POINTER(Args), ctypes.c_int]
    return lib
