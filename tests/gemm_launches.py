"""Which kernels a matrix product runs, as the library's planner describes them
(on the current device; for 256 CUs, those of an MI355X, without one)."""
import ctypes

import paper_2602_06063_amd as q4

_describe = q4.lib.q4nx_internal_gemm_launches
_describe.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.c_char_p, ctypes.c_int]
_describe.restype = ctypes.c_int

FORMATS = (q4.Q4NX_WEIGHTS_Q4NX, q4.Q4NX_WEIGHTS_MXFP4, q4.Q4NX_WEIGHTS_BF16)


def launches(fmt, M, N, K, work=False):
    """Such as "ks 80x64", "tile 256x192 + tile 128x128", "dequant + split4 256x256"."""
    text = ctypes.create_string_buffer(256)
    assert _describe(fmt, M, N, K, int(work), text, len(text)) >= 0
    return text.value.decode()
