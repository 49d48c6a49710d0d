"""The rules that pick a projection's kernel, shape and K slices (csrc/launch_rule.h), on the CPU."""
import ctypes

import pytest

from tests.test_abi_host import HOST_LIB

STREAM = (0, 0, 0, 0)


def gemm_pick(bf16, n, nt, kb, parts, norm):
    """(waves, tiles per wave, K-blocks per chunk, slices) of the panel kernel; zeros: the streaming kernel."""
    lib = ctypes.CDLL(HOST_LIB)
    out = (ctypes.c_int32 * 4)()
    lib.sprh_gemm_pick(int(not bf16), n, nt, kb, parts, int(norm), out)
    return tuple(out)


# (bf16, rows, weight tiles, K-blocks, parts, fused norm, us streamed, us on the panel kernel), measured on MI355X.
MEASURED = [
    # fp32, models of 256, 1024 and 4096 features
    (False, 9, 48, 16, 1, True, 3.1, 5.6), (False, 16, 16, 43, 1, False, 4.8, 12.9), (False, 64, 48, 16, 1, True, 6.2, 11.2),
    (False, 24, 352, 64, 1, True, 15.4, 19.6), (False, 64, 352, 64, 1, True, 30.5, 28.6),
    (False, 24, 64, 64, 1, False, 6.2, 8.7), (False, 64, 64, 176, 1, False, 21.0, 17.6),
    (False, 16, 1376, 256, 1, True, 69.5, 83.6), (False, 24, 1376, 256, 1, True, 162.3, 106.5),
    (False, 64, 2000, 256, 1, True, 501.2, 178.9),
    # bf16, models of 256, 1024, 2048 and 4096 features
    (True, 9, 48, 8, 3, True, 3.0, 3.9), (True, 64, 16, 22, 2, False, 6.0, 7.7), (True, 9, 192, 32, 3, True, 4.9, 7.2),
    (True, 24, 64, 32, 2, False, 4.8, 6.9), (True, 64, 64, 88, 2, False, 14.5, 10.8),
    (True, 9, 128, 64, 2, False, 5.0, 6.9), (True, 24, 384, 64, 3, True, 13.5, 11.9),
    (True, 9, 2000, 64, 2, True, 21.1, 26.0), (True, 9, 1024, 96, 2, True, 18.4, 17.8),
    (True, 9, 256, 128, 2, False, 8.3, 9.5), (True, 32, 256, 128, 2, False, 12.7, 11.2),
    (True, 16, 256, 344, 2, False, 22.8, 17.9), (True, 24, 256, 344, 2, False, 27.0, 21.6),
    (True, 64, 1376, 128, 2, True, 92.3, 38.1),
    # bf16, at most 8 rows: large matrices on both sides of the panel kernel's one-round range
    (True, 1, 2304, 256, 2, True, 96.6, 102.4), (True, 1, 2560, 256, 2, True, 104.2, 105.9),
    (True, 1, 2688, 256, 2, True, 113.5, 108.4), (True, 8, 3584, 256, 2, True, 139.7, 132.4),
    (True, 1, 3200, 192, 2, True, 95.0, 90.9), (True, 1, 4608, 256, 2, True, 184.5, 209.4),
    (True, 1, 5120, 192, 2, True, 145.8, 165.3), (True, 8, 8016, 256, 2, True, 308.2, 339.6),
    (True, 1, 4608, 160, 2, True, 110.5, 134.0), (True, 8, 1376, 128, 2, True, 29.9, 30.1),
]


@pytest.mark.parametrize("bf16,n,nt,kb,parts,norm,stream_us,panel_us", MEASURED)
def test_the_faster_kernel_is_picked(bf16, n, nt, kb, parts, norm, stream_us, panel_us):
    assert (gemm_pick(bf16, n, nt, kb, parts, norm) == STREAM) == (stream_us < panel_us)
