"""The rules that pick a projection's kernel, shape and K slices (csrc/launch_rule.h), on the CPU."""
import ctypes
import random

import pytest

from tests.test_abi_host import HOST_LIB

STREAM = (0, 0, 0, 0)


ROOM = (7 << 20, 1 << 14)  # floats and counters of split-K: more than any pick below asks for


def _lib():
    lib = ctypes.CDLL(HOST_LIB)
    i, z = ctypes.c_int, ctypes.c_size_t
    lib.sprh_gemm_pick.argtypes = [i, i, i, i, i, i, z, i, ctypes.c_void_p]
    lib.sprh_tile_pick.argtypes = [i, i, i, i, z, i, ctypes.c_void_p]
    return lib


def gemm_pick(bf16, n, nt, kb, parts, norm, room=ROOM):
    """(waves, tiles per wave, K-blocks per chunk, slices) of the panel kernel; zeros: the streaming kernel."""
    out = (ctypes.c_int32 * 4)()
    _lib().sprh_gemm_pick(int(not bf16), n, nt, kb, parts, int(norm), *room, out)
    return tuple(out)


def tile_pick(nt, kb, padded_rows, parts, room=ROOM):
    """(weight tiles, row tiles, stages, slices) of the tiled prefill projection."""
    out = (ctypes.c_int32 * 4)()
    _lib().sprh_tile_pick(nt, kb, padded_rows, parts, *room, out)
    return tuple(out)


def row_tiles(n):
    t = -(-n // 16)
    return t if t <= 4 else 6 if t <= 6 else 8


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


@pytest.mark.parametrize("room", [(0, 0), (64 << 10, 256), (300 << 10, 4096), (1 << 20, 4096), (4 << 20, 100), (7 << 20, 1 << 14)])
def test_split_k_fits_the_room(room):
    """What a split launch writes (per group and wave: slices x fragments of 256 floats, one counter) is inside its room."""
    rng = random.Random(sum(room))
    split = 0
    for _ in range(3000):
        nt, kb = int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 11))
        n, parts, norm, bf16 = rng.randint(1, 128), rng.choice([2, 3]), rng.random() < 0.5, rng.random() < 0.8
        nw, rt, uc, s = gemm_pick(bf16, n, nt, kb, parts if bf16 else 1, norm, room)
        if s > 1:
            groups, jt = -(-nt // (nw * rt)), row_tiles(n)
            assert s <= -(-kb // uc)
            assert groups * nw <= room[1] and groups * nw * s * (rt * jt + norm * -(-jt // 4)) * 256 <= room[0]
        split += s > 1
        rows = 128 * rng.randint(1, 32)
        tn, tm, _, s = tile_pick(nt, kb, rows, parts, room)
        if s > 1:
            tiles = -(-nt // tn) * -(-(rows // 16) // tm)
            assert s <= kb and tiles * 4 <= room[1] and tiles * s * tn * tm * 256 <= room[0]
        split += s > 1
    assert (split > 0) == (room[0] > 0)
