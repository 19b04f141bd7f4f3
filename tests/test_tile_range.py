"""CPU: the range of the buffer descriptors that load operand tiles (csrc/tile_range.hpp, compiled for the
host): to the end of the dword that holds the last element of the tile, and never past the operand's."""
import ctypes
import itertools
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(HERE, "..", "paper_2201_13195_amd", "csrc", "tile_range.hpp")
SOURCE = """
#include "%s"
extern "C" int64_t range_bytes(int es, int krows, int64_t rows_left, int64_t tile_rows, int64_t ld, int64_t left, int64_t skew) {
    if (es == 2) return krows ? rmm::tile_range_bytes<2, true>(rows_left, tile_rows, ld, left, skew)
                              : rmm::tile_range_bytes<2, false>(rows_left, tile_rows, ld, left, skew);
    return krows ? rmm::tile_range_bytes<4, true>(rows_left, tile_rows, ld, left, skew)
                 : rmm::tile_range_bytes<4, false>(rows_left, tile_rows, ld, left, skew);
}
extern "C" uint32_t range_bytes_32(int es, int krows, uint32_t rows_left, uint32_t tile_rows, uint32_t ld, uint32_t left, uint32_t skew) {
    if (es == 2) return krows ? rmm::tile_range_bytes<2, true>(rows_left, tile_rows, ld, left, skew)
                              : rmm::tile_range_bytes<2, false>(rows_left, tile_rows, ld, left, skew);
    return krows ? rmm::tile_range_bytes<4, true>(rows_left, tile_rows, ld, left, skew)
                 : rmm::tile_range_bytes<4, false>(rows_left, tile_rows, ld, left, skew);
}
extern "C" uint32_t start(int y, uint32_t tile, int64_t m0, int64_t n0, int64_t columns) {
    return y ? rmm::start_of_place(m0, n0, columns) : rmm::start_of_tile(tile);
}
"""


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    where = tmp_path_factory.mktemp("range")
    src, lib = str(where / "range.cpp"), str(where / "range.so")
    with open(src, "w") as f:
        f.write(SOURCE % HEADER)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", src, "-o", lib], check=True)
    return ctypes.CDLL(lib)


@pytest.fixture(scope="module")
def range_bytes(built):
    f = built.range_bytes
    f.restype, f.argtypes = ctypes.c_int64, [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 5
    return f


@pytest.mark.parametrize("es", [2, 4])
@pytest.mark.parametrize("krows", [True, False])
def test_ranges_end_with_the_last_element(range_bytes, es, krows):
    """Operands of `outer` rows of `ld` elements at address 0, walked in tiles as the kernels walk them."""
    tile, bk = 8, 4           # (an even contraction step, as the kernels' are)
    for outer, ld in itertools.product((1, 2, 3, 7, 8, 9, 16, 17), repeat=2):
        rows, kk = (outer, ld) if krows else (ld, outer)
        end = (outer * ld * es + 3) // 4 * 4
        for row0, done in itertools.product(range(0, rows, tile), range(0, kk + 2 * bk, bk)):
            first = row0 * (ld if krows else 1) + done * (1 if krows else ld)
            skew = (first * es % 4) // es
            base, left = first * es - skew * es, min(kk - done, bk)
            reach = range_bytes(es, krows, rows - row0, tile, ld, left, skew)
            if left <= 0:
                assert reach == 0
                continue
            last = first + ((min(rows - row0, tile) - 1) * ld + left - 1 if krows else (left - 1) * ld + rows - row0 - 1)
            assert base % 4 == 0 and base + reach == (last * es + es + 3) // 4 * 4 <= end, (outer, ld, row0, done)


@pytest.mark.parametrize("es", [2, 4])
@pytest.mark.parametrize("krows", [True, False])
def test_ranges_in_32_bits_are_those_in_64(built, range_bytes, es, krows):
    """The kernels compute them in 32 bits: tiles of 128 rows (or 128 contraction rows) of up to 2^22 - 1 elements."""
    f = built.range_bytes_32
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_int, ctypes.c_int] + [ctypes.c_uint32] * 5
    most = 0
    for ld in (1, 7, 1001, (1 << 21) + 1, (1 << 22) - 1):
        for rows_left in {1, 2, 127, 128, 129, 2 ** 31 - 1} if krows else {1, ld // 2 + 1, ld}:
            for left in (0, 1, 2, 127, 128):
                for skew in ((0, 1) if es == 2 else (0,)):
                    want = range_bytes(es, krows, rows_left, 128, ld, left, skew)
                    assert f(es, krows, rows_left, 128, ld, left, skew) == want < 1 << 31, (rows_left, ld, left, skew)
                    most = max(most, want)
    assert most > 0.99 * (1 << 31) * es / 4


def test_eight_neighbouring_tiles_start_at_the_same_step(built):
    """dX and others: on tiles of any size.  Y: on 256 x 256 tiles, and every smaller tile starts as the one that it lies in."""
    rows, columns, group = 8192, 1304, 8
    starts = {}
    for edge in (256, 128, 64):
        tiles_m, tiles_n = -(-rows // edge), -(-columns // edge)
        for tile in range(tiles_m * tiles_n):                   # bands of eight tile rows, column by column
            band, in_band = divmod(tile, group * tiles_n)
            m0, n0 = (band * group + in_band % group) * edge, in_band // group * edge
            where = (ctypes.c_uint32(tile), ctypes.c_int64(m0), ctypes.c_int64(n0), ctypes.c_int64(columns))
            assert built.start(0, *where) == tile // group
            y = built.start(1, *where)
            assert y == starts.setdefault((m0 // 256, n0 // 256), y)
            if edge == 256:
                assert y == tile // group, tile
