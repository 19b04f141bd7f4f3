"""CPU: where a backward pass makes its bias gradient (a rule on sizes, asked of the built library)."""
import ctypes

import pytest

import paper_2201_13195_amd as rmm


@pytest.fixture(scope="module")
def pair_takes_colsum():
    f = rmm.load_library()._ZN3rmm26backward_pair_takes_colsumElllli     # rmm::backward_pair_takes_colsum
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int64] * 4 + [ctypes.c_int]
    return f


@pytest.mark.parametrize("kind", [rmm.GAUSSIAN, rmm.RADEMACHER])
def test_column_sums_go_where_there_is_room(pair_takes_colsum, kind):
    # dW fills the chip (256 tiles): beside the sketch work-groups, which leave room for them
    for n, d_in, d_out, k in ((16384, 1024, 4096, 1638), (32768, 1024, 4096, 1638), (16384, 4096, 1024, 1638)):
        assert pair_takes_colsum(n, d_in, d_out, k, kind), (n, d_in, d_out, k)
    # dW leaves most of it idle; the paired launch has no place left (k = 64)
    for n, d_in, d_out, k in ((4096, 768, 3072, 410), (4096, 768, 768, 410), (16384, 1024, 4096, 64)):
        assert not pair_takes_colsum(n, d_in, d_out, k, kind), (n, d_in, d_out, k)
