"""Which lines of their output the 144-channel product kernels store non-temporally, at sizes where the choices were measured
against each other: a change of a rule has to come with new measurements."""
import gpu_util as gu
import pytest

NONE, WHOLE, ALL = 0, 1, 2


# up to 16 MB all, beyond whole lines, beyond 28 MB none for fewer than 640 input channels
@pytest.mark.parametrize("M,K,N,lines", [(5120, 1152, 1152, ALL), (6144, 512, 1152, ALL), (4096, 4608, 1152, ALL), (3072, 512, 4608, WHOLE),
                                         (3072, 1152, 4608, WHOLE), (16384, 1152, 3456, WHOLE), (7168, 640, 2304, WHOLE),
                                         (11264, 512, 2304, NONE), (8192, 512, 4608, NONE)])
def test_pipelined_kernels(M, K, N, lines):
    assert gu.library_rule("_ZN4trdq4gemm13pipe144_linesElii", M, K, N) == lines


# row-major codes, K split inside the workgroup: from 9 MB on
@pytest.mark.parametrize("M,K,N,lines", [(4000, 1152, 1152, ALL), (2000, 2304, 2304, ALL), (1900, 1152, 2304, NONE), (1000, 1152, 3456, NONE),
                                         (3000, 4608, 1152, NONE)])
def test_k_split_rows(M, K, N, lines):
    assert bool(gu.library_rule("_ZN4trdq4gemm17ksplit_rows_linesElii", M, K, N) & 1) == (lines == ALL)
