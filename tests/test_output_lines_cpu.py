"""Which lines of their output the 144-channel product kernels store non-temporally, at sizes where the choices were measured
against each other: a change of a rule has to come with new measurements."""
import gpu_util as gu
import pytest

NONE, WHOLE, ALL = 0, 1, 2


# up to 20 MB all, beyond whole lines, beyond 28 MB none for fewer than 640 input channels
@pytest.mark.parametrize("M,K,N,lines", [(5120, 1152, 1152, ALL), (6144, 512, 1152, ALL), (4096, 4608, 1152, ALL), (8192, 4608, 1152, ALL), (3072, 512, 4608, WHOLE),
                                         (3072, 1152, 4608, WHOLE), (16384, 1152, 3456, WHOLE), (7168, 640, 2304, WHOLE),
                                         (11264, 512, 2304, NONE), (8192, 512, 4608, NONE)])
def test_pipelined_kernels(M, K, N, lines):
    assert gu.library_rule("_ZN4trdq4gemm13pipe144_linesElii", M, K, N) == lines


# tiled product: all lines from 8 to 20 MB (from 16 on whole ones for fewer than 640 input channels), none to 64 (128 for 1024 to 1151 input channels,
# 192 for fewer), then all, or whole ones for fewer than 768
@pytest.mark.parametrize("M,K,N,lines", [(6000, 256, 288, NONE), (9368, 256, 288, NONE), (5120, 768, 1152, ALL), (2560, 1152, 2304, ALL),
                                         (4096, 1152, 1152, ALL), (8192, 1152, 1152, ALL), (4096, 512, 2304, WHOLE), (8192, 384, 1152, WHOLE),
                                         (4096, 896, 3456, NONE), (4096, 1152, 3456, NONE), (5000, 768, 2304, NONE),
                                         (8192, 512, 2304, NONE), (8192, 768, 2304, NONE), (4096, 1152, 4608, NONE), (6144, 1536, 3456, NONE),
                                         (16384, 896, 2304, NONE), (8192, 1024, 4608, NONE), (8192, 1152, 4608, ALL), (16384, 1152, 3456, ALL),
                                         (16384, 1024, 4608, ALL), (32768, 768, 4608, ALL), (16384, 512, 4608, NONE), (32768, 512, 4608, WHOLE),
                                         (32768, 1152, 4608, ALL)])
def test_tiled_kernel(M, K, N, lines):
    assert gu.library_rule("_ZN4trdq4gemm11tiled_linesElii", M, K, N) == lines
