"""Outputs whose rows begin at any byte (u8) or any int32: the wide stores of the tile kernels' epilogues inside the
matrix, their remainders at its right edge, and the bytes beyond it."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ldc_pad", [0, 1, 5, 8])
@pytest.mark.parametrize("kernel", ["NGEMM_KERNEL_TILE_64", "NGEMM_KERNEL_TILE_128", "NGEMM_KERNEL_TILE_256", "NGEMM_KERNEL_TILE_192"])
def test_any_output_pitch(kernel, ldc_pad):
    import paper_1910_00178_amd as ng
    from gpu_util import Runner
    r = Runner()
    r.set_kernel(getattr(ng, kernel))
    rng = np.random.default_rng(ldc_pad)
    # 64 x 64: more tiles than the small-output kernel takes; K = 192: pipelined stages and, at 200, a remainder
    for M, N, K in ((1100, 1600, 200), (300, 515, 192), (260, 530, 200)):
        A = rng.integers(0, 256, size=(M, K), dtype=np.uint8)
        B = rng.integers(-128, 128, size=(N, K), dtype=np.int8)
        h, packed = r.pack(B)
        for lda_pad in (-K % 16, 1):                   # the direct-to-LDS kernels, the register-staged ones
            got = r.run(A, h, N, 131, 3, scale=0.0011, zc=120, lda_pad=lda_pad, ldc_pad=ldc_pad)
            assert np.array_equal(got, oracle.gemm_u8s8u8_requant(A, B, 131, 3, 0.0011, 120)), (M, N, K, lda_pad)
            got = r.run(A, h, N, 131, 3, lda_pad=lda_pad, ldc_pad=ldc_pad)
            assert np.array_equal(got, oracle.gemm_u8s8s32(A, B, 131, 3)), (M, N, K, lda_pad)
    r.close()
