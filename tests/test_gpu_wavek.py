"""The kernel that splits K over a workgroup's wavefronts, against the oracle, at the edges of its tiles (32 and 64
rows and columns), of its steps (64 bytes of K, dealt out to two or four wavefronts) and of the rules that choose
its forms."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def runner():
    from gpu_util import Runner
    r = Runner()
    yield r
    r.close()


# (M, N): one tile and its edges; forms of 32 x 32, 32 x 64 and 64 x 64 tiles
S16_OUT = [(1, 1), (31, 33), (33, 31), (64, 70), (600, 500), (300, 1800), (900, 900), (1000, 1500)]
# elements of K: partial steps (32 elements), fewer steps than wavefronts, one and several rounds of them
S16_K = [1, 31, 32, 40, 127, 128, 161, 300]


@pytest.mark.parametrize("K", S16_K)
def test_s16_small_outputs(runner, K):
    import torch
    import paper_1910_00178_amd as ng
    rng = np.random.default_rng(K)
    for M, N in S16_OUT:
        A = rng.integers(-32768, 32768, size=(M, K)).astype(np.int16)
        B = rng.integers(-32768, 32768, size=(N, K)).astype(np.int16)
        lda = (K + 7) // 8 * 8
        Ah = np.full((M, lda), 7777, np.int16)
        Ah[:, :K] = A
        Ad, Bd = torch.from_numpy(Ah).cuda(), torch.from_numpy(B).cuda()
        nb = ng.ngemm_packed_b_bytes_s16(K, N)
        packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
        h = ng.ngemm_pack_b_s16(runner.ctx, K, N, Bd, K, packed, nb)
        wsb = ng.ngemm_workspace_bytes(M, N, K)
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
        C = torch.full((M + 1, N + 3), -7, dtype=torch.int32, device="cuda")
        za, zb = int(rng.integers(-32768, 32768)), int(rng.integers(-32768, 32768))
        ng.ngemm_run_s16s16s32(runner.ctx, M, Ad, lda, za, h, zb, C, N + 3, ws, wsb)
        got = C.cpu().numpy()
        ng.ngemm_packed_b_free(h)
        assert np.array_equal(got[:M, :N], oracle.gemm_s16s16s32(A, B, za, zb)), (M, N)
        assert (got[M:] == -7).all() and (got[:, N:] == -7).all(), (M, N)
