"""The kernel that splits K over a workgroup's wavefronts, against the oracle, at the edges of its tiles (32 and 64
rows and columns), of its steps (64 bytes of K, dealt out to two or four wavefronts) and of the rules that choose
its forms."""
import numpy as np
import pytest

import oracle
from test_gpu_routes import launches  # noqa: F401

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


# Under a cap on workgroups: the 128 x 128 kernel and, below two of its stages, the looping form, several tiles each.  Without
# one, outputs of more than a tile per compute unit: what is left of K behind the pipelined stages of 64 elements (an odd
# full stage, a partial one, both, neither), ragged rows and columns, values at both ends of the type.
S16_LARGE_K = [128, 129, 191, 192, 209, 257, 320]
S16_LARGE = [(300, 400, K, 3) for K in [1, 40, 127] + S16_LARGE_K] + [(M, N, K, 0) for M, N in ((1500, 1700), (2049, 2111)) for K in S16_LARGE_K]


@pytest.mark.parametrize("M,N,K,cap", S16_LARGE)
def test_s16_large_tile_kernel_and_caps(runner, M, N, K, cap):
    import torch
    import paper_1910_00178_amd as ng
    rng = np.random.default_rng(M + K)
    A = rng.integers(-32768, 32768, size=(M, K)).astype(np.int16)
    B = rng.integers(-32768, 32768, size=(N, K)).astype(np.int16)
    A[::3], B[1::4] = np.where(A[::3] < 0, -32768, 32767), np.where(B[1::4] < 0, -32768, 32767)
    lda = (K + 7) // 8 * 8
    Ah = np.full((M, lda), 7777, np.int16)
    Ah[:, :K] = A
    Ad, Bd = torch.from_numpy(Ah.reshape(-1)[:(M - 1) * lda + K].copy()).cuda(), torch.from_numpy(B).cuda()
    nb = ng.ngemm_packed_b_bytes_s16(K, N)
    packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
    h = ng.ngemm_pack_b_s16(runner.ctx, K, N, Bd, K, packed, nb)
    wsb = ng.ngemm_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    C = torch.full((M + 1, N + 3), -7, dtype=torch.int32, device="cuda")
    za, zb = int(rng.integers(-32768, 32768)), int(rng.integers(-32768, 32768))
    ng.ngemm_set_max_workgroups(runner.ctx, cap)
    try:
        ng.ngemm_run_s16s16s32(runner.ctx, M, Ad, lda, za, h, zb, C, N + 3, ws, wsb)
        got = C.cpu().numpy()
    finally:
        ng.ngemm_set_max_workgroups(runner.ctx, 0)
    ng.ngemm_packed_b_free(h)
    # exact in 64 bits (|sum| < 2^41), then the low 32; float64 products of 16-bit values and sums below 2^53 are exact
    want = ((A.astype(np.float64) - za) @ (B.astype(np.float64) - zb).T).astype(np.int64).astype(np.int32)
    assert np.array_equal(want[::97], oracle.gemm_s16s16s32(np.ascontiguousarray(A[::97]), B, za, zb))
    assert np.array_equal(got[:M, :N], want)
    assert (got[M:] == -7).all() and (got[:, N:] == -7).all()


# Row and column sums beyond 2^31, which wrap like everything else: the pack's, the small-output kernel's and, under a cap,
# the row-sum launch of the 128 x 128 kernel
@pytest.mark.parametrize("cap", [0, 2])
def test_s16_sums_wrap(runner, cap):
    import torch
    import paper_1910_00178_amd as ng
    M, N, K = 290, 270, 70000
    rng = np.random.default_rng(cap)
    A, B = np.full((M, K), -32768, np.int16), np.full((N, K), 32767, np.int16)
    A[::2], B[::3] = rng.integers(-32768, 32768, size=A[::2].shape), rng.integers(-32768, 32768, size=B[::3].shape)
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    nb = ng.ngemm_packed_b_bytes_s16(K, N)
    packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
    h = ng.ngemm_pack_b_s16(runner.ctx, K, N, Bd, K, packed, nb)
    wsb = ng.ngemm_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    ng.ngemm_set_max_workgroups(runner.ctx, cap)
    try:
        ng.ngemm_run_s16s16s32(runner.ctx, M, Ad, K, 12345, h, -23456, C, N, ws, wsb)
        got = C.cpu().numpy()
    finally:
        ng.ngemm_set_max_workgroups(runner.ctx, 0)
    ng.ngemm_packed_b_free(h)
    # float64: every product below 2^33 and every sum below 2^50 is exact
    want = ((A.astype(np.float64) - 12345) @ (B.astype(np.float64) + 23456).T).astype(np.int64).astype(np.int32)
    assert abs(A[1].astype(np.int64).sum()) > 2 ** 31 and B[1].astype(np.int64).sum() > 2 ** 31
    assert np.array_equal(got, want)


# (M, N, K): every form of the 8-bit rule on 256 compute units: 32 x 32 tiles, two wavefronts per tile (M <= 32 and
# not), 32 x 64, 64 x 64 and 64 x 128 tiles, each with ragged rows, columns and partial steps
U8_CASES = [(1, 1, 1), (33, 31, 63), (64, 70, 64), (5, 300, 65), (31, 100, 129), (33, 33, 511), (70, 129, 4097), (300, 500, 200),
            (32, 9000, 70), (7, 10001, 200), (600, 700, 300), (1000, 600, 257), (520, 1000, 64), (100, 5100, 90), (500, 1900, 1100),
            (9, 33, 300), (40, 16000, 2049), (300, 4000, 3100), (1000, 1300, 3073),
            # M <= 32 with non-temporal copies of B, the partial step asked for early: four and two wavefronts, 32 x 64 tiles
            (3, 4000, 777), (16, 300, 1000), (30, 8190, 1000), (7, 9000, 900), (13, 10000, 2100), (20, 8200, 2500), (2, 17000, 2049)]


@pytest.mark.parametrize("pitch", ["padded", "tight"])
@pytest.mark.parametrize("case", U8_CASES, ids=str)
def test_u8_small_outputs(runner, case, pitch):
    import torch
    import paper_1910_00178_amd as ng
    M, N, K = case
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    A = rng.integers(0, 256, size=(M, K), dtype=np.uint8)
    B = rng.integers(-128, 128, size=(N, K), dtype=np.int8)
    handle, packed = runner.pack(B)
    pad = -K % 16 if pitch == "padded" else (1 if K % 16 == 0 else 0)      # tight: rows of any alignment
    for za, zb, ldc_pad in ((0, 0, 0), (131, 0, 1), (255, -128, 0), (7, 5, 2)):
        assert np.array_equal(runner.run(A, handle, N, za, zb, lda_pad=pad, ldc_pad=ldc_pad), oracle.gemm_u8s8s32(A, B, za, zb)), (za, zb)
        assert np.array_equal(runner.run(A, handle, N, za, zb, scale=0.0007, zc=99, lda_pad=pad, ldc_pad=ldc_pad),
                              oracle.gemm_u8s8u8_requant(A, B, za, zb, 0.0007, 99)), (za, zb)
    # per-column scales, bias, zero-points and ReLU; signed A
    scale = rng.uniform(0.0003, 0.001, N).astype(np.float32)
    bias, zbv = rng.integers(-9999, 9999, N).astype(np.int32), rng.integers(-128, 128, N).astype(np.int32)
    lda = K + pad
    Ah = np.full((M, lda), 201, np.uint8)
    Ah[:, :K] = A
    Ad, sd, bd, zd = (torch.from_numpy(x).cuda() for x in (Ah, scale, bias, zbv))
    wsb = ng.ngemm_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    C8 = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    for zc, relu in ((3, True), (1 << 24, False)):          # the second takes the 64-bit form of the arithmetic
        ng.ngemm_run_u8s8u8_requant_channel(runner.ctx, M, Ad, lda, 77, handle, 0, zd, sd, bd, relu, zc, C8, N, ws, wsb)
        want = oracle.gemm_u8s8u8_requant_channel(A, B, 77, 0, scale, zc, zb_vec=zbv, bias=bias, relu=relu)
        assert np.array_equal(C8.cpu().numpy(), want), (zc, relu)
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    ng.ngemm_run_s8s8s32(runner.ctx, M, Ad, lda, -5, handle, 9, C, N, ws, wsb)
    assert np.array_equal(C.cpu().numpy(), oracle.gemm_s8s8s32(A.view(np.int8), B, -5, 9))
    ng.ngemm_packed_b_free(handle)


# Unpacked B: the forms above on the caller's storage, and the 64 x 64 (1100 x 1600) and 128 x 128 (1600 x 1700 with a
# long K) tiles that form both operands' sums
RAW_CASES = [(1, 1, 1), (33, 31, 63), (31, 100, 129), (300, 500, 200), (32, 9000, 70), (7, 10001, 200), (600, 700, 300),
             (500, 1900, 1100), (1100, 1600, 100), (1111, 1601, 64), (1600, 1700, 1041), (30, 17000, 4100), (300, 4000, 3100)]


@pytest.mark.parametrize("case", RAW_CASES, ids=str)
def test_unpacked_sums_in_kernel(runner, case):
    import torch
    import paper_1910_00178_amd as ng
    M, N, K = case
    rng = np.random.default_rng(M * 5 + N * 3 + K)
    pitch = (K + 15) // 16 * 16 + 16
    Ah, Bh = rng.integers(0, 256, size=(M, pitch), dtype=np.uint8), rng.integers(-128, 128, size=(N, pitch), dtype=np.int8)
    A, B = np.ascontiguousarray(Ah[:, :K]), np.ascontiguousarray(Bh[:, :K])
    Ad, Bd = torch.from_numpy(Ah).cuda(), torch.from_numpy(Bh).cuda()
    wsb = ng.ngemm_unpacked_workspace_bytes(M, N, K)
    ws = torch.full((wsb,), 0xC3, dtype=torch.uint8, device="cuda")
    for za, zb in ((128, 0), (0, 0), (128, -7), (200, 127)):
        C = torch.full((M + 1, N + 1), -7, dtype=torch.int32, device="cuda")
        ng.ngemm_run_u8s8s32_unpacked(runner.ctx, M, N, K, Ad, pitch, za, Bd, pitch, zb, C, N + 1, ws, wsb)
        got = C.cpu().numpy()
        want = oracle.gemm_u8s8s32(A, B, za, zb)
        assert np.array_equal(got[:M, :N], want), (za, zb)
        assert (got[M:] == -7).all() and (got[:, N:] == -7).all()


def test_forced_skinny_stays_refused_beyond_its_rows(runner):
    import torch
    import paper_1910_00178_amd as ng
    M, N, K = 33, 64, 64
    A = torch.zeros((M, K), dtype=torch.uint8, device="cuda")
    B = torch.zeros((N, K), dtype=torch.int8, device="cuda")
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    wsb = ng.ngemm_unpacked_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    runner.set_kernel(ng.NGEMM_KERNEL_SKINNY)
    try:
        with pytest.raises(ng.NgemmError):
            ng.ngemm_run_u8s8s32_unpacked(runner.ctx, M, N, K, A, K, 0, B, K, 0, C, N, ws, wsb)
    finally:
        runner.set_kernel(ng.NGEMM_KERNEL_AUTO)


# Every number of steps of a wavefront around the ends of its ring (four or two wavefronts, 64 bytes a step): the steps that are laid out one by one,
# the first that are asked for at once, K ending in any of them, within 16 bytes and not; rows of any alignment, whose A comes through registers,
# and aligned ones.  The allocation ends with the last byte of A.
@pytest.mark.parametrize("pad", [0, 1], ids=["aligned", "tight"])
@pytest.mark.parametrize("M,N", [(40, 1100), (13, 8300)])
def test_u8_every_number_of_steps(runner, M, N, pad):
    import torch
    rng = np.random.default_rng(M)
    Kmax = 64 * (56 if N < 8192 else 30)
    B = rng.integers(-128, 128, size=(N, Kmax), dtype=np.int8)
    A = rng.integers(0, 256, size=(M, Kmax), dtype=np.uint8)
    Bd = torch.from_numpy(B).cuda().double()
    for k, K in enumerate(sorted({64 * q + r for q in range(Kmax // 64) for r in ((0, 9, 53) if q % 3 else (23, 32))} - {0})):
        if k % (1 if N < 8192 else 2): continue
        if pad and K % 16 == 0: K += 3
        K = min(K, Kmax - 1)
        za, zb = 131, (0, 5)[k % 2]
        h, packed = runner.pack(np.ascontiguousarray(B[:, :K]))
        got = runner.run(np.ascontiguousarray(A[:, :K]), h, N, za=za, zb=zb, lda_pad=0 if pad else -K % 16)
        want = ((torch.from_numpy(A[:, :K]).cuda().double() - za) @ (Bd[:, :K] - zb).t()).long().int().cpu().numpy()
        assert np.array_equal(got, want), (K, zb)
        import paper_1910_00178_amd as ng
        ng.ngemm_packed_b_free(h)


# At most one step per wavefront, aligned rows: a branch of its own, in which K ends in any byte of the step or not at all.  The allocations end with
# the last byte of the last row.
@pytest.mark.parametrize("op", ["u8", "s16", "unpacked"])
@pytest.mark.parametrize("M,N", [(1, 70), (17, 33), (40, 96)])
def test_one_step_per_wavefront(runner, op, M, N):
    import torch
    import paper_1910_00178_amd as ng
    gen = torch.Generator(device="cuda").manual_seed(M)
    ta, tb, elems = (torch.int16, torch.int16, 8) if op == "s16" else (torch.uint8, torch.int8, 16)
    ia, ib = torch.iinfo(ta), torch.iinfo(tb)
    size, pack, run = (ng.ngemm_packed_b_bytes_s16, ng.ngemm_pack_b_s16, ng.ngemm_run_s16s16s32) if op == "s16" else \
        (ng.ngemm_packed_b_bytes, ng.ngemm_pack_b, ng.ngemm_run_u8s8s32)
    wsb = ng.ngemm_unpacked_workspace_bytes(M, N, 300) + ng.ngemm_workspace_bytes(M, N, 300)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    for K in range(1, 17 * elems + 1):
        ld = (K + elems - 1) // elems * elems
        A = torch.randint(ia.min, ia.max + 1, ((M - 1) * ld + K,), generator=gen, device="cuda", dtype=ta)
        B = torch.randint(ib.min, ib.max + 1, ((N - 1) * ld + K,), generator=gen, device="cuda", dtype=tb)
        C = torch.full((M + 1, N + 1), -7, dtype=torch.int32, device="cuda")
        za, zb = ((131, 0), (131, 5), (128, -3))[K % 3]
        if op == "unpacked":
            ng.ngemm_run_u8s8s32_unpacked(runner.ctx, M, N, K, A, ld, za, B, ld, zb, C, N + 1, ws, wsb)
        else:
            packed = torch.empty(size(K, N), dtype=torch.uint8, device="cuda")
            h = pack(runner.ctx, K, N, B, ld, packed, packed.numel())
            run(runner.ctx, M, A, ld, za, h, zb, C, N + 1, ws, wsb)
            ng.ngemm_packed_b_free(h)
        _check(A.as_strided((M, K), (ld, 1)), B.as_strided((N, K), (ld, 1)), za, zb, C)


# The same for the forms with a ring of three (32 x 64, 64 x 64 and 64 x 128 tiles of four wavefronts, aligned rows): other steps laid out, another first wait.
# From the smallest K that the rules give them over all that the last steps, the parity of the first fragments and the ring can meet; packed B and the
# caller's.  The allocations end with the last byte.
THREE = [(600, 700, 1, "gemm_wavek_kernel<1, 1, 2, 4, 3,"), (700, 1400, 1025, "gemm_wavek_kernel<1, 2, 2, 4, 3,"), (200, 6000, 3072, "gemm_wavek_kernel<1, 2, 4, 4, 3,")]


@pytest.mark.parametrize("M,N,first,kernel", THREE)
@pytest.mark.parametrize("raw", [False, True], ids=["packed", "unpacked"])
def test_u8_every_number_of_steps_of_a_ring_of_three(runner, launches, M, N, first, kernel, raw):  # noqa: F811
    import torch
    import paper_1910_00178_amd as ng
    gen = torch.Generator(device="cuda").manual_seed(M)
    most = first + 64 * 37
    Aall = torch.randint(0, 256, (M, most), generator=gen, device="cuda", dtype=torch.uint8)
    Ball = torch.randint(-128, 128, (N, most), generator=gen, device="cuda", dtype=torch.int8)
    Ad, Bd = Aall.double(), Ball.double()
    wsb = ng.ngemm_unpacked_workspace_bytes(M, N, most) + ng.ngemm_workspace_bytes(M, N, most)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    for n, K in enumerate(first + 64 * q + r for q in range(36) for r in ((0, 9, 53) if q % 3 else (23, 32))):
        za, zb, ld = 131, (0, 5)[n % 2], (K + 15) // 16 * 16
        A, B = (torch.zeros((X.shape[0], ld), dtype=X.dtype, device="cuda") for X in (Aall, Ball))
        A[:, :K], B[:, :K] = Aall[:, :K], Ball[:, :K]
        A, B = A.view(-1)[:(M - 1) * ld + K].clone(), B.view(-1)[:(N - 1) * ld + K].clone()
        C = torch.full((M + 1, N + 1), -7, dtype=torch.int32, device="cuda")
        if not raw:
            nb = ng.ngemm_packed_b_bytes(K, N)
            packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
            h = ng.ngemm_pack_b(runner.ctx, K, N, B, ld, packed, nb)

        def call(stream):
            if raw:
                ng.ngemm_run_u8s8s32_unpacked(runner.ctx, M, N, K, A, ld, za, B, ld, zb, C, N + 1, ws, wsb, stream)
            else:
                ng.ngemm_run_u8s8s32(runner.ctx, M, A, ld, za, h, zb, C, N + 1, ws, wsb, stream)
        if n % 16 == 0:
            torch.cuda.synchronize()
            names = [name for name, _ in launches(call)]
            assert len(names) == 1 and names[0].startswith(kernel), (K, names)
        call(None)
        want = ((Ad[:, :K] - za) @ (Bd[:, :K] - zb).t()).int()
        assert torch.equal(C[:M, :N], want) and bool((C[M:] == -7).all()) and bool((C[:, N:] == -7).all()), (K, zb)
        if not raw: ng.ngemm_packed_b_free(h)


# Rows of any alignment, long, two 32 x 64 tiles to a unit: from K = 2048 on every other step waits for all of its loads.  Every number of steps
# modulo the four that are laid out, on both sides of the line, the first and last number of tiles that it holds for.
@pytest.mark.parametrize("M,N", [(13, 16384), (13, 16385), (12, 49152), (300, 3000)])
def test_long_unaligned_rows_two_tiles_to_a_unit(runner, launches, M, N):  # noqa: F811
    import torch
    import paper_1910_00178_amd as ng
    gen = torch.Generator(device="cuda").manual_seed(N)
    wsb = ng.ngemm_workspace_bytes(M, N, 2700)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    for K in (2047, 2049, 2111, 2175, 2241, 2300, 2367, 2431, 2497, 2570, 2625):
        A = torch.randint(0, 256, (M * K,), generator=gen, device="cuda", dtype=torch.uint8)
        B = torch.randint(-128, 128, (N, K), generator=gen, device="cuda", dtype=torch.int8)
        packed = torch.empty(ng.ngemm_packed_b_bytes(K, N), dtype=torch.uint8, device="cuda")
        h = ng.ngemm_pack_b(runner.ctx, K, N, B, K, packed, packed.numel())
        C = torch.full((M + 1, N + 1), -7, dtype=torch.int32, device="cuda")
        zb = (0, 5)[K & 2 and 1]
        call = lambda stream: ng.ngemm_run_u8s8s32(runner.ctx, M, A, K, 131, h, zb, C, N + 1, ws, wsb, stream)
        torch.cuda.synchronize()
        names = [name for name, _ in launches(call)]
        kernel = "gemm_wavek_drain_kernel<1, 2, 2, 4," if N != 16384 and K >= 2048 else "gemm_wavek_kernel<1, 1, 2, 2, 4," if M <= 32 else "gemm_"
        assert len(names) == 1 and names[0].startswith(kernel), (K, names)
        call(None)
        _check(A.view(M, K), B, 131, zb, C)
        ng.ngemm_packed_b_free(h)


# Pitches at which a tile's rows lie further apart than the kernel counts: its forms with addresses of 64 bits serve them, for 64 x 64 tiles of 16-bit
# operands the looping one; unpacked rows of any alignment are packed first.  "line": 16 KiB to either side of where the rule lies (2^31 - 8192 bytes over 64 rows of A, 128 of an unpacked
# B); "far": the last row is 4 GiB and more from the first, so that an offset of 32 bits would name another one.
FAR = [("u8", 3, 70, 200), ("u8", 40, 70, 200), ("u8 any", 40, 70, 201), ("s16", 3, 70, 100), ("s16", 40, 70, 100), ("s16", 40, 70, 300), ("s16", 70, 10944, 100), ("s16", 70, 10944, 300), ("u8", 40, 12000, 300),
       ("u8", 100, 8000, 1400), ("raw", 5, 70, 192),
       ("raw", 40, 70, 192), ("raw B", 40, 5, 192), ("raw B", 40, 70, 192), ("raw any", 40, 70, 191)]


@pytest.mark.parametrize("op,M,N,K", FAR)
@pytest.mark.parametrize("where", ["near the line", "past the line", "far"])
def test_rows_far_apart(runner, launches, op, M, N, K, where):  # noqa: F811
    import torch
    import paper_1910_00178_amd as ng
    size, of_b = 2 if op == "s16" else 1, op == "raw B"
    rows = N if of_b else M
    line = ((1 << 31) - 8192) // (128 if of_b else 64)
    ld = {"near the line": line - 16384, "past the line": line + 16384, "far": max((1 << 32) // (rows - 1) // 16 * 16 + 16, line + 16384)}[where] // 16 * 16 // size
    if op.endswith("any"): ld += 3
    assert where != "far" or (rows - 1) * ld * size >= 1 << 32
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    ta, tb = (torch.int16, torch.int16) if op == "s16" else (torch.uint8, torch.int8)
    ia, ib = torch.iinfo(ta), torch.iinfo(tb)
    A = torch.randint(ia.min, ia.max + 1, (M, K), generator=gen, device="cuda", dtype=ta)
    B = torch.randint(ib.min, ib.max + 1, (N, K), generator=gen, device="cuda", dtype=tb)
    far = torch.empty((rows - 1) * ld + K, dtype=tb if of_b else ta, device="cuda")
    far.as_strided((rows, K), (ld, 1)).copy_(B if of_b else A)
    C = torch.full((M + 1, N + 2), -7, dtype=torch.int32, device="cuda")
    h = None
    if op.startswith("raw"):
        wsb = ng.ngemm_unpacked_workspace_bytes(M, N, K)
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
        Ad, lda, Bd, ldb = (A, K, far, ld) if of_b else (far, ld, B, K)

        def call(stream):
            ng.ngemm_run_u8s8s32_unpacked(runner.ctx, M, N, K, Ad, lda, 37, Bd, ldb, 3, C, N + 2, ws, wsb, stream)
    else:
        size_of, pack, run = (ng.ngemm_packed_b_bytes_s16, ng.ngemm_pack_b_s16, ng.ngemm_run_s16s16s32) if op == "s16" else \
            (ng.ngemm_packed_b_bytes, ng.ngemm_pack_b, ng.ngemm_run_u8s8s32)
        nb = size_of(K, N)
        packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
        h = pack(runner.ctx, K, N, B, K, packed, nb)
        wsb = ng.ngemm_workspace_bytes(M, N, K)
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")

        def call(stream):
            run(runner.ctx, M, far, ld, 37, h, 3, C, N + 2, ws, wsb, stream)
    names = [name for name, _ in launches(call)]
    near = where == "near the line"
    looping = op == "s16" and N > 10000 and not near
    assert names[-1].startswith("gemm_wavek_kernel<" if near or looping else "gemm_wavek_far_kernel<"), names
    assert names[-1].endswith(", true>") or not looping, names
    assert (len(names) > 1) == (op == "raw any" and not near), names
    torch.cuda.synchronize()
    call(0)
    torch.cuda.synchronize()
    if h is not None:
        ng.ngemm_packed_b_free(h)
    want = ((A.double() - 37) @ (B.double() - 3).t()).long()
    want = ((want + 2**31) % 2**32 - 2**31).int()
    assert torch.equal(C[:M, :N], want) and bool((C[M:] == -7).all()) and bool((C[:, N:] == -7).all())


# Panels: a K of 2^24 - 64 is the first whose columns are too long (u8 outputs with a zero-point per column, which the K split over workgroups does not serve).
@pytest.mark.parametrize("K,near", [((1 << 24) - 192, True), ((1 << 24) - 64, False)])
def test_panels_far_apart(runner, launches, K, near):  # noqa: F811
    import torch
    import paper_1910_00178_amd as ng
    M, N = 33, 40
    A = torch.randint(0, 256, (M, K), device="cuda", dtype=torch.uint8)
    B = torch.randint(-128, 128, (N, K), device="cuda", dtype=torch.int8)
    zb = torch.randint(-9, 9, (N,), device="cuda", dtype=torch.int32)
    scales = torch.full((N,), 2.0 ** -24, device="cuda")
    nb = ng.ngemm_packed_b_bytes(K, N)
    packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
    h = ng.ngemm_pack_b(runner.ctx, K, N, B, K, packed, nb)
    wsb = ng.ngemm_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    C = torch.full((M + 1, N), 77, dtype=torch.uint8, device="cuda")

    def call(stream):
        ng.ngemm_run_u8s8u8_requant_channel(runner.ctx, M, A, K, 37, h, 0, zb, scales, None, False, 128, C, N, ws, wsb, stream)
    names = [name for name, _ in launches(call)]
    assert len(names) == 1 and names[0].startswith("gemm_wavek_kernel<" if near else "gemm_wavek_far_kernel<"), names
    torch.cuda.synchronize()
    call(0)
    sums = torch.zeros((M, N), dtype=torch.float64, device="cuda")           # (whole numbers below 2^53: exact)
    for k in range(0, K, 1 << 20):
        sums += (A[:, k:k + (1 << 20)].double() - 37) @ (B[:, k:k + (1 << 20)].double() - zb[:, None]).t()
    sums = (sums.long() + 2**31) % 2**32 - 2**31
    want = (torch.round(sums.float() * 2.0 ** -24).double() + 128).clamp(0, 255).to(torch.uint8)
    torch.cuda.synchronize()
    assert torch.equal(C[:M], want) and bool((C[M:] == 77).all())
    ng.ngemm_packed_b_free(h)


# (M, N, K, zero-point, output, kernel): each line of the rules that give a call 32 x 64 or 64 x 64 tiles of four wavefronts, on both sides
W12, W22 = "gemm_wavek_kernel<%d, 1, 2, 4, 3,", "gemm_wavek_kernel<%d, 2, 2, 4, 3,"
FORMS = [(661, 1469, 784, 0, "s32", W12 % 1), (661, 1469, 1025, 0, "s32", W22 % 1), (480, 2048, 4096, 0, "s32", W22 % 1),
         (480, 2048, 4097, 0, "s32", "gemm_tile_deep_kernel<1,"), (480, 2048, 3072, 0, "u8", W22 % 1), (480, 2048, 3073, 0, "u8", "gemm_tile_deep_kernel<1,"),
         (224, 3904, 383, 3, "s32", "gemm_tile_dma_kernel<64, 64,"), (224, 3904, 384, 3, "s32", W12 % 1), (224, 3904, 256, 3, "u8", W12 % 1),
         (412, 2492, 1472, 3, "s32", W12 % 1), (160, 5696, 3008, 0, "s32", W12 % 1), (160, 5696, 191, 0, "s32", "gemm_tile_dma_kernel<64, 64,"),
         (303, 2046, 2047, 5, "s16", W12 % 2), (303, 2046, 2048, 5, "s16", W22 % 2), (640, 1664, 2500, 5, "s16", "gemm_wavek_kernel<2, 2, 2, 2, 4,")]


@pytest.mark.parametrize("case", FORMS, ids=str)
def test_forms_and_their_lines(runner, launches, case):  # noqa: F811
    import torch
    import paper_1910_00178_amd as ng
    M, N, K, zb, op, want = case
    gen = torch.Generator(device="cuda").manual_seed(K)
    ta, tb = (torch.int16, torch.int16) if op == "s16" else (torch.uint8, torch.int8)
    ia, ib, ld = torch.iinfo(ta), torch.iinfo(tb), (K + 15) // 16 * 16
    A = torch.randint(ia.min, ia.max + 1, (M, ld), generator=gen, device="cuda", dtype=ta)
    B = torch.randint(ib.min, ib.max + 1, (N, K), generator=gen, device="cuda", dtype=tb)
    nb = (ng.ngemm_packed_b_bytes_s16 if op == "s16" else ng.ngemm_packed_b_bytes)(K, N)
    packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
    h = (ng.ngemm_pack_b_s16 if op == "s16" else ng.ngemm_pack_b)(runner.ctx, K, N, B, K, packed, nb)
    wsb = ng.ngemm_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    C = torch.full((M + 1, N + 3), 77, dtype=torch.uint8 if op == "u8" else torch.int32, device="cuda")
    scale = 2.0 ** -12

    def call(stream):
        if op == "u8":
            ng.ngemm_run_u8s8u8_requant(runner.ctx, M, A, ld, 37, h, zb, scale, 128, C, N + 3, ws, wsb, stream)
        else:
            (ng.ngemm_run_s16s16s32 if op == "s16" else ng.ngemm_run_u8s8s32)(runner.ctx, M, A, ld, 37, h, zb, C, N + 3, ws, wsb, stream)
    got = launches(call)
    assert len(got) == 1 and got[0][0].startswith(want), got
    call(0)
    sums = ((A[:, :K].double() - 37) @ (B.double() - zb).t()).long()
    sums = (sums + 2**31) % 2**32 - 2**31
    exact = (torch.round(sums.float() * scale).double() + 128).clamp(0, 255).to(torch.uint8) if op == "u8" else sums.int()
    torch.cuda.synchronize()
    assert torch.equal(C[:M, :N], exact) and bool((C[M:] == 77).all()) and bool((C[:, N:] == 77).all())
    ng.ngemm_packed_b_free(h)


RAW11, RAW12 = "gemm_wavek_kernel<1, 1, 1, 4, 4, false, %s, true, true,", "gemm_wavek_kernel<1, 1, 2, 2, 4, false, %s, true, true,"
# (M, N, K, kernel or None: B is packed first), both sides of the lines of the rule
RAW_ANY = [(1, 1, 1, RAW11), (33, 65, 15, RAW11), (512, 512, 77, RAW11), (512, 1024, 1024, RAW11), (512, 1024, 1025, RAW12), (512, 1025, 1024, RAW12),
           (30, 17000, 190, RAW12), (1024, 1024, 1030, RAW12), (1024, 1024, 3072, RAW12), (1024, 1024, 3073, None), (1024, 1056, 255, RAW12),
           (1024, 1056, 257, None), (2048, 1024, 250, RAW12), (2048, 1030, 250, None), (8, 512, 6144, RAW11), (8, 512, 6145, None), (9, 512, 6145, RAW11),
           (8, 513, 6145, RAW11), (40, 70, 8192, RAW11), (40, 70, 8193, None)]


@pytest.mark.parametrize("M,N,K,kernel", RAW_ANY)
def test_unpacked_rows_of_any_alignment(runner, launches, M, N, K, kernel):  # noqa: F811
    import torch
    import paper_1910_00178_amd as ng
    wsb = ng.ngemm_unpacked_workspace_bytes(M, N, K)
    ws = torch.full((wsb,), 0xC3, dtype=torch.uint8, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    for pa, pb, za, zb in ((K + K % 2 + 1, K + 5, 128, 0), (K + K % 2 + 1, (K + 15) // 16 * 16, 37, -7)):      # the second: only A's rows are unaligned
        A = torch.randint(0, 256, (M, pa), generator=gen, device="cuda", dtype=torch.uint8).reshape(-1)[:(M - 1) * pa + K].clone()
        B = torch.randint(-128, 128, (N, pb), generator=gen, device="cuda", dtype=torch.int8).reshape(-1)[:(N - 1) * pb + K].clone()
        C = torch.full((M + 1, N + 1), -7, dtype=torch.int32, device="cuda")
        call = lambda stream: ng.ngemm_run_u8s8s32_unpacked(runner.ctx, M, N, K, A, pa, za, B, pb, zb, C, N + 1, ws, wsb, stream)
        names = [name for name, _ in launches(lambda stream: call(stream.cuda_stream))]
        if kernel:
            assert len(names) == 1 and kernel % ("true" if zb else "false") in names[0], names
        else:
            assert len(names) > 1, names
        call(None)
        _check(A.as_strided((M, K), (pa, 1)), B.as_strided((N, K), (pb, 1)), za, zb, C)


@pytest.mark.parametrize("M,N", [(1, 70), (35, 33), (100, 66)])
def test_unpacked_every_number_of_steps(runner, M, N):
    """K from one byte to past every number of steps that the kernel treats by itself, either operand ending with its last row."""
    import torch
    import paper_1910_00178_amd as ng
    wsb = ng.ngemm_unpacked_workspace_bytes(M, N, 4000)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(M)
    for K in list(range(1, 40)) + [64 * s + d for s in range(1, 46) for d in (-1, 0, 1, 17)]:
        A = torch.randint(0, 256, (M * K,), generator=gen, device="cuda", dtype=torch.uint8)
        B = torch.randint(-128, 128, (N * K + 1,), generator=gen, device="cuda", dtype=torch.int8)[1:]          # (unaligned for every K)
        C = torch.full((M + 1, N + 1), -7, dtype=torch.int32, device="cuda")
        ng.ngemm_run_u8s8s32_unpacked(runner.ctx, M, N, K, A, K, 3, B, K, (0, 5)[K & 1], C, N + 1, ws, wsb)
        _check(A.view(M, K), B.view(N, K), 3, (0, 5)[K & 1], C)


def _check(A, B, za, zb, C):
    import torch
    M, N = A.shape[0], B.shape[0]
    want = ((A.double() - za) @ (B.double() - zb).t()).long()
    want = ((want + 2**31) % 2**32 - 2**31).int()
    assert torch.equal(C[:M, :N], want) and bool((C[M:] == -7).all()) and bool((C[:, N:] == -7).all()), (A.shape, B.shape)
