"""gemm_mid_kernel against the oracle, in all its forms: edges of its tiles (64 and 128 rows, 128 to 256 columns), K of one stage (64 bytes),
of fewer stages than its ring, of partial stages and of a last chunk that ends inside 16 bytes, rows of A with any alignment (the
allocation ends with the last row), each output and operand type."""
import numpy as np
import pytest

import oracle
from test_gpu_routes import Problem, ctx, launches  # noqa: F401

pytestmark = pytest.mark.gpu

W64x128, W64x192, W128, W192, W256 = "2, 4, 2, 2, 6", "2, 6, 2, 2, 4", "4, 4, 2, 2, 4", "4, 6, 2, 2, 4", "4, 4, 2, 4, 6"
# (M, N, K, pitch of A: 0 = K, which form)
SHAPES = [(802, 4624, 64, 64, W64x128), (387, 2314, 1537, 1552, W64x128), (802, 4624, 79, 0, W64x128), (1100, 1300, 1663, 0, W64x128),
          (4727, 774, 65, 80, W64x192), (386, 4727, 781, 784, W64x192), (385, 4755, 773, 0, W64x192), (1701, 1537, 1600, 1603, W64x192),
          (4712, 1185, 64, 64, W128), (3279, 775, 774, 784, W128), (2918, 1314, 643, 0, W128),
          (4524, 1935, 65, 80, W192), (2725, 3339, 193, 208, W192), (3490, 2519, 77, 0, W192), (2368, 4629, 343, 0, W192),
          (1824, 3322, 774, 784, W256), (3268, 1799, 131, 0, W256), (1930, 3100, 1000, 1001, W256),
          # stages enough for two passes of the steady loop and more, every number of stages modulo its unrolling for the 128 x 192 tiles
          (2388, 2307, 901, 912, W192), (2242, 2144, 1000, 1008, W192), (2116, 1936, 1025, 1040, W192), (835, 4621, 1100, 1104, W192),
          (4880, 1737, 901, 0, W192), (4891, 1752, 965, 0, W192), (4875, 1744, 1027, 0, W192), (2882, 1028, 901, 0, W128),
          (4694, 1168, 1157, 1168, W256), (3279, 1160, 1157, 0, W256)]


@pytest.fixture(scope="module")
def runner():
    from gpu_util import Runner
    r = Runner()
    yield r
    r.close()


def steady_passes(form, K, aligned):
    """Passes of the kernel's steady loop: NS stages in the ring, AD register sets for unaligned rows, U stages a pass."""
    ns, nst, t, n = int(form.split(", ")[-1]), -(-K // 64), 0, 0
    ad = 4 if ns % 4 == 0 else 3
    u, ahead = ns if aligned or ns % ad == 0 else ns * ad, ns if aligned else max(ns, ad + 2)
    u = u if u % 2 == 0 else 2 * u
    while t + u - 1 + ahead < nst - 1:
        t, n = t + u, n + 1
    return n


@pytest.mark.parametrize("form", [W64x128, W64x192, W128, W192, W256])
@pytest.mark.parametrize("aligned", [True, False])
def test_the_shapes_run_the_steady_loops(form, aligned):
    mine = [(steady_passes(form, K, aligned), -(-K // 64)) for M, N, K, pitch, f in SHAPES if f == form and ((pitch or K) % 16 == 0) == aligned]
    assert max(n for n, _ in mine) >= 2, mine
    if form == W192:
        assert len({nst % 4 for n, nst in mine if n >= 2}) >= (4 if aligned else 3), mine


@pytest.mark.parametrize("case", SHAPES, ids=str)
def test_forms_against_the_oracle(runner, ctx, launches, case):  # noqa: F811
    M, N, K, pitch, form = case
    import paper_1910_00178_amd as ng
    p = Problem(ctx, M, N, K, pitch or K)
    for u8, zb in ((False, 0), (False, -5), (True, 0), (True, -5)):
        got = launches(p.run_u8(zb) if u8 else p.run(zb))
        want = ["gemm_mid_kernel<MidCfg<%s>, %s>" % (form, ", ".join(str(x).lower() for x in (u8, zb != 0, (pitch or K) % 16 != 0)))]
        assert [name for name, _ in got] == want, got
    ng.ngemm_packed_b_free(p.h)
    rng = np.random.default_rng(M * 7 + K)
    A, B = rng.integers(0, 256, size=(M, K), dtype=np.uint8), rng.integers(-128, 128, size=(N, K), dtype=np.int8)
    A[::5], B[1::7] = 255, -128
    h, _ = runner.pack(B)
    pad = (pitch or K) - K
    for za, zb, ldc_pad in ((7, 0, 0), (200, -5, 3)):
        C = oracle.gemm_u8s8s32(A, B, za, zb)
        assert np.array_equal(runner.run(A, h, N, za=za, zb=zb, lda_pad=pad, ldc_pad=ldc_pad), C)
        scale = np.float32(60.0 / np.sqrt(K) / 5000)
        assert np.array_equal(runner.run(A, h, N, za=za, zb=zb, scale=float(scale), zc=128, lda_pad=pad, ldc_pad=ldc_pad),
                              oracle.requant_s32u8(C, float(scale), 128))
    ng.ngemm_packed_b_free(h)


def test_u8_rows_that_end_inside_16_bytes(runner, ctx, launches):  # noqa: F811
    """u8 rows of every length modulo 16, to the byte: what follows a row keeps its contents."""
    import paper_1910_00178_amd as ng
    M, K, top = 1500, 67, 2336
    rng = np.random.default_rng(16)
    A, B = rng.integers(0, 256, size=(M, K), dtype=np.uint8), rng.integers(-128, 128, size=(top, K), dtype=np.int8)
    want = oracle.requant_s32u8(oracle.gemm_u8s8s32(A, B, 9, 5), 0.0015, 128)
    for N in range(top - 16, top + 1):
        p = Problem(ctx, M, N, K)
        got = launches(p.run_u8(5))
        assert len(got) == 1 and got[0][0].startswith("gemm_mid_kernel<"), got
        ng.ngemm_packed_b_free(p.h)
        h, _ = runner.pack(B[:N])
        assert np.array_equal(runner.run(A, h, N, za=9, zb=5, scale=0.0015, zc=128, lda_pad=13, ldc_pad=1), want[:, :N]), N
        ng.ngemm_packed_b_free(h)


# (M, N, K, pitch of A: 0 = whole 16 bytes, u8 output, zero-point of B, kernel): each line of the rule that gives a call to gemm_mid_kernel, on both sides
BORDERS = [
    (28544, 64, 960, 0, False, 0, "gemm_tile_dma_kernel<64, 64,"), (28544, 65, 960, 0, False, 0, "gemm_mid"),
    (2112, 1300, 768, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"), (2112, 1300, 768, 0, False, 0, "gemm_mid"),
    (2112, 1300, 1000, 0, False, 3, "gemm_mid"), (1024, 2560, 832, 0, True, 3, "gemm_mid"), (1024, 2561, 832, 0, True, 3, "gemm_tile_dma_kernel<64, 64,"),
    (1024, 3072, 768, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"), (1757, 1881, 512, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"),
    (1757, 1881, 641, 0, False, 3, "gemm_mid"), (1757, 1881, 512, 0, False, 0, "gemm_mid"),
    (1100, 1300, 1536, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"), (1100, 1300, 1537, 0, False, 3, "gemm_mid"),
    (47, 32253, 960, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"), (64, 17000, 1100, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"),
    (64, 17000, 1600, 0, False, 3, "gemm_mid"), (65, 8500, 1600, 0, False, 3, "gemm_mid"), (47, 45376, 891, 891, False, 3, "gemm_tile_kernel<64, 64,"),
    (47, 17000, 1771, 1771, False, 3, "gemm_mid"), (38465, 19, 128, 0, True, 0, "gemm_tile_dma_kernel<128, 128,"),
    (38465, 49, 128, 0, True, 0, "gemm_mid"), (38465, 49, 128, 0, True, 3, "gemm_tile_dma_kernel<128, 128,"), (38465, 19, 128, 0, False, 0, "gemm_mid"),
    (48289, 128, 397, 397, False, 3, "gemm_tile_kernel<128, 128,"), (48289, 129, 397, 397, False, 3, "gemm_mid"),
    (3826, 5056, 192, 0, False, 3, "gemm_tile_dma_kernel<128, 128,"), (3826, 5057, 192, 0, False, 3, "gemm_mid"),
    (33280, 128, 3392, 0, False, 0, "gemm_tile_x64_kernel<"), (33280, 128, 3392, 0, False, 3, "gemm_mid"),
    (64, 29000, 800, 0, False, 0, "gemm_mid"), (64, 29000, 768, 0, False, 0, "gemm_tile_dma_kernel<64, 64,"), (64, 29000, 2368, 0, False, 3, "gemm_mid"),
    (64, 29000, 2304, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"), (256, 9000, 832, 0, False, 3, "gemm_mid"),
    (320, 9000, 832, 0, False, 3, "gemm_tile_dma_kernel<64, 64,"), (320, 27686, 1792, 0, False, 3, "gemm_tile_x64_kernel<"),
    (320, 27686, 1792, 0, True, 3, "gemm_mid"), (704, 13149, 1179, 0, False, 0, "gemm_tile_x64_kernel<"),
]


@pytest.mark.parametrize("case", BORDERS, ids=str)
def test_which_calls_the_kernel_serves(ctx, launches, case):  # noqa: F811
    import paper_1910_00178_amd as ng
    M, N, K, pitch, u8, zb, want = case
    p = Problem(ctx, M, N, K, pitch or None)
    got = launches(p.run_u8(zb) if u8 else p.run(zb))
    assert got[-1][0].startswith(want), got
    ng.ngemm_packed_b_free(p.h)


def test_where_the_kernels_before_stay(ctx, launches):  # noqa: F811
    """A cap below the unit count, rows or panels too far apart for 32-bit offsets, and a shape that the time model leaves to the large tiles."""
    import paper_1910_00178_amd as ng
    p = Problem(ctx, 1024, 3072, 1000)
    assert launches(p.run())[0][0].startswith("gemm_mid_kernel<")
    ng.ngemm_set_max_workgroups(ctx, 100)
    try:
        got = launches(p.run())
    finally:
        ng.ngemm_set_max_workgroups(ctx, 0)
    assert got[0][0].startswith("gemm_tile_dma_kernel<64, 64,") and got[0][1] <= 400, got
    far = (1 << 32) // 255 // 16 * 16                       # captured only: no row but the first is there
    for lda, name in ((far - 4096, "gemm_mid_kernel<"), (far, "gemm_tile_dma_kernel<64, 64,")):
        got = launches(lambda st: ng.ngemm_run_u8s8s32(ctx, p.M, p.A, lda, 7, p.h, 0, p.C, p.N, p.ws, p.wsb, st))
        assert got[0][0].startswith(name), (lda, got)
    ng.ngemm_packed_b_free(p.h)
    for shape, name in (((4736, 3072, 768), "gemm_tile_x64_kernel<"), ((2048, 4096, 1024), "gemm_mid_kernel<")):
        p = Problem(ctx, *shape)
        assert launches(p.run())[-1][0].startswith(name), shape
        ng.ngemm_packed_b_free(p.h)


def test_a_tuned_shape_takes_what_the_tuner_found(launches):  # noqa: F811
    """3000 x 3001 x 448 with a zero-point: a fifth faster than any kernel that can be forced.  Later calls of the shape take it, other outputs
    and zero-points too; what the rule says against 64 x 64 tiles (K of 257 .. 640, columns that share lines of C) does not count then."""
    import paper_1910_00178_amd as ng
    own = ng.ngemm_create(0)
    p = Problem(own, 3000, 3001, 448)
    best = ng.ngemm_tune_u8s8s32(own, p.M, p.A, p.lda, 7, p.h, 3, p.C, p.N, p.ws, p.wsb)
    assert best != ng.NGEMM_KERNEL_AUTO and ng.ngemm_tuned_kernel(own, p.M, p.N, p.K) == best
    tuned = [launches(call)[-1][0] for call in (p.run(3), p.run(0), p.run_u8(3))]
    assert all(t.startswith("gemm_mid_kernel<") for t in tuned), tuned
    ng.ngemm_set_kernel(own, best)
    assert not launches(p.run(3))[-1][0].startswith("gemm_mid_kernel<")
    ng.ngemm_packed_b_free(p.h)
    ng.ngemm_destroy(own)


def test_more_tiles_than_a_launch_takes(ctx, launches):  # noqa: F811
    """A launch takes less than 2^32 threads: a form with 2^24 tiles (128 x 128, here of 184 GB of u8 beside 46 GB of A) is not launched.
    Captured only: the addresses are those of small buffers that nothing reads."""
    import paper_1910_00178_amd as ng
    M, N, K = 715827883, 257, 64
    p = Problem(ctx, 64, N, K)
    got = launches(lambda st: ng.ngemm_run_u8s8u8_requant(ctx, M, p.A, K, 7, p.h, 0, 0.01, 3, p.C, N, p.ws, 0, st))
    assert len(got) == 1 and got[0][1] * (512 if W256 in got[0][0] else 256) < 1 << 32, got
    ng.ngemm_packed_b_free(p.h)


@pytest.mark.parametrize("K,pitch", [(770, 784), (773, 773)])
def test_other_operands_and_per_column_terms(runner, launches, K, pitch):  # noqa: F811
    """Signed A and unsigned B with zero-points, a zero-point, bias and scale per column, a zero-point of C beyond binary32."""
    import torch
    import paper_1910_00178_amd as ng
    M, N = 1500, 1605
    rng = np.random.default_rng(K)
    ctx = runner.ctx                                         # noqa: F811
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()

    def rows(x):
        full = np.full((x.shape[0], pitch), 99, x.dtype)
        full[:, :K] = x
        return dev(full.reshape(-1)[:(x.shape[0] - 1) * pitch + K])
    Au, As = rng.integers(0, 256, size=(M, K), dtype=np.uint8), rng.integers(-128, 128, size=(M, K), dtype=np.int8)
    Bs, Bu = rng.integers(-128, 128, size=(N, K), dtype=np.int8), rng.integers(0, 256, size=(N, K), dtype=np.uint8)
    nb = ng.ngemm_packed_b_bytes(K, N)
    ps, pu = (torch.empty(nb, dtype=torch.uint8, device="cuda") for _ in range(2))
    hs, hu = ng.ngemm_pack_b(ctx, K, N, dev(Bs), K, ps, nb), ng.ngemm_pack_b_u8(ctx, K, N, dev(Bu), K, pu, nb)
    wsb = ng.ngemm_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    As_d, Au_d = rows(As), rows(Au)

    def run(call):
        got = launches(lambda st: call(st))
        assert len(got) == 1 and got[0][0].startswith("gemm_mid_kernel<"), got
        call(None)
    run(lambda st: ng.ngemm_run_s8s8s32(ctx, M, As_d, pitch, -5, hs, 9, C, N, ws, wsb, st))
    assert np.array_equal(C.cpu().numpy(), oracle.gemm_s8s8s32(As, Bs, -5, 9))
    run(lambda st: ng.ngemm_run_u8u8s32(ctx, M, Au_d, pitch, 131, hu, 120, C, N, ws, wsb, st))
    assert np.array_equal(C.cpu().numpy(), oracle.gemm_u8u8s32(Au, Bu, 131, 120))
    zbv, bias = rng.integers(-8, 9, N).astype(np.int32), rng.integers(-3000, 3000, N).astype(np.int32)
    scale = (rng.random(N) * 1e-3 + 1e-4).astype(np.float32)
    zb_d, scale_d, bias_d = dev(zbv), dev(scale), dev(bias)
    D = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    for zc, relu in ((128, False), (-(1 << 30), False), (3, True)):
        run(lambda st: ng.ngemm_run_u8s8u8_requant_channel(ctx, M, Au_d, pitch, 128, hs, 0, zb_d, scale_d, bias_d, int(relu), zc, D, N, ws, wsb, st))
        assert np.array_equal(D.cpu().numpy(), oracle.gemm_u8s8u8_requant_channel(Au, Bs, 128, 0, scale, zc, zb_vec=zbv, bias=bias, relu=relu))
    ng.ngemm_packed_b_free(hs)
    ng.ngemm_packed_b_free(hu)


@pytest.mark.parametrize("wide", [False, True])
def test_grouped_tiles(runner, launches, wide):  # noqa: F811
    """Tiled members of a batch: K of none, one, two ... stages of 64 bytes to well past the ring and its unrolled loop, with and without a
    last chunk that ends inside 16 bytes, edges of the 64 x 64 tiles, rows of any alignment, a skinny member in front; one member
    whose rows are too far apart for 32-bit offsets takes the whole group to the kernel with 64-bit addresses."""
    import torch
    import paper_1910_00178_amd as ng
    rng = np.random.default_rng(31)
    ks = [0, 1, 15, 16, 17, 63, 64, 65, 80, 127, 128, 129, 191, 257, 320, 383, 449, 513, 640, 705, 769, 1000, 1100, 1663]
    shapes = [((33, 64, 65, 129)[i % 4], (1, 31, 64, 65, 130)[i % 5], k, k + (0, 3, 16)[i % 3]) for i, k in enumerate(ks)]
    shapes += [(7, 100, 700, 701)] + ([(35, 40, 16, 1 << 27)] if wide else [])
    items, want, outs, keep, handles = [], [], [], [], []
    for t, (M, N, K, pitch) in enumerate(shapes):
        A, B = rng.integers(0, 256, size=(M, K), dtype=np.uint8), rng.integers(-128, 128, size=(N, K), dtype=np.int8)
        za, zb = int(rng.integers(0, 256)), 0 if t % 3 == 0 else int(rng.integers(-128, 128))
        h, packed = runner.pack(B)
        flat = torch.empty(max(16, (M - 1) * pitch + K), dtype=torch.uint8, device="cuda")          # ends with the last row
        if K:
            flat.as_strided((M, K), (pitch, 1)).copy_(torch.from_numpy(A))
        C = torch.full((M + 1, N + 1), -9, dtype=torch.int32, device="cuda")
        items.append((M, flat, max(pitch, 1), za, zb, h, C, N + 1))
        want.append(oracle.gemm_u8s8s32(A, B, za, zb))
        outs.append(C)
        keep += [flat, packed]
        handles.append(h)
    problems = ng.make_problems(items)
    got = launches(lambda stream: ng.ngemm_run_batched_u8s8s32(runner.ctx, problems, None, 0, stream.cuda_stream))
    assert [name.split("<")[0] for name, _ in got] == ["gemm_group_kernel" if wide else "gemm_group_mid_kernel"], got
    ng.ngemm_run_batched_u8s8s32(runner.ctx, problems)
    torch.cuda.synchronize()
    for shape, C, w in zip(shapes, outs, want):
        c = C.cpu().numpy()
        assert np.array_equal(c[:-1, :-1], w), shape
        assert (c[-1] == -9).all() and (c[:, -1] == -9).all(), shape
    for h in handles:
        ng.ngemm_packed_b_free(h)


@pytest.mark.parametrize("shapes,want", [
    ([(100, 200, 640)], "gemm_group_kernel"), ([(100, 200, 192)], "gemm_group_mid_kernel"), ([(100, 200, 1537)], "gemm_group_mid_kernel"),
    ([(64, 64, 700)] * 30 + [(16, 500, 3000)], "gemm_group_kernel"), ([(64, 64, 700)] * 30 + [(64, 64, 1600)], "gemm_group_mid_kernel"),
    ([(1024, 1024, 1024)], "gemm_group_kernel"), ([(1024, 1024, 1025)], "gemm_group_mid_kernel"), ([(1024, 1025, 1024)], "gemm_group_mid_kernel")], ids=str)
def test_grouped_tiles_of_few_short_chains(runner, launches, shapes, want):  # noqa: F811
    import torch
    import paper_1910_00178_amd as ng
    items, keep, handles = [], [], []
    for M, N, K in shapes:
        A, C = torch.zeros((M, K), dtype=torch.uint8, device="cuda"), torch.empty((M, N), dtype=torch.int32, device="cuda")
        h, packed = runner.pack(np.zeros((N, K), np.int8))
        items.append((M, A, K, 7, 3, h, C, N))
        keep += [A, C, packed]
        handles.append(h)
    problems = ng.make_problems(items)
    got = launches(lambda stream: ng.ngemm_run_batched_u8s8s32(runner.ctx, problems, None, 0, stream.cuda_stream))
    assert [name.split("<")[0] for name, _ in got] == [want], got
    for h in handles:
        ng.ngemm_packed_b_free(h)


@pytest.mark.parametrize("shapes,small", [
    ([((33, 5, 64, 1, 65)[i % 5], (1, 31, 33, 64, 130)[i % 4 + i // 16], k) for i, k in enumerate([0, 1, 15, 16, 63, 64, 65, 127, 129, 192, 255, 256, 257, 320, 449, 513, 700, 1000, 1025, 1279, 1535, 1536])], True),
    ([(40, 70, 4113), (3, 200, 3001), (97, 33, 2048), (65, 65, 0), (32, 32, 130), (33, 1, 2111)], True),
    ([(40, 70, 4113), (35, 40, 16)], "far apart"),                                            # the second one's rows
    ([(64, 8192, 300)], True), ([(64, 8193, 300)], False), ([(33, 100, 257)], True), ([(33, 100, 256)], False), ([(33, 100, 1537)], False),
    ([(33, 100, 2047)], False), ([(32, 100, 700)] * 3, False),
    # two rounds: the tiles with more than a third of the longest K have to fit the first
    ([(512, 1024, 2048)], True), ([(512, 1025, 2048)], False), ([(512, 2048, 2048)], False), ([(512, 1024, 2048), (512, 1024, 682)], True),
    ([(512, 1024, 2048), (512, 1024, 683)], False), ([(512, 1024, 2048), (512, 1025, 682)], False),
    ([(33, 40, 300 + i) for i in range(80)], True),
    # members of up to eight rows and up to K = 1024 do not count as long
    ([(33, 100, 256), (8, 40, 1024)], False), ([(33, 100, 256), (9, 40, 300)], True), ([(33, 100, 64), (8, 40, 1025)], True),
    ([(33, 100, 64), (1, 300, 2048)], True)], ids=lambda s: str(s) if isinstance(s, (bool, str)) else "%dx%s" % (len(s), s[0]))
def test_grouped_small_tiles(runner, launches, shapes, small):  # noqa: F811
    """Batches of few tiles: 32 x 32 tiles with K shared by four wavefronts.  K of every remainder of a step, of fewer steps than wavefronts, none at all;
    rows of any alignment, members with M <= 32 among the others, more members than one launch holds, both sides of the lines of the rule."""
    import torch
    import paper_1910_00178_amd as ng
    rng = np.random.default_rng(len(shapes))
    items, want, outs, keep, handles = [], [], [], [], []
    for t, (M, N, K) in enumerate(shapes):
        pitch = (1 << 27) if small == "far apart" and t else max(1, K + (0, 3, 16)[t % 3])
        A, B = rng.integers(0, 256, size=(M, K), dtype=np.uint8), rng.integers(-128, 128, size=(N, K), dtype=np.int8)
        za, zb = int(rng.integers(0, 256)), 0 if t % 3 == 0 else int(rng.integers(-128, 128))
        h, packed = runner.pack(B)
        flat = torch.empty(max(16, (M - 1) * pitch + K), dtype=torch.uint8, device="cuda")          # ends with the last row
        if K:
            flat.as_strided((M, K), (pitch, 1)).copy_(torch.from_numpy(A))
        C = torch.full((M + 1, N + 1), -9, dtype=torch.int32, device="cuda")
        items.append((M, flat, pitch, za, zb, h, C, N + 1))
        want.append(oracle.gemm_u8s8s32(A, B, za, zb))
        outs.append(C)
        keep += [flat, packed]
        handles.append(h)
    problems = ng.make_problems(items)
    got = launches(lambda stream: ng.ngemm_run_batched_u8s8s32(runner.ctx, problems, None, 0, stream.cuda_stream))
    assert all(("gemm_group_kernel<32" in name) == (small is True) for name, _ in got), got
    ng.ngemm_run_batched_u8s8s32(runner.ctx, problems)
    torch.cuda.synchronize()
    for shape, C, w in zip(shapes, outs, want):
        c = C.cpu().numpy()
        assert np.array_equal(c[:-1, :-1], w), shape
        assert (c[-1] == -9).all() and (c[:, -1] == -9).all(), shape
    for h in handles:
        ng.ngemm_packed_b_free(h)


@pytest.mark.parametrize("M,N,K,in_kernel", [(1541, 1500, 128, True), (1665, 1409, 133, True), (1537, 1537, 191, True), (2047, 2050, 192, True),
                                             (1600, 1600, 333, True), (1541, 1500, 2560, True), (1541, 1500, 2561, False), (4097, 2049, 1344, False)])
def test_s16_row_sums(ctx, launches, M, N, K, in_kernel):  # noqa: F811
    """The 128 x 128 kernel of 16-bit operands forms the row sums itself while a unit works through 40 stages of 64 elements at most: K of an even and an
    odd number of stages, with a partial one, several tiles per workgroup, extreme values; a launch of their own beyond."""
    import torch
    import paper_1910_00178_amd as ng
    rng = np.random.default_rng(M + K)
    A, B = (rng.integers(-32768, 32768, size=(n, K)).astype(np.int16) for n in (M, N))
    A[::3], A[1::9] = -32768, 32767
    lda = (K + 7) // 8 * 8
    Ah = np.full((M, lda), 7777, np.int16)
    Ah[:, :K] = A
    Ad, Bd = torch.from_numpy(Ah.reshape(-1)[:(M - 1) * lda + K].copy()).cuda(), torch.from_numpy(B).cuda()
    nb, wsb = ng.ngemm_packed_b_bytes_s16(K, N), ng.ngemm_workspace_bytes(M, N, K)
    packed, ws = torch.empty(nb, dtype=torch.uint8, device="cuda"), torch.empty(wsb, dtype=torch.uint8, device="cuda")
    h = ng.ngemm_pack_b_s16(ctx, K, N, Bd, K, packed, nb)
    C = torch.full((M + 1, N + 3), -7, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    got = launches(lambda st: ng.ngemm_run_s16s16s32(ctx, M, Ad, lda, -321, h, 20000, C, N + 3, ws, wsb, st))
    assert [name for name, _ in got] == (["gemm_s16_tile_kernel<true>"] if in_kernel else ["rowsum_s16_kernel", "gemm_s16_tile_kernel<false>"]), got
    ng.ngemm_run_s16s16s32(ctx, M, Ad, lda, -321, h, 20000, C, N + 3, ws, wsb)
    got = C.cpu().numpy()
    ng.ngemm_packed_b_free(h)
    # products below 2^33, sums below 2^45: exact in binary64, then the low 32 bits
    want = ((A.astype(np.float64) + 321) @ (B.astype(np.float64) - 20000).T).astype(np.int64).astype(np.int32)
    assert np.array_equal(got[:M, :N], want)
    assert (got[M:] == -7).all() and (got[:, N:] == -7).all()
