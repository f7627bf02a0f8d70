"""Which kernel a call launches: the calls are captured into a graph that is never run, and the names and grids of the
graph's kernel nodes are looked at.  A kernel that a caller forced is the one that runs, so the tests that force a
kernel run the kernel they name."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")                 # before the library: both then use torch's HIP runtime


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNode(ctypes.Structure):                     # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


@pytest.fixture(scope="module")
def launches():
    """launches(call) -> [(kernel name, workgroups)] of what call(stream) launches; nothing is executed."""
    import paper_1910_00178_amd as ng
    hip = ctypes.CDLL(ng.LIB_PATH)                       # the HIP runtime that the library itself is bound to
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    demangle = ctypes.CDLL("libstdc++.so.6").__cxa_demangle
    demangle.restype = ctypes.c_char_p
    stream = torch.cuda.Stream()

    def ok(code):
        assert code == 0, code

    def run(call):
        st, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(0)
        ok(hip.hipStreamBeginCapture(st, 2))             # relaxed
        try:
            call(stream)
        finally:
            ended = hip.hipStreamEndCapture(st, ctypes.byref(graph))
        ok(ended)
        ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)))
        nodes = (ctypes.c_void_p * n.value)()
        ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)))
        out = []
        for node in nodes:
            p = _KernelNode()
            ok(hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)))
            name = hip.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), st)
            full = demangle(name, None, None, None) or name
            out.append((full.decode().replace("void ", "").split("(")[0].replace("ngemm::", ""), p.grid.x))
        ok(hip.hipGraphDestroy(graph))
        return out

    return run


def is_kernel(name, want):
    """The same kernel; template arguments behind those of `want` may be anything."""
    return name == want or name.startswith(want[:-1] + ",")


class Problem:
    """Operands of one 8-bit product (contents do not matter: nothing is run)."""

    def __init__(self, ctx, M, N, K, pitch=None):
        import paper_1910_00178_amd as ng
        self.ng, self.ctx, self.M, self.N, self.K = ng, ctx, M, N, K
        self.lda = pitch or (K + 15) // 16 * 16
        self.A = torch.zeros((M, self.lda), dtype=torch.uint8, device="cuda")
        self.B = torch.zeros((N, self.lda), dtype=torch.int8, device="cuda")
        nb = ng.ngemm_packed_b_bytes(K, N)
        self.packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
        self.h = ng.ngemm_pack_b(ctx, K, N, self.B, self.lda, self.packed, nb)
        self.C = torch.empty((M, N), dtype=torch.int32, device="cuda")
        self.wsb = ng.ngemm_workspace_bytes(M, N, K)
        self.ws = torch.empty(self.wsb, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()

    def run(self, zb=0):
        return lambda st: self.ng.ngemm_run_u8s8s32(self.ctx, self.M, self.A, self.lda, 7, self.h, zb, self.C, self.N, self.ws, self.wsb, st)

    def run_u8(self, zb=0):
        return lambda st: self.ng.ngemm_run_u8s8u8_requant(self.ctx, self.M, self.A, self.lda, 7, self.h, zb, 0.01, 3, self.C, 4 * self.N,
                                                           self.ws, self.wsb, st)


@pytest.fixture(scope="module")
def ctx():
    import paper_1910_00178_amd as ng
    c = ng.ngemm_create(0)
    yield c
    ng.ngemm_destroy(c)


# (kernel, M, N, K, pitch, zero-point of B, what runs): shapes that the automatic choice gives to the kernel that splits K
# over wavefronts
FORCED = [
    ("SKINNY", 16, 4096, 1024, None, 0, "gemm_skinny_kernel<false, 1>"),
    ("SKINNY", 17, 32840, 2112, None, 3, "gemm_skinny_kernel<false, 4>"),
    ("SKINNY", 9, 65600, 2048, None, 3, "gemm_stream_skinny_kernel<false>"),
    ("SKINNY", 20, 4096, 1025, 1025, 3, "gemm_skinny_kernel<false, 1>"),
    ("TILE_64", 64, 4096, 4096, None, 0, "gemm_tile_deep_kernel<1, 4, 4, false, 0, false>"),
    ("TILE_64", 64, 4096, 4096, None, 3, "gemm_tile_deep_kernel<1, 4, 4, false, 0, true>"),
    ("TILE_64", 300, 200, 200, None, 3, "gemm_tile_dma_kernel<64, 64, 2, 2, 4, false, false, true>"),
    ("TILE_64", 64, 1000, 4097, 4097, 3, "gemm_tile_kernel<64, 64, 2, 2, 64, false, true>"),
    ("TILE_128", 512, 4096, 4096, None, 3, "gemm_tile_deep_kernel<2, 2, 4, false, 0, true>"),
    ("SPLIT_K", 40, 4000, 3000, None, 0, "gemm_tile_deep_kernel<1, 4, 4, false, 1, false>"),
    # what a forced K split cannot serve: the 64 x 64 tiles, the streaming kernel
    ("SPLIT_K", 64, 1000, 1024, None, 3, "gemm_tile_deep_kernel<1, 4, 4, false, 0, true>"),
    ("SPLIT_K", 16, 1000, 1024, None, 3, "gemm_skinny_kernel<false, 1>"),
]


@pytest.mark.parametrize("case", FORCED, ids=str)
def test_a_forced_kernel_is_the_one_that_runs(ctx, launches, case):
    import paper_1910_00178_amd as ng
    kernel, M, N, K, pitch, zb, want = case
    p = Problem(ctx, M, N, K, pitch)
    ng.ngemm_set_kernel(ctx, getattr(ng, "NGEMM_KERNEL_" + kernel))
    try:
        got = launches(p.run(zb))
    finally:
        ng.ngemm_set_kernel(ctx, ng.NGEMM_KERNEL_AUTO)
    assert is_kernel(got[-1][0], want), got
    automatic = launches(p.run(zb))
    assert [name.split("<")[0] for name, _ in automatic] == ["gemm_wavek_kernel"], automatic
    ng.ngemm_packed_b_free(p.h)


@pytest.mark.parametrize("M,kernel,want", [(16, "SKINNY", "gemm_skinny_kernel<"), (500, "TILE_64", "gemm_tile_dma_kernel<64, 64,"),
                                           (500, "TILE_128", "gemm_tile_dma_kernel<128, 128,")])
def test_a_forced_kernel_on_unpacked_operands(ctx, launches, M, kernel, want):
    import paper_1910_00178_amd as ng
    N, K = 700, 1024
    p = Problem(ctx, M, N, K)
    wsb = ng.ngemm_unpacked_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    call = lambda st: ng.ngemm_run_u8s8s32_unpacked(ctx, M, N, K, p.A, p.lda, 7, p.B, p.lda, 3, p.C, N, ws, wsb, st)
    ng.ngemm_set_kernel(ctx, getattr(ng, "NGEMM_KERNEL_" + kernel))
    try:
        got = launches(call)
    finally:
        ng.ngemm_set_kernel(ctx, ng.NGEMM_KERNEL_AUTO)
    assert got[-1][0].startswith(want), got
    assert [name.split("<")[0] for name, _ in launches(call)] == ["gemm_wavek_kernel"]
    ng.ngemm_packed_b_free(p.h)


def test_tuning_chooses_among_all_of_them(ctx, launches):
    """The tuner reports a kernel that can be forced, and where the kernel that splits K over wavefronts beat it by far
    (64 x 4096 x 4096: 7 us against 10 and more) later calls take that one."""
    import paper_1910_00178_amd as ng
    own = ng.ngemm_create(0)
    p = Problem(own, 64, 4096, 4096)
    best = ng.ngemm_tune_u8s8s32(own, p.M, p.A, p.lda, 7, p.h, 3, p.C, p.N, p.ws, p.wsb)
    assert best in (ng.NGEMM_KERNEL_TILE_64, ng.NGEMM_KERNEL_TILE_128, ng.NGEMM_KERNEL_SPLIT_K)
    assert ng.ngemm_tuned_kernel(own, p.M, p.N, p.K) == best
    assert launches(p.run(3))[0][0].startswith("gemm_wavek_kernel<"), best
    ng.ngemm_set_kernel(own, best)
    assert not any(name.startswith("gemm_wavek_kernel<") for name, _ in launches(p.run(3)))
    ng.ngemm_packed_b_free(p.h)
    ng.ngemm_destroy(own)


# M <= 32 (M, N, K, what runs): which calls stream a weight, measured with the weight in cache and in memory: from memory the
# plain copies of the kernel that splits K over wavefronts lose up to 20 % to the streaming kernel
SKINNY = [
    (1, 4096, 1024, "gemm_wavek_kernel<1, 1, 1, 4, 4, false, false, false, false, true>"),       # non-temporal copies (the last)
    (16, 1024, 512, "gemm_wavek_kernel<1, 1, 1, 2, 4, false, false, false, false, true>"),
    (16, 4096, 4096, "gemm_wavek_kernel<1, 1, 1, 4, 4, false, false, false, false, false>"),
    (8, 8192, 4096, "gemm_wavek_kernel<1, 1, 1, 4, 4, false, false, false, false, true>"),
    (16, 8192, 4096, "gemm_wavek_kernel<1, 1, 1, 4, 4, false, false, false, false, false>"),
    (8, 16384, 1024, "gemm_wavek_kernel<1, 1, 1, 2, 4, false, false, false, false, true>"),
    (8, 16384, 2048, "gemm_skinny_kernel<false, 1>"),
    (16, 16384, 2048, "gemm_wavek_kernel<1, 1, 2, 4, 3, false, false, false, false, true>"),
    (32, 16384, 2048, "gemm_wavek_kernel<1, 1, 2, 4, 3, false, false, false, false, false>"),
    (4, 32768, 256, "gemm_skinny_kernel<false, 1>"),
    (4, 32768, 2048, "gemm_wavek_kernel<1, 1, 1, 2, 4, false, false, false, false, true>"),
    (8, 32768, 2048, "gemm_wavek_kernel<1, 1, 1, 2, 4, false, false, false, false, false>"),
    (16, 24576, 4096, "gemm_skinny_kernel<false, 1>"),
    (16, 32768, 4096, "gemm_wavek_kernel<1, 1, 2, 4, 3, false, false, false, false, false>"),
]


@pytest.mark.parametrize("case", SKINNY, ids=str)
def test_weights_from_memory(ctx, launches, case):
    import paper_1910_00178_amd as ng
    M, N, K, want = case
    p = Problem(ctx, M, N, K)
    got = launches(p.run())
    assert len(got) == 1 and is_kernel(got[0][0], want), got
    ng.ngemm_packed_b_free(p.h)


# rows of A that are not 16-byte aligned, 9 .. 32 of them
UNALIGNED = [
    (16, 4096, 513, "gemm_skinny_kernel<false, 1>"),
    (16, 1024, 1025, "gemm_skinny_kernel<false, 1>"),
    (16, 4096, 2047, "gemm_wavek_kernel<1, 1, 1, 4, 4, false, false, false, true, false>"),
    (17, 4096, 513, "gemm_wavek_kernel<1, 1, 1, 4, 4, false, false, false, true, false>"),
    (16, 16384, 1025, "gemm_wavek_kernel<1, 1, 2, 2, 4, false, false, false, true, false>"),
    (9, 16384, 4097, "gemm_skinny_kernel<false, 1>"),
    (12, 16384, 4097, "gemm_wavek_kernel<1, 1, 2, 2, 4, false, false, false, true, false>"),
    (9, 32767, 2047, "gemm_wavek_kernel<1, 1, 2, 2, 4, false, false, false, true, false>"),
]


@pytest.mark.parametrize("case", UNALIGNED, ids=str)
def test_unaligned_rows(ctx, launches, case):
    import paper_1910_00178_amd as ng
    M, N, K, want = case
    p = Problem(ctx, M, N, K, pitch=K)
    got = launches(p.run())
    assert len(got) == 1 and is_kernel(got[0][0], want), got
    ng.ngemm_packed_b_free(p.h)


# K split over workgroups: from K = 8192 on for int32 outputs of few tiles (weights from memory: 64 x 1024 x 8192 12.9 us without)
SPLIT = [(64, 1024, 8192, False, True), (64, 1024, 8128, False, False), (64, 1024, 8192, True, False), (64, 1024, 9216, True, True),
         (32, 2048, 8192, False, True), (64, 2048, 8192, False, False), (64, 2048, 9216, False, True)]


@pytest.mark.parametrize("M,N,K,u8,split", SPLIT)
def test_k_split(ctx, launches, M, N, K, u8, split):
    import paper_1910_00178_amd as ng
    p = Problem(ctx, M, N, K)
    got = launches(p.run_u8() if u8 else p.run())
    want = ["gemm_tile_deep_kernel", "splitk_reduce_kernel"] if u8 else ["zero_c_kernel", "gemm_tile_deep_kernel"]
    assert [name.split("<")[0] for name, _ in got] == (want if split else ["gemm_wavek_kernel"]), got
    ng.ngemm_packed_b_free(p.h)


# 128 x 128 tiles where 64 x 64 ones need a third round of two per compute unit and K is long (1536 x 1408 x 3584: 16.6 / 19.4 us)
THIRD_ROUND = [(1536, 1408, 2560, "gemm_tile_deep_kernel<2, 2, 4, false, 0, false>"), (1536, 1408, 2048, "gemm_tile_dma_kernel<64, 64, 2, 2, 4, false, false, false>"),
               (1472, 1408, 3584, "gemm_wavek_kernel<1, 2, 4, 4, 3, false, false, false, false, false>")]


@pytest.mark.parametrize("case", THIRD_ROUND, ids=str)
def test_third_round_of_small_tiles(ctx, launches, case):
    import paper_1910_00178_amd as ng
    M, N, K, want = case
    p = Problem(ctx, M, N, K)
    got = launches(p.run())
    assert len(got) == 1 and is_kernel(got[0][0], want), got
    ng.ngemm_packed_b_free(p.h)


def s16_call(ctx, M, N, K):
    import paper_1910_00178_amd as ng
    lda = (K + 7) // 8 * 8
    A, B = (torch.zeros((rows, lda), dtype=torch.int16, device="cuda") for rows in (M, N))
    nb = ng.ngemm_packed_b_bytes_s16(K, N)
    packed = torch.empty(nb, dtype=torch.uint8, device="cuda")
    h = ng.ngemm_pack_b_s16(ctx, K, N, B, lda, packed, nb)
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    wsb = ng.ngemm_workspace_bytes(M, N, K)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    return lambda st, keep=(A, B, packed): ng.ngemm_run_s16s16s32(ctx, M, A, lda, 7, h, 3, C, N, ws, wsb, st)


# (M, N, K, entry point, cap, what runs, workgroups at most): 64 x 64 tiles of four to a unit count four for one
CAPPED = [(64, 4096, 4096, "s32", 3, "gemm_tile_deep_kernel<1,", 3), (500, 768, 768, "u8", 7, "gemm_tile_deep_kernel<1,", 7),
          (300, 200, 200, "s32", 5, "gemm_tile_dma_kernel<64, 64,", 20), (512, 4096, 4096, "s32", 9, "gemm_tile_deep_kernel<2,", 9),
          (1024, 768, 768, "s32", 0, "gemm_wavek_kernel<1, 1, 1, 2,", 768), (64, 96, 1000, "s32", 6, "gemm_wavek_kernel<1, 1, 1, 4,", 6),
          (500, 700, 1024, "unpacked", 3, "gemm_tile_dma_kernel<64, 64,", 12), (512, 768, 768, "s16", 2, "gemm_s16_tile_kernel", 2),
          (512, 768, 100, "s16", 2, "gemm_wavek_kernel<2, 2, 2, 2, 4, false, true, false, false, false, true>", 2),
          (60, 60, 100, "s16", 4, "gemm_wavek_kernel<2, 1, 1, 4,", 4), (512, 768, 768, "s16", 0, "gemm_wavek_kernel<2, 1, 2, 4,", 192),
          # shapes that no form of the kernel that splits K serves (its form 0 was asked how many tiles it has)
          (1024, 3072, 1000, "s32", 100, "gemm_tile_dma_kernel<64, 64,", 400), (1000, 3000, 300, "u8", 31, "gemm_tile_dma_kernel<64, 64,", 124),
          (1100, 1300, 1500, "unpacked", 31, "gemm_tile_dma_kernel<64, 64,", 124), (2048, 2048, 200, "unpacked", 31, "gemm_tile_dma_kernel<128, 128,", 62),
          (3072, 3072, 1024, "unpacked", 50, "gemm_tile_x64_kernel<true", 50)]


@pytest.mark.parametrize("case", CAPPED, ids=str)
def test_cap_on_workgroups(ctx, launches, case):
    import paper_1910_00178_amd as ng
    M, N, K, op, cap, want, most = case
    if op == "s16":
        call = s16_call(ctx, M, N, K)
    else:
        p = Problem(ctx, M, N, K)
        wsb = ng.ngemm_unpacked_workspace_bytes(M, N, K)
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
        call = {"s32": p.run(3), "u8": p.run_u8(3), "unpacked": lambda st: ng.ngemm_run_u8s8s32_unpacked(
            ctx, M, N, K, p.A, p.lda, 7, p.B, p.lda, 3, p.C, N, ws, wsb, st)}[op]
    ng.ngemm_set_max_workgroups(ctx, cap)
    try:
        got = launches(call)
    finally:
        ng.ngemm_set_max_workgroups(ctx, 0)
    assert got[-1][0].startswith(want) and got[-1][1] <= most, got
