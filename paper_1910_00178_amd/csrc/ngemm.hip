// Host side of the C ABI declared in include/ngemm.h: argument validation, kernel
// selection and launches.  Every step of the path runs in the kernels of
// ngemm_kernels.h; there is no CPU fallback.
#include "ngemm.h"
#include "ngemm_kernels.h"
#include "ngemm_mid.h"

#include <hip/hip_runtime.h>
#include <cmath>
#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

using namespace ngemm;

// Scratch memory of ngemm_run_u8s8s32_static, the entry point for callers that cannot allocate:
// the row sums of A that a zero-point of B needs (4 bytes per row), in the device image of the
// library instead of a caller's workspace.  Every GPU the library runs on holds its own copy of
// the array until the process ends.  In host code the name below only stands for the symbol: the
// device address of a GPU's copy comes from hipGetSymbolAddress (ngemm_create keeps it in the
// context), and only that address is ever handed to a kernel.
constexpr int64_t kStaticMaxM = 65536;
constexpr size_t kStaticScratchBytes = (size_t)kStaticMaxM * 4;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

struct ngemm_ctx {
    uint32_t magic;
    int device;
    int num_cus;
    int num_xcd;             // XCDs (L2 domains) of the device; workgroup ids go round them in turn
    int force_kernel;
    int max_workgroups;      // 0 = one per compute unit
    void *static_scratch;    // device address of this device's copy of `scratch`
    // kernels found fastest by ngemm_tune_u8s8s32, by shape; consulted before the shape heuristic
    struct Tuned {
        int64_t M, N, K;
        int kernel;          // the fastest of NGEMM_KERNEL_*
        bool wavek;          // what only the automatic choice launches (gemm_wavek_kernel, gemm_mid_kernel) was faster still
    };
    std::vector<Tuned> tuned;
};

struct ngemm_packed_b {
    uint32_t magic;
    int device;
    int64_t K, N, Kp, Np;
    const uint8_t *data;     // device, caller-owned
    size_t bytes;
    int32_t b_shift;         // 0: packed from int8; 128: packed from uint8, stored as B - 128
    int32_t elem_bytes;      // 1: 8-bit operand; 2: int16 operand packed as two byte planes
};

namespace {

constexpr uint32_t kCtxMagic = 0x4e47454du;   // "NGEM"
constexpr uint32_t kPackMagic = 0x4e47504bu;  // "NGPK"
constexpr int64_t kMaxDim = 0x7fffffff - 4096;
constexpr int kSkinnyMaxM = 32;
constexpr int BK256 = 64;                        // stage depth of the 256 x 256 configuration
constexpr int kStages256 = 4;                    // ring depth of its direct-to-LDS form

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// gemm_tile_x64_kernel addresses its copies with 32-bit offsets from the tile's first row (panel,
// column): `rows` rows of `pitch` bytes, `extent` bytes used of the last one
inline bool x64_offsets_fit(int64_t rows, int64_t pitch, int64_t extent)
{
    return pitch < (1ll << 32) && (rows - 1) * pitch + extent + 4096 < (1ll << 32);
}

// gemm_wavek_kernel counts in 31 bits, from a row of at most 64 of A and from one of at most four panels of 32 columns of B
// (unpacked: rows of it); what lies further apart takes the same forms with addresses of 64 bits (launch_wavek_far_form)
inline bool wavek_offsets_fit(int64_t lda_bytes, int64_t kbytes, int64_t Kp, int64_t ldb = 0)
{
    constexpr int64_t most = (1ll << 31) - 8192;
    return lda_bytes < most / 64 && 64 * lda_bytes + kbytes < most && Kp < most / 128 && ldb < most / 128 && 128 * ldb + kbytes < most;
}

struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) return;
        ok = (prev == dev) || (hipSetDevice(dev) == hipSuccess);
        if (prev == dev) prev = -1;
        // the launches below are checked with hipGetLastError(): drop an error that other code on
        // this thread left behind, so that it is not reported as one of ours
        (void)hipGetLastError();
    }
    ~DeviceGuard()
    {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

bool ctx_ok(const ngemm_ctx *c) { return c && c->magic == kCtxMagic; }
bool pack_ok(const ngemm_packed_b *b) { return b && b->magic == kPackMagic; }

template <int BM, int BN, int WGM, int WGN, int BK>
hipError_t launch_tile(const GemmParams &p0, bool requant, hipStream_t st, bool rows = false)
{
    using Cfg = TileCfg<BM, BN, WGM, WGN, BK>;
    GemmParams p = p0;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n)), block(WGM * WGN * 64);
    const size_t smem = Cfg::kLdsBytes;
    if constexpr (BM < 256) {
        // the form that adds up the row sums itself (64 x 64 and 128 x 128 tiles)
        static_assert(Cfg::kLdsBytes <= 64 * 1024, "needs no LDS attribute");
        if (rows) {
            if (requant)
                hipLaunchKernelGGL((gemm_tile_kernel<BM, BN, WGM, WGN, BK, true, true>), grid, block, smem, st, args_of(p));
            else
                hipLaunchKernelGGL((gemm_tile_kernel<BM, BN, WGM, WGN, BK, false, true>), grid, block, smem, st, args_of(p));
            return hipGetLastError();
        }
    }
    if (requant)
        hipLaunchKernelGGL((gemm_tile_kernel<BM, BN, WGM, WGN, BK, true>), grid, block, smem, st, args_of(p));
    else
        hipLaunchKernelGGL((gemm_tile_kernel<BM, BN, WGM, WGN, BK, false>), grid, block, smem, st, args_of(p));
    return hipGetLastError();
}

// Kernels whose LDS need exceeds the 64 KiB default must be opted in once per device.
template <int BM, int BN, int WGM, int WGN, int BK>
hipError_t allow_big_lds()
{
    using Cfg = TileCfg<BM, BN, WGM, WGN, BK>;
    if (Cfg::kLdsBytes <= 64 * 1024) return hipSuccess;
    hipError_t e = hipFuncSetAttribute((const void *)gemm_tile_kernel<BM, BN, WGM, WGN, BK, true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kLdsBytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)gemm_tile_kernel<BM, BN, WGM, WGN, BK, false>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kLdsBytes);
}

template <int BM, int BN, int WGM, int WGN, int NSTAGE = 4>
hipError_t launch_tile_dma(const GemmParams &p0, bool requant, int num_cus, hipStream_t st,
                           const RawB *rawb = nullptr, bool rows = false)
{
    using Cfg = DmaCfg<BM, BN, WGM, WGN, NSTAGE>;
    GemmParams p = p0;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    // Persistent workgroups: as many as can be resident (the 256 x 256 configuration fills a
    // compute unit's registers and LDS with one workgroup, the smaller ones leave room for more).
    const int ntiles = p.tiles_m * p.tiles_n;
    const int per_cu = BM >= 256 ? 1 : (BM >= 128 ? 2 : 4);
    const int nwg = ntiles < num_cus * per_cu ? ntiles : num_cus * per_cu;
    dim3 grid((unsigned)nwg), block(WGM * WGN * 64);
    const size_t smem = Cfg::kLdsBytes;
    const GemmArgs args = rawb ? args_of_raw(p, *rawb, nwg) : args_of(p, nwg);
    if (rawb) {      // unpacked B: int32 output only; `rows`: the sums of both operands are formed in the kernel
        if constexpr (BM < 256) {
            if (rows) {
                hipLaunchKernelGGL((gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, false, true, true>), grid, block, smem, st, args);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, false, true>), grid, block, smem, st, args);
        return hipGetLastError();
    }
    if constexpr (BM < 256) {
        // the form that adds up the row sums itself (64 x 64 and 128 x 128 tiles)
        static_assert(Cfg::kLdsBytes <= 64 * 1024, "needs no LDS attribute");
        if (rows) {
            if (requant)
                hipLaunchKernelGGL((gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, true, false, true>), grid, block, smem, st, args);
            else
                hipLaunchKernelGGL((gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, false, false, true>), grid, block, smem, st, args);
            return hipGetLastError();
        }
    }
    if (requant)
        hipLaunchKernelGGL((gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, true>), grid, block, smem, st, args);
    else
        hipLaunchKernelGGL((gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, false>), grid, block, smem, st, args);
    return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int NSTAGE = 4>
hipError_t allow_big_lds_dma()
{
    using Cfg = DmaCfg<BM, BN, WGM, WGN, NSTAGE>;
    if (Cfg::kLdsBytes <= 64 * 1024) return hipSuccess;
    hipError_t e = hipFuncSetAttribute((const void *)gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kLdsBytes);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void *)gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, false, true>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kLdsBytes);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void *)gemm_tile_dma_kernel<BM, BN, WGM, WGN, NSTAGE, false>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kLdsBytes);
}

// Small tiles with the long pipeline: one workgroup per compute unit (the ring takes 128 KiB).
// T = 1: 64 x 64 tiles, stages of 256 bytes of K; T = 2: 128 x 128 tiles, stages of 128 bytes.
constexpr int kDeepStages = 4;
template <int T>
constexpr int kDeepSub = T == 1 ? 4 : 2;

// `rows`: the kernel forms the row sums itself (a zero-point of B is there; no row-sum pass ran)
template <int T>
hipError_t launch_tile_deep(const GemmParams &p0, bool requant, bool rows, int num_cus, hipStream_t st)
{
    using Cfg = DeepCfg<T, kDeepSub<T>, kDeepStages>;
    GemmParams p = p0;
    p.tiles_m = (p.M + Cfg::BMN - 1) / Cfg::BMN;
    p.tiles_n = (p.N + Cfg::BMN - 1) / Cfg::BMN;
    const int ntiles = p.tiles_m * p.tiles_n;
    const int nwg = ntiles < num_cus ? ntiles : num_cus;
    const dim3 grid((unsigned)nwg), block(256);
    const GemmArgs args = args_of(p, nwg);
    if (requant && rows)
        hipLaunchKernelGGL((gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, true, 0, true>), grid, block, Cfg::kLdsBytes, st, args);
    else if (requant)
        hipLaunchKernelGGL((gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, true>), grid, block, Cfg::kLdsBytes, st, args);
    else if (rows)
        hipLaunchKernelGGL((gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, false, 0, true>), grid, block, Cfg::kLdsBytes, st, args);
    else
        hipLaunchKernelGGL((gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, false>), grid, block, Cfg::kLdsBytes, st, args);
    return hipGetLastError();
}

// K split over workgroups for outputs that leave most compute units without a tile (64 x 64 tiles,
// int32 output): S = the number of parts that brings the grid up to the unit count, each part a
// multiple of 256 bytes of K (whole stages of the long pipeline) and at least kSplitMinChunk long.
// With room in the workspace the parts store their partial tiles there and a second kernel sums them
// and finishes the epilogue (any output type); without it C is cleared first and every part adds its
// partial tile with atomic adds (int32 outputs; exact in any order).
constexpr int kSplitMinChunk = 1024;
constexpr int kSplitMaxUnits = 256;        // (tile, part) units of a K split: one per compute unit at most
int splitk_parts(int64_t M, int64_t N, int64_t K, int num_cus, int *kchunk)
{
    const int64_t ntiles = ((M + 63) / 64) * ((N + 63) / 64);
    if (num_cus > kSplitMaxUnits) num_cus = kSplitMaxUnits;
    int64_t S = ntiles > 0 ? num_cus / ntiles : 1;
    if (S * kSplitMinChunk > K) S = K / kSplitMinChunk;
    if (S < 2) return 1;
    const int64_t chunk = round_up((K + S - 1) / S, 256);
    *kchunk = (int)chunk;
    return (int)((K + chunk - 1) / chunk);         // every part holds at least one byte of K
}

// Bytes of the partial results of a K split into `parts`.
size_t splitk_part_bytes(int64_t M, int64_t N, int parts)
{
    return (size_t)round_up((int64_t)parts * M * splitk_part_pitch(N) * 4, 256);
}

// part_ws: room for the partial results (splitk_part_bytes), or nullptr for the atomic form.
hipError_t launch_tile_deep_splitk(const GemmParams &p0, int parts, int kchunk, bool rows, bool requant, int32_t *part_ws,
                                   int num_cus, hipStream_t st)
{
    using Cfg = DeepCfg<1, kDeepSub<1>, kDeepStages>;
    GemmParams p = p0;
    p.tiles_m = (p.M + 63) / 64;
    p.tiles_n = (p.N + 63) / 64;
    p.ksplit = parts;
    p.kchunk = kchunk;
    p.part_ws = part_ws;
    const int nunits = p.tiles_m * p.tiles_n * parts;
    const int nwg = nunits < num_cus ? nunits : num_cus;
    const dim3 grid((unsigned)nwg), block(256);
    const GemmArgs args = args_of(p, nwg);
    if (part_ws) {
        if (rows)
            hipLaunchKernelGGL((gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 2, true>), grid, block, Cfg::kLdsBytes, st, args);
        else
            hipLaunchKernelGGL((gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 2, false>), grid, block, Cfg::kLdsBytes, st, args);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const int nw = parts < kReduceWaves ? parts : kReduceWaves;
        const int64_t lanes = (int64_t)p.M * (splitk_part_pitch(p.N) / 4);
        const dim3 rgrid((unsigned)((lanes + 63) / 64)), rblock(64 * nw);
        if (requant)
            hipLaunchKernelGGL(splitk_reduce_kernel<true>, rgrid, rblock, 0, st, args_of(p, nw));
        else
            hipLaunchKernelGGL(splitk_reduce_kernel<false>, rgrid, rblock, 0, st, args_of(p, nw));
        return hipGetLastError();
    }
    const int64_t segs = (p.N + 1023) / 1024;
    hipLaunchKernelGGL(zero_c_kernel, dim3((unsigned)(p.M * segs)), dim3(256), 0, st, (int32_t *)p.C, p.ldc, p.N, (int)segs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (rows)
        hipLaunchKernelGGL((gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 1, true>), grid, block, Cfg::kLdsBytes, st, args);
    else
        hipLaunchKernelGGL((gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 1, false>), grid, block, Cfg::kLdsBytes, st, args);
    return hipGetLastError();
}

template <int T>
hipError_t allow_big_lds_deep()
{
    using Cfg = DeepCfg<T, kDeepSub<T>, kDeepStages>;
    const void *forms[] = {
        (const void *)gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, false>,
        (const void *)gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, true>,
        (const void *)gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, false, 0, true>,
        (const void *)gemm_tile_deep_kernel<T, kDeepSub<T>, kDeepStages, true, 0, true>,
        (const void *)gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 1, false>,
        (const void *)gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 1, true>,
        (const void *)gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 2, false>,
        (const void *)gemm_tile_deep_kernel<1, kDeepSub<1>, kDeepStages, false, 2, true>,
    };
    for (const void *f : forms) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, Cfg::kLdsBytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int P>
void launch_skinny_p(const GemmParams &p, bool requant, int nwaves, size_t smem, hipStream_t st)
{
    dim3 grid((unsigned)((p.npanels + P - 1) / P)), block(nwaves * 64);
    if (requant)
        hipLaunchKernelGGL((gemm_skinny_kernel<true, P>), grid, block, smem, st, args_of(p, nwaves));
    else
        hipLaunchKernelGGL((gemm_skinny_kernel<false, P>), grid, block, smem, st, args_of(p, nwaves));
}

// The streaming kernel (a panel per wavefront, A in LDS) can serve a problem when its A fits the
// 64 KiB of LDS a kernel gets without asking and there is a K to stream.
bool stream_can_serve(int64_t M, int64_t Kp)
{
    return Kp >= 64 && stream_lds_bytes((int)M, Kp, kStreamMaxChunk, 0) <= kStreamMaxLds;
}

// LDS of a streaming launch for one problem: what it needs, plus room to park the sums of all but
// the last panel of each wavefront as far as the 64 KiB allow.
int stream_launch_lds(int M, int64_t Kp, int chunk)
{
    const int per_wave = chunk / kStreamWaves - 1;
    int64_t want = stream_lds_bytes(M, Kp, chunk, per_wave > 0 ? per_wave : 0);
    return (int)(want < kStreamMaxLds ? want : kStreamMaxLds);
}

// Panels per workgroup of the streaming kernel for `panels` panels in all: R per wavefront, one
// as long as that makes no more than eight rounds of resident wavefronts (16 per compute unit):
// short-lived workgroups handed out by the dispatcher even out what a static share cannot
// (measured on 59 x 128 panels: R = 1, 1888 workgroups, 5.6 TB/s; R = 2, 944, one round, 5.45;
// on 84 x 128: R = 1 5.6, R = 2 5.5).
int stream_chunk(int64_t panels, int num_cus)
{
    const int64_t max_waves = (int64_t)num_cus * 128;
    int64_t R = (panels + max_waves - 1) / max_waves;
    R = R < 1 ? 1 : (R > kStreamMaxChunk / kStreamWaves ? kStreamMaxChunk / kStreamWaves : R);
    return (int)(kStreamWaves * R);
}

hipError_t launch_skinny(const GemmParams &p, bool requant, int num_cus, hipStream_t st)
{
    if (p.npanels >= 8 * num_cus && stream_can_serve(p.M, p.Kp)) {
        const int chunk = stream_chunk(p.npanels, num_cus);
        const dim3 grid((unsigned)((p.npanels + chunk - 1) / chunk)), block(kStreamWaves * 64);
        const int smem = stream_launch_lds(p.M, p.Kp, chunk);
        GemmArgs args = args_of(p);
        args.kchunk = chunk;
        args.ksplit = smem;
        if (requant)
            hipLaunchKernelGGL(gemm_stream_skinny_kernel<true>, grid, block, (size_t)smem, st, args);
        else
            hipLaunchKernelGGL(gemm_stream_skinny_kernel<false>, grid, block, (size_t)smem, st, args);
        return hipGetLastError();
    }
    const int nslices = p.Kp / 32;
    int nwaves = 1;
    while (nwaves < 8 && nwaves * 4 <= nslices) nwaves *= 2;    // at least two fragments per wavefront, at most 8 wavefronts
    const int nregs = 4 * ((p.M + 7) / 8);
    const size_t smem = nwaves > 1 ? (size_t)nwaves * nregs * 64 * sizeof(int) : 0;
    // panels per workgroup: share an A fragment between panels when the output is wide enough to
    // still give every compute unit several workgroups (only worth it once A's rows are many)
    // (measured at N = 32768, K = 8192: M = 32 gains 30 % with four panels, M = 16 12 % with two;
    // at N = 16384 a workgroup per panel is still the fastest)
    if (p.M > 16 && p.npanels >= 4 * num_cus)
        launch_skinny_p<4>(p, requant, nwaves, smem, st);
    else if (p.M > 4 && p.npanels >= 4 * num_cus)
        launch_skinny_p<2>(p, requant, nwaves, smem, st);
    else
        launch_skinny_p<1>(p, requant, nwaves, smem, st);
    return hipGetLastError();
}

int workgroup_budget(const ngemm_ctx *ctx)
{
    const int cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    return (ctx->max_workgroups > 0 && ctx->max_workgroups < cus) ? ctx->max_workgroups : cus;
}

// Rows that copies into LDS can fetch: 16-byte aligned.
inline bool rows_aligned(const void *A, int64_t lda) { return (((uintptr_t)A | (uintptr_t)lda) & 15) == 0; }

// Shape heuristic: the 256 x 256 configuration when it fills at least half of the compute units
// (3072^3, 144 tiles: 35 us against 47 us with 128 x 128; 2048 x 4096 x 1024, 128 tiles: a tie),
// the 128 x 128 one when every unit still gets a workgroup, else 64 x 64 (measured on 18 shapes
// from 16 x 512 x 512 to 4096^3: the smallest tile wins as long as the larger ones leave units
// idle; ngemm_tune_u8s8s32 settles the borderline cases by measurement).
int choose_kernel(const ngemm_ctx *ctx, int64_t M, int64_t N, int64_t K, bool aligned, bool requant)
{
    auto tiles = [&](int64_t b) { return ((M + b - 1) / b) * ((N + b - 1) / b); };
    const int64_t cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    // Few tiles and a long K: spread K over the idle units.  The launch that clears C and the atomic adds have
    // to pay off: against 64 x 64 tiles (48 shapes) the split wins from K = 8192 on up to 96 of them and from 12288 up to
    // 128.  Against the kernel that splits K over a workgroup's wavefronts (wavek_form) it depends on where the weight
    // is (us, that kernel / the split, the same weight in cache, then every byte from memory):
    //   64 x 1024 x 6144 5.5 / 7.1 and 10.5 / 9.4, x 8192 6.3 / 7.4 and 12.9 / 9.6, x 9216 6.8 / 7.7 and 14.1 / 10.0
    //   256 x 256 x 8192 8.6 / 8.7 and 11.1 / 9.8, x 9216 9.4 / 8.8 and 12.1 / 10.0, x 16384 9.7 / 10.0 (u8 10.2 / 10.6)
    //   32 x 2048 x 8192 6.3 / 7.5 and 14.2 / 9.8; u8 outputs, whose partial sums go through the workspace:
    //   64 x 256 x 8192 6.5 / 8.4 and 12.7 / 10.6, 64 x 64 x 8192 6.5 / 8.1 and 8.6 / 8.9
    // so int32 outputs of up to a quarter of a 32 x 32 tile per unit split from K = 8192 on and u8 ones and larger ones
    // (64 x 2048 x 8192 7.2 / 9.5 and 13.6 / 11.8, x 9216 9.1 / 9.7 and 14.8 / 11.6; 512 x 256 x 9216 9.3 / 10.7 and 10.8 / 11.0) from 9216.
    const int64_t split_min_k = tiles(32) * 4 <= cus && !requant ? 8192 : 9216;
    const int64_t t64 = tiles(64), step = 3 * cus / 16;
    if (M <= kSkinnyMaxM) {
        if (K >= split_min_k && t64 * 8 <= cus) return NGEMM_KERNEL_SPLIT_K;
        return NGEMM_KERNEL_SKINNY;
    }
    if (t64 * 2 <= cus && K >= split_min_k && K >= 4096 * ((t64 + step - 1) / step)) return NGEMM_KERNEL_SPLIT_K;
    const int64_t t192 = ((M + 191) / 192) * ((N + 255) / 256);
    // The large tiles pay off from 0.7 of the compute units filled with K >= 512 (4096 x 4096 x 256: 16.5 / 15.0), from 0.5 with K >= 1024,
    // from 0.4 with K >= 2048: their fill and epilogue want stages to spread over (us, large against
    // 128 x 128 tiles: 3072 x 3072 x 512 13.2 / 15.0, 2560 x 2560 x 512 10.8 / 9.6, 2176 x 2176 x 1024
    // 13.4 / 12.1, 2304^3 20.8 / 22.5, 2560^3 24.0 / 26.6).
    const int64_t big = tiles(256) > t192 ? tiles(256) : t192;
    // Only where 128 x 128 tiles would not give every unit one at most (256 x 16384 x 4096, 64 tiles of 256 rows or 128
    // of 192, half of them rows that do not exist: 35.2 us, 128 x 128 tiles 26).
    if (tiles(128) > cus && ((big * 10 >= cus * 7 && K >= 512) || (big * 2 >= cus && K >= 1024) || (big * 5 >= cus * 2 && K >= 2048))) {
        if (!aligned) {
            // The 256 x 256 tiles are staged through registers then and pay off only when they fill most of every
            // round of compute units; else 128 x 128 tiles, which also form the row sums (us, 128 / 256, zero-point
            // of B: 2047 x 3071 x 1537, 96 tiles of 256 25.8 / 40.5, 3001 x 3003 x 1001, 144 tiles 29.1 / 34.3,
            // 4097^3, 289 tiles 129 / 145, 8191 x 4095 x 2047, 512 tiles 128 / 115).
            const int64_t rounds = (tiles(256) + cus - 1) / cus;
            return tiles(256) * 100 < 58 * rounds * cus ? NGEMM_KERNEL_TILE_128 : NGEMM_KERNEL_TILE_256;
        }
        // The large tiles take what is left of K behind their even number of stages without pipelining, 4 us and
        // more per tile; 128 x 128 tiles that all are resident at once (two per unit) lose less by it (us, 128 against
        // the large ones: 2047 x 3071 x 1537 23.1 / 24.3, u8 23.4 / 27.6; 700 x 8000 x 1500 20.4 / 22.1, u8 21.1 / 26.7;
        // 1000 x 7000 x 3000 33.4 / 34.0, u8 34.0 / 35.9; 2304 x 2304 x 2304, whole stages 24.2 / 22.0).
        if (K % 64 != 0 && tiles(128) <= 2 * cus) return NGEMM_KERNEL_TILE_128;
        // rounds of resident workgroups times the rows of a tile: 192 x 256 tiles when they fill more of the
        // compute units for less time (3072^3: 144 tiles of 256 rows against 192 of 192, one round each;
        // 2560^3: 100 against 140, 29.3 us against 24.0 us, 128 x 128 tiles 26.6 us)
        const int64_t r256 = (tiles(256) + cus - 1) / cus * 256, r192 = (t192 + cus - 1) / cus * 192;
        return r192 < r256 ? NGEMM_KERNEL_TILE_192 : NGEMM_KERNEL_TILE_256;
    }
    // (us, 128 x 128 against 64 x 64 tiles; 1536^3, 144 tiles of 128 x 128, inputs changing from call to call, 12.2 / 12.7;
    // the same inputs: 1408 x 1408, 121 tiles, K = 1024 8.3 / 7.1, 2048 11.7 / 10.9, 3072 15.7 / 14.3 (the kernel behind TILE_64
    // there splits K over wavefronts); 1024 x 2048 x 2048, 128 tiles 11.9 / 10.8 and with a zero-point or u8 output 13.6 / 11.9;
    // 1024^3, 64 tiles 7.9 / 5.5; 1536 x 1536 x 512 6.9 / 6.4.  Once 64 x 64 tiles need a third round of two per unit the larger ones
    // win from K = 2560 on: 1536 x 1408, 132 tiles, 14.4 / 15.4, u8 16.0 / 15.9, 3584 16.6 / 19.4, u8 18.3 / 20.1; 1400 x 1500 x 2048
    // 12.6 / 12.7 and u8 14.2 / 12.9.)
    // Not for M <= 64, which would leave half of every tile empty (64 x 16384 x 4096 18.6 / 14.5 us).
    if (M > 64 && (tiles(128) >= cus || (tiles(128) * 20 >= cus * 11 && K >= 1024) || (tiles(128) * 5 >= cus * 2 && K >= 4096) ||
                   (t64 > 2 * cus && tiles(128) * 2 >= cus && K >= 2560)))
        return NGEMM_KERNEL_TILE_128;
    return NGEMM_KERNEL_TILE_64;
}

// Pack and column sums.  kbytes: bytes of a column that exist, Kp: bytes of a packed one.
// Columns of up to 2 KiB: one workgroup of 512 threads per panel walks the whole column, so the sums are
// stored and no launch has to clear them (us, against parts of 512 bytes with a clearing launch: 64 x 64
// 5.4 -> 3.9, 768 x 768 5.9 -> 4.1, 4096 columns of 2048 7.8 -> 6.9).  Longer columns: workgroups of 256
// threads, sums added to cleared memory; parts of one block (512 bytes) for the 8-bit operand (4096 columns of
// 4096: 9.9 against 10.5 with two), of two for the 16-bit one, the second on its way while the first is turned
// (4096 columns of 8192 bytes 13.7 against 16.0).  A workgroup per whole long column leaves compute units idle
// (1024 columns of 8192 bytes: 17 us in the place of 8).
template <int ELEM, int NT, int PER>
ngemm_status launch_pack_blocks(const uint8_t *B, int64_t ldb_bytes, int64_t kbytes, int64_t N, int64_t Kp, int64_t Np, uint32_t b_xor,
                                uint8_t *packed, int32_t *colsum, hipStream_t st)
{
    constexpr int KB = 2 * NT;
    const int64_t panels = Np / 32, nblocks = (Kp + KB - 1) / KB, nparts = (nblocks + PER - 1) / PER;
    if (panels * nparts > 0x7fffffff) return NGEMM_ERR_BAD_SHAPE;
    if (nparts != 1) {                               // several parts add up, and K = 0 has no block that would store
        hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)((Np + 255) / 256)), dim3(256), 0, st, colsum, (int)Np);
        if (hipGetLastError() != hipSuccess) return NGEMM_ERR_DEVICE;
        if (nparts == 0) return NGEMM_OK;
    }
    hipLaunchKernelGGL((pack_b_kernel<NT, ELEM, PER>), dim3((unsigned)(panels * nparts)), dim3(NT), 0, st, B, ldb_bytes, kbytes, (int)N,
                       (int)(Kp / 32), (int)nblocks, (int)nparts, b_xor, packed, colsum);
    return hipGetLastError() == hipSuccess ? NGEMM_OK : NGEMM_ERR_DEVICE;
}

template <int ELEM>
ngemm_status launch_pack(const uint8_t *B, int64_t ldb_bytes, int64_t kbytes, int64_t N, int64_t Kp, int64_t Np, uint32_t b_xor,
                         uint8_t *packed, int32_t *colsum, hipStream_t st)
{
    // (the runtime takes less than 2^32 threads in a launch: the widest operands need the smaller workgroups)
    if (Kp <= 2048 && Np / 32 * 512 < (1ll << 32)) return launch_pack_blocks<ELEM, 512, 2>(B, ldb_bytes, kbytes, N, Kp, Np, b_xor, packed, colsum, st);
    return launch_pack_blocks<ELEM, 256, ELEM>(B, ldb_bytes, kbytes, N, Kp, Np, b_xor, packed, colsum, st);
}

// Forms of the kernel that splits K over a workgroup's wavefronts (gemm_wavek_kernel): tile in units of
// 32 x 32, wavefronts, ring depth.
template <int TM_, int TN_, int NW_, int RING_>
struct WaveKForm {
    static constexpr int TM = TM_, TN = TN_, NW = NW_, RING = RING_;
};
using WaveK11 = WaveKForm<1, 1, 4, 4>;       // 64 KiB of LDS: two workgroups per compute unit
using WaveK12 = WaveKForm<1, 2, 4, 3>;       // 72 KiB
using WaveK22 = WaveKForm<2, 2, 2, 4>;       // 64 KiB (16-bit operands)
using WaveK11Short = WaveKForm<1, 1, 2, 4>;  // 32 KiB: five workgroups per compute unit
using WaveK22Long = WaveKForm<2, 2, 4, 3>;   // 96 KiB: one
using WaveK24 = WaveKForm<2, 4, 4, 3>;       // 144 KiB: one
using WaveK12Short = WaveKForm<1, 2, 2, 4>;  // 48 KiB (A through registers)

template <class F, int ELEM, bool REQUANT, bool ROWS, bool BRAW = false, bool AREG = false, bool NT = false>
hipError_t launch_wavek(const GemmParams &p0, hipStream_t st, const RawB *rawb = nullptr)
{
    GemmParams p = p0;
    p.tiles_m = (p.M + F::TM * 32 - 1) / (F::TM * 32);
    p.tiles_n = (p.N + F::TN * 32 - 1) / (F::TN * 32);
    hipLaunchKernelGGL((gemm_wavek_kernel<ELEM, F::TM, F::TN, F::NW, F::RING, REQUANT, ROWS, BRAW, AREG, NT>), dim3((unsigned)(p.tiles_m * p.tiles_n)),
                       dim3(F::NW * 64), (WaveKCfg<F::TM, F::TN, F::NW, F::RING>::kLdsBytes), st, rawb ? args_of_raw(p, *rawb) : args_of(p));
    return hipGetLastError();
}

template <class F, int ELEM, bool REQUANT, bool ROWS, bool BRAW = false, bool NT = false>
hipError_t allow_big_lds_wavek()
{
    constexpr int lds = WaveKCfg<F::TM, F::TN, F::NW, F::RING>::kLdsBytes;
    if (lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute((const void *)gemm_wavek_kernel<ELEM, F::TM, F::TN, F::NW, F::RING, REQUANT, ROWS, BRAW, false, NT>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

template <class F>
hipError_t allow_big_lds_wavek_u8()
{
    hipError_t e = allow_big_lds_wavek<F, 1, false, false>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, false, true>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, true, false>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, true, true>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, false, false, true>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, false, true, true>();
    return e;
}

template <class F>
hipError_t allow_big_lds_wavek_nt()
{
    hipError_t e = allow_big_lds_wavek<F, 1, false, false, false, true>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, false, true, false, true>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, true, false, false, true>();
    if (e == hipSuccess) e = allow_big_lds_wavek<F, 1, true, true, false, true>();
    return e;
}

// M <= 32, aligned rows: the form (10 TM + TN of its tile, 1 for WaveK11Short), or 0: the streaming kernel is faster.  A weight
// may be read again and again from cache or come from memory on every call, so the lines lie where neither loses much:
// us in a graph, one weight / three in turn / 768 MiB of them in turn (every byte from memory), streaming kernel,
// then this one (copies as wavek_nt says):
//  * a 32 x 32 tile per compute unit at most: 16 x 1024 x 1024 3.68 / 3.59 / 3.98, 3.23 / 3.14 / 3.71; 8 x 8192 x 4096
//    6.7 / 8.2 / 8.9, 5.9 / 7.3 / 8.0.  Two wavefronts are enough up to K = 512 (1 x 4096 x 512 3.42 with four, 3.35 with two);
//  * up to two tiles per unit and up to eight rows: 1 x 16384 x 1024 4.2 / 5.0 / 5.6, 4.0 / 5.0 / 5.7, but 1 x 16384 x 4096
//    10.6 / 11.6 / 12.7, 10.7 / 12.0 / 13.2 and 8 x 16384 x 2048 5.9 / 7.1 / 7.8, 5.7 / 7.5 / 8.2: half of what this kernel copies
//    is A.  More rows: 16 x 16384 x 4096 13.3 / 13.8 / 14.6, 11.1 / 12.5 / 13.5; two panels per workgroup from K = 2048
//    on (32 x 16384 x 2048 6.5 / 8.4 / 10.4 with one, 6.0 / 8.6 / 9.6 with two; 16 x 16384 x 512 3.5 / 3.4 / 4.7 and 3.7 / 3.6 / 4.9);
//  * more tiles and up to 64 MiB of weight: 8 x 32768 x 1024 8.8 / 10.8 / 11.6, 6.0 / 8.3 / 9.9; 1 x 32768 x 2048
//    12.5 / 13.1 / 14.1, 12.3 / 13.2 / 14.2; not for a few rows and the shortest K (1 x 32768 x 256 4.0 / 3.9 / 4.8, 4.0 / 3.9 / 5.2; 1 x 32768 x 300
//    4.8 / 5.1 / 5.9, 4.4 / 4.9 / 7.0; at 512 it is 7.6 / 8.2 (in cache, from memory), 4.4 / 6.8);
//  * larger ones, more than eight rows: 32 x 32768 x 4096 27.3 / 28.2 / 29.8, 22.3 / 27.9 / 28.7, but not the widest and deepest
//    (32 x 32768 x 8192 51, 60), and up to 16 rows only if the last round of units is nearly full (16 x 24576 x 4096, 1.5 rounds,
//    18.9 / 19.7 / 20.6, 17.7 / 22.6 / 23.4; 16 x 32768 x 4096, two rounds, 26.7 / 28.9 / 29.6, 21.4 / 26.3 / 27.3).
int wavek_skinny_form(int64_t M, int64_t N, int64_t K, int64_t cus)
{
    const int64_t t32 = (N + 31) / 32;
    if (t32 <= cus) return K <= 512 ? 1 : 11;
    if (t32 <= 2 * cus) return M <= 8 && K > 1024 ? 0 : K >= 2048 ? 12 : 1;
    if (N * K <= (64ll << 20)) return t32 > 4 * cus || (M <= 4 && K <= 320) ? 0 : 1;
    const int64_t wgs = (N + 63) / 64, rounds = (wgs + cus - 1) / cus;
    if (M <= 16 && wgs * 10 < rounds * cus * 8) return 0;
    return M > 8 && K <= 4096 ? 12 : 0;
}

// Whether that form copies B non-temporally.  From memory this is always faster (1 x 4096 x 1024 3.73 against 4.39 us,
// 16 x 16384 x 4096 13.5 / 15.1), but a weight that the next call could have found in cache is not kept there (three in
// turn, us, non-temporal / plain: 16 x 4096 x 4096 6.6 / 5.7, 32 x 8192 x 8192 15.6 / 13.0).  Weights of up to 8 MiB
// stay in cache all the same (8 x 4096 x 2048 3.58 / 3.58; from memory 4.7 / 5.4).  Beyond, where most units stream and the plain
// copies lose to the streaming kernel (three in turn and from memory, non-temporal / plain / streaming kernel):
// 8 x 8192 x 2048 4.9 / 5.5 / 5.5 and 5.4 / 6.1 / 6.1, 8 x 8192 x 4096 7.3 / 7.7 / 8.2 and 8.0 / 9.1 / 8.9, 16 x 16384 x 2048
// 7.7 / 8.1 / 7.8 and 8.4 / 9.3 / 8.6, 1 x 32768 x 2048 13.2 / 12.2 / 13.1 and 14.2 / 16.6 / 14.1.
bool wavek_nt(int64_t M, int64_t N, int64_t K, int64_t cus)
{
    if (M > kSkinnyMaxM) return false;
    const int64_t t32 = (N + 31) / 32;
    if (N * K <= (8ll << 20)) return true;
    if (M > 16) return false;
    if (t32 <= cus) return 2 * t32 > cus && (N * K <= (16ll << 20) || M <= 8);
    return N * K <= (64ll << 20) && (t32 <= 2 * cus || (M <= 4 && K >= 2048));
}

// The form that serves an 8-bit problem with aligned rows of A, or 0: the other kernels are faster.  us in a graph, this
// kernel / the others (at z: with a zero-point of B, whose row sums cost the others more):
//  * a 32 x 32 tile per compute unit at most: 64 x 4096 x 4096 7.0 / 10.2 (z 7.1 / 12.5), 33 x 4096 x 1024
//    3.8 / 5.2;
//  * 32 x 64 tiles, one per compute unit at most: 128 x 4096 x 4096 8.5 / 10.4, 512 x 768 x 3072 7.1 / 8.6,
//    512 x 768 x 768 4.4 / 5.1;
//  * a K of up to 1024 and up to three 32 x 32 tiles per unit: 1024 x 768 x 768 5.0 / 5.5, 700 x 900 x 600
//    6.3 / 6.5; at four tiles per unit (1024 x 1024 x 256 4.6 / 4.4) and below K = 256 it is a tie or a loss;
//  * 64 x 128 tiles, one per compute unit at most, and a long K, in the place of 128 x 128 tiles on half of the units or
//    of two rounds of 64 x 64: 512 x 4096 x 4096 16.8 / 19.3 (z 18.0 / 21.9), 128 x 16384 x 4096 18.1 / 20.2 (z 20.4 /
//    23.0); at K = 2048 it is a tie (1024 x 2048 x 2048 12.0 / 11.9);
//  * 64 x 64 tiles, one per unit at most, and a long K: with row sums 256 x 4096 x 4096 z 11.8 / 13.7, 384 x 2048 x 2048 z 8.3 / 9.0.
// The next three lines come from 9900 shapes of 257 to 760 tiles of 32 x 64 timed with these forms and with the kernels before, a third
// of them with every byte of B from memory, where the gains are the same or larger (averages; z, u8: a zero-point of B, u8 outputs):
//  * the same tiles without row sums: int32 1.08 x up to K = 2048, 1.05 up to 3072, 1.02 up to 4096, 1.00 beyond (480 x 2048 x 2369 9.0 / 8.1); u8
//    1.04, 1.015 and 1.00 x;
//  * 32 x 64 tiles where there are more than three of 32 x 32 per unit and a K of up to 1024: 1.04-1.14 x (661 x 1469 x 784
//    6.8 / 5.7, 224 x 3904 x 819 z 6.6 / 5.6), only with row sums, int32 and K < 384 1.00;
//  * 32 x 64 tiles, two per unit, in the place of two rounds of 64 x 64: 1.07-1.27 x (412 x 2492 x 1472 z 9.6 / 7.6, 160 x 5696 x 3008 13.5 / 11.8),
//    beyond K = 6144 1.03 (from memory 1.00); plain int32 problems also in the place of 64 x 128 tiles (1.05-1.3 x).  With more tiles 0.80-1.02 x.
//    From K = 1536 on the others are gemm_mid_kernel's (1.05-1.3 x is left there).
int wavek_form(int64_t M, int64_t N, int64_t K, bool rows, bool requant, int64_t cus)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t t32 = tiles(32, 32), t64 = tiles(64, 64);
    if (M <= kSkinnyMaxM) return wavek_skinny_form(M, N, K, cus);
    if (t32 <= cus) return 11;
    if (tiles(32, 64) <= cus) return 12;
    if (K >= 256 && K <= 1024 && t32 <= 3 * cus && t64 <= cus) return 1;
    if (K >= (rows && !requant ? 384 : 256) && K <= 1024 && t64 <= cus) return 12;
    const bool plain = !rows && !requant && K % 64 == 0;
    if (K >= 192 && K <= 6144 && t64 > cus && tiles(32, 64) <= 2 * cus && (K < 1536 || plain)) return 12;
    if (K > 1024 && t64 <= cus && (rows || K <= (requant ? 3072 : 4096))) return 22;
    if (K >= 3072 && t64 > cus && tiles(64, 128) <= cus) return 24;
    return 0;
}

template <class F, bool NT = false>
hipError_t launch_wavek_u8(const GemmParams &p, bool requant, bool rows, hipStream_t st)
{
    if (requant) return rows ? launch_wavek<F, 1, true, true, false, false, NT>(p, st) : launch_wavek<F, 1, true, false, false, false, NT>(p, st);
    return rows ? launch_wavek<F, 1, false, true, false, false, NT>(p, st) : launch_wavek<F, 1, false, false, false, false, NT>(p, st);
}

hipError_t launch_wavek_form(int form, const GemmParams &p, bool requant, bool rows, bool nt, hipStream_t st)
{
    if (nt) {
        if (form == 1) return launch_wavek_u8<WaveK11Short, true>(p, requant, rows, st);
        if (form == 11) return launch_wavek_u8<WaveK11, true>(p, requant, rows, st);
        if (form == 12) return launch_wavek_u8<WaveK12, true>(p, requant, rows, st);
    }
    switch (form) {
    case 1: return launch_wavek_u8<WaveK11Short>(p, requant, rows, st);
    case 11: return launch_wavek_u8<WaveK11>(p, requant, rows, st);
    case 12: return launch_wavek_u8<WaveK12>(p, requant, rows, st);
    case 24: return launch_wavek_u8<WaveK24>(p, requant, rows, st);
    default: return launch_wavek_u8<WaveK22Long>(p, requant, rows, st);
    }
}

// Rows of A with any alignment (A through registers).  us in a graph, this kernel / the others; where there are three pairs
// for one weight / three in turn / every byte from memory, as above:
//  * up to eight rows the skinny kernel's direct loads of A cost little (1 x 4096 x 1025 4.3 / 4.3, 2 x 300 x 8191 12.8 / 10.3);
//    up to 16 that holds for one tile per unit and a K of up to 1500 (12 x 8191 x 1025 5.5 / 4.9, 5.4 / 5.1, 7.1 / 5.8;
//    16 x 4096 x 513 4.5 / 4.2, 4.4 / 4.1, 5.6 / 4.5; 16 x 4096 x 2047 6.0 / 6.7, 5.9 / 7.1, 8.1 / 7.5; 16 x 16384 x 1025
//    5.6 / 7.3, 7.5 / 7.9, 9.0 / 8.0), and below 12 for two (9 x 16384 x 4097 14.4 / 15.3, 14.3 / 14.7, 19.5 / 15.6; 12 rows
//    15.0 / 18.0, 14.9 / 17.5, 20.4 / 18.5);
//  * a 32 x 32 tile per compute unit at most: 64 x 4096 x 4097 9.9 / 23.7, 32 x 4096 x 4097 9.8 / 18.5,
//    64 x 1024 x 1025 5.2 / 6.1;
//  * 32 x 64 tiles of two wavefronts: M <= 32 beyond that (16 x 32767 x 2047 14.4 / 19.4, 16 x 16384 x 4097 15.6 /
//    22.6), one per unit (128 x 4096 x 4097 13.8 / 23.8, 256 x 1025 x 1025 6.3 / 6.7), two per unit with a long K
//    (256 x 4096 x 4097 16.8 / 24.2, 48 x 16384 x 2049 12.0 / 14.6, but 200 x 4096 x 1001 8.1 / 6.8).
int wavek_areg_form(int64_t M, int64_t N, int64_t K, int64_t cus)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t t32 = tiles(32, 32);
    if (M <= 8 || (M <= 16 && K <= 1500 && t32 <= cus) || (M < 12 && t32 > cus && t32 <= 2 * cus)) return 0;
    if (t32 <= cus) return 11;
    if (M <= kSkinnyMaxM || tiles(32, 64) <= cus || (K >= 2048 && tiles(32, 64) <= 2 * cus)) return 12;
    return 0;
}

template <class F>
hipError_t launch_wavek_areg(const GemmParams &p, bool requant, bool rows, hipStream_t st)
{
    if (requant) return rows ? launch_wavek<F, 1, true, true, false, true>(p, st) : launch_wavek<F, 1, true, false, false, true>(p, st);
    return rows ? launch_wavek<F, 1, false, true, false, true>(p, st) : launch_wavek<F, 1, false, false, false, true>(p, st);
}

// Whether the 32 x 64 tiles wait for all of their loads in every other step.  A's steps are halves of 128-byte lines, and the other half is wanted by
// the tile's other wavefront a step later.  With two or three tiles to a unit and four steps of each on their way the vector cache has lost the line by then,
// and calls with a long K took up to 8 % longer than with half as many.  With one tile to a unit, and with a fourth of a unit's tiles in a round
// of their own, the deeper pipeline is worth more.  Averages of 6500 drawn calls, the kernel before this pipeline over (deep / waiting):
// 257 to 512 tiles, M <= 32: K = 2000 .. 3000 1.03 / 1.07, 4000 .. 8000 0.98 / 1.04, M > 32: 1.08 / 1.12, 1.01 / 1.07; 513 to 768: K = 2000 .. 3000
// 1.06 / 1.06, 3000 .. 4500 1.04 / 1.05; up to 256: 1.2-1.37 / 1.08-1.14; 769 to 1023: 1.17-1.22 / 1.12-1.15.  Below K = 2048 it is a tie.
bool wavek_areg_drains(int64_t M, int64_t N, int64_t K, int64_t cus)
{
    const int64_t t64 = ((M + 31) / 32) * ((N + 63) / 64);
    return t64 > cus && t64 <= 3 * cus && K >= 2048;
}

template <class F>
hipError_t launch_wavek_drain(const GemmParams &p, bool requant, bool rows, hipStream_t st)
{
    auto go = [&](auto kernel) {
        const int64_t tiles = ((int64_t)(p.M + F::TM * 32 - 1) / (F::TM * 32)) * ((p.N + F::TN * 32 - 1) / (F::TN * 32));
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(F::NW * 64), (WaveKCfg<F::TM, F::TN, F::NW, F::RING>::kLdsBytes), st, args_of(p));
        return hipGetLastError();
    };
    if (requant) return rows ? go(gemm_wavek_drain_kernel<F::TM, F::TN, F::NW, F::RING, true, true>) : go(gemm_wavek_drain_kernel<F::TM, F::TN, F::NW, F::RING, true, false>);
    return rows ? go(gemm_wavek_drain_kernel<F::TM, F::TN, F::NW, F::RING, false, true>) : go(gemm_wavek_drain_kernel<F::TM, F::TN, F::NW, F::RING, false, false>);
}

hipError_t launch_wavek_areg_form(int form, const GemmParams &p, bool requant, bool rows, int64_t cus, hipStream_t st)
{
    if (form == 11) return launch_wavek_areg<WaveK11>(p, requant, rows, st);
    return wavek_areg_drains(p.M, p.N, p.K, cus) ? launch_wavek_drain<WaveK12Short>(p, requant, rows, st) : launch_wavek_areg<WaveK12Short>(p, requant, rows, st);
}

// The forms with addresses of 64 bits: 32 x 32 and 32 x 64 tiles of four wavefronts (rows of any alignment: of two), which serve forms 1 and 22 as well; they
// form the row sums whether a zero-point needs them or not.  Instead of 64 x 128 tiles the kernels before run.
template <class F, int ELEM, bool REQUANT, bool BRAW = false, bool AREG = false>
hipError_t launch_wavek_far(const GemmParams &p, hipStream_t st, const RawB *rawb = nullptr)
{
    const int64_t tiles = ((int64_t)(p.M + F::TM * 32 - 1) / (F::TM * 32)) * ((p.N + F::TN * 32 - 1) / (F::TN * 32));
    hipLaunchKernelGGL((gemm_wavek_far_kernel<ELEM, F::TM, F::TN, F::NW, F::RING, REQUANT, BRAW, AREG>), dim3((unsigned)tiles), dim3(F::NW * 64),
                       (WaveKCfg<F::TM, F::TN, F::NW, F::RING>::kLdsBytes), st, rawb ? args_of_raw(p, *rawb) : args_of(p));
    return hipGetLastError();
}

template <class F, int ELEM, bool REQUANT, bool BRAW = false>
hipError_t allow_big_lds_wavek_far()
{
    return hipFuncSetAttribute((const void *)gemm_wavek_far_kernel<ELEM, F::TM, F::TN, F::NW, F::RING, REQUANT, BRAW, false>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, WaveKCfg<F::TM, F::TN, F::NW, F::RING>::kLdsBytes);
}

template <bool REQUANT, bool BRAW = false>
hipError_t launch_wavek_far_aligned(int form, const GemmParams &p, hipStream_t st, const RawB *rawb = nullptr)
{
    return form == 11 ? launch_wavek_far<WaveK11, 1, REQUANT, BRAW>(p, st, rawb) : launch_wavek_far<WaveK12, 1, REQUANT, BRAW>(p, st, rawb);
}

hipError_t launch_wavek_far_form(int form, const GemmParams &p, bool requant, bool aligned, hipStream_t st)
{
    if (aligned) return requant ? launch_wavek_far_aligned<true>(form, p, st) : launch_wavek_far_aligned<false>(form, p, st);
    if (form == 11) return requant ? launch_wavek_far<WaveK11, 1, true, false, true>(p, st) : launch_wavek_far<WaveK11, 1, false, false, true>(p, st);
    return requant ? launch_wavek_far<WaveK12Short, 1, true, false, true>(p, st) : launch_wavek_far<WaveK12Short, 1, false, false, true>(p, st);
}

// Whether a form's workgroups, one per tile, keep within a caller's cap (budget < cus).  Up to 32 rows they need not: the
// streaming kernels, in whose place they run there, launch a workgroup per panel as well.  (Form 0, none, has no tiles to count.)
bool wavek_fits(int form, int64_t M, int64_t N, int64_t budget, int64_t cus)
{
    if (form == 0 || budget >= cus || M <= kSkinnyMaxM) return true;
    const int64_t bm = form == 1 ? 32 : form / 10 * 32, bn = form == 1 ? 32 : form % 10 * 32;
    return ((M + bm - 1) / bm) * ((N + bn - 1) / bn) <= budget;
}

// The form that takes the place of `kernel` (the streaming kernel, 64 x 64 tiles, 128 x 128 tiles with aligned rows), or 0.
// budget: workgroups that the caller allows (the kernels for unaligned rows launch one per tile whichever runs).
int wavek_form_of(int kernel, int64_t M, int64_t N, int64_t K, bool aligned, bool rows, bool requant, int64_t cus, int64_t budget)
{
    const bool small = kernel == NGEMM_KERNEL_SKINNY || kernel == NGEMM_KERNEL_TILE_64;
    if (!aligned) return small ? wavek_areg_form(M, N, K, cus) : 0;
    const int form = small || kernel == NGEMM_KERNEL_TILE_128 ? wavek_form(M, N, K, rows, requant, cus) : 0;
    return (small || form == 24) && wavek_fits(form, M, N, budget, cus) ? form : 0;
}

// Forms of gemm_mid_kernel.
using Mid256 = MidCfg<4, 4, 2, 4, 6>;        // 128 x 256, eight wavefronts, 144 KiB of LDS: one workgroup per compute unit
using Mid192 = MidCfg<4, 6, 2, 2, 4>;        // 128 x 192, 80 KiB: two
using Mid128 = MidCfg<4, 4, 2, 2, 4>;        // 128 x 128, 64 KiB
using Mid64x192 = MidCfg<2, 6, 2, 2, 4>;     // 64 KiB
using Mid64x128 = MidCfg<2, 4, 2, 2, 6>;     // 72 KiB
struct MidGroup : MidCfg<2, 2, 2, 2, 4> { static constexpr int kPerCu = 4; };      // grouped launches

template <class C>
hipError_t launch_mid(const GemmParams &p0, bool requant, bool rows, bool aligned, hipStream_t st)
{
    GemmParams p = p0;
    p.tiles_m = (p.M + C::BM - 1) / C::BM;
    p.tiles_n = (p.N + C::BN - 1) / C::BN;
    const dim3 grid((unsigned)(p.tiles_m * p.tiles_n)), block(C::kThreads);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, C::kLdsBytes, st, args_of(p));
        return hipGetLastError();
    };
    if (aligned) {
        if (requant) return rows ? go(gemm_mid_kernel<C, true, true, false>) : go(gemm_mid_kernel<C, true, false, false>);
        return rows ? go(gemm_mid_kernel<C, false, true, false>) : go(gemm_mid_kernel<C, false, false, false>);
    }
    if (requant) return rows ? go(gemm_mid_kernel<C, true, true, true>) : go(gemm_mid_kernel<C, true, false, true>);
    return rows ? go(gemm_mid_kernel<C, false, true, true>) : go(gemm_mid_kernel<C, false, false, true>);
}

hipError_t launch_mid_form(int form, const GemmParams &p, bool requant, bool rows, bool aligned, hipStream_t st)
{
    switch (form) {
    case 1: return launch_mid<Mid64x128>(p, requant, rows, aligned, st);
    case 2: return launch_mid<Mid64x192>(p, requant, rows, aligned, st);
    case 3: return launch_mid<Mid128>(p, requant, rows, aligned, st);
    case 4: return launch_mid<Mid192>(p, requant, rows, aligned, st);
    default: return launch_mid<Mid256>(p, requant, rows, aligned, st);
    }
}

template <class C>
hipError_t allow_big_lds_mid()
{
    if (C::kLdsBytes <= 64 * 1024) return hipSuccess;
    const void *forms[] = {
        (const void *)gemm_mid_kernel<C, false, false, false>, (const void *)gemm_mid_kernel<C, false, true, false>,
        (const void *)gemm_mid_kernel<C, true, false, false>,  (const void *)gemm_mid_kernel<C, true, true, false>,
        (const void *)gemm_mid_kernel<C, false, false, true>,  (const void *)gemm_mid_kernel<C, false, true, true>,
        (const void *)gemm_mid_kernel<C, true, false, true>,   (const void *)gemm_mid_kernel<C, true, true, true>,
    };
    for (const void *f : forms) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Where another kernel stays although the lines of mid_form admit a problem.  90000 shapes were drawn around those lines and beyond the sizes that its
// model was fitted to (N from 16, M from 33), 7000 of them with every weight byte from memory as well as from cache; the lines lie where neither
// loses much.  us before / with gemm_mid_kernel; z: with a zero-point of B, whose row sums cost its forms more.
// In the place of 64 x 64 tiles (t of them per unit):
//  * N <= 64, a single column of them: never (28544 x 33 x 960 9.2 / 11.8, 16512 x 39 x 3328 16.6 / 18.8);
//  * M <= 64, which leaves half of a 128-row tile empty: from a K on that grows with t and z (without z beyond 768 0.99-1.18 x in cache, 1.09-1.2 x from
//    memory; with z, t = 1.5 .. 2, K up to 1024 0.89 and 1.03, up to 2304 0.92 and 1.15, beyond 0.99 and 1.14; unaligned 47 x 16896 x 1771
//    14.7 / 11.2, 47 x 45376 x 891 z 11.2 / 12.8); beyond t = 2 without z u8 outputs only (1.03-1.07 x, int32 0.93-1.01 x);
//  * z, t <= 2: beyond K = 1536 (2432 x 512 x 2112 12.3 / 11.5; K = 1536 itself 0.95 x);
//  * z, t <= 3: also from 769 on if K is no whole number of stages (1.05 x), u8 rows are whole tiles (1024 x 2560 x 832 10.0 / 9.1) or M <= 256 (in cache
//    1.0 x, from memory 1.09 x); else 2086 x 1359 x 768 10.1 / 12.0, 642 x 3659 x 960 10.4 / 11.1;
//  * z, t > 3, M > 256 (from memory 1.18 x): not for 256 < K <= 640 and columns that share 64-byte lines of C (0.90-1.02 x), nor K = 512 (0.96 x;
//    1757 x 1881 x 512 9.8 / 11.2); the rest 1.02-1.15 x (1885 x 1856 x 283 7.9 / 7.6, 2368 x 1425 x 832 13.0 / 11.8).
// In the place of 128 x 128 tiles:
//  * narrow u8 outputs, for which their epilogue skips the columns past N: not N <= 32 and, with z, N < 64, up to K = 1536 (38465 x 19 x 128 6.5 / 7.6,
//    55276 x 37 x 64 z 7.1 / 7.7; 63872 x 49 x 64 without z 7.8 / 7.2);
//  * unaligned rows, K < 1024: not N <= 64 nor, with z and up to three tiles per unit, N <= 128, but u8 rows of whole pieces (64128 x 40 x 98
//    7.9 / 9.3, 48289 x 128 x 397 z 12.2 / 14.9; 60416 x 64 x 108 u8 8.3 / 7.3; from 1024 on 67499 x 64 x 2653 82 / 73);
//  * z, int32 rows of whole lines, four to five such tiles per unit, whole stages: their third round of two is short (3826 x 5056 x 192 19.4 / 22.1).
// In the place of the larger tiles (t of 128 x 128 per unit):
//  * 192-row ones, int32 without z, N <= 128, t <= 1.5, K > 2048: a stream of A (33280 x 128 x 3392 39.7 / 52.0; beyond t = 1.5 1.18 x);
//  * wide short int32 outputs (N >= 8 M), K > 1024, 2 < t <= 3 (192 rows) or, z, 3 < t <= 4 (256 rows): the last round of two tiles per unit is short, and
//    from memory it waits (320 x 27686 x 1792 z from cache 29.4 / 35.1, from memory 33.1 / 44.4; on average 1.00 and 0.94 x).
bool mid_stays_out(int kernel, int64_t M, int64_t N, int64_t K, bool aligned, bool rows, bool requant, int64_t cus)
{
    const int64_t t64 = ((M + 63) / 64) * ((N + 63) / 64), t128 = ((M + 127) / 128) * ((N + 127) / 128);
    const bool whole = K % 64 == 0, above_1_5 = t64 * 2 > cus * 3;
    if (kernel == NGEMM_KERNEL_TILE_64) {
        if (N <= 64) return true;
        if (M <= 64) {
            if (rows) return K <= (aligned ? (above_1_5 ? 2304 : 1536) : above_1_5 ? 1024 : 768);
            if (t64 <= 2 * cus) return aligned && K <= 768;
            return aligned ? !(requant && (!whole || N % 16 == 0)) : K <= 1024;
        }
        if (!rows) return false;
        if (t64 > 3 * cus) return M > 256 && ((K > 256 && K <= 640 && N % 16 != 0) || K == 512);
        return K <= 1536 && !(t64 > 2 * cus && K > 768 && (!whole || M <= 256 || (requant && N % 64 == 0)));
    }
    if (kernel == NGEMM_KERNEL_TILE_128) {
        if (requant && K < 1536 && (N <= 32 || (rows && N < 64))) return true;
        if (!aligned) return K < 1024 && (N <= 64 || (rows && N <= 128 && t128 <= 3 * cus)) && !(requant && N % 64 == 0);
        return rows && !requant && whole && K > 64 && N % 16 == 0 && t128 > 4 * cus && t128 <= 5 * cus;
    }
    if (requant || (kernel != NGEMM_KERNEL_TILE_192 && kernel != NGEMM_KERNEL_TILE_256) || !aligned) return false;
    const bool t192 = kernel == NGEMM_KERNEL_TILE_192;
    if (N >= 8 * M && K > 1024 && (t192 ? t128 > 2 * cus && t128 <= 3 * cus : rows && t128 > 3 * cus && t128 <= 4 * cus)) return true;
    return t192 && !rows && N <= 128 && K > 2048 && t128 * 2 <= 3 * cus;
}

// The form of gemm_mid_kernel that serves an 8-bit problem in the place of the tiled kernels, or 0.  1420 shapes were timed with every
// form and with the kernels before (M from 64, N from 256, K up to 8192, odd sizes among them, aligned and unaligned rows, int32 and u8 outputs, with
// and without a zero-point of B):
//  * outputs of more than 0.55 x 128 x 128 tiles per compute unit: 1.17 x faster on average, unaligned rows 1.15 x; a K below 768 only from 0.8
//    tiles per unit on (1.08-1.16 x there; below it, K = 576 .. 767, 0.92-0.98 x with a zero-point of B, and without one 0.97-1.14 x, aligned rows
//    of no whole stages most: a line that could be drawn closer);
//  * from one 64 x 64 tile per unit on with a long K where the kernels before pay extra: row sums, u8 outputs, K of no whole stages,
//    unaligned rows (1.1 x; 1088 x 1413 x 2112 z 12.5 / 11.0).  Plain int32 problems there are a tie or a loss;
//  * less what mid_stays_out keeps.
// Which form: the least time by a model with constants (ns) that were fitted to those shapes; its choices are within 1.5 % of the best form on
// average, in all four combinations of output type and zero-point.  n tiles that a unit works through (rounds of resident workgroups counted whole)
// cost `stage` per stage and `tile` each, all the tiles together their share of the chip's (`flow`, `out`), a workgroup alone on its unit
// `lone_stage`, `lone` on top.
// `kernel`: what would run otherwise; the 256- and 192-row tiles, which read half the bytes per matrix op but take a row-sum launch and
// what is left behind an even number of stages apart, stay by a model of the same kind where it says that they are faster (4736 x 3072 x
// 768 19.2 us against 21.7, 4096 x 4096 x 1024 25.4 / 27.2, 2662 x 3521 x 2816 z 34.9 / 39.3).  NGEMM_KERNEL_AUTO: a measurement decides, not a comparison
// with what would run.
int mid_form(int kernel, int64_t M, int64_t N, int64_t K, int64_t lda, bool aligned, bool rows, bool requant, int64_t cus, int64_t budget)
{
    if (M <= kSkinnyMaxM || K < 64 || budget < cus) return 0;          // (a workgroup per tile: not under a caller's cap)
    if (!x64_offsets_fit(256, lda, K) || !x64_offsets_fit(9, 32 * round_up(K, 64), 0)) return 0;
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const bool plain = aligned && !rows && !requant && K % 64 == 0;
    if (!(tiles(128, 128) * 20 > cus * 11 && (K >= 768 || tiles(128, 128) * 5 > cus * 4)) && !(!plain && tiles(64, 64) > cus && K >= 1536)) return 0;
    if (mid_stays_out(kernel, M, N, K, aligned, rows, requant, cus)) return 0;
    struct Form {
        int id, bm, bn, per_cu;
        int64_t fixed, stage, tile, flow, out, lone_stage, lone;
    };
    constexpr Form forms[2][5] = {{{1, 64, 128, 2, 2650, 139, 1287, 38, 315, -10, 2084},
                                  {2, 64, 192, 2, 3002, 176, 1083, 38, 1132, 9, 1022},
                                  {3, 128, 128, 2, 2577, 192, 1841, 76, 822, 16, 1132},
                                  {4, 128, 192, 2, 2219, 257, 2758, 79, 1525, 14, 2067},
                                  {5, 128, 256, 1, 1793, 313, 4811, 189, 1919, 0, 0}},
                                 // rows of A through registers
                                 {{1, 64, 128, 2, 3485, 166, 1110, 39, 312, 22, 1600},
                                  {2, 64, 192, 2, 3371, 181, 2221, 70, -227, 43, 874},
                                  {3, 128, 128, 2, 2813, 261, 2873, 56, -99, 54, 1119},
                                  {4, 128, 192, 2, 2760, 375, 2079, 12, 2048, 41, 2773},
                                  {5, 128, 256, 1, 3345, 397, 3102, 90, 2557, 0, 0}}};
    int best = 0;
    int64_t least = 0;
    const int64_t nst = (K + 63) / 64;
    for (const Form &f : forms[aligned ? 0 : 1]) {
        const int64_t t = tiles(f.bm, f.bn), whole = t / (cus * f.per_cu), rest = t - whole * cus * f.per_cu;
        if (t * (f.id == 5 ? 512 : 256) >= (1ll << 32)) continue;         // (the runtime takes less than 2^32 threads in a launch)
        const int64_t n = whole * f.per_cu + (rest + cus - 1) / cus;
        const int64_t cost = f.fixed + n * (f.stage * nst + f.tile) + t * (f.flow * nst + f.out) / cus + (n == 1 ? f.lone_stage * nst + f.lone : 0);
        if (best == 0 || cost < least) {
            best = f.id;
            least = cost;
        }
    }
    if (aligned && (kernel == NGEMM_KERNEL_TILE_256 || kernel == NGEMM_KERNEL_TILE_192)) {
        const bool t256 = kernel == NGEMM_KERNEL_TILE_256;
        const int64_t t = tiles(t256 ? 256 : 192, 256), rounds = (t + cus - 1) / cus, odd = K % 128 != 0 ? rounds : 0;
        const int64_t large = t256 ? -2142 + rounds * (324 * nst + 12043) + t * (244 * nst + 4397) / cus + (rows ? 6211 : 0) + 5828 * odd
                                   : 3533 + rounds * (283 * nst + 5802) + t * (249 * nst + 3410) / cus + (rows ? 5391 : 0) + 2809 * odd;
        if (least * 100 > large * 93) return 0;
    }
    return best;
}

// The forms that read B from the caller's storage.
template <class F, bool ANY = false>                    // ANY: rows of any alignment
hipError_t launch_wavek_raw(const GemmParams &p, bool rows, const RawB &rawb, hipStream_t st)
{
    return rows ? launch_wavek<F, 1, false, true, true, ANY>(p, st, &rawb) : launch_wavek<F, 1, false, false, true, ANY>(p, st, &rawb);
}

hipError_t launch_wavek_raw_form(int form, const GemmParams &p, bool rows, const RawB &rawb, bool aligned, hipStream_t st)
{
    if (!aligned) return form == 11 ? launch_wavek_raw<WaveK11, true>(p, rows, rawb, st) : launch_wavek_raw<WaveK12Short, true>(p, rows, rawb, st);
    switch (form) {
    case 1: return launch_wavek_raw<WaveK11Short>(p, rows, rawb, st);
    case 11: return launch_wavek_raw<WaveK11>(p, rows, rawb, st);
    case 12: return launch_wavek_raw<WaveK12>(p, rows, rawb, st);
    case 24: return launch_wavek_raw<WaveK24>(p, rows, rawb, st);
    default: return launch_wavek_raw<WaveK22Long>(p, rows, rawb, st);
    }
}

// Unpacked B.  There is no long-pipeline form of the 64 x 64 kernel for it, so the 64 x 64 form serves a long K
// without row sums too (200 x 4096 x 4096 12.1 us against 17.4), and the other way for M <= 32 packs B first.
int wavek_raw_form(int64_t M, int64_t N, int64_t K, int64_t cus)
{
    const int form = wavek_form(M, N, K, true, false, cus);
    return form == 0 && M <= kSkinnyMaxM ? 12 : form;
}

// The same with rows of any alignment, both operands through registers; 0: a pack pass first, then the kernels for packed B.  us in a graph, packed
// first / so: 1 x 996 x 909 8.3 / 4.9, 16 x 2846 x 4103 19.9 / 11.7, 64 x 2126 x 1729 14.6 / 7.2,
// 221 x 314 x 328 9.4 / 4.4, 896 x 960 x 319 9.9 / 6.0.  Averages over 12400 drawn shapes with rows of an odd pitch: 2.1 x with K of up to 512,
// 2.0 up to 1024, 1.9 up to 2048, 1.6 beyond, and 1.6 to 3.1 for M <= 32 with many panels.  Where the lines lie:
//  * 32 x 32 tiles up to one per compute unit, and up to two with K <= 1024 (32 x 64 tiles there 1.6-1.9 x, these 1.9-2.2; with a longer K the former lead);
//  * more tiles than four of 32 x 32 per unit lose the pack pass's price to reading B once per 32 rows: K of up to 256 1.23 x, 512 1.09 (some 0.95),
//    then 0.9 and less; from three on K of up to 3072 1.2-1.5 x, beyond it 0.87-1.3;
//  * up to eight rows on a few tiles, K over 6144: 0.83-1.1 x, the K split over workgroups is worth the pass; over 8192 it was not measured for others.
int wavek_raw_any_form(int64_t M, int64_t N, int64_t K, int64_t cus)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t t32 = tiles(32, 32), t64 = tiles(32, 64);
    if (K > 8192 || (K > 6144 && M <= 8 && t32 <= 16)) return 0;
    if (t32 <= cus || (K <= 1024 && t32 <= 2 * cus)) return 11;
    if (M <= kSkinnyMaxM || t64 <= cus || (K <= 3072 && t64 <= 2 * cus) || (K <= 256 && t64 <= 4 * cus)) return 12;
    return 0;
}

struct RunArgs {
    int64_t M;
    const uint8_t *A;
    int64_t lda;
    int32_t za, zb;
    const ngemm_packed_b *B;
    void *C;
    int64_t ldc;
    bool requant;
    float scale;
    int32_t zc;
    // per-column epilogue (requantising calls only)
    const float *scale_vec = nullptr;
    const int32_t *bias_vec = nullptr;
    const int32_t *zb_vec = nullptr;
    int relu = 0;
    bool a_signed = false;    // A holds int8 (s8 x s8 variant); za then lies in [-128,127]
    bool b_unsigned = false;  // B was packed from uint8 (u8 x u8 variant); zb is then the caller's zero-point - 128
    bool needs_rowsum() const { return zb != 0 || zb_vec != nullptr; }
};

// What serves a call: one of NGEMM_KERNEL_*, and whether the kernels that have no number, the one that splits K over a
// workgroup's wavefronts and gemm_mid_kernel, may take its place where their rules have a form for the call.  They may for the automatic
// choice and for shapes whose tuning found them faster; a kernel that the caller asked for is the one that runs.
struct Route {
    int kernel;
    bool wavek;
    bool measured = false;    // by the tuner: the rules against `kernel` do not apply
};

ngemm_status validate_run(const ngemm_ctx *ctx, const RunArgs &a, Route *route)
{
    if (!ctx_ok(ctx) || !pack_ok(a.B)) return NGEMM_ERR_INVALID_ARG;
    if (a.B->device != ctx->device) return NGEMM_ERR_INVALID_ARG;
    if (a.M < 0 || a.M > kMaxDim) return NGEMM_ERR_BAD_SHAPE;
    if (a.a_signed ? (a.za < -128 || a.za > 127) : (a.za < 0 || a.za > 255)) return NGEMM_ERR_INVALID_ARG;
    if ((a.B->b_shift != 0) != a.b_unsigned) return NGEMM_ERR_INVALID_ARG;   // entry point and pack disagree
    if (a.B->elem_bytes != 1) return NGEMM_ERR_INVALID_ARG;                  // a 16-bit pack: ngemm_run_s16s16s32 only
    if (a.zb < -128 || a.zb > 127) return NGEMM_ERR_INVALID_ARG;   // of the packed (signed) bytes
    if (a.requant && !a.scale_vec) {
        if (!std::isfinite(a.scale) || a.scale < 0x1p-30f || a.scale > 0x1p30f) return NGEMM_ERR_INVALID_ARG;
    }
    if (a.M == 0 || a.B->N == 0) {
        *route = Route{NGEMM_KERNEL_AUTO, false};
        return NGEMM_OK;
    }
    if (!a.C || (!a.A && a.B->K > 0)) return NGEMM_ERR_INVALID_ARG;
    if (a.lda < a.B->K || a.ldc < a.B->N) return NGEMM_ERR_BAD_SHAPE;
    Route r{ctx->force_kernel, false};
    const int64_t cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    if (r.kernel == NGEMM_KERNEL_AUTO) {
        for (const ngemm_ctx::Tuned &t : ctx->tuned)
            if (t.M == a.M && t.N == a.B->N && t.K == a.B->K) {
                r = Route{t.kernel, false};
                const int small = a.M <= kSkinnyMaxM ? NGEMM_KERNEL_SKINNY : NGEMM_KERNEL_TILE_64;
                // (its rules look at the rows' alignment and at the zero-point, which another call may have otherwise)
                if (t.wavek && (wavek_form_of(small, a.M, a.B->N, a.B->K, rows_aligned(a.A, a.lda), a.needs_rowsum(), a.requant, cus, workgroup_budget(ctx)) != 0 ||
                                mid_form(NGEMM_KERNEL_AUTO, a.M, a.B->N, a.B->K, a.lda, rows_aligned(a.A, a.lda), a.needs_rowsum(), a.requant, cus,
                                         workgroup_budget(ctx)) != 0))
                    r = Route{small, true, true};
            }
        if (r.kernel == NGEMM_KERNEL_AUTO) r = Route{choose_kernel(ctx, a.M, a.B->N, a.B->K, rows_aligned(a.A, a.lda), a.requant), true};
    }
    if (r.kernel == NGEMM_KERNEL_SKINNY && a.M > kSkinnyMaxM) return NGEMM_ERR_INVALID_ARG;
    *route = r;
    return NGEMM_OK;
}

size_t rowsum_bytes(int64_t M) { return (size_t)round_up(M * 4, 256); }

// Kernel parameters of one validated GEMM (row sums not yet attached).
GemmParams make_params(const RunArgs &a, int nxcd)
{
    const ngemm_packed_b *B = a.B;
    GemmParams p;
    std::memset(&p, 0, sizeof p);
    p.A = a.A;
    p.lda = a.lda;
    p.Bp = B->data;
    p.C = a.C;
    p.ldc = a.ldc;
    p.M = (int)a.M;
    p.N = (int)B->N;
    p.K = (int)B->K;
    p.Kp = (int)B->Kp;
    p.npanels = (int)(B->Np / 32);
    const int32_t shift = a.a_signed ? 0 : 128;      // A' = A - shift is what the matrix pipe sees
    p.a_xor = a.a_signed ? 0u : 0x80808080u;
    p.za_term = (uint32_t)(shift - a.za);
    p.zb = (uint32_t)a.zb;
    p.scale = a.scale;
    p.zc = a.zc;
    p.scale_vec = a.scale_vec;
    p.bias_vec = a.bias_vec;
    p.zb_vec = a.zb_vec;
    p.relu = a.relu;
    p.ksplit = 1;
    p.kchunk = 0;
    p.nxcd = nxcd;
    return p;
}

// Launches one validated GEMM; `ws` must hold rowsum_bytes(M) when zb != 0.  What lies beyond those
// bytes serves the K split for its partial results when there is enough of it.
ngemm_status launch_run(const RunArgs &a, Route route, int num_cus, int device_cus, int nxcd, void *ws, size_t ws_bytes,
                        hipStream_t st)
{
    const ngemm_packed_b *B = a.B;
    if (a.M == 0 || B->N == 0) return NGEMM_OK;
    GemmParams p = make_params(a, nxcd);
    const bool dma_ok = rows_aligned(a.A, a.lda);
    int kernel = route.kernel;
    int kchunk = 0, parts = 1;
    int32_t *part_ws = nullptr;
    if (kernel == NGEMM_KERNEL_SPLIT_K) {
        // aligned rows of A only; u8 outputs need the workspace form and a zero-point of B per tensor;
        // what it cannot serve goes to the 64 x 64 tiles (to the streaming kernel when M <= 32)
        parts = dma_ok ? splitk_parts(a.M, B->N, B->K, num_cus, &kchunk) : 1;
        // int32 outputs always take the atomic form (never slower: 7.0 against 7.2 us for one tile,
        // 10.4 against 15.2 for 128 tiles at K = 4096); u8 outputs need the partial results in memory
        if (a.requant && parts >= 2 && ws && ws_bytes >= rowsum_bytes(a.M) + splitk_part_bytes(a.M, B->N, parts) && !a.zb_vec)
            part_ws = (int32_t *)((uint8_t *)ws + rowsum_bytes(a.M));
        if (a.requant && !part_ws) parts = 1;
        if (parts < 2) kernel = a.M <= kSkinnyMaxM ? NGEMM_KERNEL_SKINNY : NGEMM_KERNEL_TILE_64;
    }
    const bool rows_needed = a.needs_rowsum() && B->K > 0;
    // outputs of few tiles: K split over the wavefronts of a workgroup; of many: the kernel of tiles between those of the others
    if (route.wavek) {
        const int form = wavek_form_of(kernel, a.M, B->N, B->K, dma_ok, rows_needed, a.requant, device_cus, num_cus);
        const bool far = !wavek_offsets_fit(a.lda, B->K, B->Kp);
        if (form != 0 && !(far && form == 24)) {
            const hipError_t we = far ? launch_wavek_far_form(form, p, a.requant, dma_ok, st)
                                : dma_ok ? launch_wavek_form(form, p, a.requant, rows_needed, wavek_nt(a.M, B->N, B->K, device_cus), st)
                                         : launch_wavek_areg_form(form, p, a.requant, rows_needed, device_cus, st);
            return we == hipSuccess ? NGEMM_OK : NGEMM_ERR_DEVICE;
        }
        const int mid = kernel == NGEMM_KERNEL_SPLIT_K ? 0 : mid_form(route.measured ? NGEMM_KERNEL_AUTO : kernel, a.M, B->N, B->K, a.lda, dma_ok, rows_needed,
                                                                      a.requant, device_cus, num_cus);
        if (mid != 0) return launch_mid_form(mid, p, a.requant, rows_needed, dma_ok, st) == hipSuccess ? NGEMM_OK : NGEMM_ERR_DEVICE;
    }
    // at most one tile per compute unit and a K worth pipelining: the long-pipeline variants
    const bool deep64 = kernel == NGEMM_KERNEL_TILE_64 && dma_ok && B->K >= 512 &&
                        ((a.M + 63) / 64) * ((B->N + 63) / 64) <= (int64_t)device_cus;
    const bool deep128 = kernel == NGEMM_KERNEL_TILE_128 && dma_ok && B->K >= 512 &&
                         ((a.M + 127) / 128) * ((B->N + 127) / 128) <= (int64_t)device_cus;
    // the streaming kernel and every 64 x 64 and 128 x 128 kernel (the K split is one) form the row
    // sums themselves; the 256 x 256 kernels read them from a pass of their own
    const bool rows_in_kernel = kernel == NGEMM_KERNEL_SKINNY || kernel == NGEMM_KERNEL_SPLIT_K ||
                                kernel == NGEMM_KERNEL_TILE_64 || kernel == NGEMM_KERNEL_TILE_128;
    if (rows_needed && !rows_in_kernel) {
        int32_t *rs = (int32_t *)ws;
        hipLaunchKernelGGL(rowsum_a_kernel, dim3((unsigned)((a.M + 3) / 4)), dim3(256), 0, st, a.A, a.lda,
                           (int)a.M, (int)B->K, p.a_xor, rs);
        if (hipGetLastError() != hipSuccess) return NGEMM_ERR_DEVICE;
        p.rowsum = rs;
    }
    hipError_t e;
    if (kernel == NGEMM_KERNEL_SPLIT_K)
        return launch_tile_deep_splitk(p, parts, kchunk, rows_needed, a.requant, part_ws, num_cus, st) == hipSuccess ? NGEMM_OK
                                                                                                                : NGEMM_ERR_DEVICE;
    switch (kernel) {
    case NGEMM_KERNEL_SKINNY: e = launch_skinny(p, a.requant, num_cus, st); break;
    // direct-to-LDS copies need 16-byte aligned rows of A; the register-staged kernels take the rest
    case NGEMM_KERNEL_TILE_64:
        if (deep64)
            e = launch_tile_deep<1>(p, a.requant, rows_needed, num_cus, st);
        else
            e = dma_ok ? launch_tile_dma<64, 64, 2, 2>(p, a.requant, num_cus, st, nullptr, rows_needed)
                       : launch_tile<64, 64, 2, 2, 64>(p, a.requant, st, rows_needed);
        break;
    case NGEMM_KERNEL_TILE_128:
        if (deep128)
            e = launch_tile_deep<2>(p, a.requant, rows_needed, num_cus, st);
        else
            e = dma_ok ? launch_tile_dma<128, 128, 2, 2>(p, a.requant, num_cus, st, nullptr, rows_needed)
                       : launch_tile<128, 128, 2, 2, 64>(p, a.requant, st, rows_needed);
        break;
    case NGEMM_KERNEL_TILE_192:
    case NGEMM_KERNEL_TILE_256:
        if (dma_ok && B->K >= X64Cfg::kMinK && x64_offsets_fit(256, a.lda, B->K) && x64_offsets_fit(9, 32 * round_up(B->K, 64), 0)) {
            // the 16 x 16 x 64 form of the matrix instruction; 192 x 256 tiles on request
            const int trows = kernel == NGEMM_KERNEL_TILE_192 ? 192 : 256;
            p.tiles_m = (p.M + trows - 1) / trows;
            p.tiles_n = (p.N + 255) / 256;
            const int ntiles = p.tiles_m * p.tiles_n;
            const int nwg = ntiles < num_cus ? ntiles : num_cus;
            const dim3 grid((unsigned)nwg);
            const GemmArgs args = args_of(p, nwg);
            if (trows == 192) {
                if (a.requant)
                    hipLaunchKernelGGL((gemm_tile_x64_kernel<false, true, true, 6>), grid, dim3(256), X64Cfg::kLdsBytes, st, args);
                else
                    hipLaunchKernelGGL((gemm_tile_x64_kernel<false, false, true, 6>), grid, dim3(256), X64Cfg::kLdsBytes, st, args);
            } else if (a.requant)
                hipLaunchKernelGGL((gemm_tile_x64_kernel<false, true>), grid, dim3(256), X64Cfg::kLdsBytes, st, args);
            else if (a.a_signed)      // signed A: the form without the u8 -> s8 shift
                hipLaunchKernelGGL((gemm_tile_x64_kernel<false, false, false>), grid, dim3(256), X64Cfg::kLdsBytes, st, args);
            else
                hipLaunchKernelGGL((gemm_tile_x64_kernel<false, false>), grid, dim3(256), X64Cfg::kLdsBytes, st, args);
            e = hipGetLastError();
        } else {
            e = dma_ok ? launch_tile_dma<256, 256, 2, 2, kStages256>(p, a.requant, num_cus, st)
                       : launch_tile<256, 256, 2, 2, BK256>(p, a.requant, st);
        }
        break;
    default: return NGEMM_ERR_INVALID_ARG;
    }
    return e == hipSuccess ? NGEMM_OK : NGEMM_ERR_DEVICE;
}

// A validated call on a given kernel.
ngemm_status run_route(ngemm_ctx *ctx, const RunArgs &a, Route route, void *ws, size_t ws_bytes, void *stream)
{
    if (a.M == 0 || a.B->N == 0) return NGEMM_OK;
    if (a.needs_rowsum() && a.B->K > 0) {
        if (!ws) return NGEMM_ERR_INVALID_ARG;
        if (ws_bytes < rowsum_bytes(a.M)) return NGEMM_ERR_BUFFER_TOO_SMALL;
    }
    // the kernels read and write the workspace in 16-byte pieces
    if (ws && ws_bytes > 0 && ((uintptr_t)ws & 15u) != 0) return NGEMM_ERR_INVALID_ARG;
    DeviceGuard g(ctx->device);
    if (!g.ok) return NGEMM_ERR_DEVICE;
    return launch_run(a, route, workgroup_budget(ctx), ctx->num_cus > 0 ? ctx->num_cus : 256, ctx->num_xcd, ws, ws_bytes,
                      (hipStream_t)stream);
}

ngemm_status run_common(ngemm_ctx *ctx, const RunArgs &a, void *ws, size_t ws_bytes, void *stream)
{
    Route route;
    const ngemm_status s = validate_run(ctx, a, &route);
    return s == NGEMM_OK ? run_route(ctx, a, route, ws, ws_bytes, stream) : s;
}

}  // namespace

extern "C" {

const char *ngemm_status_string(ngemm_status s)
{
    switch (s) {
    case NGEMM_OK: return "ok";
    case NGEMM_ERR_INVALID_ARG: return "invalid argument";
    case NGEMM_ERR_BAD_SHAPE: return "bad shape or leading dimension";
    case NGEMM_ERR_BUFFER_TOO_SMALL: return "buffer too small";
    case NGEMM_ERR_DEVICE: return "HIP device error";
    case NGEMM_ERR_UNSUPPORTED_ARCH: return "unsupported architecture (gfx950 required)";
    case NGEMM_ERR_STATIC_LIMIT: return "problem exceeds the static scratch of the no-allocation entry point (M > 65536)";
    }
    return "unknown status";
}

ngemm_status ngemm_create(ngemm_ctx **out, int device_ordinal)
{
    if (!out) return NGEMM_ERR_INVALID_ARG;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || device_ordinal < 0 || device_ordinal >= count) {
        (void)hipGetLastError();
        return NGEMM_ERR_DEVICE;
    }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device_ordinal) != hipSuccess) return NGEMM_ERR_DEVICE;
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return NGEMM_ERR_UNSUPPORTED_ARCH;
    ngemm_ctx *c = new (std::nothrow) ngemm_ctx;
    if (!c) return NGEMM_ERR_DEVICE;
    c->magic = kCtxMagic;
    c->device = device_ordinal;
    c->num_cus = prop.multiProcessorCount;
    // XCDs: each has an L2 of its own, and consecutive workgroup ids are dispatched to them in turn
    int nxcc = 0;
    if (hipDeviceGetAttribute(&nxcc, hipDeviceAttributeNumberOfXccs, device_ordinal) != hipSuccess || nxcc < 1) {
        (void)hipGetLastError();
        nxcc = 8;                                    // the MI355X layout
    }
    c->num_xcd = nxcc;
    c->force_kernel = NGEMM_KERNEL_AUTO;
    c->max_workgroups = 0;
    {
        DeviceGuard g(device_ordinal);
        // this device's copy of the static scratch array (every device has its own, at its own address)
        void *sp = nullptr;
        if (!g.ok || hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)) != hipSuccess || !sp) {
            (void)hipGetLastError();
            delete c;
            return NGEMM_ERR_DEVICE;
        }
        c->static_scratch = sp;
        if (allow_big_lds<256, 256, 2, 2, BK256>() != hipSuccess ||
            allow_big_lds_dma<256, 256, 2, 2, kStages256>() != hipSuccess || allow_big_lds_dma<128, 128, 2, 2>() != hipSuccess ||
            allow_big_lds_dma<64, 64, 2, 2>() != hipSuccess || allow_big_lds_deep<1>() != hipSuccess || allow_big_lds_deep<2>() != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_tile_x64_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                X64Cfg::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_tile_x64_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                X64Cfg::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_tile_x64_kernel<false, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                X64Cfg::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_tile_x64_kernel<false, false, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                X64Cfg::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_tile_x64_kernel<false, false, true, 6>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                X64Cfg::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_tile_x64_kernel<false, true, true, 6>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                X64Cfg::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_s16_tile_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                S16Cfg::kLdsBytes) != hipSuccess ||
            hipFuncSetAttribute((const void *)gemm_s16_tile_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                S16Cfg::kLdsBytes) != hipSuccess ||
            allow_big_lds_wavek<WaveK12, 2, false, true>() != hipSuccess || allow_big_lds_wavek<WaveK22Long, 2, false, true>() != hipSuccess ||
            allow_big_lds_wavek_u8<WaveK12>() != hipSuccess || allow_big_lds_wavek_nt<WaveK12>() != hipSuccess || allow_big_lds_wavek_u8<WaveK22Long>() != hipSuccess || allow_big_lds_wavek_u8<WaveK24>() != hipSuccess ||
            allow_big_lds_wavek_far<WaveK12, 2, false>() != hipSuccess || allow_big_lds_wavek_far<WaveK12, 1, false>() != hipSuccess ||
            allow_big_lds_wavek_far<WaveK12, 1, true>() != hipSuccess || allow_big_lds_wavek_far<WaveK12, 1, false, true>() != hipSuccess ||
            allow_big_lds_mid<Mid256>() != hipSuccess || allow_big_lds_mid<Mid192>() != hipSuccess || allow_big_lds_mid<Mid128>() != hipSuccess ||
            allow_big_lds_mid<Mid64x192>() != hipSuccess || allow_big_lds_mid<Mid64x128>() != hipSuccess) {
            delete c;
            return NGEMM_ERR_DEVICE;
        }
    }
    *out = c;
    return NGEMM_OK;
}

ngemm_status ngemm_destroy(ngemm_ctx *ctx)
{
    if (!ctx) return NGEMM_OK;
    if (!ctx_ok(ctx)) return NGEMM_ERR_INVALID_ARG;
    ctx->magic = 0;
    delete ctx;
    return NGEMM_OK;
}

ngemm_status ngemm_set_kernel(ngemm_ctx *ctx, int kernel)
{
    if (!ctx_ok(ctx)) return NGEMM_ERR_INVALID_ARG;
    if (kernel < NGEMM_KERNEL_AUTO || kernel >= NGEMM_KERNEL_COUNT) return NGEMM_ERR_INVALID_ARG;
    ctx->force_kernel = kernel;
    return NGEMM_OK;
}

ngemm_status ngemm_tune_u8s8s32(ngemm_ctx *ctx, int64_t M, const uint8_t *A_dev, int64_t lda, int32_t a_zero_point,
                                const ngemm_packed_b *B, int32_t b_zero_point, int32_t *C_dev, int64_t ldc,
                                void *workspace_dev, size_t workspace_bytes, void *hip_stream, int *best_kernel)
{
    if (best_kernel) *best_kernel = NGEMM_KERNEL_AUTO;
    if (!ctx_ok(ctx) || !pack_ok(B)) return NGEMM_ERR_INVALID_ARG;
    RunArgs a{M, A_dev, lda, a_zero_point, b_zero_point, B, C_dev, ldc, false, 1.0f, 0};
    const int saved = ctx->force_kernel;
    Route checked;
    ctx->force_kernel = NGEMM_KERNEL_TILE_64;         // valid for every shape: checks the arguments
    ngemm_status s = validate_run(ctx, a, &checked);
    ctx->force_kernel = saved;
    if (s != NGEMM_OK) return s;
    if (M == 0 || B->N == 0 || B->K == 0) return NGEMM_OK;   // nothing to measure
    DeviceGuard g(ctx->device);
    if (!g.ok) return NGEMM_ERR_DEVICE;
    hipStream_t st = (hipStream_t)hip_stream;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return NGEMM_ERR_DEVICE;
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return NGEMM_ERR_DEVICE;
    }
    const bool dma_ok = rows_aligned(A_dev, lda);
    const int small = M <= kSkinnyMaxM ? NGEMM_KERNEL_SKINNY : NGEMM_KERNEL_TILE_64;
    // the last one: what the automatic choice puts in the place of the kernel for small outputs (gemm_wavek_kernel, gemm_mid_kernel)
    const Route candidates[7] = {{NGEMM_KERNEL_SKINNY, false}, {NGEMM_KERNEL_TILE_64, false}, {NGEMM_KERNEL_TILE_128, false},
                                 {NGEMM_KERNEL_TILE_256, false}, {NGEMM_KERNEL_SPLIT_K, false}, {NGEMM_KERNEL_TILE_192, false},
                                 {small, true, true}};
    int best = NGEMM_KERNEL_AUTO;
    bool best_wavek = false;
    float best_ms = 0.0f;
    s = NGEMM_OK;
    for (int c = 0; c < 7 && s == NGEMM_OK; ++c) {
        const int k = candidates[c].kernel;
        if (k == NGEMM_KERNEL_SKINNY && M > kSkinnyMaxM) continue;
        // a tile far larger than the output cannot win: skip what would leave most of it empty
        if ((k == NGEMM_KERNEL_TILE_256 || k == NGEMM_KERNEL_TILE_192) && (M <= 64 || B->N <= 64)) continue;
        if (k == NGEMM_KERNEL_SPLIT_K) {
            // only where it would really split (else it is the 64 x 64 candidate once more)
            int kchunk = 0;
            if (!dma_ok || splitk_parts(M, B->N, B->K, workgroup_budget(ctx), &kchunk) < 2) continue;
        }
        const int64_t cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
        if (candidates[c].wavek && wavek_form_of(k, M, B->N, B->K, dma_ok, b_zero_point != 0, false, cus, workgroup_budget(ctx)) == 0 &&
            mid_form(NGEMM_KERNEL_AUTO, M, B->N, B->K, lda, dma_ok, b_zero_point != 0, false, cus, workgroup_budget(ctx)) == 0) continue;
        // three rounds of 50 launches after a warm-up, the fastest round counts: short kernels are
        // within the noise of one another otherwise (clock ramp, first-touch effects)
        const int warm = 5, reps = 50, rounds = 3;
        float ms = 0.0f;
        for (int round = 0; round < rounds && s == NGEMM_OK; ++round) {
            for (int r = (round == 0 ? 0 : warm); r < warm + reps && s == NGEMM_OK; ++r) {
                if (r == warm && hipEventRecord(e0, st) != hipSuccess) s = NGEMM_ERR_DEVICE;
                if (s == NGEMM_OK) s = run_route(ctx, a, candidates[c], workspace_dev, workspace_bytes, hip_stream);
            }
            float t = 0.0f;
            if (s == NGEMM_OK && (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                                  hipEventElapsedTime(&t, e0, e1) != hipSuccess))
                s = NGEMM_ERR_DEVICE;
            if (round == 0 || t < ms) ms = t;
        }
        if (s == NGEMM_OK && (best == NGEMM_KERNEL_AUTO || ms < best_ms)) {
            if (candidates[c].wavek) best_wavek = true;      // `best` stays the fastest that a caller can force
            else best = k;
            best_ms = ms;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (s != NGEMM_OK) return s;
    bool found = false;
    for (ngemm_ctx::Tuned &t : ctx->tuned)
        if (t.M == M && t.N == B->N && t.K == B->K) {
            t.kernel = best;
            t.wavek = best_wavek;
            found = true;
        }
    if (!found) {
        try {
            if (ctx->tuned.size() >= 4096) ctx->tuned.erase(ctx->tuned.begin());
            ctx->tuned.push_back(ngemm_ctx::Tuned{M, B->N, B->K, best, best_wavek});
        } catch (...) {
            return NGEMM_ERR_DEVICE;               // out of host memory: measured, but not remembered
        }
    }
    if (best_kernel) *best_kernel = best;
    return NGEMM_OK;
}

ngemm_status ngemm_tuned_kernel(const ngemm_ctx *ctx, int64_t M, int64_t N, int64_t K, int *kernel)
{
    if (!ctx_ok(ctx) || !kernel) return NGEMM_ERR_INVALID_ARG;
    *kernel = NGEMM_KERNEL_AUTO;
    for (const ngemm_ctx::Tuned &t : ctx->tuned)
        if (t.M == M && t.N == N && t.K == K) *kernel = t.kernel;
    return NGEMM_OK;
}

ngemm_status ngemm_set_max_workgroups(ngemm_ctx *ctx, int max_workgroups)
{
    if (!ctx_ok(ctx) || max_workgroups < 0) return NGEMM_ERR_INVALID_ARG;
    ctx->max_workgroups = max_workgroups;
    return NGEMM_OK;
}

size_t ngemm_packed_b_bytes(int64_t K, int64_t N)
{
    if (K < 0 || N < 0 || K > kMaxDim || N > kMaxDim) return 0;
    const int64_t Kp = round_up(K, 64), Np = round_up(N, 32);
    return (size_t)(Kp * Np + 4 * Np);
}

static ngemm_status pack_common(ngemm_ctx *ctx, int64_t K, int64_t N, const int8_t *B_dev, int64_t ldb,
                                void *packed_dev, size_t packed_bytes, void *hip_stream, ngemm_packed_b **out,
                                int32_t b_shift)
{
    if (!out) return NGEMM_ERR_INVALID_ARG;
    *out = nullptr;
    if (!ctx_ok(ctx)) return NGEMM_ERR_INVALID_ARG;
    if (K < 0 || N < 0 || K > kMaxDim || N > kMaxDim) return NGEMM_ERR_BAD_SHAPE;
    if (K > 0 && N > 0 && (!B_dev || ldb < K)) return B_dev ? NGEMM_ERR_BAD_SHAPE : NGEMM_ERR_INVALID_ARG;
    const size_t need = ngemm_packed_b_bytes(K, N);
    if (need > 0 && !packed_dev) return NGEMM_ERR_INVALID_ARG;
    if (packed_bytes < need) return NGEMM_ERR_BUFFER_TOO_SMALL;
    if (((uintptr_t)packed_dev & 15u) != 0) return NGEMM_ERR_INVALID_ARG;
    const int64_t Kp = round_up(K, 64), Np = round_up(N, 32);

    ngemm_packed_b *d = new (std::nothrow) ngemm_packed_b;
    if (!d) return NGEMM_ERR_DEVICE;
    d->magic = kPackMagic;
    d->device = ctx->device;
    d->K = K; d->N = N; d->Kp = Kp; d->Np = Np;
    d->data = (const uint8_t *)packed_dev;
    d->bytes = need;
    d->b_shift = b_shift;
    d->elem_bytes = 1;

    if (Np > 0) {
        DeviceGuard g(ctx->device);
        if (!g.ok) { delete d; return NGEMM_ERR_DEVICE; }
        hipStream_t st = (hipStream_t)hip_stream;
        int32_t *colsum = (int32_t *)((uint8_t *)packed_dev + Kp * Np);
        const ngemm_status ls = launch_pack<1>((const uint8_t *)B_dev, ldb, K, N, Kp, Np, b_shift ? 0x80808080u : 0u,
                                               (uint8_t *)packed_dev, colsum, st);
        if (ls != NGEMM_OK) { delete d; return ls; }
    }
    *out = d;
    return NGEMM_OK;
}

ngemm_status ngemm_pack_b(ngemm_ctx *ctx, int64_t K, int64_t N, const int8_t *B_dev, int64_t ldb,
                          void *packed_dev, size_t packed_bytes, void *hip_stream, ngemm_packed_b **out)
{
    return pack_common(ctx, K, N, B_dev, ldb, packed_dev, packed_bytes, hip_stream, out, 0);
}

ngemm_status ngemm_pack_b_u8(ngemm_ctx *ctx, int64_t K, int64_t N, const uint8_t *B_dev, int64_t ldb,
                             void *packed_dev, size_t packed_bytes, void *hip_stream, ngemm_packed_b **out)
{
    return pack_common(ctx, K, N, (const int8_t *)B_dev, ldb, packed_dev, packed_bytes, hip_stream, out, 128);
}

ngemm_status ngemm_packed_b_free(ngemm_packed_b *b)
{
    if (!b) return NGEMM_OK;
    if (!pack_ok(b)) return NGEMM_ERR_INVALID_ARG;
    b->magic = 0;
    delete b;
    return NGEMM_OK;
}

ngemm_status ngemm_packed_b_shape(const ngemm_packed_b *b, int64_t *K, int64_t *N)
{
    if (!pack_ok(b) || !K || !N) return NGEMM_ERR_INVALID_ARG;
    *K = b->K;
    *N = b->N;
    return NGEMM_OK;
}

size_t ngemm_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    if (M <= 0 || M > kMaxDim) return 0;
    size_t bytes = rowsum_bytes(M);
    // room for the partial results of the K split (outputs of few tiles with a long K: at most 4 MiB)
    if (N > 0 && N <= kMaxDim && K > 0 && K <= kMaxDim) {
        int kchunk = 0;
        const int parts = splitk_parts(M, N, K, kSplitMaxUnits, &kchunk);
        if (parts >= 2) bytes += splitk_part_bytes(M, N, parts);
    }
    return bytes;
}

ngemm_status ngemm_run_u8s8s32(ngemm_ctx *ctx, int64_t M, const uint8_t *A_dev, int64_t lda, int32_t a_zero_point,
                               const ngemm_packed_b *B, int32_t b_zero_point, int32_t *C_dev, int64_t ldc,
                               void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    RunArgs a{M, A_dev, lda, a_zero_point, b_zero_point, B, C_dev, ldc, false, 1.0f, 0};
    return run_common(ctx, a, workspace_dev, workspace_bytes, hip_stream);
}

ngemm_status ngemm_run_u8s8s32_static(ngemm_ctx *ctx, int64_t M, const uint8_t *A_dev, int64_t lda, int32_t a_zero_point,
                                      const ngemm_packed_b *B, int32_t b_zero_point, int32_t *C_dev, int64_t ldc,
                                      void *hip_stream)
{
    if (!ctx_ok(ctx)) return NGEMM_ERR_INVALID_ARG;
    if (M > kStaticMaxM) return NGEMM_ERR_STATIC_LIMIT;
    // ngemm_run_u8s8s32 with the row sums in this device's static array (its address, taken at
    // ngemm_create; never the symbol).  The kernel that forms them writes all M entries before
    // the GEMM kernel behind it on the stream reads them, so nothing needs clearing; room for a K
    // split's partial results is not offered (int32 outputs add their parts into C).
    RunArgs a{M, A_dev, lda, a_zero_point, b_zero_point, B, C_dev, ldc, false, 1.0f, 0};
    return run_common(ctx, a, ctx->static_scratch, kStaticScratchBytes, hip_stream);
}

ngemm_status ngemm_run_s8s8s32(ngemm_ctx *ctx, int64_t M, const int8_t *A_dev, int64_t lda, int32_t a_zero_point,
                               const ngemm_packed_b *B, int32_t b_zero_point, int32_t *C_dev, int64_t ldc,
                               void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    RunArgs a{M, (const uint8_t *)A_dev, lda, a_zero_point, b_zero_point, B, C_dev, ldc, false, 1.0f, 0};
    a.a_signed = true;
    return run_common(ctx, a, workspace_dev, workspace_bytes, hip_stream);
}

ngemm_status ngemm_run_u8u8s32(ngemm_ctx *ctx, int64_t M, const uint8_t *A_dev, int64_t lda, int32_t a_zero_point,
                               const ngemm_packed_b *B, int32_t b_zero_point, int32_t *C_dev, int64_t ldc,
                               void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    // (B - zb) == (B - 128) - (zb - 128): the packed bytes are already B - 128
    if (b_zero_point < 0 || b_zero_point > 255) return NGEMM_ERR_INVALID_ARG;
    RunArgs a{M, A_dev, lda, a_zero_point, b_zero_point - 128, B, C_dev, ldc, false, 1.0f, 0};
    a.b_unsigned = true;
    return run_common(ctx, a, workspace_dev, workspace_bytes, hip_stream);
}

ngemm_status ngemm_run_u8s8u8_requant(ngemm_ctx *ctx, int64_t M, const uint8_t *A_dev, int64_t lda,
                                      int32_t a_zero_point, const ngemm_packed_b *B, int32_t b_zero_point,
                                      float scale, int32_t c_zero_point, uint8_t *C_dev, int64_t ldc,
                                      void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    RunArgs a{M, A_dev, lda, a_zero_point, b_zero_point, B, C_dev, ldc, true, scale, c_zero_point};
    return run_common(ctx, a, workspace_dev, workspace_bytes, hip_stream);
}

ngemm_status ngemm_run_u8s8u8_requant_channel(ngemm_ctx *ctx, int64_t M, const uint8_t *A_dev, int64_t lda,
                                              int32_t a_zero_point, const ngemm_packed_b *B, int32_t b_zero_point,
                                              const int32_t *b_zero_points_dev, const float *scales_dev,
                                              const int32_t *bias_dev, int32_t relu, int32_t c_zero_point,
                                              uint8_t *C_dev, int64_t ldc, void *workspace_dev,
                                              size_t workspace_bytes, void *hip_stream)
{
    if (!scales_dev) return NGEMM_ERR_INVALID_ARG;
    RunArgs a{M, A_dev, lda, a_zero_point, b_zero_point, B, C_dev, ldc, true, 1.0f, c_zero_point};
    a.scale_vec = scales_dev;
    a.bias_vec = bias_dev;
    a.zb_vec = b_zero_points_dev;
    a.relu = relu ? 1 : 0;
    return run_common(ctx, a, workspace_dev, workspace_bytes, hip_stream);
}

size_t ngemm_packed_b_bytes_s16(int64_t K, int64_t N)
{
    if (K < 0 || N < 0 || K > kMaxDim / 2 || N > kMaxDim) return 0;
    const int64_t Kp = 2 * round_up(K, 32), Np = round_up(N, 32);
    return (size_t)(Kp * Np + 4 * Np);
}

ngemm_status ngemm_pack_b_s16(ngemm_ctx *ctx, int64_t K, int64_t N, const int16_t *B_dev, int64_t ldb,
                              void *packed_dev, size_t packed_bytes, void *hip_stream, ngemm_packed_b **out)
{
    if (!out) return NGEMM_ERR_INVALID_ARG;
    *out = nullptr;
    if (!ctx_ok(ctx)) return NGEMM_ERR_INVALID_ARG;
    if (K < 0 || N < 0 || K > kMaxDim / 2 || N > kMaxDim) return NGEMM_ERR_BAD_SHAPE;
    if (K > 0 && N > 0 && (!B_dev || ldb < K)) return B_dev ? NGEMM_ERR_BAD_SHAPE : NGEMM_ERR_INVALID_ARG;
    if (((uintptr_t)B_dev & 1u) != 0) return NGEMM_ERR_INVALID_ARG;
    const size_t need = ngemm_packed_b_bytes_s16(K, N);
    if (need > 0 && !packed_dev) return NGEMM_ERR_INVALID_ARG;
    if (packed_bytes < need) return NGEMM_ERR_BUFFER_TOO_SMALL;
    if (((uintptr_t)packed_dev & 15u) != 0) return NGEMM_ERR_INVALID_ARG;
    const int64_t Kp = 2 * round_up(K, 32), Np = round_up(N, 32);
    ngemm_packed_b *d = new (std::nothrow) ngemm_packed_b;
    if (!d) return NGEMM_ERR_DEVICE;
    d->magic = kPackMagic;
    d->device = ctx->device;
    d->K = K; d->N = N; d->Kp = Kp; d->Np = Np;
    d->data = (const uint8_t *)packed_dev;
    d->bytes = need;
    d->b_shift = 0;
    d->elem_bytes = 2;
    if (Np > 0) {
        DeviceGuard g(ctx->device);
        if (!g.ok) { delete d; return NGEMM_ERR_DEVICE; }
        hipStream_t st = (hipStream_t)hip_stream;
        int32_t *colsum = (int32_t *)((uint8_t *)packed_dev + Kp * Np);
        const ngemm_status ls = launch_pack<2>((const uint8_t *)B_dev, 2 * ldb, 2 * K, N, Kp, Np, 0u, (uint8_t *)packed_dev, colsum, st);
        if (ls != NGEMM_OK) { delete d; return ls; }
    }
    *out = d;
    return NGEMM_OK;
}

ngemm_status ngemm_run_s16s16s32(ngemm_ctx *ctx, int64_t M, const int16_t *A_dev, int64_t lda, int32_t a_zero_point,
                                 const ngemm_packed_b *B, int32_t b_zero_point, int32_t *C_dev, int64_t ldc,
                                 void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    if (!ctx_ok(ctx) || !pack_ok(B) || B->elem_bytes != 2 || B->device != ctx->device) return NGEMM_ERR_INVALID_ARG;
    if (M < 0 || M > kMaxDim) return NGEMM_ERR_BAD_SHAPE;
    if (a_zero_point < -32768 || a_zero_point > 32767 || b_zero_point < -32768 || b_zero_point > 32767)
        return NGEMM_ERR_INVALID_ARG;
    if (M == 0 || B->N == 0) return NGEMM_OK;
    if (!C_dev || (!A_dev && B->K > 0)) return NGEMM_ERR_INVALID_ARG;
    if (lda < B->K || ldc < B->N) return NGEMM_ERR_BAD_SHAPE;
    // the kernel copies rows of A straight into LDS in 16-byte pieces
    if ((((uintptr_t)A_dev | (uintptr_t)(lda * 2)) & 15) != 0) return NGEMM_ERR_INVALID_ARG;
    if (B->K > 0) {
        if (!workspace_dev) return NGEMM_ERR_INVALID_ARG;
        if (workspace_bytes < rowsum_bytes(M)) return NGEMM_ERR_BUFFER_TOO_SMALL;
    }
    DeviceGuard g(ctx->device);
    if (!g.ok) return NGEMM_ERR_DEVICE;
    hipStream_t st = (hipStream_t)hip_stream;
    GemmParams p;
    std::memset(&p, 0, sizeof p);
    p.A = (const uint8_t *)A_dev;
    p.lda = lda * 2;
    p.Bp = B->data;
    p.C = C_dev;
    p.ldc = ldc;
    p.M = (int)M; p.N = (int)B->N; p.K = (int)B->K; p.Kp = (int)B->Kp;
    p.npanels = (int)(B->Np / 32);
    // sum (a-za)(b-zb) = sum (a-128)(b-128) + (128-za) colsum'[j] - (zb-128) rowsum'[i] - (zb-128)(128-za) K
    p.za_term = (uint32_t)(128 - a_zero_point);
    p.zb = (uint32_t)(b_zero_point - 128);
    p.nxcd = ctx->num_xcd;
    // Small outputs run the kernel that splits K over a workgroup's wavefronts (no row-sum launch, tiles small
    // enough to spread over the compute units): 32 x 32 tiles while there is a compute unit for each, 32 x 64 up
    // to two per unit, 64 x 64 up to two per unit while 128 x 128 tiles would fill less than half of the units;
    // larger ones, and what a K of less than two stages leaves to them, the 128 x 128 kernel.  us, against the
    // 128 x 128 kernel: 16 x 4096 x 4096 8.5 / 45.6, 64 x 4096 x 4096 11.1 / 46.0, 512 x 768 x 768 5.8 / 15.0,
    // 1024^3 9.8 / 17.6, 512 x 3072 x 768 11.5 / 15.4, 1024 x 2048 x 1024 14.0 / 17.8, but 1024 x 3072 x 1024
    // 24.8 / 19.6 and 1536^3 27 / 24.9.  From K = 2048 on 64 x 64 tiles of four wavefronts, one per unit at most, in the place of two of 32 x 64: 1.06 x up to
    // K = 3072, 1.11 beyond (303 x 2046 x 3824 22.1 / 19.1), from memory the same; at 1536 0.97.
    // Under a caller's cap only those whose workgroups, one per tile, keep within it; the 128 x 128 kernel and, below its K,
    // the looping form walk several tiles per workgroup.
    const int64_t cus = ctx->num_cus > 0 ? ctx->num_cus : 256, budget = workgroup_budget(ctx);
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((B->N + bn - 1) / bn); };
    const bool near = wavek_offsets_fit(p.lda, 2 * B->K, B->Kp);       // else the forms with addresses of 64 bits, the looping one for 64 x 64 tiles
    auto fits = [&](int64_t n) { return budget >= cus || n <= budget; };
    hipError_t e;
    if (tiles(32, 32) <= cus && fits(tiles(32, 32))) {
        e = near ? launch_wavek<WaveK11, 2, false, true>(p, st) : launch_wavek_far<WaveK11, 2, false>(p, st);
    } else if (near && tiles(32, 64) > cus && tiles(64, 64) <= cus && B->K >= 2048 && fits(tiles(64, 64))) {
        e = launch_wavek<WaveK22Long, 2, false, true>(p, st);
    } else if (tiles(32, 64) <= 2 * cus && fits(tiles(32, 64))) {
        e = near ? launch_wavek<WaveK12, 2, false, true>(p, st) : launch_wavek_far<WaveK12, 2, false>(p, st);
    } else if ((B->K < S16Cfg::kMinK && (!near || !fits(tiles(64, 64)))) ||
               (!near && tiles(64, 64) <= 2 * cus && tiles(128, 128) * 2 <= cus && fits(tiles(64, 64)))) {
        p.tiles_m = (int)((M + 63) / 64);
        p.tiles_n = (int)((B->N + 63) / 64);
        const int64_t most = budget >= cus ? 2 * cus : budget, nwg = tiles(64, 64) < most ? tiles(64, 64) : most;      // (two to a unit)
        hipLaunchKernelGGL((gemm_wavek_kernel<2, 2, 2, WaveK22::NW, WaveK22::RING, false, true, false, false, false, true>), dim3((unsigned)nwg),
                           dim3(WaveK22::NW * 64), (WaveKCfg<2, 2, WaveK22::NW, WaveK22::RING>::kLdsBytes), st, args_of(p, (int)nwg));
        e = hipGetLastError();
    } else if (B->K < S16Cfg::kMinK || (tiles(64, 64) <= 2 * cus && tiles(128, 128) * 2 <= cus && fits(tiles(64, 64)))) {
        e = launch_wavek<WaveK22, 2, false, true>(p, st);
    } else {
        p.tiles_m = (int)((M + 127) / 128);
        p.tiles_n = (int)((B->N + 127) / 128);
        const int64_t ntiles = (int64_t)p.tiles_m * p.tiles_n, grid = ntiles < budget ? ntiles : budget;
        // The row sums: in the kernel while that costs clearly less (40 ns per stage, 0.14 us per tile) than a launch of their own (2.3 us and 0.12 per
        // MB of A).  3800 drawn shapes, launch over kernel: up to 8 stages per unit 1.10-1.16 x, 32 1.03, 40 1.025 (0.976 at worst, many short tiles),
        // 64 1.01, 80 1.006, beyond 100 0.99.
        if ((ntiles + grid - 1) / grid * ((B->K + 63) / 64) <= 40) {
            hipLaunchKernelGGL(gemm_s16_tile_kernel<true>, dim3((unsigned)grid), dim3(256), S16Cfg::kLdsBytes, st, args_of(p, (int)grid));
        } else {
            int32_t *rs = (int32_t *)workspace_dev;
            hipLaunchKernelGGL(rowsum_s16_kernel, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, st, A_dev, lda, (int)M, (int)B->K, rs);
            if (hipGetLastError() != hipSuccess) return NGEMM_ERR_DEVICE;
            p.rowsum = rs;
            hipLaunchKernelGGL(gemm_s16_tile_kernel<false>, dim3((unsigned)grid), dim3(256), S16Cfg::kLdsBytes, st, args_of(p, (int)grid));
        }
        e = hipGetLastError();
    }
    return e == hipSuccess ? NGEMM_OK : NGEMM_ERR_DEVICE;
}

size_t ngemm_unpacked_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    if (M < 0 || N < 0 || K < 0 || M > kMaxDim || N > kMaxDim || K > kMaxDim) return 0;
    return (size_t)round_up((int64_t)ngemm_packed_b_bytes(K, N), 256) + rowsum_bytes(M > 0 ? M : 1);
}

ngemm_status ngemm_run_u8s8s32_unpacked(ngemm_ctx *ctx, int64_t M, int64_t N, int64_t K, const uint8_t *A_dev,
                                        int64_t lda, int32_t a_zero_point, const int8_t *B_dev, int64_t ldb,
                                        int32_t b_zero_point, int32_t *C_dev, int64_t ldc, void *workspace_dev,
                                        size_t workspace_bytes, void *hip_stream)
{
    if (!ctx_ok(ctx)) return NGEMM_ERR_INVALID_ARG;
    if (M < 0 || N < 0 || K < 0 || M > kMaxDim || N > kMaxDim || K > kMaxDim) return NGEMM_ERR_BAD_SHAPE;
    if (a_zero_point < 0 || a_zero_point > 255 || b_zero_point < -128 || b_zero_point > 127)
        return NGEMM_ERR_INVALID_ARG;
    if (M == 0 || N == 0) return NGEMM_OK;
    if (!C_dev || (K > 0 && (!A_dev || !B_dev))) return NGEMM_ERR_INVALID_ARG;
    if (lda < K || ldb < K || ldc < N) return NGEMM_ERR_BAD_SHAPE;
    if (!workspace_dev || ((uintptr_t)workspace_dev & 15u) != 0) return NGEMM_ERR_INVALID_ARG;
    if (workspace_bytes < ngemm_unpacked_workspace_bytes(M, N, K)) return NGEMM_ERR_BUFFER_TOO_SMALL;
    // Rows of both operands 16-byte aligned: no pack pass.  The kernels read B from the caller's storage with the
    // same copies as A; all but the 256 x 256 ones form the sums of its columns themselves.  Other rows: none either for
    // small outputs, where one kernel takes both operands through registers.
    int kernel = ctx->force_kernel == NGEMM_KERNEL_AUTO ? choose_kernel(ctx, M, N, K, rows_aligned(A_dev, lda), false) : ctx->force_kernel;
    if (kernel == NGEMM_KERNEL_SPLIT_K)                                     // the K split reads a packed B only
        kernel = M <= kSkinnyMaxM ? NGEMM_KERNEL_SKINNY : NGEMM_KERNEL_TILE_64;
    const bool aligned = (((uintptr_t)A_dev | (uintptr_t)lda | (uintptr_t)B_dev | (uintptr_t)ldb) & 15) == 0;
    const int64_t cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    const bool small_kernel = kernel == NGEMM_KERNEL_TILE_64 || kernel == NGEMM_KERNEL_TILE_128 || kernel == NGEMM_KERNEL_SKINNY;
    // the kernel that splits K over a workgroup's wavefronts: of the automatic choice only
    int form = K == 0 || !small_kernel || ctx->force_kernel != NGEMM_KERNEL_AUTO ? 0
               : aligned ? wavek_raw_form(M, N, K, cus) : wavek_raw_any_form(M, N, K, cus);
    const bool near = wavek_offsets_fit(lda, K, 0, ldb);
    if ((kernel == NGEMM_KERNEL_TILE_128 && form != 24) || !wavek_fits(form, M, N, workgroup_budget(ctx), cus) || (!near && (!aligned || form == 24))) form = 0;
    if (form != 0 || (aligned && K > 0 && kernel != NGEMM_KERNEL_SKINNY)) {
        DeviceGuard g(ctx->device);
        if (!g.ok) return NGEMM_ERR_DEVICE;
        hipStream_t st = (hipStream_t)hip_stream;
        ngemm_packed_b shape;                         // sizes only: nothing is packed
        shape.magic = kPackMagic; shape.device = ctx->device;
        shape.K = K; shape.N = N; shape.Kp = round_up(K, 64); shape.Np = round_up(N, 32);
        shape.data = nullptr; shape.bytes = 0; shape.b_shift = 0; shape.elem_bytes = 1;
        RunArgs a{M, A_dev, lda, a_zero_point, b_zero_point, &shape, C_dev, ldc, false, 1.0f, 0};
        GemmParams p = make_params(a, ctx->num_xcd);
        int32_t *colsum = (int32_t *)workspace_dev;
        int32_t *rowsum = (int32_t *)((uint8_t *)workspace_dev + round_up(shape.Np * 4, 256));
        p.Bp = nullptr;
        p.colsum = colsum;
        const RawB rawb{(const uint8_t *)B_dev, ldb};
        if (form != 0) {
            const hipError_t we = near ? launch_wavek_raw_form(form, p, b_zero_point != 0, rawb, aligned, st)
                                       : launch_wavek_far_aligned<false, true>(form, p, st, &rawb);
            return we == hipSuccess ? NGEMM_OK : NGEMM_ERR_DEVICE;
        }
        // The sums of B's columns (without weight at a_zero_point = 128) and of A's rows (at b_zero_point = 0): the
        // 64 x 64 and 128 x 128 kernels form them, the larger ones read them from passes of their own.
        const bool sums = p.za_term != 0 || b_zero_point != 0;
        const bool sums_in_kernel = kernel == NGEMM_KERNEL_TILE_64 || kernel == NGEMM_KERNEL_TILE_128;
        if (p.za_term != 0 && !sums_in_kernel) {
            hipLaunchKernelGGL(rowsum_a_kernel, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, st, (const uint8_t *)B_dev,
                               ldb, (int)N, (int)K, 0u, colsum);
            if (hipGetLastError() != hipSuccess) return NGEMM_ERR_DEVICE;
        }
        if (b_zero_point != 0 && !sums_in_kernel) {
            hipLaunchKernelGGL(rowsum_a_kernel, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, st, A_dev, lda, (int)M,
                               (int)K, p.a_xor, rowsum);
            if (hipGetLastError() != hipSuccess) return NGEMM_ERR_DEVICE;
            p.rowsum = rowsum;
        }
        const int budget = workgroup_budget(ctx);
        hipError_t e;
        if (kernel == NGEMM_KERNEL_TILE_64) e = launch_tile_dma<64, 64, 2, 2>(p, false, budget, st, &rawb, sums);
        else if (kernel == NGEMM_KERNEL_TILE_128) e = launch_tile_dma<128, 128, 2, 2>(p, false, budget, st, &rawb, sums);
        else if (K >= X64Cfg::kMinK && x64_offsets_fit(256, lda, K) && x64_offsets_fit(256, ldb, K)) {
            p.tiles_m = (int)((M + 255) / 256);
            p.tiles_n = (int)((N + 255) / 256);
            const int ntiles = p.tiles_m * p.tiles_n;
            const int nwg = ntiles < budget ? ntiles : budget;
            hipLaunchKernelGGL(gemm_tile_x64_kernel<true>, dim3((unsigned)nwg), dim3(256), X64Cfg::kLdsBytes, st, args_of_raw(p, rawb, nwg));
            e = hipGetLastError();
        } else e = launch_tile_dma<256, 256, 2, 2, kStages256>(p, false, budget, st, &rawb);
        return e == hipSuccess ? NGEMM_OK : NGEMM_ERR_DEVICE;
    }
    const size_t pb = (size_t)round_up((int64_t)ngemm_packed_b_bytes(K, N), 256);
    ngemm_packed_b *h = nullptr;
    ngemm_status s = ngemm_pack_b(ctx, K, N, B_dev, ldb, workspace_dev, pb, hip_stream, &h);
    if (s != NGEMM_OK) return s;
    s = ngemm_run_u8s8s32(ctx, M, A_dev, lda, a_zero_point, h, b_zero_point, C_dev, ldc,
                          (uint8_t *)workspace_dev + pb, workspace_bytes - pb, hip_stream);
    ngemm_packed_b_free(h);      // the descriptor only: the kernels already hold the device addresses
    return s;
}

size_t ngemm_batched_workspace_bytes(int count, const ngemm_problem *problems)
{
    (void)count;
    (void)problems;
    return 0;                    // the grouped kernels form the row sums they need themselves
}

ngemm_status ngemm_run_batched_u8s8s32(ngemm_ctx *ctx, int count, const ngemm_problem *problems,
                                       void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    (void)workspace_dev;
    (void)workspace_bytes;
    if (!ctx_ok(ctx) || count < 0 || (count > 0 && !problems)) return NGEMM_ERR_INVALID_ARG;
    for (int t = 0; t < count; ++t) {
        const ngemm_problem &q = problems[t];
        RunArgs a{q.M, q.A_dev, q.lda, q.a_zero_point, q.b_zero_point, q.B, q.C_dev, q.ldc, false, 1.0f, 0};
        Route route;
        ngemm_status s = validate_run(ctx, a, &route);
        if (s != NGEMM_OK) return s;
    }
    DeviceGuard g(ctx->device);
    if (!g.ok) return NGEMM_ERR_DEVICE;
    hipStream_t st = (hipStream_t)hip_stream;

    // Grouped launches: the members' parameters ride in the kernel argument block, up to
    // kGroupMax per launch; one grid covers the panels of a group's skinny members and the 64 x 64
    // tiles of its members with M > 32.  Launch count, not arithmetic, is what a batch of small odd
    // shapes costs (and two launches run one after the other, however few compute units each can use),
    // so there is no launch for the row sums either: both bodies form them from the A fragments they
    // read anyway.
    GroupParams grp;
    grp.count = 0;
    grp.nxcd = ctx->num_xcd;
    grp.first_tile = 0;
    grp.unit_start[0] = 0;
    const int cus = ctx->num_cus > 0 ? ctx->num_cus : 256;
    using TCfg = TileCfg<64, 64, 2, 2, 64>;
    // small_tiles: every member by 32 x 32 tiles (below).
    // gemm_group_mid_kernel counts in 32 bits from a tile's first row and panel; a group with a member that has more keeps the kernel
    // with 64-bit addresses.
    bool wide = false, small_tiles = false;
    auto flush = [&]() -> hipError_t {
        if (grp.count == 0) return hipSuccess;
        const unsigned grid = (unsigned)grp.unit_start[grp.count];
        if (grid > 0) {
            if (small_tiles) {
                hipLaunchKernelGGL((gemm_group_kernel<32, 32, 1, 4, 64>), dim3(grid), dim3(256), (WaveKCfg<1, 1, 4, 4>::kLdsBytes), st, grp);
            } else if (grp.first_tile == grp.count) {
                // skinny members only.  Wavefronts per panel: eight hide latency when the panels are
                // few; with several panels per compute unit anyway, fewer wavefronts with more
                // fragments each spend less on the final sum across wavefronts
                const unsigned nw = grid >= 8u * cus ? 2 : (grid >= 4u * cus ? 4 : 8);
                grp.nwaves = (int)nw;
                hipLaunchKernelGGL(gemm_group_skinny_kernel, dim3(grid), dim3(64 * nw), (size_t)(nw * 16 * 64 * 4), st, grp);
            } else {
                const size_t lds = std::max((size_t)TCfg::kLdsBytes, (size_t)(4 * 16 * 64 * 4));
                // Few tiles and a K around the 11 stages from which gemm_group_mid_kernel has a steady loop: a workgroup alone on its unit waits longer
                // per stage there (in a graph, gemm_group_kernel is 1.12 x as fast on up to 64 tiles with K = 512 .. 640, 1.04 x with 1280, 1.05 x on up
                // to 256 tiles with K = 640 .. 1024; outside of these lines the other one, 1.0-1.3 x).  Most such groups take the 32 x 32 tiles (below).  The
                // members with the longest K come first.
                const int tiles = grp.unit_start[grp.count] - grp.unit_start[grp.first_tile], longest = grp.prob[grp.first_tile].K;
                const bool short_chains = (tiles <= cus / 4 && longest > 192 && longest <= 1536) || (tiles <= cus && longest > 256 && longest <= 1024);
                if (wide || short_chains) hipLaunchKernelGGL((gemm_group_kernel<64, 64, 2, 2, 64>), dim3(grid), dim3(256), lds, st, grp);
                else hipLaunchKernelGGL((gemm_group_mid_kernel<MidGroup>), dim3(grid), dim3(256), MidGroup::kLdsBytes, st, grp);
            }
        }
        grp.count = 0;
        grp.first_tile = 0;
        grp.unit_start[0] = 0;
        wide = false;
        return hipGetLastError();
    };
    // The streaming kernel's group: up to kStreamGroupMax members; unit_start collects panel counts
    // until the launch, which turns them into chunks of panels sized for the whole group.
    StreamGroupParams stream;
    stream.count = 0;
    stream.nxcd = ctx->num_xcd;
    stream.unit_start[0] = 0;
    auto flush_stream = [&]() -> hipError_t {
        if (stream.count == 0) return hipSuccess;
        const int chunk = stream_chunk(stream.unit_start[stream.count], cus);
        int lds = 0, units = 0;
        for (int t = 0; t < stream.count; ++t) {
            const int panels = stream.unit_start[t + 1] - stream.unit_start[t];
            stream.unit_start[t] = units;
            units += (panels + chunk - 1) / chunk;
            lds = std::max(lds, stream_launch_lds((int)(stream.mzz[t] & 63u), round_up(stream.K[t], 64), chunk));
        }
        stream.unit_start[stream.count] = units;
        stream.chunk = chunk;
        stream.lds_bytes = lds;
        if (units > 0)
            hipLaunchKernelGGL(gemm_group_stream_kernel, dim3((unsigned)units), dim3(kStreamWaves * 64), (size_t)lds, st, stream);
        stream.count = 0;
        stream.unit_start[0] = 0;
        return hipGetLastError();
    };
    auto push_stream = [&](const GemmParams &p) {
        const int t = stream.count;
        stream.A[t] = p.A; stream.Bp[t] = p.Bp; stream.C[t] = p.C;
        stream.lda[t] = (int)p.lda; stream.ldc[t] = (int)p.ldc;
        stream.N[t] = p.N; stream.K[t] = p.K;
        stream.mzz[t] = stream_pack_mzz(p.M, p.za_term, p.zb);
        stream.unit_start[t + 1] = stream.unit_start[t] + p.npanels;
        ++stream.count;
    };
    auto push = [&](const GemmParams &p, int64_t units, bool is_skinny) {
        GroupMember &m = grp.prob[grp.count];        // the rest is rebuilt on the device
        m.A = p.A; m.Bp = p.Bp; m.C = p.C;
        m.lda = p.lda; m.ldc = p.ldc;
        m.M = p.M; m.N = p.N; m.K = p.K;
        m.za_term = (int16_t)(int32_t)p.za_term;     // 128 - za and zb: small signed values
        m.zb = (int16_t)(int32_t)p.zb;
        grp.unit_start[grp.count + 1] = grp.unit_start[grp.count] + (int)units;
        ++grp.count;
        if (is_skinny) grp.first_tile = grp.count;   // the skinny members of a group come first
    };
    constexpr int64_t kMaxGrid = 1 << 30;
    // Members with the longest K first: a workgroup's time grows with K, and the grid is handed out
    // in order, so the long ones start at once and the many short ones fill in around them.
    struct Pending { GemmParams p; int64_t units; };
    std::vector<Pending> tile_members, skinny_members, stream_members;
    try {
        tile_members.reserve((size_t)count);
        skinny_members.reserve((size_t)count);
        stream_members.reserve((size_t)count);
    } catch (...) {
        return NGEMM_ERR_DEVICE;                   // out of host memory; nothing was launched
    }
    for (int t = 0; t < count; ++t) {
        const ngemm_problem &q = problems[t];
        if (q.M == 0 || q.B->N == 0) continue;
        RunArgs a{q.M, q.A_dev, q.lda, q.a_zero_point, q.b_zero_point, q.B, q.C_dev, q.ldc, false, 1.0f, 0};
        const GemmParams p = make_params(a, ctx->num_xcd);
        if (q.M <= kSkinnyMaxM && stream_can_serve(p.M, p.Kp) && q.lda <= 0x7fffffff && q.ldc <= 0x7fffffff)
            stream_members.push_back(Pending{p, p.npanels});
        else if (q.M <= kSkinnyMaxM)
            skinny_members.push_back(Pending{p, p.npanels});
        else
            tile_members.push_back(Pending{p, (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64)});
    }
    // The streaming kernel pays off once its members have panels for every compute unit several
    // times over; a few panels are better served by the kernel that splits K over wavefronts.
    int64_t stream_panels = 0;
    for (const Pending &m : stream_members) stream_panels += m.units;
    if (stream_panels < 4 * (int64_t)cus) {
        skinny_members.insert(skinny_members.end(), stream_members.begin(), stream_members.end());
        stream_members.clear();
    }
    auto longer_k = [](const Pending &x, const Pending &y) { return x.p.K > y.p.K; };
    // Tiles of 32 x 32 for every member, K shared by four wavefronts, while the chip holds them all at once, two workgroups to a compute
    // unit, and up to twice as many, in two rounds, where the chains are long.  In a graph, on drawn batches with a member of M > 32, the other kernels' time over this
    // one's: 1.02-1.05 on up to 512 tiles with a longest K of 65 to 256, 1.12 up to 512, 1.22 up to 1024, 1.27 up to 1536; 1.4-1.5 from 2048 on, up
    // to 1024 tiles; on 513 to 1024 tiles with K up to 1024 0.9, and from 1025 tiles on 0.5-0.8 (K over 2048: 1.15).  Between 1536 and 2048 the 64 x 64
    // tiles stay (on 1460 drawn batches 1.35 x on up to 512 tiles, 1.2 up to 768 and 1.1 up to 1024, one in eight of those slower: left there).  Groups of skinny members alone do not gain (0.9-1.0): their panels have eight wavefronts to a workgroup already.  Up to K = 1024 a
    // member of up to eight rows is no long chain: as a panel it takes no longer than here, so the line is drawn by the others.  (Batches whose only K over
    // 256 was such a member's ran at 0.89-1.15 x, 1.01 on average; with a longer K, or more rows, at 1.0-1.3.)
    // In two rounds they lead only while the second one is short, that is while the tiles with more than a third of the longest K fit the first: of 5100 drawn
    // batches with a K of 2048 and more on 513 to 1024 tiles, those 1.22 x, the others 0.92 (512 x 2048 x 2048 alone 0.75).
    int64_t tiles32 = 0, longest = 0, chain = 0, long32 = 0;
    bool near = true;
    for (const std::vector<Pending> *v : {&tile_members, &skinny_members})
        for (const Pending &m : *v) {
            tiles32 += (int64_t)((m.p.M + 31) / 32) * m.p.npanels;
            longest = std::max<int64_t>(longest, m.p.K);
            if (m.p.M > 8 || m.p.K > 1024) chain = std::max<int64_t>(chain, m.p.K);
            near = near && wavek_offsets_fit(m.p.lda, m.p.K, m.p.Kp);
        }
    for (const std::vector<Pending> *v : {&tile_members, &skinny_members})
        for (const Pending &m : *v)
            if (3 * (int64_t)m.p.K > longest) long32 += (int64_t)((m.p.M + 31) / 32) * m.p.npanels;
    if (!tile_members.empty() && stream_members.empty() && near &&
        ((chain > 256 && longest <= 1536 && tiles32 <= 2 * cus) || (longest >= 2048 && tiles32 <= 4 * cus && long32 <= 2 * cus))) {
        small_tiles = true;
        skinny_members.insert(skinny_members.end(), tile_members.begin(), tile_members.end());
        tile_members.clear();
        for (Pending &m : skinny_members) m.units = (int64_t)((m.p.M + 31) / 32) * m.p.npanels;
    }
    std::stable_sort(tile_members.begin(), tile_members.end(), longer_k);
    std::stable_sort(skinny_members.begin(), skinny_members.end(), longer_k);
    // skinny members first: in a grid that also holds tiles they start with the launch (the longest
    // of them take as long as all the tiles together)
    for (const Pending &m : skinny_members) {
        if (grp.count == kGroupMax || grp.unit_start[grp.count] + m.units > kMaxGrid)
            if (flush() != hipSuccess) return NGEMM_ERR_DEVICE;
        push(m.p, m.units, true);
    }
    for (const Pending &m : tile_members) {
        if (grp.count == kGroupMax || grp.unit_start[grp.count] + m.units > kMaxGrid)
            if (flush() != hipSuccess) return NGEMM_ERR_DEVICE;
        wide = wide || !x64_offsets_fit(256, m.p.lda, m.p.K) || !x64_offsets_fit(9, 32 * (int64_t)m.p.Kp, 0);
        push(m.p, m.units, false);
    }
    for (const Pending &m : stream_members) {
        if (stream.count == kStreamGroupMax || stream.unit_start[stream.count] + m.units > kMaxGrid)
            if (flush_stream() != hipSuccess) return NGEMM_ERR_DEVICE;
        push_stream(m.p);
    }
    if (flush() != hipSuccess) return NGEMM_ERR_DEVICE;
    if (flush_stream() != hipSuccess) return NGEMM_ERR_DEVICE;
    return NGEMM_OK;
}

}  // extern "C"
