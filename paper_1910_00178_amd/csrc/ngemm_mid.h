// Device kernel for outputs of one to some rounds of workgroups and for rows of A with any alignment; mid_form in ngemm.hip, which alone
// includes this, says which calls it serves.
//
// What bounded such calls: 64 x 64 and 128 x 128 tiles of the older kernels pull 128 bytes per byte of K and tile through a unit's path
// from L2 (120-155 GB/s) with a barrier per 64 bytes; the 256-row tiles leave units idle (2048 x 4096: 176 tiles of 192 x 256) and
// take what is left behind an even number of stages without pipelining; the u8 epilogue read three column arrays from LDS for every
// four values; row sums were a launch of their own.  Here:
//  * tiles from 64 x 128 to 128 x 256 on v_mfma_i32_16x16x64_i8, a wavefront 16 RM x 16 RN of them; two workgroups per unit (but for
//    128 x 256), so that one's fill and epilogue lie under the other's matrix ops;
//  * A and B are copied memory -> LDS in stages of 64 bytes of K, a ring of NS of them, one barrier per stage; both operands lie there
//    so that a fragment read is one conflict-free 16-byte read per lane; fragments of the next stage are read between the matrix ops;
//  * K needs no whole stages: B is padded with zeros, so what A holds behind its K does not matter, and the last stage runs
//    like the others (only the 16 bytes in which the last row of all ends are fetched apart);
//  * the row sums of a zero-point of B are formed once per byte of A, by the wavefront that brings it, with v_sad_u8 (a v_dot4 runs on the
//    matrix pipe and holds it up: 35 cycles per pair with a matrix op against 19);
//  * AREG: rows of A with any alignment, which copies into LDS cannot fetch, come through registers, AD stages ahead;
//  * the u8 output is requantised where it lies in the accumulators, with the column terms in registers, and leaves through LDS in
//    16-byte pieces of whole rows.
// Time stamps in a copy of the loop: no wait for copies to land, 50-150 of a stage's 640-900 cycles at the barrier; 512 are matrix ops (16 of 16 cycles
// for each of two wavefronts on a SIMD).
// Tried: stages of 128 bytes (the same), 64 x 128 of a 128 x 256 tile per wavefront (registers spill or move to the accumulation file),
// the shift of A as an exclusive or on LDS (29 cycles each: slower), priorities for one of two workgroups (nothing).
// us in a graph, the kernels before / here: 2048 x 4096 x 1024 with a zero-point 19.9 / 16.6 (128 x 128 tiles of this kernel: 1.0 POP/s, half of the
// time the launch and 32 MiB of C), 2048 x 3072 x 1536 18.3 / 15.7, 1024 x 3072 x 768 u8 9.0 / 7.7, 1088 x 1413 x 2112 z 12.4 / 11.7; unaligned
// rows: 2047 x 3071 x 1537 z 24.5 / 22.0, 2368 x 4629 x 1343 36.6 / 27.9.
#pragma once
#include "ngemm_kernels.h"

namespace ngemm {

// Wavefront: RM x RN blocks of 16 x 16; workgroup: WGM x WGN wavefronts; NS stages in the ring.
template <int RM_, int RN_, int WGM_, int WGN_, int NS_>
struct MidCfg {
    static constexpr int RM = RM_, RN = RN_, WGM = WGM_, WGN = WGN_, NS = NS_;
    static constexpr int NW = WGM * WGN, kThreads = NW * 64;
    static constexpr int BM = WGM * RM * 16, BN = WGN * RN * 16;
    static constexpr int AITEMS = BM / 16, BITEMS = BN / 16;   // KiB of A and B per stage
    static constexpr int kABytes = BM * 64, kStage = (BM + BN) * 64;
    static constexpr int kPatchRow = RN * 64 + 16;
    static constexpr int kPatch = 16 * kPatchRow;              // per wavefront
    static constexpr int kRow8 = BN + 16;
    static constexpr int kEpi32 = NW * kPatch + BM * 4, kEpi8 = BM * kRow8 + 3 * BN * 4 + BM * 4;
    static constexpr int kEpi = kEpi32 > kEpi8 ? kEpi32 : kEpi8;
    static constexpr int kLdsBytes = NS * kStage > kEpi ? NS * kStage : kEpi;
    static constexpr int kPerCu = kLdsBytes <= 80 * 1024 || NW == 4 ? 2 : 1;
    static constexpr int AD = NS % 4 == 0 ? 4 : 3;             // register sets for A of unaligned rows
    static_assert(kLdsBytes <= 160 * 1024, "LDS of a compute unit");
    static_assert(NS >= 3, "ring");
    static_assert(BN % 32 == 0 && BN <= kThreads, "whole panels, a thread per column");
    static_assert(AITEMS % NW == 0 && BITEMS % NW == 0 && AITEMS / NW <= 4 && BITEMS / NW <= 4, "as many copies for every wavefront");
    static constexpr int kCopyBias = 3 * 1024;                 // lane offsets carry it, the descriptors' bases lack it
};

// f(IntC<U>) && ... && f(IntC<R - 1>)
template <int U, int R, class F>
__device__ __forceinline__ bool all_of(F &&f)
{
    if constexpr (U < R) return f(IntC<U>{}) && all_of<U + 1, R>(f);
    else return true;
}

// One workgroup tile (`tile` in the XCD-aware order of tile_of_block) of the problem `p`.  K >= 16, AREG: any K.
template <class C, bool REQUANT, bool ROWS, bool AREG>
__device__ __forceinline__ void mid_body(const GemmParams &p, int tile, uint8_t *lds)
{
    constexpr int RM = C::RM, RN = C::RN, WGN = C::WGN, NW = C::NW, NS = C::NS, NM = RM * RN, NT = C::kThreads, NR = RM + RN;
    constexpr int AC = C::AITEMS / NW, BC = C::BITEMS / NW;          // KiB of A and B per wavefront and stage
    constexpr int PER = AC + BC, NC = AREG ? BC : PER;               // vector memory instructions, copies into LDS among them
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    int tm, tn;
    tile_of_block(tile, p.tiles_m, p.tiles_n, p.nxcd, tm, tn);
    const int m0 = tm * C::BM, n0 = tn * C::BN;
    const int nst = p.Kp / 64;                               // stages of 64 bytes of K
    const int nfrag = p.Kp / 32;
    const int klast = (nst - 1) * 64;                        // K offset of the last one

    // ---- loader ----
    // Items of a KiB, one copy each.  A: 16 rows x 64 bytes of K, chunk c of row r in 16-byte slot 4 r + (c + r / 2) % 4.  B: a
    // fragment of the matrix op, 16 columns x 64 bytes of K, gathered from the two packed fragments by the copy's lanes.
    // A wavefront's items of an operand are neighbours in LDS: their copies share the LDS base (M0) and carry 1024 * i as
    // immediate offset, which counts for the memory address as well (the lane offsets take it back, + kCopyBias, never negative; the
    // descriptors' bases start kCopyBias early, an address only).
    // (arrays of dependent size here make the host pass drop the kernel: PER and AC places are used)
    uint32_t voff[8], a_last[4];                             // this lane's offset from the tile's first row (panel); A: in the last stage
    bool fix[4];                                             // its 16 bytes of the last stage reach past the end of the last row: fixv
    v4i fixv[4];
    const int a_row = lane >> 2, a_chunk = ((lane & 3) - (a_row >> 1)) & 3;
    const uint8_t *a_tile = p.A + (int64_t)m0 * p.lda;
    const uint8_t *b_tile = p.Bp + (int64_t)(n0 / 32) * nfrag * kFragBytes;
#pragma unroll
    for (int i = 0; i < AC; ++i) {
        int grow = m0 + (wave * AC + i) * 16 + a_row;
        grow = grow < p.M ? grow : p.M - 1;                  // rows past M: read a valid row, never stored
        const uint32_t row = (uint32_t)(grow - m0) * (uint32_t)p.lda, bias = AREG ? 0u : (uint32_t)(C::kCopyBias - 1024 * i);
        voff[i] = row + (uint32_t)(a_chunk * 16) + bias;
        const int k0 = klast + a_chunk * 16, valid = p.K - k0;
        fix[i] = (valid > 0 && valid < 16 && grow == p.M - 1) || (AREG && nst == 1);     // (a row may be shorter than 16 bytes)
        a_last[i] = row + bias + (valid <= 0 || fix[i] ? 0u : (uint32_t)k0);
        fixv[i] = v4i{0, 0, 0, 0};
        if (fix[i]) fixv[i] = valid >= 16 ? load16_any(a_tile + row + k0) : load16_partial(a_tile + row + k0, valid < 0 ? 0 : valid);
    }
#pragma unroll
    for (int i = 0; i < BC; ++i) {
        const int q = lane >> 4, item = wave * BC + i;
        int pnl = n0 / 32 + (item >> 1);
        pnl = pnl < p.npanels ? pnl : p.npanels - 1;         // panels past N: read a valid one, never stored
        voff[AC + i] = (uint32_t)(pnl - n0 / 32) * (uint32_t)(nfrag * kFragBytes) + (uint32_t)((q >> 1) * 1024 + (q & 1) * 512 + (item & 1) * 256 + (lane & 15) * 16) +
                       (uint32_t)(C::kCopyBias - 1024 * i);
    }
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void *)((uintptr_t)a_tile - C::kCopyBias), (short)0, -1, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc((void *)((uintptr_t)b_tile - C::kCopyBias), (short)0, -1, 0x00020000);
    // the column terms: asked for now, needed behind the loop
    constexpr int LPR = RN * 4 <= 8 ? 8 : RN * 4 <= 16 ? 16 : 32, RPI = 64 / LPR;       // read-back: lanes per row (RN * 4 of them store), rows per instruction
    const int bcol = n0 + wn * RN * 16 + 4 * (lane % LPR);
    int4 cs = {0, 0, 0, 0};
    int32_t cs1 = 0, bias1 = 0;
    uint32_t zb1 = p.zb;
    float sc1 = p.scale;
    if (REQUANT) {
        const int col = n0 + tid;
        if (tid < C::BN && col < p.N) {
            cs1 = p.colsum[col];
            if (p.bias_vec) bias1 = p.bias_vec[col];
            if (p.zb_vec) zb1 = (uint32_t)p.zb_vec[col];
            if (p.scale_vec) sc1 = p.scale_vec[col];
        }
    } else if (bcol < p.N && lane % LPR < RN * 4) {
        cs = *(const int4 *)(p.colsum + bcol);
    }
    auto dma1 = [&](auto n, int t, int slot) {               // copy n of stage t into the ring: A's, then B's
        constexpr int I = decltype(n)::value + (AREG ? AC : 0);
        if constexpr (I < AC) {
            const bool at_end = t == nst - 1;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lptr_t)(lds + slot * C::kStage + wave * AC * 1024), 16, at_end ? a_last[I] : voff[I],
                                                     at_end ? 0 : t * 64, I * 1024, 0);
        } else {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lptr_t)(lds + slot * C::kStage + C::kABytes + wave * BC * 1024), 16, voff[I], t * 2048,
                                                     (I - AC) * 1024, 0);
        }
    };
    auto dma1_full = [&](auto n, int t, int slot) {          // the same of a stage that is not the last
        constexpr int I = decltype(n)::value + (AREG ? AC : 0);
        if constexpr (I < AC)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (lptr_t)(lds + slot * C::kStage + wave * AC * 1024), 16, voff[I], t * 64, I * 1024, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lptr_t)(lds + slot * C::kStage + C::kABytes + wave * BC * 1024), 16, voff[I], t * 2048,
                                                     (I - AC) * 1024, 0);
    };
    constexpr int AD = C::AD;                                // AREG: register sets, stage t in set t % AD
    v4i va[AD][AC];
    auto load_a = [&](auto set, int t) {
        constexpr int S = decltype(set)::value;
#pragma unroll
        for (int i = 0; i < AC; ++i) va[S][i] = load16_any(t < nst - 1 ? a_tile + t * 64 + voff[i] : a_tile + a_last[i]);
    };
    // The row sums that a zero-point of B needs, once per byte of A, by the wavefront that brings it: sums of absolute differences of
    // unsigned bytes (signed ones 128 up), less 128 per byte at the end.  (A dot product with ones runs on the matrix pipe.)
    uint32_t rs[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) rs[i] = 0u;
    const uint32_t to_unsigned = p.a_xor ^ 0x80808080u;
    auto add_row = [&](int i, uint32_t word, uint32_t exist) { rs[i] = __builtin_amdgcn_sad_u8((word ^ to_unsigned) & exist, 0u, rs[i]); };
    auto exist_of = [&](int t) { return ~bytes_from(p.K - (t * 64 + a_chunk * 16)); };      // ones in this lane's bytes of stage t that exist
    auto a_place = [&](int i, int slot) { return lds + slot * C::kStage + (wave * AC + i) * 1024; };
    v4i own[4];
    auto read_own = [&](int i, int slot) { own[i] = *(const v4i *)(a_place(i, slot) + lane * 16); };
    // AREG: A is shifted to signed bytes on its way into LDS (else behind the fragment reads)
    auto write_a = [&](auto set, int slot, int t) {
        constexpr int S = decltype(set)::value;
#pragma unroll
        for (int i = 0; i < AC; ++i) {
            const v4i a = t == nst - 1 && fix[i] ? fixv[i] : va[S][i];       // (the piece that ends inside 16 bytes of the last row)
            if (ROWS) {
                const v4i e = exist_of(t);
#pragma unroll
                for (int w = 0; w < 4; ++w) add_row(i, (uint32_t)a[w], (uint32_t)e[w]);
            }
            *(v4i *)(a_place(i, slot) + lane * 16) = shift_u8_to_s8(a, p.a_xor);
        }
    };
    auto write_a_full = [&](auto set, int slot) {             // the same of a stage that is not the last
        constexpr int S = decltype(set)::value;
#pragma unroll
        for (int i = 0; i < AC; ++i) {
            if (ROWS) {
#pragma unroll
                for (int w = 0; w < 4; ++w) add_row(i, (uint32_t)va[S][i][w], 0xffffffffu);
            }
            *(v4i *)(a_place(i, slot) + lane * 16) = shift_u8_to_s8(va[S][i], p.a_xor);
        }
    };
    const bool fixes = (p.K & 15) != 0 && m0 + C::BM >= p.M;       // (one tile row)
    auto apply_fix = [&](int slot) {                          // the last stage's pieces that end inside 16 bytes of the last row
#pragma unroll
        for (int i = 0; i < AC; ++i)
            if (fix[i]) *(v4i *)(a_place(i, slot) + lane * 16) = fixv[i];
    };
    auto own_rows = [&](int t, int slot) {                    // (not in the steady loop)
        const v4i e = exist_of(t);
#pragma unroll
        for (int i = 0; i < AC; ++i) {
            read_own(i, slot);
#pragma unroll
            for (int w = 0; w < 4; ++w) add_row(i, (uint32_t)own[i][w], (uint32_t)e[w]);
        }
    };

    // ---- fragments ----
    v4i fa[2][RM], fb[2][RN];                                 // of two stages
    const int r16 = lane & 15, c4 = lane >> 4;
    const int a_off = wm * RM * 1024 + (4 * r16 + ((c4 + (r16 >> 1)) & 3)) * 16;
    const int b_off = C::kABytes + wn * RN * 1024 + lane * 16;
    auto read_one = [&](auto x, const uint8_t *base, int n) {        // in the order of their use: A's block 0, B, the rest of A
        constexpr int X = decltype(x)::value;
        if (n == 0) fa[X][0] = *(const v4i *)(base + a_off);
        else if (n <= RN) fb[X][n - 1] = *(const v4i *)(base + b_off + (n - 1) * 1024);
        else fa[X][n - RN] = *(const v4i *)(base + a_off + (n - RN) * 1024);
    };
    v4i acc[RM][RN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) acc[i][j] = v4i{0, 0, 0, 0};
    // The matrix ops of stage x of a double one; `gap(m)` goes between them.
    auto stage = [&](auto x, auto &&gap) {
        constexpr int X = decltype(x)::value;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            acc[m / RN][m % RN] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[X][m % RN], fa[X][m / RN], acc[m / RN][m % RN], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            gap(m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto read_gap = [&](auto x, const uint8_t *base, int m) {     // fragment reads: four in three gaps, from the first one on
#pragma unroll
        for (int n = 0; n < NR; ++n)
            if (n * 3 / 4 == m) read_one(x, base, n);
    };
    static_assert((NR - 1) * 3 / 4 < NM, "a place for every read");
    // Shifts: A's block i + 1 in the gaps of block i, block 0 of the next stage in those of the last one.
    auto shift_gap = [&](auto x, auto other, int m) {
        constexpr int X = decltype(x)::value, O = decltype(other)::value;
        const int i = m / RN, j = m % RN;
        if (AREG) return;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if (w * RN / 4 == j) {
                if (i + 1 < RM) fa[X][i + 1][w] ^= (int)p.a_xor;
                else fa[O][0][w] ^= (int)p.a_xor;
            }
    };
    constexpr int RG = (NR * 3 + 3) / 4, CG = RG + PER <= NM ? RG : NM - PER > 0 ? NM - PER : 0;      // copies: one per gap behind the reads

    // ---- prologue ----
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (AREG) {
        if (nst > 1) static_for<0, AD>([&](auto u) { load_a(u, decltype(u)::value); });
    }
#pragma unroll
    for (int t = 0; t < NS; ++t)
        if (t < nst) static_for<0, NC>([&](auto n) { dma1(n, t, t); });
    if constexpr (AREG) {
        write_a(IntC<0>{}, 0, 0);
        if (nst > 1) {
            write_a(IntC<1>{}, 1, 1);
            load_a(IntC<0>{}, AD);
            load_a(IntC<1>{}, AD + 1);
            wait_vmcnt<2 * AC>();
        } else wait_vmcnt<0>();                                 // (all first copies: once per tile)
    } else {
        if (nst >= NS) wait_vmcnt<(NS - 1) * NC>();
        else wait_vmcnt<0>();
        if (fixes && nst == 1) apply_fix(0);
        if (ROWS) own_rows(0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < NR; ++n) read_one(IntC<0>{}, lds, n);
    if (!AREG) fa[0][0] = shift_u8_to_s8(fa[0][0], p.a_xor);

    // ---- main loop: stage t in place t % NS of the ring, its fragments in set t % 2 ----
    // At the barrier stage t + 1 has landed for every wavefront and the place of stage t is read.  Between the matrix ops of t: the
    // fragments of t + 1 are read, stage t + NS is requested into that place.
    int t = 0;
    auto steady = [&](auto u) {
        constexpr int V = decltype(u)::value, X = V & 1, P2 = (V + 2) % AD, S0 = V % NS, S1 = (V + 1) % NS, S2 = (V + 2) % NS;
        const uint8_t *nxt = lds + S1 * C::kStage;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        if constexpr (AREG) wait_vmcnt<(NS - 2 < AD - 1 ? NS - 2 : AD - 1) * PER>();
        else wait_vmcnt<(NS - 2) * PER>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (AREG) write_a_full(IntC<P2>{}, S2);     // A of t + 2
        __builtin_amdgcn_sched_barrier(0);
        stage(IntC<X>{}, [&](int m) {
            read_gap(IntC<X ^ 1>{}, nxt, m);
            static_for<0, PER>([&](auto n) {
                constexpr int I = decltype(n)::value;
                if ((CG + I < NM - 1 ? CG + I : NM - 1) == m) {
                    if constexpr (AREG && I < AC) va[P2][I] = load16_any(a_tile + (t + V + 2 + AD) * 64 + voff[I]);
                    else dma1_full(IntC<I - (AREG ? AC : 0)>{}, t + V + NS, S0);
                }
            });
            shift_gap(IntC<X>{}, IntC<X ^ 1>{}, m);
            if constexpr (ROWS && !AREG) {                    // of t + 1
#pragma unroll
                for (int i = 0; i < AC; ++i)
                    if (m == NM / 4 + i) read_own(i, S1);
#pragma unroll
                for (int w = 0; w < 4 * AC; ++w)
                    if (NM / 2 + w * (NM / 2) / (4 * AC) == m) add_row(w >> 2, (uint32_t)own[w >> 2][w & 3], 0xffffffffu);
            }
        });
    };
    // AREG: the last stages but one.  As many loads as in the steady loop, so that the waits are counted there as well; what lies past
    // the end is one address for all lanes.
    auto finish_areg = [&](auto u) -> bool {
        constexpr int V = decltype(u)::value, X = V & 1, P2 = (V + 2) % AD, S0 = V % NS, S1 = (V + 1) % NS, S2 = (V + 2) % NS;
        if (t + 1 >= nst) return false;
        const uint8_t *nxt = lds + S1 * C::kStage;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        wait_vmcnt<(NS - 2 < AD - 1 ? NS - 2 : AD - 1) * PER>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (t + 2 < nst) write_a(IntC<P2>{}, S2, t + 2);
        __builtin_amdgcn_sched_barrier(0);
        const int ta = t + 2 + AD, tb = t + NS;
        static_for<0, PER>([&](auto n) {
            constexpr int I = decltype(n)::value;
            if constexpr (I < AC) {
                const uint32_t at = ta < nst - 1 ? voff[I] + (uint32_t)(ta * 64) : ta == nst - 1 ? a_last[I] : 0u;
                va[P2][I] = load16_any(a_tile + at);
            } else {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, (lptr_t)(lds + S0 * C::kStage + C::kABytes + wave * BC * 1024), 16,
                                                         tb < nst ? voff[I] : (uint32_t)C::kCopyBias, tb < nst ? tb * 2048 : 0, (I - AC) * 1024, 0);
            }
        });
        __builtin_amdgcn_sched_barrier(0);
        stage(IntC<X>{}, [&](int m) { read_gap(IntC<X ^ 1>{}, nxt, m); });
        ++t;
        return true;
    };
    auto finish = [&](auto u) {                               // the last stages
        constexpr int V = decltype(u)::value, X = V & 1, S0 = V % NS, S1 = (V + 1) % NS;
        const uint8_t *nxt = lds + S1 * C::kStage;
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < nst) {
            const int y = nst - 2 - t;                        // stages behind t + 1 on their way
            if (y >= NS - 2) wait_vmcnt<(NS - 2) * NC>();
            else if (y == 1) wait_vmcnt<NC>();
            else if (NS > 4 && y == 2) wait_vmcnt<2 * NC>();
            else if (NS > 5 && y == 3) wait_vmcnt<3 * NC>();
            else wait_vmcnt<0>();
            if (fixes && t + 1 == nst - 1) apply_fix(S1);
            if (ROWS) own_rows(t + 1, S1);
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_s_barrier();
            if (t + NS < nst) static_for<0, NC>([&](auto n) { dma1(n, t + NS, S0); });
        }
        __builtin_amdgcn_sched_barrier(0);
        stage(IntC<X>{}, [&](int m) {
            read_gap(IntC<X ^ 1>{}, nxt, m);                  // (past the end: a place nobody needs)
            shift_gap(IntC<X>{}, IntC<X ^ 1>{}, m);
        });
        ++t;
    };
    // steady while the stages requested, the rows of A of t + V + 2 + AD among them, are not the last
    constexpr int U1 = AREG && NS % AD != 0 ? NS * AD : NS, U = U1 % 2 == 0 ? U1 : 2 * U1, AHEAD = AREG && AD + 2 > NS ? AD + 2 : NS;
    static_assert(U % NS == 0 && U % 2 == 0 && (!AREG || U % AD == 0), "static places and sets");
    static_assert(AHEAD >= NS && (!AREG || AHEAD >= AD + 2), "no request past the last stage but one");
    for (; t + U - 1 + AHEAD < nst - 1; t += U) static_for<0, U>(steady);
    if constexpr (AREG) {
        while (all_of<0, U>(finish_areg)) {}
        if (nst == 0) {                                       // (a grouped member of K = 0)
        } else if ((t & 1) == 0) stage(IntC<0>{}, [](int) {});
        else stage(IntC<1>{}, [](int) {});
    } else {
        while (t < nst) {
            static_for<0, U>([&](auto u) {
                if (t < nst) finish(u);
            });
        }
    }

    // ---- epilogue ----
    wait_vmcnt<0>();
    __syncthreads();                                          // every wavefront is done with the ring
    uint32_t rsum[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) rsum[i] = 0u;
    uint32_t *rsx = (uint32_t *)(lds + (REQUANT ? C::BM * C::kRow8 + 3 * C::BN * 4 : NW * C::kPatch));
    if (ROWS) {
#pragma unroll
        for (int i = 0; i < AC; ++i) {
            uint32_t v = rs[i];
            v += (uint32_t)__shfl_xor((int)v, 1, 64);
            v += (uint32_t)__shfl_xor((int)v, 2, 64);
            if ((lane & 3) == 0) rsx[(wave * AC + i) * 16 + a_row] = v - 128u * (uint32_t)p.K;
        }
    }
    if constexpr (REQUANT) {
        uint32_t *cterm = (uint32_t *)(lds + C::BM * C::kRow8);
        if (tid < C::BN) {
            cterm[tid] = p.za_term * (uint32_t)cs1 + (uint32_t)bias1;
            cterm[C::BN + tid] = zb1;
            ((float *)cterm)[2 * C::BN + tid] = sc1;
        }
        __syncthreads();
        if (ROWS) {
#pragma unroll
            for (int i = 0; i < RM; ++i) rsum[i] = rsx[(wm * RM + i) * 16 + r16];
        }
        uint4 cb[RN], zv[RN];
        float4 scv[RN];
#pragma unroll
        for (int j = 0; j < RN; ++j) {
            const int lcol = (wn * RN + j) * 16 + 4 * c4;
            cb[j] = *(const uint4 *)(cterm + lcol);
            zv[j] = *(const uint4 *)(cterm + C::BN + lcol);
            scv[j] = *(const float4 *)((const float *)cterm + 2 * C::BN + lcol);
        }
        const float zcf = (float)p.zc, floor_f = p.relu ? zcf : -3.402823466e38f;
        auto rows_out = [&](auto small) {
            constexpr bool SMALL = decltype(small)::value != 0;
#pragma unroll
            for (int i = 0; i < RM; ++i) {
                const uint32_t rr = rsum[i] + p.rconst;
#pragma unroll
                for (int j = 0; j < RN; ++j) {
                    int32_t c[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t cbe = e == 0 ? cb[j].x : e == 1 ? cb[j].y : e == 2 ? cb[j].z : cb[j].w;
                        const uint32_t zve = e == 0 ? zv[j].x : e == 1 ? zv[j].y : e == 2 ? zv[j].z : zv[j].w;
                        c[e] = (int32_t)((uint32_t)acc[i][j][e] + cbe - (ROWS ? zve * rr : 0u));
                    }
                    uint32_t bw;
                    if (SMALL) bw = requant4_u8_small_zc(c, scv[j], zcf, floor_f);
                    else
                        bw = (uint32_t)requant_u8(c[0], scv[j].x, p.zc, p.relu) | ((uint32_t)requant_u8(c[1], scv[j].y, p.zc, p.relu) << 8) |
                             ((uint32_t)requant_u8(c[2], scv[j].z, p.zc, p.relu) << 16) | ((uint32_t)requant_u8(c[3], scv[j].w, p.zc, p.relu) << 24);
                    *(uint32_t *)(lds + ((wm * RM + i) * 16 + r16) * C::kRow8 + (wn * RN + j) * 16 + 4 * c4) = bw;
                }
            }
        };
        if (p.zc > -8388608 && p.zc < 8388608) rows_out(IntC<1>{});
        else rows_out(IntC<0>{});
        __syncthreads();
        constexpr int CPR = C::BN / 16, TOTAL = C::BM * CPR;
        constexpr int NPASS = (TOTAL + NT - 1) / NT;
        v4i o[NPASS];
#pragma unroll
        for (int k = 0; k < NPASS; ++k) {
            const int q = tid + k * NT;
            if (q < TOTAL) o[k] = *(const v4i *)(lds + (q / CPR) * C::kRow8 + (q % CPR) * 16);
        }
#pragma unroll
        for (int k = 0; k < NPASS; ++k) {
            const int q = tid + k * NT, row = m0 + q / CPR, col = n0 + (q % CPR) * 16;
            uint8_t *dst = (uint8_t *)p.C + (int64_t)row * p.ldc + col;
            if (q < TOTAL && row < p.M && col < p.N) {
                if (col + 16 <= p.N) {
                    __builtin_memcpy(dst, &o[k], 16);
                } else {                                      // the last piece of a row: words, then bytes (u8 with a zero-point, bytes only / so:
                                                              // 5120 x 3901 x 192 22.5 / 20.4 us, 113945 x 29 x 262 22.0 / 19.6)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const uint32_t v = (uint32_t)o[k][w];
                        if (col + 4 * w + 4 <= p.N) {
                            __builtin_memcpy(dst + 4 * w, &v, 4);
                        } else {
#pragma unroll
                            for (int b = 0; b < 3; ++b)
                                if (col + 4 * w + b < p.N) dst[4 * w + b] = (uint8_t)(v >> (8 * b));
                        }
                    }
                }
            }
        }
    } else {
        if (ROWS) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < RM; ++i) rsum[i] = rsx[(wm * RM + i) * 16 + r16];
        }
        uint8_t *patch = lds + wave * C::kPatch;
        uint4 ct;
        ct.x = p.za_term * (uint32_t)cs.x; ct.y = p.za_term * (uint32_t)cs.y;
        ct.z = p.za_term * (uint32_t)cs.z; ct.w = p.za_term * (uint32_t)cs.w;
        const bool interior = m0 + (wm + 1) * RM * 16 <= p.M && n0 + (wn + 1) * RN * 16 <= p.N;
        const bool lines = (((uintptr_t)p.C | (uintptr_t)(p.ldc * 4)) & 63) == 0;
        const int lr = lane / LPR, lc = lane % LPR;
        const bool storing = LPR == RN * 4 || lc < RN * 4;
#pragma unroll
        for (int i = 0; i < RM; ++i) {
            const uint32_t row_term = p.kconst - (ROWS ? p.zb * rsum[i] : 0u);
#pragma unroll
            for (int j = 0; j < RN; ++j) {
                v4i v = acc[i][j];
                v.x = (int)((uint32_t)v.x + row_term); v.y = (int)((uint32_t)v.y + row_term);
                v.z = (int)((uint32_t)v.z + row_term); v.w = (int)((uint32_t)v.w + row_term);
                *(v4i *)(patch + r16 * C::kPatchRow + (16 * j + 4 * c4) * 4) = v;
            }
            constexpr int NPASS = 16 / RPI;
            v4i o[NPASS];
#pragma unroll
            for (int q = 0; q < NPASS; ++q) {
                if (storing) o[q] = *(const v4i *)(patch + (RPI * q + lr) * C::kPatchRow + lc * 16);
            }
#pragma unroll
            for (int q = 0; q < NPASS; ++q) {
                o[q].x = (int)((uint32_t)o[q].x + ct.x); o[q].y = (int)((uint32_t)o[q].y + ct.y);
                o[q].z = (int)((uint32_t)o[q].z + ct.z); o[q].w = (int)((uint32_t)o[q].w + ct.w);
            }
            const int row0 = m0 + (wm * RM + i) * 16 + lr;
            int32_t *dst = (int32_t *)p.C + (int64_t)row0 * p.ldc + bcol;
            if (interior && lines) {
#pragma unroll
                for (int q = 0; q < NPASS; ++q, dst += RPI * p.ldc)
                    if (storing) __builtin_nontemporal_store(o[q], (v4i_a4 *)dst);
            } else {
#pragma unroll
                for (int q = 0; q < NPASS; ++q, dst += RPI * p.ldc) {
                    const v4i v = o[q];
                    if (storing && row0 + RPI * q < p.M && bcol < p.N) {
                        if (bcol + 3 < p.N) {
                            __builtin_memcpy(dst, &v, 16);
                        } else {
                            dst[0] = v.x;
                            if (bcol + 1 < p.N) dst[1] = v.y;
                            if (bcol + 2 < p.N) dst[2] = v.z;
                        }
                    }
                }
            }
        }
    }
}

template <class C, bool REQUANT, bool ROWS, bool AREG>
__global__ __launch_bounds__(C::kThreads, C::NW / 4 * C::kPerCu) void gemm_mid_kernel(const GemmArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    mid_body<C, REQUANT, ROWS, AREG>(params_of<1, C::BM, C::BN>(a), blockIdx.x, lds);
}

// Grouped launches (see GroupParams): the panels of the skinny members, four wavefronts each, then the tiles of the others, whose rows
// have any alignment.  Bound by latency: a member of few tiles and a long K lasts as long as its stages, and the short ones are a prologue and an
// epilogue each, so four workgroups share a unit (64 x 64 tiles, 32 KiB, 128 registers).  The batch of 64 odd shapes (M, N to 4096, K to
// 3183; 1911 tiles and the panels) in a graph: 18.3 us on gemm_group_kernel, whose tiles are staged through registers, 16.9 here; when this was
// written, against 16.5: 128 columns per tile 17.8, two workgroups per unit 17.4, six stages and register sets 18.1.  Groups of few tiles and a short K
// stay with gemm_group_kernel (the launch says which).
template <class C>
__global__ __launch_bounds__(256, C::kPerCu) void gemm_group_mid_kernel(const GroupParams g)
{
    static_assert(C::kThreads == 256, "the skinny members' four wavefronts");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    const int q = group_find(g, blockIdx.x);
    const GemmParams p = group_member_params<C::BM, C::BN>(g.prob[q], g.nxcd);
    const int unit = blockIdx.x - g.unit_start[q];
    if (q < g.first_tile) skinny_body<false, 1, true>(p, unit, C::NW, (int *)lds);
    else mid_body<C, false, true, true>(p, unit, lds);
}

}  // namespace ngemm
