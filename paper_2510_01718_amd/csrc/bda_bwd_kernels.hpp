// Gradient kernels of the BD K/V projection (Section "BDA Training Evaluation": C is a learnable
// parameter and gradients flow through steps 2-3 of Algorithm "BD Attention Inference").
//
// With out[t, n] = c[t, off_g + (n - col0_g) % d_h] + sum_i c[t, Bbar_g(i)] C[i, n] and G = dL/d out:
//
//   latent gradient  gc[t, l] = sum_g sum_{n in group g} G[t, n] Wfull_g[l, n]
//                    Wfull_g[l, n] = C[rank_g(l), n]             for l outside the window of g
//                                  = [l - off_g == (n - col0_g) % d_h]   for l inside it
//   weight gradient  gC[i, n] = sum_t c[t, Bbar_g(i)] G[t, n]
//
// Both are GEMMs of the forward's size that contract over thousands of elements into few output tiles (T x d_c and
// (d_c - d_h) x N are small next to T x N), so a launch has about one workgroup per compute unit and each workgroup a long
// loop.  Operands go from memory to LDS by DMA through a ring of stages with counted waits and one barrier a stage; the
// waves of a workgroup share out the contraction of a stage (WK of them on the same outputs, added at the end in a fixed
// order), which keeps a wave's tile at 64 x 64 or more and with it the LDS reads below the MFMAs' time.
// The latent gradient contracts over the output columns n, along which both G and C are contiguous: rows of 128 bytes,
// read as they lie.  The weight gradient contracts over the tokens t, the slow index of c and G: whole rows, transposed by
// the LDS read.
// Bound: a stage's requests at 64 bytes a clock and compute unit beside its MFMAs, plus some 300 cycles of barrier and
// bookkeeping a stage that both waves of a SIMD spend at the same time.  Against the kernels before (register-staged copies,
// two halves of 2 x 2 waves): 8192 tokens, N = 32768, bf16: latent 381 -> 278 us, weight 282 -> 193; 4096 tokens, N = 4096,
// f16, float32 gradients: 41 -> 26 and 32 -> 24; 202 tokens, N = 30464: 193 -> 86 and 34 -> 13.
// Whichever operand is contiguous in the OUTPUT is the MFMA's row operand, so that each lane holds four consecutive
// elements of a row.
#pragma once
#include <type_traits>

#include "bda_ring.hpp"

namespace bda {

struct BwdArgs {
    const void* c;    // T x d_c latent
    const void* g;    // T x N upstream gradient
    const void* C;    // K x N coefficients (latent gradient only)
    void* out;        // gc (T x d_c) or gC (K x N)
    int64_t ldc, ldg, ldC, ldo;          // in elements
    int64_t T;
    int d_c, d_h, K;                     // K = d_c - d_h
    int n_groups;
    int m_tiles, n_tiles;                // tile grid: rows x columns of the output
    int n_stages;                        // latent gradient: stages of all groups (none straddles two)
    int tile_start[kMaxGroups + 1];      // weight gradient: first column tile of each group
    int64_t col_start[kMaxGroups + 1];   // first output column of each group
    int a_off[kMaxGroups];               // basis window start of each group
};

// The latent gradient's table of ones: row r = -32 .. 47 is 16 elements with a one at r (none outside 0 .. 15).
constexpr int kOnesFirst = -32, kOnesRows = 80, kOnesBytes = kOnesRows * 32;

template <typename X, typename OutT, typename C, typename Acc>
__device__ __forceinline__ void ring_finish(unsigned char* smem, Acc& acc, __amdgpu_buffer_rsrc_t rD, int64_t ldo, int cols_left,
                                            int wave, int wt, int wn, int kg, int lane)
{
    wait_vmcnt<0>();                           // (requests past the last stage, of loops that are not unrolled, still write zeros to the ring)
    __syncthreads();
    ring_reduce<C>(smem, acc, kg, wt * C::WN + wn, lane);
    if (C::WK > 1 && kg >= 2) return;
    static_assert(C::TN % 2 == 0 && (C::WK == 1 || C::TT % 2 == 0));
    unsigned char* const stag = smem + wave * 4096;
    const uint32_t pitch = (uint32_t)(ldo * sizeof(OutT));
    constexpr int KEPT = C::WK == 1 ? C::TT : C::TT / 2;             // token blocks of this wave, in its first accumulators
    const int row0 = wt * (32 * C::TT) + (C::WK > 1 && kg == 1 ? 32 * KEPT : 0);
#pragma unroll
    for (int ti = 0; ti < KEPT; ++ti)
#pragma unroll
        for (int n = 0; n < C::TN; n += 2)
            ring_store<X, OutT>(stag, acc[n][ti], acc[n + 1][ti], rD, pitch, row0 + 32 * ti, wn * (32 * C::TN) + 32 * n, cols_left, lane);
}

// ---------------------------------------------------------------------------------------------
// Latent gradient: BT tokens x BN latent columns, contraction over the output columns n, group by group.
// ---------------------------------------------------------------------------------------------
template <typename X, typename OutT, typename C>
__global__ __launch_bounds__(C::THREADS) void ring_latent_kernel(const BwdArgs p)
{
    constexpr int BT = C::BT, BN = C::BN, TT = C::TT, TN = C::TN, S = C::S, PT = C::PT, PN = C::PN, KSW = C::KSW, CK = C::CK;
    constexpr int RT = BT / 8, RN = BN / 8;    // requests of a block of 64 along the contraction: 8 rows of 128 bytes each
    constexpr int BLOCK = (BT + BN) * 128;     // LDS bytes of such a block: token rows, then weight rows
    static_assert(CK % 64 == 0 && RT % PT == 0 && RN % PN == 0 && BT != 192 && BN != 192);
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    typedef __attribute__((address_space(3))) unsigned char* lds_u8;
    typedef __attribute__((address_space(3))) const u32x4* lds_u32x4;

    const int tile = tile_of_block(p.m_tiles * p.n_tiles);
    if (tile < 0) return;
    const int mt = tile / p.n_tiles, nt = tile % p.n_tiles;   // the column tiles of one token tile share its G rows
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / (C::WT * C::WN), wt = wave / C::WN % C::WT, wn = wave % C::WN;
    const int l31 = lane & 31, lhi = lane >> 5;

    const int64_t t0 = (int64_t)mt * BT;
    const int64_t rows_left = p.T - t0;
    const int l0 = nt * BN;
    const int cols_left = p.d_c - l0 > BN ? BN : p.d_c - l0;
    const int64_t N = p.col_start[p.n_groups];
    const u32x4 rG = make_rsrc_words((const char*)p.g + t0 * p.ldg * 2, ((rows_left - 1) * p.ldg + N) * 2);
    const u32x4 rC = make_rsrc_words(p.C, ((int64_t)(p.K - 1) * p.ldC + N) * 2);
    const uint32_t g_pitch = (uint32_t)(p.ldg * 2), c_pitch = (uint32_t)(p.ldC * 2);
    const int d_h = p.d_h, d_c = p.d_c, n_groups = p.n_groups;

    // ---- requests: a wave's are 8 rows each of one block; a row's 16-byte piece p is stored at position p ^ tok_swz(row) ----
    const int lrow = lane >> 3, lpos = lane & 7;
    const int blk_t = wave * PT / RT, first_t = (wave * PT % RT) * 8, row_t = first_t + lrow;
    const int blk_n = wave * PN / RN, first_n = (wave * PN % RN) * 8, row_n = first_n + lrow;
    uint32_t vt[PT], vw[PN], xt[PT], xw[PN];
    auto piece = [&](int row) { return lpos ^ tok_swz<64>(row & 15); };
#pragma unroll
    for (int j = 0; j < PT; ++j) vt[j] = (uint32_t)(row_t + 8 * j) * g_pitch + (uint32_t)(blk_t * 128 + piece(row_t + 8 * j) * 16);
    int ld_g = -1, ld_rem = 0;                 // group being requested, its columns not yet asked for (of the stage being set up, too)
    uint32_t ld_soff = 0u - 2u * CK;
    auto prepare = [&]() {
        ld_rem -= CK;
        ld_soff += 2u * CK;
        if (ld_rem < CK) {
            if (ld_rem <= 0) {                 // (nothing is requested past the last group)
                ld_g = uniform(ld_g + 1);
                // (waited for in here, not by every stage where the paths meet)
                const int start = uniform((int)p.col_start[ld_g]), end = uniform((int)p.col_start[ld_g + 1]), off = uniform(p.a_off[ld_g]);
                ld_rem = end - start;
                ld_soff = (uint32_t)start * 2u;
#pragma unroll
                for (int j = 0; j < PN; ++j) {
                    const int row = row_n + 8 * j, l = l0 + row;
                    const bool ok = l < d_c && (l < off || l >= off + d_h);
                    vw[j] = ok ? (uint32_t)(l < off ? l : l - d_h) * c_pitch + (uint32_t)(blk_n * 128 + piece(row) * 16) : kBadOffset;
                }
            }
            // (columns past the group's end read as zero)
#pragma unroll
            for (int j = 0; j < PT; ++j) xt[j] = blk_t * 64 + piece(row_t + 8 * j) * 8 < ld_rem ? vt[j] : kBadOffset;
#pragma unroll
            for (int j = 0; j < PN; ++j) xw[j] = blk_n * 64 + piece(row_n + 8 * j) * 8 < ld_rem ? vw[j] : kBadOffset;
        }
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8)smem;
    const uint32_t dst_t = lds0 + (uint32_t)(blk_t * BLOCK + first_t * 128), dst_n = lds0 + (uint32_t)(blk_n * BLOCK + BT * 128 + first_n * 128);
    auto request = [&](auto jc, uint32_t slot) {
        constexpr int j = decltype(jc)::value;
        const uint32_t soff = (uint32_t)uniform((int)ld_soff);
        if constexpr (j < PT) lds_dma_imm<1024 * j>(rG, dst_t + slot, xt[j], soff);
        else lds_dma_imm<1024 * (j - PT)>(rC, dst_n + slot, xw[j - PT], soff);
    };

    // ---- fragments: k-step kg KSW + s of a stage, four to a block ----
    uint32_t a_tok[KSW], a_wgt[KSW];
#pragma unroll
    for (int s = 0; s < KSW; ++s) {
        const int ks = kg * KSW + s;
        const uint32_t at = (uint32_t)((ks >> 2) * BLOCK + ((((ks & 3) * 2 + lhi) ^ tok_swz<64>(l31 & 15)) << 4));
        a_tok[s] = lds0 + at + (uint32_t)((wt * (32 * TT) + l31) * 128);
        a_wgt[s] = lds0 + at + (uint32_t)((BT + wn * (32 * TN) + l31) * 128);
    }
    // Window rows of Wfull are staged as zeros.  Output column 16 ks + k' of a stage feeds latent column off + jk + k' with
    // weight one: a 32-column block inside the window takes its fragments from a table of ones instead, shifted by where
    // the k-step's columns fall in the block; a block that the window's edge cuts, from both.  (Ones put into the fragments
    // in registers, or products of their own, stood between every barrier and its MFMAs: 4096 tokens, N = 4096 25 -> 33 us.)
    unsigned char* const ones = smem + C::BYTES;
    for (int e = threadIdx.x; e < kOnesRows * 8; e += C::THREADS) {
        const int r = kOnesFirst + e / 8, k0 = e % 8 * 2;
        ((uint32_t*)ones)[e] = (k0 == r ? IdentityFrag<X>::one : 0u) | (k0 + 1 == r ? IdentityFrag<X>::one << 16 : 0u);
    }
    const uint32_t a_ones = lds0 + (uint32_t)(C::BYTES + (l31 - kOnesFirst) * 32 + lhi * 16);
    const uint32_t a_zeros = lds0 + (uint32_t)(C::BYTES + l31 * 32 + lhi * 16);   // 32 of its rows without a one
    const int colm0 = l0 + wn * (32 * TN);     // first latent column of this wave
    const int period = d_h * 32, step = CK % d_h * 32;
    int rd_g = -1, rd_left = 0, place = 0, at = 0;   // group being read, its stages left; 32 x: the wave's first column of the stage in its head, window start - colm0
    bool inside[TN], all_inside = false, cut = false, meets = false;   // blocks inside the window; all of them; some block is cut by its edge; some block has to do with it
    auto enter_group = [&]() {
        rd_g = uniform(rd_g + 1);
        if (rd_g >= n_groups) return;
        const int start = uniform((int)p.col_start[rd_g]), end = uniform((int)p.col_start[rd_g + 1]), off = uniform(p.a_off[rd_g]);
        rd_left = (end - start + CK - 1) / CK;
        place = 16 * kg * KSW % d_h * 32;
        at = (off - colm0) * 32;
        cut = meets = false;
        all_inside = true;
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            const int b = off - colm0 - 32 * ni;     // the window's start in the block
            inside[ni] = b <= 0 && 32 <= b + d_h;
            const bool touched = b < 32 && b + d_h > 0;
            all_inside = all_inside && inside[ni];
            cut = cut || (touched && !inside[ni]);
            meets = meets || touched;
        }
    };
    enter_group();
    f32x16 acc[TN][TT];
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int ti = 0; ti < TT; ++ti)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ni][ti][r] = 0.0f;
    u32x4 fw[2][TN], ft[2][TT];
    auto next = [&]() {
        place += step;
        if (place >= period) place -= period;
        if (--rd_left == 0) enter_group();
    };
    auto read = [&](auto setc, auto sc, uint32_t slot) {
        constexpr int Q = decltype(setc)::value, s = decltype(sc)::value;
        if (!meets) {
#pragma unroll
            for (int ti = 0; ti < TT; ++ti) ft[Q][ti] = *(lds_u32x4)(uintptr_t)(a_tok[s] + slot + ti * (32 * 128));
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) fw[Q][ni] = *(lds_u32x4)(uintptr_t)(a_wgt[s] + slot + ni * (32 * 128));
        } else {
            int d0 = place + 16 * 32 * s;
            if (d0 >= period) d0 -= period;
            // Nothing but zeros to multiply with: not with the tokens, which need not be finite.  (Per wave, for the price of an
            // address.  Per block of 32, tokens masked in registers, 4096 tokens, N = 4096 took 29.6 us instead of 26.5; skipped
            // MFMAs make the compiler move the accumulators.)
            const bool idle = all_inside && (at + d0 <= -16 * 32 || at + d0 >= 32 * TN * 32);
#pragma unroll
            for (int ti = 0; ti < TT; ++ti) ft[Q][ti] = *(lds_u32x4)(uintptr_t)(idle ? a_zeros : a_tok[s] + slot + (uint32_t)(ti * (32 * 128)));
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
                int d = at + d0 - 32 * 32 * ni;      // 32 x: where the k-step's columns begin in the block
                d = d < -16 * 32 ? -16 * 32 : d > 32 * 32 ? 32 * 32 : d;
                const uint32_t from = inside[ni] ? a_ones - (uint32_t)d : a_wgt[s] + slot + (uint32_t)(ni * (32 * 128));
                fw[Q][ni] = *(lds_u32x4)(uintptr_t)from;
                if (cut && !inside[ni]) fw[Q][ni] |= *(lds_u32x4)(uintptr_t)(a_ones - (uint32_t)d);
            }
        }
    };
    auto multiply = [&](auto setc, auto&& between) {
        constexpr int Q = decltype(setc)::value;
        static_for<TN>([&](auto ni) {
            static_for<TT>([&](auto ti) {
                constexpr int n = decltype(ni)::value, t = decltype(ti)::value;
                acc[n][t] = X::mfma(fw[Q][n], ft[Q][t], acc[n][t]);
                between(std::integral_constant<int, n * TT + t>{});
            });
        });
    };
    ring_loop<C>(p.n_stages, prepare, request, read, next, multiply);
    const __amdgpu_buffer_rsrc_t rD = make_rsrc((char*)p.out + (t0 * p.ldo + l0) * (int64_t)sizeof(OutT),
                                                ((rows_left - 1) * p.ldo + cols_left) * (int64_t)sizeof(OutT));
    ring_finish<X, OutT, C>(smem, acc, rD, p.ldo, cols_left, wave, wt, wn, kg, lane);
}

// ---------------------------------------------------------------------------------------------
// Weight gradient: BT rows of C x BN columns, contraction over the tokens in stages of CK.
// ---------------------------------------------------------------------------------------------
template <typename X, typename OutT, typename C>
__global__ __launch_bounds__(C::THREADS) void ring_weight_kernel(const BwdArgs p)
{
    constexpr int BT = C::BT, BN = C::BN, TT = C::TT, TN = C::TN, S = C::S, PT = C::PT, PN = C::PN, KSW = C::KSW, CK = C::CK;
    constexpr int PITCH_T = C::PAD_T * 2, PITCH_N = C::PAD_N * 2, PPR_T = PITCH_T / 16, PPR_N = PITCH_N / 16;
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    typedef __attribute__((address_space(3))) unsigned char* lds_u8;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const int tile = tile_of_block(p.m_tiles * p.n_tiles);
    if (tile < 0) return;
    const int nt = tile / p.m_tiles, mt = tile % p.m_tiles;   // the row tiles of one column tile share its G columns
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / (C::WT * C::WN), wt = wave / C::WN % C::WT, wn = wave % C::WN;

    int g = 0;
    while (g + 1 < p.n_groups && nt >= p.tile_start[g + 1]) ++g;
    const int64_t n0 = p.col_start[g] + (int64_t)(nt - p.tile_start[g]) * BN;
    const int cols_left = (int)((p.col_start[g + 1] - n0) > BN ? BN : (p.col_start[g + 1] - n0));
    const int i0 = mt * BT;
    const int rows_left = p.K - i0 > BT ? BT : p.K - i0;
    const int a_off = p.a_off[g];
    const int64_t T = p.T;
    const int64_t c_pitch = p.ldc * 2, g_pitch = p.ldg * 2;

    // ---- requests: piece 64 q + lane of the staged operand in memory order, its row's pieces swizzled ----
    uint32_t vt[PT], vw[PN];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int e = (wave * PT + j) * 64 + lane, row = e / PPR_T, piece = (e % PPR_T) ^ transpose_swz(PITCH_T, row);
        const int i = i0 + piece * 8;                               // row of C
        vt[j] = piece * 8 < rows_left ? (uint32_t)row * (uint32_t)c_pitch + (uint32_t)(i < a_off ? i : i + p.d_h) * 2u : kBadOffset;
    }
#pragma unroll
    for (int j = 0; j < PN; ++j) {
        const int e = (wave * PN + j) * 64 + lane, row = e / PPR_N, piece = (e % PPR_N) ^ transpose_swz(PITCH_N, row);
        vw[j] = piece * 8 < cols_left ? (uint32_t)row * (uint32_t)g_pitch + (uint32_t)piece * 16u : kBadOffset;
    }
    // The descriptors move along with the stages and end with a stage's last token, so that token rows past T read as zero.
    const int n_stages = (int)((T + CK - 1) / CK), n_full = (int)(T / CK), tail = (int)(T % CK);
    const uint32_t c_full = (uint32_t)(CK - 1) * (uint32_t)c_pitch + (uint32_t)p.d_c * 2u;
    const uint32_t c_tail = tail ? (uint32_t)(tail - 1) * (uint32_t)c_pitch + (uint32_t)p.d_c * 2u : 0u;
    const uint32_t g_full = (uint32_t)(CK - 1) * (uint32_t)g_pitch + (uint32_t)cols_left * 2u;
    const uint32_t g_tail = tail ? (uint32_t)(tail - 1) * (uint32_t)g_pitch + (uint32_t)cols_left * 2u : 0u;
    const char* c_ptr = (const char*)p.c;
    const char* g_ptr = (const char*)p.g + n0 * 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8)smem;
    const uint32_t dst_t = lds0 + (uint32_t)(wave * PT * 1024), dst_w = lds0 + (uint32_t)(C::TOK_BYTES + wave * PN * 1024);
    u32x4 rA = make_rsrc_words(c_ptr - CK * c_pitch, c_full), rB = make_rsrc_words(g_ptr - CK * g_pitch, g_full);
    const uint64_t c_step = (uint64_t)(CK * c_pitch), g_step = (uint64_t)(CK * g_pitch);
    int ld_left = n_full + 1;                  // full stages not yet set up, plus one
    auto move = [](u32x4& r, uint64_t step) {
        const uint64_t at = ((uint64_t)r[1] << 32 | r[0]) + step;
        r[0] = (uint32_t)at;
        r[1] = (uint32_t)(at >> 32) & 0xffffu;
    };
    auto prepare = [&]() {
        move(rA, c_step);
        move(rB, g_step);
        if (--ld_left <= 0) {                  // the stage that T cuts, then nothing
            rA[2] = ld_left == 0 ? c_tail : 0u;
            rB[2] = ld_left == 0 ? g_tail : 0u;
        }
    };
    auto request = [&](auto jc, uint32_t slot) {
        constexpr int j = decltype(jc)::value;
        if constexpr (j < PT) lds_dma_imm<1024 * j>(rA, dst_t + slot, vt[j], 0u);
        else lds_dma_imm<1024 * (j - PT)>(rB, dst_w + slot, vw[j - PT], 0u);
    };

    // ---- fragments: transposing reads (see transpose_swz); the swizzle is a constant of the lane ----
    const int c_s = lane & 15, c_q = lane >> 4;
    const int fr_row = 8 * (c_q >> 1) + (c_s >> 2), fr_col = 16 * (c_q & 1) + 4 * (c_s & 3);
    uint32_t a_tok[TT], a_wgt[TN];
#pragma unroll
    for (int ti = 0; ti < TT; ++ti) {
        const int cb = (wt * (32 * TT) + 32 * ti + fr_col) * 2;
        a_tok[ti] = lds0 + (uint32_t)((16 * KSW * kg + fr_row) * PITCH_T + (((cb >> 4) ^ transpose_swz(PITCH_T, fr_row)) << 4) + (cb & 15));
    }
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
        const int cb = (wn * (32 * TN) + 32 * ni + fr_col) * 2;
        a_wgt[ni] = lds0 + (uint32_t)(C::TOK_BYTES + (16 * KSW * kg + fr_row) * PITCH_N + (((cb >> 4) ^ transpose_swz(PITCH_N, fr_row)) << 4) + (cb & 15));
    }
    auto frag = [&](uint32_t addr, int pitch) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)addr);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(addr + 4 * pitch));
        const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
        return (u32x4){lo2[0], lo2[1], hi2[0], hi2[1]};
    };
    // A wave that has a tile to itself sums its even and its odd k-steps apart, so that no float32 sum runs over more than
    // half of the tokens.  (8192 tokens, float32 gradients: 4.0e-7 from 64 bits; in one sum 5.7e-7, in the same 197 us for N = 32768.)
    constexpr int SUMS = C::WK == 1 ? 2 : 1;
    static_assert(SUMS == 1 || KSW % 2 == 0);
    f32x16 acc[SUMS][TN][TT];
#pragma unroll
    for (int q = 0; q < SUMS; ++q)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[q][ni][ti][r] = 0.0f;
    u32x4 fw[2][TN], ft[2][TT];
    auto next = [] {};
    auto read = [&](auto setc, auto sc, uint32_t slot) {
        constexpr int Q = decltype(setc)::value, s = decltype(sc)::value;
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) fw[Q][ni] = frag(a_wgt[ni] + slot + 16 * s * PITCH_N, PITCH_N);
#pragma unroll
        for (int ti = 0; ti < TT; ++ti) ft[Q][ti] = frag(a_tok[ti] + slot + 16 * s * PITCH_T, PITCH_T);
    };
    auto multiply = [&](auto setc, auto&& between) {
        constexpr int Q = decltype(setc)::value;
        static_for<TN>([&](auto ni) {
            static_for<TT>([&](auto ti) {
                constexpr int n = decltype(ni)::value, t = decltype(ti)::value;
                acc[Q % SUMS][n][t] = X::mfma(fw[Q][n], ft[Q][t], acc[Q % SUMS][n][t]);
                between(std::integral_constant<int, n * TT + t>{});
            });
        });
    };
    ring_loop<C>(n_stages, prepare, request, read, next, multiply);
    if constexpr (SUMS == 2) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[0][ni][ti][r] += acc[SUMS - 1][ni][ti][r];
    }
    const __amdgpu_buffer_rsrc_t rD = make_rsrc((char*)p.out + ((int64_t)i0 * p.ldo + n0) * (int64_t)sizeof(OutT),
                                                ((int64_t)(rows_left - 1) * p.ldo + cols_left) * (int64_t)sizeof(OutT));
    ring_finish<X, OutT, C>(smem, acc[0], rD, p.ldo, cols_left, wave, wt, wn, kg, lane);
}

}  // namespace bda
