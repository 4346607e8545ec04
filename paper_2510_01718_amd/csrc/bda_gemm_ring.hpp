// Forward kernel for 16-bit shapes that the lean streaming kernel does not take, from about a round of its tiles up.
//
//   D[t, n] = ident(t, n) + sum_{k < K} A[t, acol_g(k)] * B[k, n]        (see bda_gemm_kernels.hpp)
//
// The gradients' ring (bda_ring.hpp): stages of 64 along the contraction, token rows of 128 bytes as they lie, weight rows
// transposed by the LDS read; two halves of 2 x 2 waves take half of every stage each, so a float32 sum is as long as in
// gemm_mid_kernel.  The identity slice is loaded as 8 bytes per lane and 8 x 32 results beside the sum of the halves and added
// in float32 before the one rounding; results leave in whole lines.
// Most contractions here are 2 .. 10 stages, so that a tile is as much its first requests and its stores as its products: two
// workgroups share a compute unit and cover one another's.  (Longer ones come too, products without an identity slice above all:
// the time grows by 0.0025 us a tile and stage up to the 64 stages measured.)
// Bound there by those latencies still (MFMA pipes busy 16 % of the time).  Against 64 x 64
// tiles copied through registers and the streaming kernel: T = 3001, K = 288, N = 2304, float32 results 23.8 -> 14.3 us; T = 2720,
// K = 384, N = 2432 23.1 -> 13.3; T = 868, K = 352, N = 16640 41 -> 27.
#pragma once
#include "bda_ring.hpp"

namespace bda {

template <typename X, typename OutT, typename C>
__global__ __launch_bounds__(C::THREADS, 4) void gemm_ring_kernel(const GemmArgs p)
{
    constexpr int BT = C::BT, BN = C::BN, TT = C::TT, TN = C::TN, PT = C::PT, PN = C::PN, KSW = C::KSW;
    constexpr int PITCH_N = BN * 2, PPR_N = PITCH_N / 16;
    static_assert(C::CK == 64 && C::WK == 2 && C::S == 2 && TN == 2 && TT % 2 == 0);
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    typedef __attribute__((address_space(3))) unsigned char* lds_u8;
    typedef __attribute__((address_space(3))) const u32x4* lds_u32x4;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const int tile = tile_of_block(p.m_tiles * p.n_tiles);
    if (tile < 0) return;
    const int mt = tile / p.n_tiles, nt = tile % p.n_tiles;         // the column tiles of one token tile share its rows
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / (C::WT * C::WN), wt = wave / C::WN % C::WT, wn = wave % C::WN;
    const int l31 = lane & 31, lhi = lane >> 5;

    int g = 0;
    while (g + 1 < p.n_groups && nt >= p.tile_start[g + 1]) ++g;
    const int64_t rel0 = (int64_t)(nt - p.tile_start[g]) * BN;      // column inside the group
    const int64_t n0 = p.col_start[g] + rel0;
    const int cols_left = (int)((p.col_start[g + 1] - n0) > BN ? BN : (p.col_start[g + 1] - n0));
    const int64_t t0 = (int64_t)mt * BT;
    const int64_t rows_left = p.M - t0;
    const int a_off = p.a_off[g], a_skip = p.a_skip, K = p.K;
    const int64_t a_range = ((rows_left - 1) * p.lda + K + a_skip) * 2;
    const u32x4 rA = make_rsrc_words((const char*)p.A + t0 * p.lda * 2, a_range);
    const u32x4 rB = make_rsrc_words((const char*)p.B + n0 * 2, ((int64_t)(K - 1) * p.ldb + cols_left) * 2);
    const uint32_t a_pitch = (uint32_t)(p.lda * 2), b_pitch = (uint32_t)(p.ldb * 2);

    // ---- requests: token rows as in ring_latent_kernel, weight rows as in ring_weight_kernel ----
    const int lrow = lane >> 3, lpos = lane & 7;
    uint32_t row_t[PT], vw[PN], xt[PT], xw[PN];
    int k_t[PT];                               // the piece's first k of the next stage
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        const int row = 8 * (wave * PT + j) + lrow;
        row_t[j] = (uint32_t)row * a_pitch;
        k_t[j] = (lpos ^ tok_swz<64>(row & 15)) * 8;
    }
#pragma unroll
    for (int j = 0; j < PN; ++j) {
        const int e = (wave * PN + j) * 64 + lane, row = e / PPR_N, piece = (e % PPR_N) ^ transpose_swz(PITCH_N, row);
        vw[j] = piece * 8 < cols_left ? (uint32_t)row * b_pitch + (uint32_t)piece * 16u : kBadOffset;
    }
    uint32_t w_at = 0;                         // bytes from the first weight row to the stage's
    auto prepare = [&]() {
        const bool live = w_at < kBadOffset;   // (a stage past the last reads zeros: its rows lie beyond both ranges)
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int k = k_t[j];
            xt[j] = k < K ? row_t[j] + (uint32_t)(k < a_off ? k : k + a_skip) * 2u : kBadOffset;
            k_t[j] = k + 64;
        }
#pragma unroll
        for (int j = 0; j < PN; ++j) xw[j] = live && vw[j] != kBadOffset ? vw[j] + w_at : kBadOffset;
        if (live) w_at += 64u * b_pitch;
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8)smem;
    const uint32_t dst_t = lds0 + (uint32_t)(wave * PT * 1024), dst_w = lds0 + (uint32_t)(C::TOK_BYTES + wave * PN * 1024);
    auto request = [&](auto jc, uint32_t slot) {
        constexpr int j = decltype(jc)::value;
        if constexpr (j < PT) lds_dma_imm<1024 * j>(rA, dst_t + slot, xt[j], 0u);
        else lds_dma_imm<1024 * (j - PT)>(rB, dst_w + slot, xw[j - PT], 0u);
    };

    // ---- fragments ----
    uint32_t a_tok[KSW], a_wgt[TN];
#pragma unroll
    for (int s = 0; s < KSW; ++s)
        a_tok[s] = lds0 + (uint32_t)((wt * (32 * TT) + l31) * 128 + ((((kg * KSW + s) * 2 + lhi) ^ tok_swz<64>(l31 & 15)) << 4));
    const int c_s = lane & 15, c_q = lane >> 4;
    const int fr_row = 8 * (c_q >> 1) + (c_s >> 2), fr_col = 16 * (c_q & 1) + 4 * (c_s & 3);
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
        const int cb = (wn * (32 * TN) + 32 * ni + fr_col) * 2;
        a_wgt[ni] = lds0 + (uint32_t)(C::TOK_BYTES + (16 * KSW * kg + fr_row) * PITCH_N + (((cb >> 4) ^ transpose_swz(PITCH_N, fr_row)) << 4) + (cb & 15));
    }
    auto frag = [&](uint32_t addr) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)addr);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(addr + 4 * PITCH_N));
        const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
        return (u32x4){lo2[0], lo2[1], hi2[0], hi2[1]};
    };
    f32x16 acc[TN][TT];
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int ti = 0; ti < TT; ++ti)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ni][ti][r] = 0.0f;
    u32x4 fw[2][TN], ft[2][TT];
    auto read = [&](auto setc, auto sc, uint32_t slot) {
        constexpr int Q = decltype(setc)::value, s = decltype(sc)::value;
#pragma unroll
        for (int ti = 0; ti < TT; ++ti) ft[Q][ti] = *(lds_u32x4)(uintptr_t)(a_tok[s] + slot + ti * (32 * 128));
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) fw[Q][ni] = frag(a_wgt[ni] + slot + 16 * s * PITCH_N);
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
    ring_loop<C>((K + 63) >> 6, prepare, request, read, [] {}, multiply);

    // identity slice of the blocks that this wave keeps: columns 8 rg + 4 lhi .. + 3 of each 32 x 32 tile
    constexpr int KEPT = TT / 2;
    const int row0 = wt * (32 * TT) + (kg == 1 ? 32 * KEPT : 0);
    wait_vmcnt<0>();                           // requests past the last stage still write zeros to the ring
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rI = make_rsrc((const char*)p.A + t0 * p.lda * 2, a_range);
    u32x2 id[TN][KEPT][4];
    if (p.ident) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            const int j0 = a_off + (int)((rel0 + wn * (32 * TN) + ni * 32) % p.d_h);
#pragma unroll
            for (int ti = 0; ti < KEPT; ++ti)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
                    id[ni][ti][rg] = __builtin_amdgcn_raw_buffer_load_b64(rI, (uint32_t)(row0 + ti * 32 + l31) * a_pitch + (uint32_t)(j0 + rg * 8 + lhi * 4) * 2u, 0, 0);
        }
    }
    ring_reduce<C>(smem, acc, kg, wt * C::WN + wn, lane);
    if (p.ident) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < KEPT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t v = id[ni][ti][r >> 2][(r >> 1) & 1];
                    acc[ni][ti][r] += X::to_f32((uint16_t)(r & 1 ? v >> 16 : v));
                }
    }
    const __amdgpu_buffer_rsrc_t rD = make_rsrc((char*)p.D + (t0 * p.ldd + n0) * (int64_t)sizeof(OutT),
                                                ((rows_left - 1) * p.ldd + cols_left) * (int64_t)sizeof(OutT));
#pragma unroll
    for (int ti = 0; ti < KEPT; ++ti)
        ring_store<X, OutT, kStreamStoreAux>(smem + wave * 4096, acc[0][ti], acc[1][ti], rD, (uint32_t)(p.ldd * sizeof(OutT)), row0 + 32 * ti,
                                             wn * (32 * TN), cols_left, lane);
}

}  // namespace bda
