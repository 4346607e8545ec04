// Forward kernel for 16-bit shapes that the lean streaming kernel does not take (contractions or head widths that
// are not multiples of 64, groups that are not multiples of 256 columns), up to a few rounds of 128 x 128 tiles.
//
//   D[t, n] = ident(t, n) + sum_{k < K} A[t, acol_g(k)] * B[k, n]        (see bda_gemm_kernels.hpp)
//
// Such launches are bound by what a tile takes from its first load to its last store: a tile of 256 x 256 is on
// few compute units and each of its stages has decisions per lane.  Here a workgroup is 8 waves = 2 halves of
// 2 x 2 waves that take alternate chunks of 64 of the contraction and whose float32 sums are added through LDS in a
// fixed order; the first four chunks are requested before the first wait, so a
// contraction of 256 waits for memory once; 64 x 64 tiles leave two workgroups on a compute unit, which cover one
// another's prologue and epilogue.  The identity slice costs no stages: it is loaded as 8 bytes per lane and
// 8 x 32 results while the halves are added, and summed in float32 before the one rounding.
#pragma once
#include <type_traits>

#include "bda_gemm_kernels.hpp"

namespace bda {

template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Tiles are dealt to the dies in contiguous runs (workgroup b runs on die b % 8), so that tiles
// that are neighbours in the run order -- they share one operand -- meet in the same L2.
__device__ __forceinline__ int tile_of_block(int total)
{
    const int per_xcd = (total + kNumXcd - 1) / kNumXcd;
    const int slot = blockIdx.x / kNumXcd;
    const int tile = (blockIdx.x % kNumXcd) * per_xcd + slot;
    return (slot < per_xcd && tile < total) ? tile : -1;
}

// Operands whose contraction index is the slow one in memory keep their rows in LDS, unpadded; their MFMA fragments come from
// ds_read_b64_tr_b16: each lane names four consecutive columns of one row and receives four consecutive rows of one column.
// Piece p (16 bytes) of row r sits at p ^ transpose_swz(r), so that the four rows one such read touches (64 bytes each) fall
// into different quarters of the 256-byte bank line: rows of an odd number of 128 bytes pair up in a line and the pair
// number picks the half; rows of whole lines pick the quarter by their number.  (The counter of bank conflicts: four cycles
// per active one with 8 x 8 blocks transposed in registers, 0.8 with rows padded by 32 bytes, none so.)
__host__ __device__ constexpr int transpose_swz(int pitch, int r) { return pitch % 256 == 128 ? ((r >> 1) & 1) * 4 : (r & 3) * 4; }

template <typename X, typename OutT, int TT, int TN>
__device__ __forceinline__ void mid_epilogue(const f32x16 (&acc)[TN][TT], __amdgpu_buffer_rsrc_t rD, int64_t ldo,
                                             int cols_left, int wt, int wn, int l31, int lhi)
{
    const uint32_t ep_lane = (uint32_t)(wt * (32 * TT) + l31) * (uint32_t)(ldo * sizeof(OutT)) +
                             (uint32_t)(wn * (32 * TN) + lhi * 4) * (uint32_t)sizeof(OutT);
    const uint32_t ep_row_step = 32u * (uint32_t)(ldo * sizeof(OutT));
#pragma unroll
    for (int ti = 0; ti < TT; ++ti) {
        const uint32_t row_off = ep_lane + (uint32_t)ti * ep_row_step;
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const int c0 = ni * 32 + rg * 8;
                if (wn * (32 * TN) + c0 >= cols_left) continue;   // uniform per wave: widths are multiples of 8
                const uint32_t off = row_off + (uint32_t)c0 * (uint32_t)sizeof(OutT);
                if constexpr (sizeof(OutT) == 4) {
                    const float e0 = acc[ni][ti][rg * 4 + 0], e1 = acc[ni][ti][rg * 4 + 1];
                    const float e2 = acc[ni][ti][rg * 4 + 2], e3 = acc[ni][ti][rg * 4 + 3];
                    const f32x4 vf = {e0, e1, e2, e3};
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, vf), rD, off, 0, 0);
                } else {
                    u32x2 v;
                    v[0] = X::pack2(acc[ni][ti][rg * 4 + 0], acc[ni][ti][rg * 4 + 1]);
                    v[1] = X::pack2(acc[ni][ti][rg * 4 + 2], acc[ni][ti][rg * 4 + 3]);
                    __builtin_amdgcn_raw_buffer_store_b64(v, rD, off, 0, 0);
                }
            }
        }
    }
}

// One staged chunk: 4 k-steps of TT x TN MFMAs.  read(ks, fw, ft) fetches the fragments of a step from LDS; they
// are requested a step (one tile per wave: two steps) before their MFMAs, so that the reads' latency runs beside
// the MFMAs instead of between them.
template <typename X, int TT, int TN, typename Read>
__device__ __forceinline__ void mid_mma_chunk(f32x16 (&acc)[TN][TT], Read&& read)
{
    constexpr int AHEAD = TT * TN == 1 ? 2 : 1, SETS = AHEAD + 1;
    u32x4 fw[SETS][TN], ft[SETS][TT];
#pragma unroll
    for (int ks = 0; ks < AHEAD; ++ks) read(ks, fw[ks], ft[ks]);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        if (ks + AHEAD < 4) read(ks + AHEAD, fw[(ks + AHEAD) % SETS], ft[(ks + AHEAD) % SETS]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < TT; ++ti) acc[ni][ti] = X::mfma(fw[ks % SETS][ni], ft[ks % SETS][ti], acc[ni][ti]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Adds half 1's accumulators to half 0's through LDS (all 8 waves call this after the last chunk).
template <int TT, int TN>
__device__ __forceinline__ void mid_reduce_halves(unsigned char* smem, f32x16 (&acc)[TN][TT], int half, int w4, int lane)
{
    __syncthreads();   // every wave is done reading the staged tiles
    float* x = (float*)smem + (w4 * (TT * TN * 16)) * 64 + lane;
    if (half == 1) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) x[((ni * TT + ti) * 16 + r) * 64] = acc[ni][ti][r];
    }
    __syncthreads();
    if (half == 0) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[ni][ti][r] += x[((ni * TT + ti) * 16 + r) * 64];
    }
}


template <int TT, int TN>
struct MidLds {
    static constexpr int BT = 64 * TT, BN = 64 * TN;
    static constexpr int WGT_PITCH = BN * 2;
    static constexpr int TOK_STAGE = BT * kRowBytes, WGT_STAGE = 64 * WGT_PITCH;
    static constexpr int WGT_BASE = 2 * TOK_STAGE;
    static constexpr int HALF = 2 * (TOK_STAGE + WGT_STAGE);
    static constexpr int BYTES = 2 * HALF;
    static_assert(4 * TT * TN * 16 * 64 * 4 <= BYTES, "accumulator exchange must fit the staging memory");
    static_assert(BYTES <= 160 * 1024);
};

template <typename X, typename OutT, int TT, int TN>
__global__ __launch_bounds__(512, TT * TN > 1 ? 2 : 4) void gemm_mid_kernel(const GemmArgs p)
{
    using L = MidLds<TT, TN>;
    constexpr int BT = L::BT, BN = L::BN;
    constexpr int TOK_LOADS = BT / 32;
    constexpr int WGT_PER_ROW = BN / 8, WGT_LOADS = 64 * WGT_PER_ROW / 256, WGT_ROWS_PER_PASS = 256 / WGT_PER_ROW;
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
    typedef __attribute__((address_space(3))) unsigned char* lds_u8;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int tile = tile_of_block(p.m_tiles * p.n_tiles);
    if (tile < 0) return;
    const int mt = tile / p.n_tiles, nt = tile % p.n_tiles;         // the column tiles of one token tile share its rows

    const int tid = threadIdx.x & 255;                              // thread within its half
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave >> 2, w4 = wave & 3;
    const int wt = w4 >> 1, wn = w4 & 1;
    const int l31 = lane & 31, lhi = lane >> 5;
    unsigned char* const lds = smem + half * L::HALF;

    int g = 0;
    while (g + 1 < p.n_groups && nt >= p.tile_start[g + 1]) ++g;
    const int64_t rel0 = (int64_t)(nt - p.tile_start[g]) * BN;      // column inside the group
    const int64_t n0 = p.col_start[g] + rel0;
    const int cols_left = (int)((p.col_start[g + 1] - n0) > BN ? BN : (p.col_start[g + 1] - n0));
    const int64_t t0 = (int64_t)mt * BT;
    const int64_t rows_left = p.M - t0;
    const int a_off = p.a_off[g];

    const __amdgpu_buffer_rsrc_t rA = make_rsrc((const char*)p.A + t0 * p.lda * 2, ((rows_left - 1) * p.lda + p.K + p.a_skip) * 2);
    const __amdgpu_buffer_rsrc_t rB = make_rsrc((const char*)p.B + n0 * 2, ((int64_t)(p.K - 1) * p.ldb + cols_left) * 2);
    const __amdgpu_buffer_rsrc_t rD = make_rsrc((char*)p.D + (t0 * p.ldd + n0) * (int64_t)sizeof(OutT),
                                                ((rows_left - 1) * p.ldd + cols_left) * (int64_t)sizeof(OutT));

    // this thread's pieces: 16 bytes of token rows trow + 32 i, and of weight rows wrow + i rows per pass
    const int tq = tid & 7, trow = tid >> 3;
    const uint32_t a_pitch = (uint32_t)(p.lda * 2), b_pitch = (uint32_t)(p.ldb * 2);
    const uint32_t tok_base = (uint32_t)trow * a_pitch;
    const int wpiece = tid % WGT_PER_ROW, wrow = tid / WGT_PER_ROW;
    const uint32_t wgt_base = wpiece * 8 < cols_left ? (uint32_t)wrow * b_pitch + (uint32_t)wpiece * 16u : kBadOffset;
    const uint32_t wgt_lds = (uint32_t)(wrow * L::WGT_PITCH + ((wpiece ^ transpose_swz(L::WGT_PITCH, wrow)) * 16));
    const int n_chunks = (p.K + 63) >> 6;
    const int n_it = (n_chunks + 1) >> 1;                           // chunks of this half: 2 it + half

    u32x4 tok_reg[2][TOK_LOADS], wgt_reg[2][WGT_LOADS];
    auto load_chunk = [&](auto set, int it) {                       // past the last chunk: nothing (zeros)
        constexpr int S = decltype(set)::value;
        const int kc = 2 * it + half, k = kc * 64 + tq * 8;
        const bool live = kc < n_chunks;
        uint32_t ta = k < p.K ? tok_base + (uint32_t)(k < a_off ? k : k + p.a_skip) * 2u : kBadOffset;
        uint32_t wa = live && wgt_base != kBadOffset ? wgt_base + (uint32_t)(kc * 64) * b_pitch : kBadOffset;
        asm volatile("" : "+v"(ta), "+v"(wa));                      // one load, not one per branch
#pragma unroll
        for (int i = 0; i < TOK_LOADS; ++i)
            tok_reg[S][i] = __builtin_amdgcn_raw_buffer_load_b128(rA, ta == kBadOffset ? ta : ta + (uint32_t)(32 * i) * a_pitch, 0, 0);
#pragma unroll
        for (int i = 0; i < WGT_LOADS; ++i)
            wgt_reg[S][i] = __builtin_amdgcn_raw_buffer_load_b128(rB, wa == kBadOffset ? wa : wa + (uint32_t)(i * WGT_ROWS_PER_PASS) * b_pitch, 0, 0);
    };
    auto store_chunk = [&](auto set) {
        constexpr int S = decltype(set)::value;
        unsigned char* tok_s = lds + S * L::TOK_STAGE;
        unsigned char* wgt_s = lds + L::WGT_BASE + S * L::WGT_STAGE + wgt_lds;
#pragma unroll
        for (int i = 0; i < TOK_LOADS; ++i) *(u32x4*)(tok_s + lds_off(trow + 32 * i, tq)) = tok_reg[S][i];
#pragma unroll
        for (int i = 0; i < WGT_LOADS; ++i) *(u32x4*)(wgt_s + i * WGT_ROWS_PER_PASS * L::WGT_PITCH) = wgt_reg[S][i];
    };

    f32x16 acc[TN][TT];
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int ti = 0; ti < TT; ++ti)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ni][ti][r] = 0.0f;

    // weight fragments: transposing reads, see transpose_swz
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8)lds;
    const int c_s = lane & 15, c_q = lane >> 4;
    const int fr_row = 8 * (c_q >> 1) + (c_s >> 2), fr_col = 16 * (c_q & 1) + 4 * (c_s & 3);
    uint32_t a_wgt[TN];
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
        const int cb = (wn * (32 * TN) + 32 * ni + fr_col) * 2;
        a_wgt[ni] = lds0 + (uint32_t)(L::WGT_BASE + fr_row * L::WGT_PITCH + (((cb >> 4) ^ transpose_swz(L::WGT_PITCH, fr_row)) << 4) + (cb & 15));
    }
    auto wgt_frag = [&](uint32_t addr) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)addr);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(addr + 4 * L::WGT_PITCH));
        const u32x2 lo2 = __builtin_bit_cast(u32x2, lo), hi2 = __builtin_bit_cast(u32x2, hi);
        return (u32x4){lo2[0], lo2[1], hi2[0], hi2[1]};
    };
    const int tok_rd = (wt * (32 * TT) + l31) * kRowBytes + lhi * 16;

    // this half's chunk `it`, in LDS stage and (until stored) register set it % 2
    auto iteration = [&](auto set, int it) {
        constexpr int S = decltype(set)::value;
        load_chunk(set, it + 2);
        const unsigned char* const tok_s = lds + tok_rd + S * L::TOK_STAGE;
        mid_mma_chunk<X, TT, TN>(acc, [&](int ks, u32x4 (&fw)[TN], u32x4 (&ft)[TT]) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) fw[ni] = wgt_frag(a_wgt[ni] + S * L::WGT_STAGE + 16 * ks * L::WGT_PITCH);
#pragma unroll
            for (int ti = 0; ti < TT; ++ti) ft[ti] = *(const u32x4*)(tok_s + ti * 32 * kRowBytes + ks * 32);
        });
        store_chunk(std::integral_constant<int, 1 - S>{});          // into the stage of chunk it - 1, free since the last barrier
        __syncthreads();
    };
    const std::integral_constant<int, 0> set0;
    const std::integral_constant<int, 1> set1;
    load_chunk(set0, 0);
    load_chunk(set1, 1);
    store_chunk(set0);
    __syncthreads();
    // (one way round the loop only, so that the compiler's count of loads in flight is exact)
    for (int it = 0;;) {
        iteration(set0, it);
        if (++it >= n_it) break;
        iteration(set1, it);
        if (++it >= n_it) break;
    }

    // identity slice: columns 8 rg + 4 lhi .. + 3 of each 32 x 32 tile, requested before the halves are added
    u32x2 id[TN][TT][4];
    const bool ident = p.ident && half == 0;
    if (ident) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            const int j0 = a_off + (int)((rel0 + wn * (32 * TN) + ni * 32) % p.d_h);
#pragma unroll
            for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
                    id[ni][ti][rg] = __builtin_amdgcn_raw_buffer_load_b64(
                        rA, (uint32_t)(wt * (32 * TT) + ti * 32 + l31) * a_pitch + (uint32_t)(j0 + rg * 8 + lhi * 4) * 2u, 0, 0);
        }
    }
    mid_reduce_halves<TT, TN>(smem, acc, half, w4, lane);
    if (half != 0) return;
    if (ident) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t v = id[ni][ti][r >> 2][(r >> 1) & 1];
                    acc[ni][ti][r] += X::to_f32((uint16_t)(r & 1 ? v >> 16 : v));
                }
    }
    mid_epilogue<X, OutT, TT, TN>(acc, rD, p.ldd, cols_left, wt, wn, l31, lhi);
}

}  // namespace bda
