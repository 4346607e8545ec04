// General kernels: any element type, shape, pitch and alignment, and every float32 call.  One kernel for the
// three products of the BD K/V projection (out[t, n], gc[t, l] and gC[i, n] below), on the float32 matrix
// instructions:
//
//   Forward   out[t, n] = ident(t, n) + sum_k A[t, acol_g(k)] B[k, n]     (also the dense and the linear layer's)
//   Latent    gc[t, l]  = sum_n G[t, n] Wfull_g[l, n]                      (Wfull: see bda_bwd_kernels.hpp)
//   Weight    gC[i, n]  = sum_t c[t, Bbar_g(i)] G[t, n]
//
// Products and sums are float32: v_mfma_f32_32x32x2 is a chain of float32 FMAs, at twice the rate of the
// vector unit's (256 against 128 FLOP per cycle and compute unit).  16-bit inputs are widened on their way to
// LDS, which is exact.
//
// A workgroup is KS groups of WT x WN waves.  All of them stage a chunk of BK = KS KPG contraction elements,
// group s multiplies elements s KPG .. of every chunk into its own accumulators, and the groups are added
// through LDS in a fixed order at the end.  The groups give a compute unit the waves that a small output tile
// has not (gC of 448 x 1024 is 112 tiles of 64 x 64 over a contraction of thousands), and shorter sums.
// An operand that is contiguous along the contraction lies in LDS as [x][k] and is read as 16 bytes = four
// k-steps; one that is contiguous along the output lies as [k][x] and is read four bytes at a time.  Element e
// of lane half h is contraction element 4 h + e in both.  The pitches (BK + 4 and BX + 8 words, of 64 banks)
// keep either read free of bank conflicts.  LDS carries a quarter of what it could (a 32 x 32 x 2 product
// takes 64 cycles and 512 bytes), so the kernel is bound by the matrix rate; the next chunk is fetched into
// registers meanwhile.  A layer's float32 training step (4096 tokens, d_c = 512, d_h = 64, N = 1024), forward and
// both gradients: 1123 us with vector FMAs, 64 x 64 tiles and no prefetch, 140 us now (42, 49 and 50; 24 each at
// the matrix rate), and half the error against float64.
// VEC: float32 operands and results aligned to 16 bytes with pitches, window, widths and group boundaries of
// multiples of 4, fetched as 16-byte pieces through buffer descriptors that end with the operand; otherwise
// element by element with guards.
#pragma once
#include <type_traits>

#include "bda_gemm_kernels.hpp"
#include "bda_internal.h"

namespace bda {

enum class Product { Forward, Latent, Weight };

struct GeneralArgs {
    const void* tok;                     // operand of the output's rows: A or c; Latent: G
    const void* wgt;                     // operand of its columns: B or C; Weight: G
    void* out;
    int64_t ld_tok, ld_wgt, ld_out;      // in elements
    int64_t rows, len;                   // rows of the output, contraction length
    int d_c;                             // columns of a latent row (K for a dense product)
    int d_h, skip, ident;                // head width; Forward: skipped columns of A, identity slice
    int n_groups, m_tiles, n_tiles;
    int tile_start[kMaxGroups + 1];      // first column tile of each group (Latent: of the one range of columns)
    int64_t col_start[kMaxGroups + 1];   // first column of each group
    int off[kMaxGroups];                 // basis window start of each group
};

template <typename InT>
struct RawOf {
    static __device__ __forceinline__ uint32_t load(const InT* p) { return p->b; }
    static __device__ __forceinline__ float value(uint32_t b) { const InT v{(uint16_t)b}; return load_as_f32(&v); }
    static constexpr uint32_t one = std::is_same_v<InT, RawF16> ? 0x3C00u : 0x3F80u;
};
template <>
struct RawOf<float> {
    static __device__ __forceinline__ uint32_t load(const float* p) { return __builtin_bit_cast(uint32_t, *p); }
    static __device__ __forceinline__ float value(uint32_t b) { return __builtin_bit_cast(float, b); }
    static constexpr uint32_t one = 0x3F800000u;
};

template <Product P, int TT, int TN, int WT, int WN, int KS, int KPG>
struct GeneralTile {
    static constexpr int BT = 32 * TT * WT, BN = 32 * TN * WN, BK = KS * KPG, THREADS = 64 * WT * WN * KS;
    static constexpr bool TOK_KC = P != Product::Weight, WGT_KC = P == Product::Latent;   // contiguous along the contraction
    static constexpr int TOK_PITCH = TOK_KC ? BK + 4 : BT + 8, WGT_PITCH = WGT_KC ? BK + 4 : BN + 8;   // words
    static constexpr int TOK_STAGE = (TOK_KC ? BT : BK) * TOK_PITCH, WGT_STAGE = (WGT_KC ? BN : BK) * WGT_PITCH;
    static constexpr int STAGE = TOK_STAGE + WGT_STAGE;
    static constexpr int TOK_PPR = (TOK_KC ? BK : BT) / 4, WGT_PPR = (WGT_KC ? BK : BN) / 4;           // pieces of four per LDS row
    static constexpr int TOK_RPP = THREADS / TOK_PPR, WGT_RPP = THREADS / WGT_PPR;                     // LDS rows per pass
    static constexpr int TOK_LOADS = (TOK_KC ? BT : BK) / TOK_RPP, WGT_LOADS = (WGT_KC ? BN : BK) / WGT_RPP;
    static constexpr int SETS = TT * TN > 1 || KS == 1 ? 1 : 2;   // register sets: chunks in flight beyond the one being multiplied
    static constexpr int STAGES = KS == 1 ? 1 : 2;                // of LDS
    static constexpr int SUMS = (KS - 1) * WT * WN * TT * TN * 16 * 64;
    static constexpr int LDS_BYTES = 4 * (STAGES * STAGE > SUMS ? STAGES * STAGE : SUMS);
    static_assert(THREADS % TOK_PPR == 0 && THREADS % WGT_PPR == 0 && KPG % 8 == 0 && (KS > 1 || (TT * TN == 1 && KPG == 16)));
    static_assert(TOK_LOADS * TOK_RPP == (TOK_KC ? BT : BK) && WGT_LOADS * WGT_RPP == (WGT_KC ? BN : BK));
    static_assert(LDS_BYTES <= 160 * 1024);
};

template <Product P, typename InT, typename OutT, bool VEC, int TT, int TN, int WT, int WN, int KS, int KPG>
__global__ __launch_bounds__(64 * WT * WN * KS, TT * TN > 1 ? 2 : 4) void general_kernel(const GeneralArgs p)
{
    using L = GeneralTile<P, TT, TN, WT, WN, KS, KPG>;
    using Raw = RawOf<InT>;
    static_assert(!VEC || (std::is_same_v<InT, float> && std::is_same_v<OutT, float>));
    extern __shared__ __attribute__((aligned(16))) float gsm[];

    // Tiles are dealt to the dies in contiguous runs (workgroup b runs on die b % 8); neighbours in a run share
    // the operand of the larger dimension.
    const int64_t total = (int64_t)p.m_tiles * p.n_tiles, block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (block >= total) return;
    const int64_t per_xcd = total / kNumXcd, extra = total % kNumXcd, xcd = block % kNumXcd;
    const int64_t tile = xcd * per_xcd + (xcd < extra ? xcd : extra) + block / kNumXcd;
    const int mt = (int)(P == Product::Weight ? tile % p.m_tiles : tile / p.n_tiles);
    const int nt = (int)(P == Product::Weight ? tile / p.m_tiles : tile % p.n_tiles);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / (WT * WN), w = wave % (WT * WN);
    const int wt = w / WN, wn = w % WN;
    const int l31 = lane & 31, lhi = lane >> 5;

    int g = 0;
    if constexpr (P != Product::Latent)
        while (g + 1 < p.n_groups && nt >= p.tile_start[g + 1]) ++g;
    const int64_t n0 = P == Product::Latent ? (int64_t)nt * L::BN : p.col_start[g] + (int64_t)(nt - p.tile_start[g]) * L::BN;
    const int64_t n_end = P == Product::Latent ? p.d_c : p.col_start[g + 1];
    const int cols_left = (int)(n_end - n0 > L::BN ? L::BN : n_end - n0);
    const int64_t m0 = (int64_t)mt * L::BT;
    const int rows_left = (int)(p.rows - m0 > L::BT ? L::BT : p.rows - m0);
    const int off = P == Product::Latent ? 0 : p.off[g];
    const InT* const tok = (const InT*)p.tok;
    const InT* const wgt = (const InT*)p.wgt;

    // this thread's pieces of either tile: LDS row (+ pass x rows per pass) and first element of four
    const int tok_row = tid / L::TOK_PPR, tok_e = tid % L::TOK_PPR * 4;
    const int wgt_row = tid / L::WGT_PPR, wgt_e = tid % L::WGT_PPR * 4;
    u32x4 tok_reg[L::SETS][L::TOK_LOADS], wgt_reg[L::SETS][L::WGT_LOADS];
    int win_off[L::SETS], win_j[L::SETS]; // Latent: window and window column of the fetched chunks' pieces

    auto latent_col = [&](int k) { return k < off ? k : k + p.skip; };   // of the k-th column outside the window
    auto load_vec = [&](auto set, int64_t k0) {         // past the last chunk: ranges of 0
        constexpr int S = decltype(set)::value % L::SETS;
        const int k_left = (int)(p.len - k0 > L::BK ? L::BK : p.len - k0 > 0 ? p.len - k0 : 0);
        {
            // KC: rows of the tile; otherwise: rows of the chunk
            const __amdgpu_buffer_rsrc_t r = L::TOK_KC
                ? make_rsrc(tok + m0 * p.ld_tok, ((int64_t)(rows_left - 1) * p.ld_tok + (P == Product::Latent ? p.len : p.d_c)) * 4)
                : make_rsrc(tok + k0 * p.ld_tok, ((int64_t)(k_left - 1) * p.ld_tok + p.d_c) * 4);
            const int k = (int)k0 + tok_e;
            const int col = P == Product::Latent ? k : latent_col(P == Product::Weight ? (int)m0 + tok_e : k);
            const bool ok = L::TOK_KC ? tok_e < k_left : tok_e < rows_left;
#pragma unroll
            for (int i = 0; i < L::TOK_LOADS; ++i) {
                uint32_t voff = ok ? (uint32_t)((tok_row + i * L::TOK_RPP) * (int)p.ld_tok + col) * 4u : kBadOffset;
                asm volatile("" : "+v"(voff));               // one load, not one per branch
                tok_reg[S][i] = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
            }
        }
        if constexpr (P == Product::Latent) {
            const __amdgpu_buffer_rsrc_t r = make_rsrc(wgt, ((int64_t)(p.d_c - p.d_h - 1) * p.ld_wgt + p.len) * 4);
            const int n = (int)k0 + wgt_e;
            int gg = 0;
            while (gg + 1 < p.n_groups && n >= p.col_start[gg + 1]) ++gg;
            win_off[S] = p.off[gg];
            win_j[S] = (n - (int)p.col_start[gg]) % p.d_h;
#pragma unroll
            for (int i = 0; i < L::WGT_LOADS; ++i) {
                const int l = (int)n0 + wgt_row + i * L::WGT_RPP;
                const bool ok = wgt_e < k_left && l < p.d_c && (l < win_off[S] || l >= win_off[S] + p.d_h);
                uint32_t voff = ok ? ((uint32_t)(l < win_off[S] ? l : l - p.d_h) * (uint32_t)p.ld_wgt + (uint32_t)n) * 4u : kBadOffset;
                asm volatile("" : "+v"(voff));               // one load, not one per branch
                wgt_reg[S][i] = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
            }
        } else {
            const __amdgpu_buffer_rsrc_t r = make_rsrc(wgt + k0 * p.ld_wgt + n0, ((int64_t)(k_left - 1) * p.ld_wgt + cols_left) * 4);
#pragma unroll
            for (int i = 0; i < L::WGT_LOADS; ++i) {
                uint32_t voff = wgt_e < cols_left ? (uint32_t)((wgt_row + i * L::WGT_RPP) * (int)p.ld_wgt + wgt_e) * 4u : kBadOffset;
                asm volatile("" : "+v"(voff));               // one load, not one per branch
                wgt_reg[S][i] = __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
            }
        }
    };
    auto load_elements = [&](auto set, int64_t k0) {
        constexpr int S = decltype(set)::value % L::SETS;
#pragma unroll
        for (int i = 0; i < L::TOK_LOADS; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = tok_row + i * L::TOK_RPP, x = L::TOK_KC ? r : tok_e + e;
                const int64_t k = k0 + (L::TOK_KC ? tok_e + e : r);
                uint32_t v = 0;
                if (x < rows_left && k < p.len) {
                    if constexpr (P == Product::Forward) v = Raw::load(tok + (m0 + x) * p.ld_tok + latent_col((int)k));
                    else if constexpr (P == Product::Latent) v = Raw::load(tok + (m0 + x) * p.ld_tok + k);
                    else v = Raw::load(tok + k * p.ld_tok + latent_col((int)m0 + x));
                }
                tok_reg[S][i][e] = v;
            }
#pragma unroll
        for (int i = 0; i < L::WGT_LOADS; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = wgt_row + i * L::WGT_RPP, x = L::WGT_KC ? r : wgt_e + e;
                const int64_t k = k0 + (L::WGT_KC ? wgt_e + e : r);
                uint32_t v = 0;
                if (x < cols_left && k < p.len) {
                    if constexpr (P == Product::Latent) {
                        int gg = 0;
                        while (gg + 1 < p.n_groups && k >= p.col_start[gg + 1]) ++gg;
                        const int l = (int)n0 + x, o = p.off[gg];
                        if (l >= o && l < o + p.d_h) v = l - o == (int)((k - p.col_start[gg]) % p.d_h) ? Raw::one : 0u;
                        else v = Raw::load(wgt + (int64_t)(l < o ? l : l - p.d_h) * p.ld_wgt + k);
                    } else {
                        v = Raw::load(wgt + k * p.ld_wgt + n0 + x);
                    }
                }
                wgt_reg[S][i][e] = v;
            }
    };
    auto load_chunk = [&](auto set, int c) {
        if constexpr (VEC) load_vec(set, (int64_t)c * L::BK);
        else load_elements(set, (int64_t)c * L::BK);
    };
    auto store_chunk = [&](auto set) {
        constexpr int S = decltype(set)::value % L::SETS;
        float* const tok_s = gsm + decltype(set)::value * L::STAGE;
        float* const wgt_s = tok_s + L::TOK_STAGE;
#pragma unroll
        for (int i = 0; i < L::TOK_LOADS; ++i) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = Raw::value(tok_reg[S][i][e]);
            *(f32x4*)(tok_s + (tok_row + i * L::TOK_RPP) * L::TOK_PITCH + tok_e) = v;
        }
#pragma unroll
        for (int i = 0; i < L::WGT_LOADS; ++i) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = Raw::value(wgt_reg[S][i][e]);
            if constexpr (VEC && P == Product::Latent) {
                const int x = (int)n0 + wgt_row + i * L::WGT_RPP - win_off[S];   // window row of Wfull, where it is one
                const int d = x >= 0 && x < p.d_h ? x - win_j[S] : -1;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = d == e ? 1.0f : v[e];
            }
            *(f32x4*)(wgt_s + (wgt_row + i * L::WGT_RPP) * L::WGT_PITCH + wgt_e) = v;
        }
    };

    f32x16 acc[TN][TT];
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int ti = 0; ti < TT; ++ti)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ni][ti][r] = 0.0f;

    // four consecutive k-steps of one 32-wide fragment
    auto frag = [&](const float* s, int pitch, bool kc, int x, int k) -> f32x4 {
        if (kc) return *(const f32x4*)(s + x * pitch + k);
        return (f32x4){s[k * pitch + x], s[(k + 1) * pitch + x], s[(k + 2) * pitch + x], s[(k + 3) * pitch + x]};
    };
    const int n_chunks = (int)((p.len + L::BK - 1) / L::BK);
    f32x4 fw[2][TN], ft[2][TT];                         // fragments of one step and the next
    auto read = [&](const float* tok_s, int s) {
        const float* const wgt_s = tok_s + L::TOK_STAGE;
        const int k = kg * KPG + 8 * s + 4 * lhi;
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) fw[s & 1][ni] = frag(wgt_s, L::WGT_PITCH, L::WGT_KC, (wn * TN + ni) * 32 + l31, k);
#pragma unroll
        for (int ti = 0; ti < TT; ++ti) ft[s & 1][ti] = frag(tok_s, L::TOK_PITCH, L::TOK_KC, (wt * TT + ti) * 32 + l31, k);
    };
    auto multiply = [&](int s, auto&& sum) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int ti = 0; ti < TT; ++ti)
                    sum(ni, ti) = VEC ? __builtin_amdgcn_mfma_f32_32x32x2f32(fw[s & 1][ni][e], ft[s & 1][ti][e], sum(ni, ti), 0, 0, 0)
                                      : __builtin_amdgcn_mfma_f32_32x32x2f32(ft[s & 1][ti][e], fw[s & 1][ni][e], sum(ni, ti), 0, 0, 0);
    };
    // Chunk c, in LDS half c % 2 (and, until it was stored there, register set c % SETS).  Where a wave has one
    // 32 x 32 tile the fragments of a step are requested before the products of the step before it; four tiles
    // give the compiler enough products between two steps' reads.
    auto iteration = [&](auto set, int c) {
        constexpr int S = decltype(set)::value;
        constexpr bool AHEAD = L::SETS == 2;
        const float* const tok_s = gsm + S * L::STAGE;
        if (AHEAD) read(tok_s, 0);
        load_chunk(std::integral_constant<int, (S + L::SETS) % 2>{}, c + L::SETS);
#pragma unroll
        for (int s = 0; s < KPG / 8; ++s) {
            if (!AHEAD) read(tok_s, s);
            else if (s + 1 < KPG / 8) read(tok_s, s + 1);
            else store_chunk(std::integral_constant<int, 1 - S>{});   // into the half of chunk c - 1, free since the last barrier
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
            multiply(s, [&](int ni, int ti) -> f32x16& { return acc[ni][ti]; });
            if (AHEAD) __builtin_amdgcn_sched_barrier(0);
        }
        if (!AHEAD) store_chunk(std::integral_constant<int, 1 - S>{});
        __syncthreads();
    };
    const std::integral_constant<int, 0> set0;
    const std::integral_constant<int, 1> set1;
    load_chunk(set0, 0);
    if constexpr (L::STAGES == 1) {
        // a chunk or a few: as little code as there can be (a launch of one chunk pays for fetching it).  Each of a chunk's
        // two steps has a sum of its own, which is added to the total: sums of 8, as short as the k-groups of the other
        // tiles have them or shorter.
        for (int c = 0;;) {
            store_chunk(set0);
            __syncthreads();
            if (++c < n_chunks) load_chunk(set0, c);
            f32x16 sums[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
#pragma unroll
                for (int r = 0; r < 16; ++r) sums[s][r] = 0.0f;
                read(gsm, s);
                multiply(s, [&](int, int) -> f32x16& { return sums[s]; });
            }
            acc[0][0] += sums[0] + sums[1];
            if (c >= n_chunks) break;
            __syncthreads();
        }
    } else {
        if (L::SETS == 2) load_chunk(set1, 1);
        store_chunk(set0);
        __syncthreads();
        // (one way round the loop only, so that the compiler's count of loads in flight is exact)
        if (n_chunks > 0)
            for (int c = 0;;) {
                iteration(set0, c);
                if (++c >= n_chunks) break;
                iteration(set1, c);
                if (++c >= n_chunks) break;
            }
    }

    if constexpr (KS > 1) {
        auto slot = [&](int s) { return gsm + ((s - 1) * WT * WN + w) * (TT * TN * 16 * 64) + lane; };
        if (kg > 0) {
            float* const x = slot(kg);
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[((ni * TT + ti) * 16 + r) * 64] = acc[ni][ti][r];
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll 1
        for (int s = 1; s < KS; ++s) {
            const float* const x = slot(s);
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[ni][ti][r] += x[((ni * TT + ti) * 16 + r) * 64];
        }
    }

    if constexpr (VEC) {
        // a lane holds columns 8 rg + 4 lhi .. + 3 of row l31 of each 32 x 32 tile
#pragma unroll
        for (int ti = 0; ti < TT; ++ti) {
            const int row = (wt * TT + ti) * 32 + l31;
            if (row >= rows_left) continue;
            const InT* const a_row = tok + (m0 + row) * p.ld_tok + off;    // Forward: the row's window
            OutT* const o_row = (OutT*)p.out + (m0 + row) * p.ld_out + n0;
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    const int col = (wn * TN + ni) * 32 + rg * 8 + lhi * 4;
                    if (col >= cols_left) continue;                        // widths are multiples of four
                    const float e0 = acc[ni][ti][rg * 4 + 0], e1 = acc[ni][ti][rg * 4 + 1];
                    const float e2 = acc[ni][ti][rg * 4 + 2], e3 = acc[ni][ti][rg * 4 + 3];
                    f32x4 v = {e0, e1, e2, e3};
                    if (P == Product::Forward && p.ident) {
                        const f32x4 id = *(const f32x4*)(a_row + (int)((n0 - p.col_start[g] + col) % p.d_h));
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += id[e];
                    }
                    *(f32x4*)(o_row + col) = v;
                }
        }
    } else {
        // a lane holds rows 8 rg + 4 lhi + e of column l31: one store is two rows of 32 consecutive elements (with the
        // VEC kernels' order an element of each of 32 rows: bf16, 8192 x 8001 over 8 elements 299 us against 57)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) {
            const int col = (wn * TN + ni) * 32 + l31;
            if (col >= cols_left) continue;
            const int j = P == Product::Forward && p.ident ? (int)((n0 - p.col_start[g] + col) % p.d_h) : 0;
            const InT* const a_col = tok + m0 * p.ld_tok + off + j;        // Forward: the column of the window
            OutT* const o_col = (OutT*)p.out + m0 * p.ld_out + n0 + col;
#pragma unroll
            for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = (wt * TT + ti) * 32 + (r >> 2) * 8 + lhi * 4 + (r & 3);
                    if (row >= rows_left) continue;
                    float v = acc[ni][ti][r];
                    if (P == Product::Forward && p.ident) v += load_as_f32(a_col + row * p.ld_tok);
                    store_from_f32(o_col + row * p.ld_out, v);
                }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Launch.  Workgroup tiles, in 32 x 32 units per wave, waves, k-groups and contraction elements per group and
// chunk (VEC kernels; the element-wise ones have 64 x 64 and 32 x 32 with two and eight groups, and the short one):
//   0   128 x 128   2 x 2 per wave, 2 x 2 waves, 2 groups of 32
//   1    64 x  64   1 x 1, 2 x 2, 2 groups of 32
//   2    64 x  32   1 x 1, 2 x 1, 4 groups of 16
//   3    32 x  32   1 x 1, 1 x 1, 8 groups of 16
//   4    64 x  64   1 x 1, 2 x 2, 1 group of 16: contractions of less than a chunk of the others, or of a few
// ---------------------------------------------------------------------------------------------
constexpr int kGeneralTiles = 4, kGeneralShort = 4;
constexpr int kGeneralBT[] = {128, 64, 64, 32, 64}, kGeneralBN[] = {128, 64, 32, 32, 64};

// The tile with the least time over the 256 compute units: rounds x matrix time x a factor for what the smaller
// ones spend beside it.  Measured, us (float32, 4096 tokens, d_c = 512, d_h = 64, N = 1024; tiles 0 / 1 / 2 / 3):
// forward (256 .. 4096 tiles) 42 / 46 / 53 / 71, latent gradient (128 .. 2048) 82 / 55 / 63 / 74, weight gradient
// (32 .. 448) 280 / 87 / 51 / 48; one token, forward 34 / 13 / 9.4 / 7.8.
// Up to 48 contraction elements (64 element by element) the k-groups have little to share and a launch is its loads
// and stores.  Short tile against the best of the others (geometric means over outputs of 1 x 64 .. 8192 x 8001;
// float32 in 16-byte pieces / element by element): 8 elements 0.75 / 0.56, 32 0.87 / 0.69, 48 0.91 / 0.73, 64 1.05 / 0.85.
// Element by element and with more than 256 tiles of 64 x 64, longer contractions take it too: there the loads are the
// time, the other tiles fetch up to two chunks of 64 or 128 for little more than one, and 32 x 32 tiles fetch everything
// twice as often.  us, the others / short: forward, bf16, 95 elements and 288 tiles 27.8 / 13.7, 107 and 532 40.0 / 19.2;
// float32, 125 and 517 35.1 / 20.6; f16, 226 and 324 35.3 / 24.6.  The limits are where it stops being faster (188 and 363
// 19.6 / 21.7, 252 and 378 23.9 / 26.0); the latent gradient's are lower for its look at the windows (100 and 384
// 17.4 / 21.8, 201 and 280 35.3 / 37.4; but 92 and 1115 41.6 / 29.9, 150 and 1032 58.8 / 45.8).
constexpr double kGeneralCost[kGeneralTiles] = {1.4, 1.6, 1.8, 2.2};
inline int general_tile(Product prod, int64_t rows, int64_t len, const int64_t* group_cols, int G, bool vec)
{
    if (len <= (vec ? 48 : 64)) return kGeneralShort;
    int best = 0;
    double best_cost = 0.0;
    for (int i = 0; i < kGeneralTiles; ++i) {
        if (!vec && i != 1 && i != 3) continue;
        int64_t nt = 0;
        for (int g = 0; g < G; ++g) nt += (group_cols[g] + kGeneralBN[i] - 1) / kGeneralBN[i];
        const int64_t tiles = (rows + kGeneralBT[i] - 1) / kGeneralBT[i] * nt;
        const double cost = (double)((tiles + 255) / 256) * kGeneralBT[i] * kGeneralBN[i] * kGeneralCost[i];
        if (best_cost == 0.0 || cost < best_cost) { best_cost = cost; best = i; }
    }
    if (!vec) {
        int64_t tiles = 0;
        for (int g = 0; g < G; ++g) tiles += (rows + 63) / 64 * ((group_cols[g] + 63) / 64);
        const int most = prod == Product::Latent ? (best == 3 || tiles > 512 ? 160 : 80) : best == 3 ? 300 : tiles <= 512 ? 112 : 200;
        if (tiles > 256 && len <= most) return kGeneralShort;
    }
    return best;
}

inline void general_tiles(GeneralArgs& a, const int64_t* group_cols, int G, int tile)
{
    a.tile_start[0] = 0;
    for (int g = 0; g < G; ++g) a.tile_start[g + 1] = a.tile_start[g] + (int)((group_cols[g] + kGeneralBN[tile] - 1) / kGeneralBN[tile]);
    a.n_tiles = a.tile_start[G];
    a.m_tiles = (int)((a.rows + kGeneralBT[tile] - 1) / kGeneralBT[tile]);
}

// 16-byte pieces throughout, and 32-bit offsets inside a tile, a chunk (256 rows at most) and, for Latent, all of C.
inline bool general_vec(const GeneralArgs& a, Product prod, const int64_t* group_cols, int G)
{
    const int64_t max_ld = (int64_t)1 << 20;
    bool ok = aligned(a.tok, 16) && aligned(a.wgt, 16) && aligned(a.out, 16) && a.ld_tok % 4 == 0 && a.ld_wgt % 4 == 0 &&
              a.ld_out % 4 == 0 && a.ld_tok < max_ld && a.ld_wgt < max_ld && a.d_c % 4 == 0 && a.d_h % 4 == 0 && a.skip % 4 == 0;
    if (prod == Product::Forward) ok = ok && a.len % 4 == 0;
    if (prod == Product::Latent) ok = ok && (int64_t)(a.d_c - a.d_h) * a.ld_wgt * 4 < ((int64_t)1 << 31);
    for (int g = 0; g < a.n_groups; ++g) ok = ok && a.off[g] % 4 == 0 && a.col_start[g + 1] % 4 == 0;
    for (int g = 0; g < G; ++g) ok = ok && group_cols[g] % 4 == 0;
    return ok;
}

template <Product P, int TILE, typename F>
auto with_general_tile(F&& f)
{
    if constexpr (TILE == 0) return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{},
                                      std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{}, std::integral_constant<int, 32>{});
    else if constexpr (TILE == 1) return f(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{},
                                           std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{}, std::integral_constant<int, 32>{});
    else if constexpr (TILE == 2) return f(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{},
                                           std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{}, std::integral_constant<int, 16>{});
    else if constexpr (TILE == 3) return f(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{},
                                           std::integral_constant<int, 1>{}, std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{});
    else return f(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{},
                  std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
}

// Workgroups of a launch: one per tile (a few more where they do not fit one grid dimension).
inline dim3 general_grid(const GeneralArgs& a)
{
    const int64_t total = (int64_t)a.m_tiles * a.n_tiles, x = total < (1 << 20) ? total : 1 << 20;
    return dim3((uint32_t)x, (uint32_t)((total + x - 1) / x));
}

// launch(kernel, threads, lds bytes, limit state, tile): makes the launch, or describes it.
template <Product P, typename InT, typename OutT, bool VEC, int TILE, typename Launch>
int launch_general_tile(Launch&& launch)
{
    return with_general_tile<P, TILE>([&](auto tt, auto tn, auto wt, auto wn, auto ks, auto kpg) {
        static LdsLimitState once;
        using L = GeneralTile<P, tt.value, tn.value, wt.value, wn.value, ks.value, kpg.value>;
        static_assert(L::BT == kGeneralBT[TILE] && L::BN == kGeneralBN[TILE]);
        return launch(general_kernel<P, InT, OutT, VEC, tt.value, tn.value, wt.value, wn.value, ks.value, kpg.value>, (int)L::THREADS,
                      (int)L::LDS_BYTES, once, TILE);
    });
}

template <Product P, typename InT, typename OutT, typename Launch>
int launch_general_typed(GeneralArgs& a, const int64_t* group_cols, int G, Launch&& launch)
{
    bool vec = false;
    if constexpr (std::is_same_v<InT, float>) vec = general_vec(a, P, group_cols, G);
    const int tile = general_tile(P, a.rows, a.len, group_cols, G, vec);
    general_tiles(a, group_cols, G, tile);
    if constexpr (std::is_same_v<InT, float>)
        if (vec) {
            if (tile == 0) return launch_general_tile<P, InT, OutT, true, 0>(launch);
            if (tile == 1) return launch_general_tile<P, InT, OutT, true, 1>(launch);
            if (tile == 2) return launch_general_tile<P, InT, OutT, true, 2>(launch);
            if (tile == 3) return launch_general_tile<P, InT, OutT, true, 3>(launch);
            return launch_general_tile<P, InT, OutT, true, 4>(launch);
        }
    if (tile == 1) return launch_general_tile<P, InT, OutT, false, 1>(launch);
    if (tile == 3) return launch_general_tile<P, InT, OutT, false, 3>(launch);
    return launch_general_tile<P, InT, OutT, false, 4>(launch);
}

// Fills in the tile grid of `a` and calls `launch` with the kernel for these types.
template <Product P, typename Launch>
int launch_general(GeneralArgs& a, const int64_t* group_cols, int G, int dtype, int out_dtype, Launch&& launch)
{
    if ((a.rows + 63) / 64 > 65535) return fail(BDA_EINVAL, "general kernel: too many rows (%lld)", (long long)a.rows);
    if (dtype == BDA_F32 && out_dtype == BDA_F32) return launch_general_typed<P, float, float>(a, group_cols, G, launch);
    if (dtype == BDA_F16 && out_dtype == BDA_F16) return launch_general_typed<P, RawF16, RawF16>(a, group_cols, G, launch);
    if (dtype == BDA_F16 && out_dtype == BDA_F32) return launch_general_typed<P, RawF16, float>(a, group_cols, G, launch);
    if (dtype == BDA_BF16 && out_dtype == BDA_BF16) return launch_general_typed<P, RawBF16, RawBF16>(a, group_cols, G, launch);
    if (dtype == BDA_BF16 && out_dtype == BDA_F32) return launch_general_typed<P, RawBF16, float>(a, group_cols, G, launch);
    return fail(BDA_EDTYPE, "unsupported element types %d/%d", dtype, out_dtype);
}

}  // namespace bda
