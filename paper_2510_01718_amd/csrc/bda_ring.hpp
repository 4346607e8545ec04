// Matrix products from a ring of LDS stages that DMA fills: tile shapes, main loop, sum over the waves that share a tile and
// stores, for the gradient kernels and the forward kernel of 16-bit shapes off the 64 grid.
#pragma once
#include <type_traits>

#include "bda_gemm_mid.hpp"
#include "bda_gemm_plain.hpp"

namespace bda {

// A workgroup's tile: BT x BN outputs, rows along the MFMA's columns; WT x WN waves side by side, each of them WK times
// for a share of every stage's contraction; stages of CK elements in a ring of S slots.
template <int BT_, int BN_, int WT_, int WN_, int WK_, int CK_, int S_>
struct RingShape {
    static constexpr int BT = BT_, BN = BN_, WT = WT_, WN = WN_, WK = WK_, CK = CK_, S = S_;
    static constexpr int NW = WT * WN * WK, THREADS = 64 * NW;
    static constexpr int TT = BT / (32 * WT), TN = BN / (32 * WN);
    static constexpr int KSW = CK / 16 / WK;                         // k-steps of 16 per wave and stage
    static constexpr int PAD_T = BT == 192 && CK == 32 ? 256 : BT, PAD_N = BN;   // (so that the requests divide evenly)
    static constexpr int PT = PAD_T * CK * 2 / 1024 / NW, PN = PAD_N * CK * 2 / 1024 / NW;   // 1 KiB requests per wave and stage
    static constexpr int TOK_BYTES = PAD_T * CK * 2, STAGE = TOK_BYTES + PAD_N * CK * 2;
    static constexpr int BYTES = S * STAGE;
    static constexpr int ACC_BYTES = TT * TN * 16 * 64 * 4;          // a wave's accumulators
    static_assert(BT % (32 * WT) == 0 && BN % (32 * WN) == 0 && CK % (16 * WK) == 0 && S >= 2);
    static_assert(PT * NW * 1024 == TOK_BYTES && PN * NW * 1024 == STAGE - TOK_BYTES, "requests divide evenly");
    static_assert(WK == 1 || ((WK == 2 || WK == 4 || WK == 8) && WT * WN * (WK / 2) * ACC_BYTES <= BYTES), "accumulator exchange");
    static_assert(NW * 4096 <= BYTES && BYTES <= 160 * 1024);
};

// A value that is the same in every lane, in a scalar register for certain.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Adds the accumulators of the WK waves that share a tile through LDS (every wave calls this with nothing in flight).
// Afterwards waves kg = 0 and 1 hold the sums of the lower and the upper half of the token blocks in their first
// accumulators; the order of the additions is fixed.
template <typename C, typename Acc>
__device__ __forceinline__ void ring_reduce(unsigned char* smem, Acc& acc, int kg, int tile_wave, int lane)
{
    constexpr int TT = C::TT, TN = C::TN, TILES = C::WT * C::WN;
#pragma unroll
    for (int n = C::WK / 2; n >= 2; n /= 2) {                        // groups n .. 2 n - 1 -> 0 .. n - 1
        float* x = (float*)(smem + ((kg & (n - 1)) * TILES + tile_wave) * C::ACC_BYTES) + lane;
        if (kg >= n && kg < 2 * n) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                    for (int r = 0; r < 16; ++r) x[((ni * TT + ti) * 16 + r) * 64] = acc[ni][ti][r];
        }
        __syncthreads();
        if (kg < n) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int ti = 0; ti < TT; ++ti)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[ni][ti][r] += x[((ni * TT + ti) * 16 + r) * 64];
        }
        __syncthreads();
    }
    if constexpr (C::WK >= 2) {                                      // groups 0 and 1 keep a half of the token blocks each
        constexpr int HT = TT / 2;
        float* x = (float*)(smem + tile_wave * C::ACC_BYTES) + lane;
        float* const mine = x + (kg == 1 ? TN * HT * 16 * 64 : 0);
        float* const theirs = x + (kg == 1 ? 0 : TN * HT * 16 * 64);
        // (selected value by value: a branch per group makes the compiler index the accumulators, which puts them in memory)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int ti = 0; ti < HT; ++ti)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float lo = acc[ni][ti][r], hi = acc[ni][ti + HT][r];
                    acc[ni][ti][r] = kg == 1 ? hi : lo;
                    acc[ni][ti + HT][r] = kg == 1 ? lo : hi;
                }
        if (kg < 2) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int ti = 0; ti < HT; ++ti)
#pragma unroll
                    for (int r = 0; r < 16; ++r) theirs[((ni * HT + ti) * 16 + r) * 64] = acc[ni][ti + HT][r];
        }
        __syncthreads();
        if (kg < 2) {
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int ti = 0; ti < HT; ++ti)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[ni][ti][r] += mine[((ni * HT + ti) * 16 + r) * 64];
        }
        __syncthreads();
    }
}

// Stores a wave's 32 x 64 block (two accumulators side by side) through 4 KiB of LDS of its own, so that eight lanes
// write a 128-byte line; float32 results 32 columns at a time.  row0 / col0: of the block inside the tile.
template <typename X, typename OutT, int AUX = 0>
__device__ __forceinline__ void ring_store(unsigned char* stag, const f32x16& a0, const f32x16& a1, __amdgpu_buffer_rsrc_t rD, uint32_t pitch,
                                           int row0, int col0, int cols_left, int lane)
{
    const int e31 = lane & 31, st_sw = (e31 ^ (e31 >> 3)) & 7, st_wr = e31 * 128, rd_row = lane >> 3, rd_chunk = lane & 7;
    if constexpr (sizeof(OutT) == 4) {
#pragma unroll
        for (int nn = 0; nn < 2; ++nn) {
            const f32x16& a = nn ? a1 : a0;
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const f32x4 v = {a[rg * 4 + 0], a[rg * 4 + 1], a[rg * 4 + 2], a[rg * 4 + 3]};
                *(u32x4*)(stag + st_wr + (((2 * rg + (lane >> 5)) ^ st_sw) << 4)) = __builtin_bit_cast(u32x4, v);
            }
            const int c = col0 + nn * 32 + rd_chunk * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = j * 8 + rd_row;
                const u32x4 v = *(const u32x4*)(stag + row * 128 + ((rd_chunk ^ ((row ^ (row >> 3)) & 7)) << 4));
                uint32_t off = c < cols_left ? (uint32_t)(row0 + row) * pitch + (uint32_t)c * 4u : kBadOffset;
                asm volatile("" : "+v"(off));
                __builtin_amdgcn_raw_buffer_store_b128(v, rD, off, 0, AUX);
            }
        }
    } else {
#pragma unroll
        for (int nn = 0; nn < 2; ++nn) {
            const f32x16& a = nn ? a1 : a0;
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                uint32_t xv[2], yv[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    xv[q] = X::pack2(a[(2 * pr) * 4 + 2 * q], a[(2 * pr) * 4 + 2 * q + 1]);
                    yv[q] = X::pack2(a[(2 * pr + 1) * 4 + 2 * q], a[(2 * pr + 1) * 4 + 2 * q + 1]);
                }
                const u32x2 s0 = __builtin_amdgcn_permlane32_swap(xv[0], yv[0], false, false);
                const u32x2 s1 = __builtin_amdgcn_permlane32_swap(xv[1], yv[1], false, false);
                *(u32x4*)(stag + st_wr + (((nn * 4 + pr * 2 + (lane >> 5)) ^ st_sw) << 4)) = (u32x4){s0[0], s1[0], s0[1], s1[1]};
            }
        }
        const int c = col0 + rd_chunk * 8;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = j * 8 + rd_row;
            const u32x4 v = *(const u32x4*)(stag + row * 128 + ((rd_chunk ^ ((row ^ (row >> 3)) & 7)) << 4));
            uint32_t off = c < cols_left ? (uint32_t)(row0 + row) * pitch + (uint32_t)c * 2u : kBadOffset;
            asm volatile("" : "+v"(off));
            __builtin_amdgcn_raw_buffer_store_b128(v, rD, off, 0, AUX);
        }
    }
}

// Waits until at most the requests of the last `stages` stages are in flight; more than MAX of them cannot be.
template <int P, int MAX>
__device__ __forceinline__ void wait_stages(int stages)
{
    if constexpr (MAX <= 0) wait_vmcnt<0>();
    else if (stages >= MAX) wait_vmcnt<P * MAX>();
    else wait_stages<P, MAX - 1>(stages);
}

// The main loop.  Stage k lies in slot k % S; all of the ring is requested before the first stage.  One k-step of fragments
// is read ahead of the MFMAs, across the stages' boundary: a wave passes the barrier that ends stage k with its last
// k-step in registers, reads the first of stage k + 1 and puts its requests for stage k + S, which takes the slot just
// freed, between the MFMAs (in front of them they held the MFMAs up: the unit that takes them works through all waves'
// requests at 64 bytes a clock).
// Beside its reads, requests and MFMAs a stage should do no more than a few scalar instructions: both waves of a SIMD do them at
// the same time, right behind the barrier, with nothing to multiply.  Stages of one k-step are unrolled over the slots, which makes
// LDS addresses constants (latent gradient, 1024 tokens, N = 32768 104 -> 86 us); longer ones are not: with several ways out of the
// loop the compiler moves the accumulators about, which those tiles have no registers for.
// Unrolled, the last stages are a loop of their own that requests nothing past the end.  Such requests (zeros, which the
// kernel waits for before its LDS takes the sums) cost S stages of LDS writes, 0.4 us of a launch of 6; with the question in
// every stage a long loop took 12 % more.  It asks once a stage, behind the MFMAs: between them it split the stage into pieces that
// the compiler does not schedule across (weight gradient, 425 tokens, N = 768 6.06 -> 5.81 us, 167 tokens, N = 160 5.10 -> 4.98).
// (After the last stage a slot that was never filled may be read; nothing is multiplied with it.)
//   prepare()  sets up the requests of the next stage to be asked for      request(j, slot)  issues the j-th of them
//   read(set, s, slot)  fetches k-step s of the stage being read           next()  goes on to the next stage to be read
//   multiply(set, f)  the k-step's MFMAs, with f(i) after the i-th         (slot: its first byte)
template <typename C, typename Prepare, typename Request, typename Read, typename Next, typename Multiply>
__device__ __forceinline__ void ring_loop(int n_stages, Prepare&& prepare, Request&& request, Read&& read, Next&& next, Multiply&& multiply)
{
    constexpr int P = C::PT + C::PN, M = C::TT * C::TN, PER = (P + M - 1) / M, S = C::S, KSW = C::KSW;
    constexpr bool UNROLLED = KSW == 1;
    const std::integral_constant<int, 0> zero;
    if (n_stages <= 0) return;
#pragma unroll 1
    for (int k = 0; k < S && (!UNROLLED || k < n_stages); ++k) {
        prepare();
        static_for<P>([&](auto j) { request(j, (uint32_t)k * (uint32_t)C::STAGE); });
    }
    wait_stages<P, S - 1>(UNROLLED ? n_stages - 1 : S - 1);
    __syncthreads();
    read(zero, zero, 0u);
    // first: the set that holds the stage's first k-step; last: whether the end may be within S stages; left: stages to go, if so
    auto stage = [&](auto first, uint32_t slot, uint32_t next_slot, auto last, int left) {
        constexpr bool LAST = decltype(last)::value;
        static_for<KSW>([&](auto sc) {
            constexpr int s = decltype(sc)::value, Q = (decltype(first)::value + s) % 2;
            const std::integral_constant<int, Q> now;
            const std::integral_constant<int, 1 - Q> other;
            if constexpr (s + 1 < KSW) {
                read(other, std::integral_constant<int, s + 1>{}, slot);
                __builtin_amdgcn_sched_barrier(0);
                multiply(now, [](auto) {});
            } else {
                wait_stages<P, S - 2>(LAST ? left - 2 : S - 2);
                __syncthreads();
                next();
                read(other, zero, next_slot);
                if constexpr (!LAST) prepare();
                __builtin_amdgcn_sched_barrier(0);
                multiply(now, [&](auto i) {
                    constexpr int I = decltype(i)::value;
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (!LAST && I * PER < P)
                        static_for<PER>([&](auto jj) {
                            constexpr int j = I * PER + decltype(jj)::value;
                            if constexpr (j < P) request(std::integral_constant<int, j>{}, slot);
                        });
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (LAST)
                    if (left > S) {
                        prepare();
                        static_for<P>([&](auto j) { request(j, slot); });
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    if constexpr (UNROLLED) {
        constexpr int U = S % 2 == 1 ? 2 * S : S;                    // stages until slot and set repeat
        static_assert(U <= 6);
        auto turn = [&](auto ic, auto last, int left) {
            constexpr int I = decltype(ic)::value;
            stage(std::integral_constant<int, I % 2>{}, (uint32_t)(I % S * C::STAGE), (uint32_t)((I + 1) % S * C::STAGE), last, left);
        };
        int left = n_stages;
        for (; left >= S + U; left -= U) static_for<U>([&](auto i) { turn(i, std::false_type{}, 0); });
        for (;;) {
#define BDA_RING_STAGE(I)                                                       \
    if constexpr (I < U) {                                                      \
        turn(std::integral_constant<int, I>{}, std::true_type{}, left);         \
        if (--left == 0) break;                                                 \
    }
            BDA_RING_STAGE(0) BDA_RING_STAGE(1) BDA_RING_STAGE(2) BDA_RING_STAGE(3) BDA_RING_STAGE(4) BDA_RING_STAGE(5)
#undef BDA_RING_STAGE
        }
    } else {
        static_assert(KSW % 2 == 0);
        uint32_t slot = 0;
        for (int left = n_stages; left > 0; --left) {
            const uint32_t next_slot = slot == (uint32_t)((S - 1) * C::STAGE) ? 0u : slot + (uint32_t)C::STAGE;
            stage(zero, slot, next_slot, std::false_type{}, 0);
            slot = next_slot;
        }
    }
}

}  // namespace bda
