// Device entry point for the gradients of the BD K/V projection: validation, tile grids, launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bda_bwd_kernels.hpp"
#include "bda_gemm_f32.hpp"
#include "bda_internal.h"

namespace bda {
namespace {

// (same contract as set_max_lds of the forward launchers: per device, retried after a failure)
template <typename K>
int allow_lds(K kernel, int bytes, LdsLimitState& state)
{
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return fail(BDA_EHIP, "hipGetDevice: %s", hipGetErrorString(err));
    const bool tracked = dev >= 0 && dev < LdsLimitState::kMaxDevices;
    if (tracked && state.done[dev].load(std::memory_order_acquire)) return BDA_OK;
    err = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (err != hipSuccess) return fail(BDA_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(err));
    if (tracked) state.done[dev].store(true, std::memory_order_release);
    return BDA_OK;
}

int launched()
{
    hipError_t err = hipGetLastError();
    return err == hipSuccess ? BDA_OK : fail(BDA_EHIP, "kernel launch: %s", hipGetErrorString(err));
}

// The gradients' tiles, largest first but for the last.
typedef RingShape<128, 128, 1, 2, 4, 64, 4> LatentLarge;
typedef RingShape<64, 128, 1, 2, 4, 64, 4> LatentMiddle;
typedef RingShape<64, 64, 1, 1, 8, 128, 4> LatentSmall;
typedef RingShape<64, 64, 1, 1, 4, 64, 3> LatentShort;
typedef RingShape<192, 256, 2, 4, 1, 32, 5> WeightLarge;
typedef RingShape<128, 256, 2, 4, 1, 32, 6> WeightMiddle;
typedef RingShape<64, 128, 1, 2, 4, 64, 4> WeightSmall;
typedef RingShape<64, 64, 1, 1, 4, 64, 4> WeightSmallest;
typedef RingShape<128, 128, 1, 2, 4, 64, 4> WeightSquare;

// Tile grid of shape C: its number of tiles; rows x group_cols = extent of the output.
template <typename C>
int64_t ring_grid(BwdArgs& a, int64_t rows, const int64_t* group_cols, int G)
{
    int64_t n_tiles = 0;
    a.tile_start[0] = 0;
    for (int g = 0; g < G; ++g) {
        n_tiles += (group_cols[g] + C::BN - 1) / C::BN;
        a.tile_start[g + 1] = (int)n_tiles;
    }
    const int64_t m_tiles = (rows + C::BT - 1) / C::BT;
    a.n_tiles = (int)n_tiles;
    a.m_tiles = (int)m_tiles;
    return m_tiles * n_tiles;
}

template <typename X, typename OutT, typename C, bool WEIGHT>
int launch_ring(BwdArgs& a, int64_t rows, const int64_t* group_cols, int G, hipStream_t st)
{
    static LdsLimitState once;
    const int64_t total = ring_grid<C>(a, rows, group_cols, G);
    const int64_t grid = kNumXcd * ((total + kNumXcd - 1) / kNumXcd);
    if (grid * C::THREADS >= (int64_t)1 << 32) return fail(BDA_EINVAL, "gradient of %lld tiles: too many for a launch", (long long)total);
    if constexpr (!WEIGHT) {
        a.n_stages = 0;
        for (int g = 0; g < a.n_groups; ++g) a.n_stages += (int)((a.col_start[g + 1] - a.col_start[g] + C::CK - 1) / C::CK);
    }
    constexpr int lds = WEIGHT ? C::BYTES : C::BYTES + kOnesBytes;
    const auto kern = [] {
        if constexpr (WEIGHT) return ring_weight_kernel<X, OutT, C>;
        else return ring_latent_kernel<X, OutT, C>;
    }();
    if (int rc = allow_lds(kern, lds, once)) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(C::THREADS), lds, st, a);
    return launched();
}

// The tile whose rounds over the 256 compute units (a workgroup each; two of the weight gradient's smallest, three of the
// latent gradient's shortest) are estimated to take the least.  The estimates are us measured over the tiles: per 64 elements of the
// contraction, and what a round takes beside them (first requests, sum over the waves, stores; less where it is the only one).
// The weight gradient's stages also take longer the more compute units work (requests wait for one another, and the clock falls), so
// a round's stage has a part for its share of the units.  Fitted to 550 drawn launches (rms 8 to 12 %), over which the rule is 0.1 % behind the
// fastest tile on average and at most 7 %.
// A wrong tile: 4096 tokens, d_c = 512, N = 4096 latent 33 / 26 / 34 us with the large, middle, small one; 1024 tokens 31 / 22 / 17; 8192 tokens,
// N = 32768 276 / 387 / 441; weight, 4096 tokens, K = 384, N = 4096 65 / 42 / 23 / 24 / 28.5 with the five, 300 tokens, K = 128, N = 32768
// 11.6 / 9.3 / 12.4 / 12.4 / 10.3.  The square one is for few rows of C or few columns, where 256 columns leave half of the units empty: 8192
// tokens, K = 128, N = 32768 131 / 130 / 147 / 172 / 101, K = 256, N = 16384 125 / 98 / 102 / 130 / 72, K = 384, N = 8192 123 / 80 / 74 / 83 / 53
// (register-staged tiles of 128 x 128 took 108, 86 and 84).
// Few output columns: 18 tokens, N = 64 6.9 / 5.4 / 5.6 / 5.1 with the four latent tiles, 912 tokens, N = 160 8.2 / 6.4 / 6.3 / 5.8, 20000
// tokens, d_c = 160, N = 512 20.3 / 20.6 / 24.5 / 14.4; from N of about 600 on the eight waves are ahead (9 tokens, N = 2048 12.7 against 14.9).
// Register-staged 64 x 64 tiles, which served N up to 512 before, took 5.3, 5.9 and 25.7 there; between N = 256 and 512 they
// were up to 1.2 us ahead (1199 tokens, N = 512 6.9 against 7.2; 2 tokens, d_c = 600 6.9 and 7.8; 19 tokens, N = 512 6.7 and 7.9).  Weight
// gradients of 160 to 450 tokens are up to 0.5 us behind them as well (400 tokens, N = 256 5.2 and 5.7), all others level or ahead.
// Neither gap is the ring's depth: with six slots, or one loop body in place of six, both took longer.
template <typename X, typename OutT, bool WEIGHT>
int launch_sized(BwdArgs& a, int64_t rows, const int64_t* group_cols, int G, hipStream_t st)
{
    auto rounds = [](int64_t tiles, int64_t slots) { return (double)((tiles + slots - 1) / slots); };
    int pick = tile_policy() - 1;              // 1, 2, ...: that tile, from the largest (testing hook)
    if constexpr (WEIGHT) {
        if (pick < 0 || pick > 4) {
            const double chunks = (double)((a.T + 63) / 64);
            auto cost = [&](int64_t tiles, double start, double stage, double crowd) {   // stage + crowd: of a round that all units work in
                const int64_t rest = tiles % 256;
                return (double)(tiles / 256) * (start + chunks * (stage + crowd)) + (rest ? start + chunks * (stage + crowd * (double)rest / 256.0) : 0.0);
            };
            const int64_t smallest = ring_grid<WeightSmallest>(a, rows, group_cols, G), rest = smallest % 512;
            const double two = 5.0 + 0.42 * chunks;   // a round with two workgroups on some unit
            const double tile_cost[5] = {cost(ring_grid<WeightLarge>(a, rows, group_cols, G), 5.7, 0.88, 0.35),
                                         cost(ring_grid<WeightMiddle>(a, rows, group_cols, G), 4.8, 0.55, 0.345),
                                         cost(ring_grid<WeightSmall>(a, rows, group_cols, G), 4.8, 0.22, 0.175),
                                         (double)(smallest / 512) * two + (rest > 256 ? two : cost(rest, 4.4, 0.156, 0.09)),
                                         cost(ring_grid<WeightSquare>(a, rows, group_cols, G), 6.6, 0.305, 0.205)};
            pick = 0;
            for (int i = 1; i < 5; ++i)
                if (tile_cost[i] < tile_cost[pick]) pick = i;
        }
        switch (pick) {
        case 0: return launch_ring<X, OutT, WeightLarge, true>(a, rows, group_cols, G, st);
        case 1: return launch_ring<X, OutT, WeightMiddle, true>(a, rows, group_cols, G, st);
        case 2: return launch_ring<X, OutT, WeightSmall, true>(a, rows, group_cols, G, st);
        case 3: return launch_ring<X, OutT, WeightSmallest, true>(a, rows, group_cols, G, st);
        default: return launch_ring<X, OutT, WeightSquare, true>(a, rows, group_cols, G, st);
        }
    } else {
        if (pick < 0 || pick > 3) {
            double stages = 0.0;               // of 64 columns
            for (int g = 0; g < a.n_groups; ++g) stages += (double)((a.col_start[g + 1] - a.col_start[g] + 63) / 64);
            auto cost = [&](double r, double one, double each, double stage) { return r == 1.0 ? one + stage * stages : r * (each + stage * stages); };
            const double n_short = (double)ring_grid<LatentShort>(a, rows, group_cols, G) / 256.0, one_short = 1.0 + 0.28 * stages;
            const double tile_cost[4] = {cost(rounds(ring_grid<LatentLarge>(a, rows, group_cols, G), 256), 3.1, 4.5, 0.42),
                                         cost(rounds(ring_grid<LatentMiddle>(a, rows, group_cols, G), 256), 1.4, 3.2, 0.31),
                                         cost(rounds(ring_grid<LatentSmall>(a, rows, group_cols, G), 256), 1.8, 3.4, 0.21),
                                         n_short <= 1.0 ? one_short : std::max(one_short, n_short * (1.2 + 0.2 * stages))};
            pick = 0;
            for (int i = 1; i < 4; ++i)
                if (tile_cost[i] < tile_cost[pick]) pick = i;
        }
        switch (pick) {
        case 0: return launch_ring<X, OutT, LatentLarge, false>(a, rows, group_cols, G, st);
        case 1: return launch_ring<X, OutT, LatentMiddle, false>(a, rows, group_cols, G, st);
        case 2: return launch_ring<X, OutT, LatentSmall, false>(a, rows, group_cols, G, st);
        default: return launch_ring<X, OutT, LatentShort, false>(a, rows, group_cols, G, st);
        }
    }
}

template <bool WEIGHT>
int launch_fast(BwdArgs& a, int64_t rows, const int64_t* group_cols, int G, int dtype, int out_dtype, hipStream_t st)
{
    if (dtype == BDA_F16 && out_dtype == BDA_F16) return launch_sized<F16, uint16_t, WEIGHT>(a, rows, group_cols, G, st);
    if (dtype == BDA_F16 && out_dtype == BDA_F32) return launch_sized<F16, float, WEIGHT>(a, rows, group_cols, G, st);
    if (dtype == BDA_BF16 && out_dtype == BDA_BF16) return launch_sized<BF16, uint16_t, WEIGHT>(a, rows, group_cols, G, st);
    if (dtype == BDA_BF16 && out_dtype == BDA_F32) return launch_sized<BF16, float, WEIGHT>(a, rows, group_cols, G, st);
    return fail(BDA_EDTYPE, "unsupported dtype/grad_dtype pair %d/%d", dtype, out_dtype);
}

template <Product P>
int run_general(GeneralArgs& p, const int64_t* out_cols, int G, int dtype, int out_dtype, hipStream_t st)
{
    return launch_general<P>(p, out_cols, G, dtype, out_dtype, [&](auto kern, int threads, int lds, LdsLimitState& once, int) {
        if (int rc = allow_lds(kern, lds, once)) return rc;
        hipLaunchKernelGGL(kern, general_grid(p), dim3(threads), lds, st, p);
        return launched();
    });
}

}  // namespace
}  // namespace bda

using namespace bda;

extern "C" int bda_kv_project_backward_ex(const void* c, int64_t ldc, const void* d_out, int64_t ld_dout,
                                          const void* C, int64_t ldC, int64_t T, int d_c, int d_h, int G,
                                          const int* H, const int* basis_offset, void* grad_c, int64_t ld_gc,
                                          void* grad_C, int64_t ld_gC, bda_dtype dtype, bda_dtype grad_dtype,
                                          void* stream, int tile_policy)
{
    clear_error();
    if (int rc = check_policy("bda_kv_project_backward_ex", tile_policy)) return rc;
    PolicyScope scope(tile_policy);
    return bda_kv_project_backward(c, ldc, d_out, ld_dout, C, ldC, T, d_c, d_h, G, H, basis_offset, grad_c, ld_gc,
                                   grad_C, ld_gC, dtype, grad_dtype, stream);
}

extern "C" int bda_kv_project_backward(const void* c, int64_t ldc, const void* d_out, int64_t ld_dout,
                                       const void* C, int64_t ldC, int64_t T, int d_c, int d_h, int G,
                                       const int* H, const int* basis_offset, void* grad_c, int64_t ld_gc,
                                       void* grad_C, int64_t ld_gC, bda_dtype dtype, bda_dtype grad_dtype,
                                       void* stream)
{
    clear_error();
    const char* fn = "bda_kv_project_backward";
    if (dtype != BDA_F32 && dtype != BDA_F16 && dtype != BDA_BF16) return fail(BDA_EDTYPE, "%s: bad dtype %d", fn, dtype);
    if (grad_dtype != dtype && grad_dtype != BDA_F32) return fail(BDA_EDTYPE, "%s: grad_dtype must equal dtype or be BDA_F32 (got %d/%d)", fn, dtype, grad_dtype);
    if (T < 0 || d_c <= 0 || d_h <= 0 || d_h >= d_c) return fail(BDA_EINVAL, "%s: need T >= 0 and 0 < d_h < d_c (T=%lld d_c=%d d_h=%d)", fn, (long long)T, d_c, d_h);
    if (G <= 0 || G > BDA_MAX_GROUPS || !H || !basis_offset) return fail(BDA_EINVAL, "%s: need 1 <= G <= %d and non-NULL H, basis_offset", fn, BDA_MAX_GROUPS);
    int64_t N = 0;
    int64_t cols[BDA_MAX_GROUPS];
    for (int g = 0; g < G; ++g) {
        if (H[g] <= 0) return fail(BDA_EINVAL, "%s: H[%d]=%d", fn, g, H[g]);
        if (basis_offset[g] < 0 || basis_offset[g] > d_c - d_h) return fail(BDA_EINVAL, "%s: basis_offset[%d]=%d outside [0, %d]", fn, g, basis_offset[g], d_c - d_h);
        cols[g] = (int64_t)H[g] * d_h;
        N += cols[g];
    }
    if (!grad_c && !grad_C) return BDA_OK;
    const int K = d_c - d_h;
    if (T > 0 && !d_out) return fail(BDA_EINVAL, "%s: NULL d_out", fn);
    if (ld_dout < N) return fail(BDA_EINVAL, "%s: ld_dout=%lld < N=%lld", fn, (long long)ld_dout, (long long)N);
    if (grad_c && T > 0 && !C) return fail(BDA_EINVAL, "%s: grad_c needs C", fn);
    if (grad_c && (ldC < N || ld_gc < d_c)) return fail(BDA_EINVAL, "%s: leading dimension too small (ldC=%lld ld_gc=%lld, N=%lld d_c=%d)", fn, (long long)ldC, (long long)ld_gc, (long long)N, d_c);
    if (grad_C && T > 0 && !c) return fail(BDA_EINVAL, "%s: grad_C needs c", fn);
    if (grad_C && (ldc < d_c || ld_gC < N)) return fail(BDA_EINVAL, "%s: leading dimension too small (ldc=%lld ld_gC=%lld, d_c=%d N=%lld)", fn, (long long)ldc, (long long)ld_gC, d_c, (long long)N);
    const size_t esz = dtype_size(dtype), gsz = dtype_size(grad_dtype);
    const Span s_c = span_of(grad_C ? c : nullptr, T, d_c, ldc, esz), s_g = span_of(d_out, T, N, ld_dout, esz);
    const Span s_C = span_of(grad_c ? C : nullptr, K, N, ldC, esz);
    const Span s_gc = span_of(grad_c, T, d_c, ld_gc, gsz), s_gC = span_of(grad_C, K, N, ld_gC, gsz);
    if (overlaps(s_gc, s_c) || overlaps(s_gc, s_g) || overlaps(s_gc, s_C) || overlaps(s_gC, s_c) ||
        overlaps(s_gC, s_g) || overlaps(s_gC, s_C) || overlaps(s_gc, s_gC))
        return fail(BDA_EINVAL, "%s: a gradient overlaps an input or the other gradient", fn);

    BwdArgs a{};
    a.c = c; a.g = d_out; a.C = C;
    a.ldc = ldc; a.ldg = ld_dout; a.ldC = ldC;
    a.T = T; a.d_c = d_c; a.d_h = d_h; a.K = K; a.n_groups = G;
    a.col_start[0] = 0;
    for (int g = 0; g < G; ++g) {
        a.col_start[g + 1] = a.col_start[g] + cols[g];
        a.a_off[g] = basis_offset[g];
    }
    hipStream_t st = (hipStream_t)stream;
    GeneralArgs p{};
    p.d_c = d_c; p.d_h = d_h; p.n_groups = G;
    for (int g = 0; g < G; ++g) {
        p.col_start[g + 1] = a.col_start[g + 1];
        p.off[g] = basis_offset[g];
    }

    const int64_t max_ld = (int64_t)1 << 21;   // 32-bit buffer offsets inside one tile
    bool fast = (dtype == BDA_F16 || dtype == BDA_BF16) && aligned(d_out, 16) && ld_dout % 8 == 0 && ld_dout < max_ld &&
                d_c % 8 == 0 && d_h % 32 == 0 && N < ((int64_t)1 << 30);
    for (int g = 0; g < G; ++g) fast = fast && basis_offset[g] % 8 == 0;

    if (grad_c && T > 0) {
        a.out = grad_c; a.ldo = ld_gc;
        const bool f = fast && aligned(C, 16) && aligned(grad_c, gsz == 4 ? 16 : 8) && ldC % 8 == 0 && ld_gc % 8 == 0 &&
                       ld_gc < max_ld && (int64_t)K * ldC * 2 < ((int64_t)1 << 31);
        int rc;
        const int64_t latent_cols[1] = {d_c};
        if (f) {
            rc = launch_fast<false>(a, T, latent_cols, 1, dtype, grad_dtype, st);
        } else {
            p.tok = d_out; p.wgt = C; p.out = grad_c;
            p.ld_tok = ld_dout; p.ld_wgt = ldC; p.ld_out = ld_gc;
            p.rows = T; p.len = N;
            rc = run_general<Product::Latent>(p, latent_cols, 1, dtype, grad_dtype, st);
        }
        if (rc) return rc;
    }
    if (grad_C) {
        a.out = grad_C; a.ldo = ld_gC;
        const bool f = fast && (T == 0 || aligned(c, 16)) && aligned(grad_C, gsz == 4 ? 16 : 8) && ldc % 8 == 0 &&
                       ldc < max_ld && ld_gC % 8 == 0 && ld_gC < max_ld;
        if (f) return launch_fast<true>(a, K, cols, G, dtype, grad_dtype, st);
        p.tok = c; p.wgt = d_out; p.out = grad_C;
        p.ld_tok = ldc; p.ld_wgt = ld_dout; p.ld_out = ld_gC;
        p.rows = K; p.len = T; p.skip = d_h;
        return run_general<Product::Weight>(p, cols, G, dtype, grad_dtype, st);
    }
    return BDA_OK;
}
