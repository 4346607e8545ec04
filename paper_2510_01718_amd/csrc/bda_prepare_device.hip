// GPU preparation of one projection (Algorithm "BD Attention Preparation (QK)", Appendix "BD for VO in
// MHA", Algorithm "BD Decomposition (Row)" for the window choice, Appendix "Residual-Min with Offset
// Search" for the candidate windows).  Float64 throughout:
//   invert_kernel    C_h = W_h[Bbar,:] W_h[B,:]^{-1} for d_h <= 128, one workgroup per head (several when
//                    there are few heads: each inverts for itself and takes a share of the rows): the
//                    basis block is inverted in LDS by Gauss-Jordan elimination with partial (row) pivoting
//                    in panels of 16 columns, then the d_c - d_h rows outside the window are multiplied by
//                    the inverse on the matrix cores and stored rounded to the requested type;
//   prepare_wide_kernel   the same for d_h up to 256 with the block in the caller's workspace (the row
//                    interchanges are undone as column interchanges at the end);
//   strip_kernel     with a companion and d_c up to 512: the companion block, W_q^h W_h[B,:]^T or W_h[B,:] W_o^h,
//                    rounded the same way, and the Frobenius reconstruction errors of the stored form of one
//                    head for all candidate windows of the launch, as partial sums of squares (a fixed number
//                    of parts per head, each summed in a fixed order);
//   measure_kernel   the same for the shapes nearly every projection has (whole tiles, windows that start on
//                    multiples of 16, aligned rows, 16-bit results), without per-lane decisions;
//   side_kernel, residual_kernel   the same in two steps, one window per launch: wider latents, and errors
//                    without a companion;
//   select_kernel    per candidate window the mean over heads of the residuals, the smallest mean
//                    (earlier candidate on ties, NaN as +inf), the chosen window start.
//   copy_kernel      the chosen window's stored C from where the search kept it to C.
// A search prepares and measures its candidate windows, as many per launch as the caller's outputs can hold
// stored C's (see Slot), selects, and either copies the chosen window's C, where the companion output could hold
// every candidate, or prepares that window once more, whose start it reads from device memory: nothing comes
// back to the host in between.
// The host routine bda_prepare solves with an orthogonal factorisation instead of forming the inverse;
// the two agree to a small multiple of cond(W_h[B,:]) * 2^-53.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "bda_internal.h"

// Scratch memory of bda_prepare_device_static, the entry point for callers that cannot allocate: part of
// the code object, so every GPU the library runs on holds its own copy from the moment the code is loaded
// there until the process ends.  Host code never uses this name as an address: it asks the runtime for
// the array's address on the current device (static_scratch below) and passes that to the kernels.
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace bda {
namespace {

template <typename T> __device__ __forceinline__ double load_as_double(const void* p, int64_t i);
template <> __device__ __forceinline__ double load_as_double<double>(const void* p, int64_t i) { return ((const double*)p)[i]; }
template <> __device__ __forceinline__ double load_as_double<float>(const void* p, int64_t i) { return (double)((const float*)p)[i]; }
template <> __device__ __forceinline__ double load_as_double<_Float16>(const void* p, int64_t i) { return (double)((const _Float16*)p)[i]; }
template <> __device__ __forceinline__ double load_as_double<__bf16>(const void* p, int64_t i)
{
    const uint32_t b = (uint32_t)((const uint16_t*)p)[i] << 16;
    return (double)__builtin_bit_cast(float, b);
}

// One rounding, to nearest even, from double to the stored type.
template <typename T> __device__ __forceinline__ void store_rounded(void* p, int64_t i, double v);
template <> __device__ __forceinline__ void store_rounded<double>(void* p, int64_t i, double v) { ((double*)p)[i] = v; }
template <> __device__ __forceinline__ void store_rounded<float>(void* p, int64_t i, double v) { ((float*)p)[i] = (float)v; }
template <> __device__ __forceinline__ void store_rounded<_Float16>(void* p, int64_t i, double v)
{
    ((_Float16*)p)[i] = (_Float16)v;          // the compiler converts f64 -> f16 with one rounding
}
template <> __device__ __forceinline__ void store_rounded<__bf16>(void* p, int64_t i, double v)
{
    // bf16 = the upper half of a float: round the double to 8 significant bits directly.  Going through
    // float first would round twice; instead the float is formed by truncation toward zero plus a
    // sticky bit, and the final rounding looks at that.
    float f = (float)v;
    if ((double)f != v) {                     // inexact: make sure the discarded part is seen below
        uint32_t b = __builtin_bit_cast(uint32_t, f);
        const bool too_big = (v >= 0) ? ((double)f > v) : ((double)f < v);
        if (too_big) b -= 1;                  // f is now v truncated toward zero ...
        b |= 1u;                              // ... with a sticky bit (never lands on a bf16 tie)
        f = __builtin_bit_cast(float, b);
    }
    uint32_t b = __builtin_bit_cast(uint32_t, f);
    if ((b & 0x7f800000u) != 0x7f800000u) b += 0x7fffu + ((b >> 16) & 1u);
    ((uint16_t*)p)[i] = (uint16_t)(b >> 16);
}

constexpr int kPrepThreads = 256;
constexpr int kPrepLdsDh = 128;               // largest head width whose basis block is inverted in registers (invert_kernel)
constexpr int kPrepMaxDh = 256;               // largest head width at all (block in the workspace)
constexpr int kPrepRows = 16;                 // rows of W_h[Bbar,:] staged per pass
constexpr int kMaxCandidates = 256;
constexpr int kMaxParts = 64;                 // workgroups per head of the residual kernel, at most (heads x parts <= 1024: about four
                                              // workgroups per compute unit, which cover one another's exposed load latency)

struct PrepArgs {
    const void* W;
    const void* side;            // companion weight (type of W) or NULL
    void* C;
    void* side_out;              // companion output (type of C) or NULL
    int* status;                 // singular_head of the public calls, or NULL
    const int* off_ptr;          // device: window start chosen by select_kernel (NULL: `off`)
    int* cand_singular;          // workspace: one flag per candidate window, or NULL
    double* partials;            // workspace: [candidate][head][part] sums of squares, or NULL
    double* mat;                 // workspace: one d_h x d_h block per workgroup of a batch (d_h > 128), or NULL
    int64_t ldw, ld_side, ldC, ld_side_out;
    int d_c, H, d_h, d_side, side_kind;
    int off, off_step, off_last; // candidate window i starts at min(off + i off_step, off_last)
    int h0;                      // first head of this launch (batches when the block lives in the workspace)
    int cand, n_cand, n_parts;   // first candidate window of this launch and their number
    int w_type, c_type;          // element types of W / side and of C / side_out
    int search, c_slots;         // candidate windows in the outputs; how many of them in C (see Slot)
    uint32_t width_magic;        // see Slot (O)
    int write_side, measure;     // strip_kernel: store the companion block; sum the reconstruction errors
    int lane_sums;               // measure_kernel: one sum per lane in LDS
};

// Start of window `z` of this launch, or -1.
__device__ __forceinline__ int window_start(const PrepArgs& a, int z = 0)
{
    if (a.off_ptr) return *a.off_ptr;
    const int o = a.off + (a.cand + z) * a.off_step;
    return o < a.off_last ? o : a.off_last;
}

// Where window `z` of a launch keeps its stored C: row kk of head h, d_h contiguous elements, begins at element
// slot_row() of the array.  The call's one window has C itself.  During a search C and the companion output are free until
// the chosen window is written and hold the candidates': C one of them (a.c_slots) and the companion output the others,
// d_c - d_h of its rows each (Q: the layout of C), or as many pieces of d_h columns of the head's own d_h rows, a column of
// pieces after the other (O: so that 16 consecutive rows from a multiple of 16 on stay together where d_h has that factor).
struct Slot {
    void* p;
    int64_t ld;
    int first;                   // rows or pieces before this window's
    uint32_t magic;              // ceil(2^32 / d_h), not read for heads of one column; 0: rows of C's layout
};
__device__ __forceinline__ Slot slot_of(const PrepArgs& a, int z)
{
    if (!a.search || z < a.c_slots) return {a.C, a.ldC, 0, 0};
    return {a.side_out, a.ld_side_out, (z - a.c_slots) * (a.d_c - a.d_h), a.side_kind == BDA_SIDE_O ? a.width_magic : 0};
}
__device__ __forceinline__ int64_t slot_row(const Slot& s, int kk, int h, int n)
{
    const int q = s.first + kk;
    if (!s.magic) return q * s.ld + (int64_t)h * n;
    const int block = n == 1 ? q : (int)__umulhi((uint32_t)q, s.magic);
    return ((int64_t)h * n + (q - block * n)) * s.ld + block * n;
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4: lane (c = lane % 16, g = lane / 16) holds A[c][g] and B[g][c] and receives
// D[4 r + g][c] in element r.
__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 acc) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0); }

// Calls f(T{}) with the C++ type of a bda_dtype (one uniform branch around a whole loop, where a kernel
// instantiated per type would only multiply the code).
template <typename F>
__device__ __forceinline__ void with_type(int type, F&& f)
{
    if (type == BDA_F32) f(float{});
    else if (type == BDA_F16) f(_Float16{});
    else if (type == BDA_BF16) f(__bf16{});
    else f(double{});
}

template <int N, typename F>
__device__ __forceinline__ void static_for_blocks(F&& f)
{
    if constexpr (N > 0) {
        static_for_blocks<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// Largest of a 32-bit value over the 64 lanes, in every lane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    auto step = [&](auto ctrl) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, true);
        v = o > v ? o : v;
    };
    step(std::integral_constant<int, 0x111>{});      // row_shr 1, 2, 4, 8: lane 15 of a row of 16 holds the row's largest
    step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{});
    step(std::integral_constant<int, 0x118>{});
    uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
#pragma unroll
    for (int l = 31; l < 64; l += 16) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)v, l);
        m = o > m ? o : m;
    }
    return m;
}

// Inverse of the basis block and C_h = W_h[Bbar,:] A^{-1}, head widths up to 32 NB (NB = 1 .. 4), 512 threads.  The block
// lies in LDS and is inverted in place by Gauss-Jordan elimination in panels of 16 columns:
//   * one wave takes the panel into registers, one or two rows a lane, and does its 16 steps there: pivot search, broadcast of
//     the pivot row (scalar registers) and update without a barrier or a trip through LDS;
//   * all waves apply the panel to the other columns on v_mfma_f64_16x16x4: with P the panel's pivot rows and G what the steps
//     left in its columns, A[i, J] (zero for i in P) + G[i, :] A[P, J].
// Rows are never interchanged: a row that has been a pivot is left out of the later searches, and the permutation is applied
// when the inverse is put in order for the product.  The pivot is the largest of the column to 13 bits of its mantissa (the
// key carries the row number in its low bits): growth is bounded as with the exact largest, up to a factor 1 + 2^-13.
// The product runs on the matrix cores too: a wave takes 16 rows of W_h[Bbar,:] straight from memory into registers (its A
// operand) against the inverse in LDS.  The pitch of 2 mod 32 doubles keeps a lane's row of a panel and 16 rows of an operand
// in different banks.
// Bound: the chain of pivots (16 heads of 128: 128 steps of some 130 instructions of one wave, 75 us; panels applied 29, product
// 18).  One step at a time over all columns, with two barriers and a row and a column through LDS each, took 146 us for 16
// heads of 128 and 172 for a search's launch; this 126 and 151.
// Error of C in float64 against one step at a time, means over some 100 blocks of 8 .. 128 columns: Gaussian blocks 0.9 to 1.2 times (32 columns
// 3.6e-15 / 3.3e-15, 128 1.9e-14 / 1.8e-14), the residual of C A 0.9 to 1.0.  Beyond one panel a badly conditioned block is further off, as the panels multiply
// by their pivot block's inverse: condition 1e6, 32 columns 6.8e-12 / 3.2e-12, 128 8.2e-12 / 6.9e-12 (cond 2^-53 is 1e-10), with a residual of 0.75 and
// 0.9 times.  Nothing of it reaches results of 16 or 32 bits.
constexpr int kInvertThreads = 512, kInvertRows = kInvertThreads / 32, kInvertWaves = kInvertThreads / 64;
template <int NB>
constexpr int invert_lds_bytes() { return 32 * NB * (32 * NB + 2) * (int)sizeof(double); }

template <int NB>
__global__ __launch_bounds__(kInvertThreads) void invert_kernel(const PrepArgs a)
{
    constexpr int NP = 32 * NB, NU = NP / kInvertRows, NV = NB, LD = NP + 2, RT = NP / 16, RPL = (NP + 63) / 64;
    constexpr int COLS = kInvertWaves / RT, CT_MAX = (RT + COLS - 1) / COLS;   // waves side by side on a row tile; column tiles of one
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    double* const inv = (double*)smem_raw;
    __shared__ double s_red[kInvertWaves];
    __shared__ int s_piv[NP], s_pos[NP], s_singular;
    const int n = a.d_h, t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int h = blockIdx.x, z = blockIdx.z;
    const int off = window_start(a, z);
    if (off < 0) return;                       // no usable window was found: nothing to prepare
    const int64_t col0 = (int64_t)h * n;
    const Slot slot = slot_of(a, z);
    const int tx = t & 31, ty = t >> 5, c = lane & 15, g = lane >> 4;

    double part = 0.0;
    with_type(a.w_type, [&](auto tag) {
        typedef decltype(tag) WT;
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int i = ty + kInvertRows * u, j = tx + 32 * v;
                const double m = (i < n && j < n) ? load_as_double<WT>(a.W, (int64_t)(off + i) * a.ldw + col0 + j) : 0.0;
                inv[i * LD + j] = m;
                part = fma(m, m, part);
            }
    });
    for (int s = 32; s >= 1; s >>= 1) part += __shfl_xor(part, s, 64);
    if (lane == 0) s_red[wave] = part;
    if (t == 0) s_singular = 0;
    if (t < NP) s_pos[t] = -1;
    __syncthreads();
    double scale = 0.0;
    for (int w = 0; w < kInvertWaves; ++w) scale += s_red[w];
    const double tiny = sqrt(scale) * n * 2.220446049250313e-16;

    bool used[RPL];                            // (wave 0) whether the lane's rows have been pivots
#pragma unroll
    for (int u = 0; u < RPL; ++u) used[u] = lane + 64 * u >= n;
    for (int k0 = 0; k0 < n; k0 += 16) {
        const int nb = n - k0 < 16 ? n - k0 : 16;
        if (wave == 0) {
            double x[RPL][16];
#pragma unroll
            for (int u = 0; u < RPL; ++u) {
                const int row = lane + 64 * u < NP ? lane + 64 * u : NP - 1;
#pragma unroll
                for (int j = 0; j < 16; j += 2) {
                    const f64x2 v = *(const f64x2*)(inv + row * LD + k0 + j);
                    x[u][j] = v[0];
                    x[u][j + 1] = v[1];
                }
            }
            bool singular = false;
            // (Unrolled over the columns.  In a loop, with the pivot's column always the first and the others moved down a place by
            // the update, the moves made a step longer than the fetch of the unrolled code does: 144 us against 126.)
            static_for_blocks<16>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                if (q >= nb || singular) return;
                uint32_t key = 0;
#pragma unroll
                for (int u = 0; u < RPL; ++u) {
                    const uint32_t hi = (uint32_t)(__builtin_bit_cast(uint64_t, x[u][q]) >> 32);
                    const uint32_t k = used[u] ? 0u : (hi & 0x7fffff80u) | (uint32_t)(127 - (lane + 64 * u));
                    key = k > key ? k : key;
                }
                const int p = 127 - (int)(wave_max_u32(key) & 127u);       // uniform: the pivot row (< n: some row is unused)
                const bool upper = RPL > 1 && p >= 64;
                const int pl = p & 63;
                double row[16];                // the pivot row, in scalar registers (a branch for its half: selects would be 32 more)
                auto broadcast = [&](const double (&from)[16]) {
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const uint64_t b = __builtin_bit_cast(uint64_t, from[j]);
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, pl);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), pl);
                        row[j] = __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
                    }
                };
                if (upper) broadcast(x[RPL - 1]);
                else broadcast(x[0]);
                const double pv = row[q];
                if (!(fabs(pv) > tiny)) { singular = true; return; }
                const double ip = 1.0 / pv;
#pragma unroll
                for (int u = 0; u < RPL; ++u) {
                    const double f = x[u][q] * ip;
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (j != q) x[u][j] = fma(-f, row[j], x[u][j]);
                    x[u][q] = -f;              // column k of the block is replaced by the inverse's
                }
                auto pivot_row = [&](double (&to)[16], bool& is_used) {
                    if (lane == pl) {
#pragma unroll
                        for (int j = 0; j < 16; ++j) to[j] = j == q ? ip : row[j] * ip;
                        is_used = true;
                    }
                };
                if (upper) pivot_row(x[RPL - 1], used[RPL - 1]);
                else pivot_row(x[0], used[0]);
                if (lane == 0) { s_piv[k0 + q] = p; s_pos[p] = k0 + q; }
            });
            if (singular && lane == 0) s_singular = 1;
#pragma unroll
            for (int u = 0; u < RPL; ++u)
                if (lane + 64 * u < NP) {
#pragma unroll
                    for (int j = 0; j < 16; j += 2) *(f64x2*)(inv + (lane + 64 * u) * LD + k0 + j) = (f64x2){x[u][j], x[u][j + 1]};
                }
        }
        __syncthreads();
        if (s_singular) break;
        const bool works = wave < RT * COLS;   // (uniform; with RT = 6 two waves are left over)
        const int rt = wave % RT, ct0 = wave / RT;
        double ga[4], pb[CT_MAX][4];
        bool pivot[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool in = 4 * s + g < nb;
            const int prow = in ? s_piv[k0 + 4 * s + g] : 0;
            ga[s] = in ? inv[(16 * rt + c) * LD + k0 + 4 * s + g] : 0.0;
#pragma unroll
            for (int i = 0; i < CT_MAX; ++i) {
                const int ct = ct0 + COLS * i;
                pb[i][s] = in && ct < RT ? inv[prow * LD + 16 * ct + c] : 0.0;
            }
            pivot[s] = s_pos[16 * rt + 4 * s + g] >= k0;
        }
        __syncthreads();                       // everybody has the pivot rows as they were
#pragma unroll
        for (int i = 0; i < CT_MAX; ++i) {
            const int ct = ct0 + COLS * i;
            if (!works || ct >= RT || 16 * ct == k0) continue;
            f64x4 acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = pivot[r] ? 0.0 : inv[(16 * rt + 4 * r + g) * LD + 16 * ct + c];
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = mfma_f64(ga[s], pb[i][s], acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) inv[(16 * rt + 4 * r + g) * LD + 16 * ct + c] = acc[r];
        }
        __syncthreads();
    }
    if (s_singular) {
        if (t == 0) {
            if (a.status) atomicMax(a.status, h + 1);
            if (a.cand_singular) a.cand_singular[a.cand + z] = 1;    // (every writer stores the same value)
        }
        return;
    }
    // storage row p_k of the result is row k of (P A)^{-1}, and A^{-1} = (P A)^{-1} P
    {
        double m[NU][NV];
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int v = 0; v < NV; ++v) m[u][v] = inv[(ty + kInvertRows * u) * LD + tx + 32 * v];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int i = ty + kInvertRows * u, j = tx + 32 * v;
                const bool in = i < n && j < n;
                inv[(i < n ? s_pos[i] : i) * LD + (j < n ? s_piv[j] : j)] = in ? m[u][v] : 0.0;
            }
    }
    __syncthreads();

    // gridDim.y workgroups per head each invert the block for themselves (the same operations in the same
    // order, so the same inverse bit for bit) and share out the row tiles of the product.
    const int K = a.d_c - n;
    for (int rt = (int)blockIdx.y + (int)gridDim.y * wave; rt * 16 < K; rt += (int)gridDim.y * (kInvertThreads / 64)) {
        const int ra = rt * 16 + c;            // this lane's row of the A operand
        const int src = ra < off ? ra : ra + n;
        double av[8 * NB];
        with_type(a.w_type, [&](auto tag) {
            typedef decltype(tag) WT;
#pragma unroll
            for (int ks = 0; ks < 8 * NB; ++ks) {
                const int k = 4 * ks + g;
                av[ks] = (ra < K && k < n) ? load_as_double<WT>(a.W, (int64_t)src * a.ldw + col0 + k) : 0.0;
            }
        });
#pragma unroll 1
        for (int jt = 0; jt < 2 * NB; jt += 2) {
            f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
            for (int ks = 0; ks < 8 * NB; ++ks) {
                const double* const b = inv + (4 * ks + g) * LD + jt * 16 + c;
                acc[0] = mfma_f64(av[ks], b[0], acc[0]);
                acc[1] = mfma_f64(av[ks], b[16], acc[1]);
            }
            with_type(a.c_type, [&](auto tag) {
                typedef decltype(tag) CT;
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = rt * 16 + 4 * r + g, j = (jt + q) * 16 + c;
                        if (row < K && j < n) store_rounded<CT>(slot.p, slot_row(slot, row, h, n) + j, acc[q][r]);
                    }
            });
        }
    }
}

// Head widths above 128: the basis block lives in the workspace (a.mat, one block per workgroup).
template <typename WT, typename CT>
__global__ __launch_bounds__(kPrepThreads) void prepare_wide_kernel(const PrepArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int n = a.d_h;
    const int ld = n;
    double* const R = (double*)smem_raw;       // kPrepRows x n staging, also scratch for the reductions
    double* const A = a.mat + (size_t)blockIdx.x * n * n;   // the basis block, then its inverse
    __shared__ int piv[kPrepMaxDh];
    __shared__ int s_pivot_row;
    __shared__ double s_pivot_val;
    __shared__ int s_singular;

    const int t = threadIdx.x;
    const int h = a.h0 + blockIdx.x;
    const int off = window_start(a);
    if (off < 0) return;                       // no usable window was found: nothing to prepare
    const int64_t col0 = (int64_t)h * n;

    // ---- basis block and its scale --------------------------------------------------------------
    double part = 0.0;
    for (int e = t; e < n * n; e += kPrepThreads) {
        const int i = e / n, j = e % n;
        const double v = load_as_double<WT>(a.W, (int64_t)(off + i) * a.ldw + col0 + j);
        A[i * ld + j] = v;
        part += v * v;
    }
    R[t] = part;
    if (t == 0) s_singular = 0;
    __syncthreads();
    if (t == 0) {
        double s = 0.0;
        for (int i = 0; i < kPrepThreads; ++i) s += R[i];
        s_pivot_val = s;
    }
    __syncthreads();
    const double tiny = sqrt(s_pivot_val) * n * 2.220446049250313e-16;
    __syncthreads();

    // ---- Gauss-Jordan inversion in place, partial pivoting ----------------------------------------
    const int row = t;
    for (int k = 0; k < n; ++k) {
        // pivot: the largest |A[i][k]|, i >= k (first such row on ties)
        if (t < 64) {
            double best = -1.0;
            int bi = k;
            for (int i = k + t; i < n; i += 64) {
                const double v = fabs(A[i * ld + k]);
                if (v > best) { best = v; bi = i; }
            }
            for (int s = 32; s >= 1; s >>= 1) {
                const double ov = __shfl_xor(best, s, 64);
                const int oi = __shfl_xor(bi, s, 64);
                if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
            }
            if (t == 0) {
                s_pivot_row = bi;
                piv[k] = bi;
                if (!(best > tiny)) s_singular = 1;
            }
        }
        __syncthreads();
        if (s_singular) break;
        const int p = s_pivot_row;
        if (p != k) {
            for (int j = t; j < n; j += kPrepThreads) {
                const double x = A[k * ld + j];
                A[k * ld + j] = A[p * ld + j];
                A[p * ld + j] = x;
            }
        }
        __syncthreads();
        const double pv = A[k * ld + k];
        const double f = (row < n) ? A[row * ld + k] : 0.0;      // multiplier of this thread's row
        __syncthreads();
        // row k becomes (row k with 1 in place of the pivot) / pivot
        const double inv = 1.0 / pv;
        for (int j = t; j < n; j += kPrepThreads) A[k * ld + j] = (j == k ? 1.0 : A[k * ld + j]) * inv;
        __syncthreads();
        if (row < n && row != k) {
            int j0 = 0;                                          // (a counter the compiler takes for one of the lane's own: the
            asm volatile("" : "+v"(j0));                         // loop is 3 to 5 % faster, 22.9 -> 21.6 ms for 4 heads of 256)
#pragma unroll 8
            for (int j = j0; j < n; ++j) {
                const double cur = (j == k) ? 0.0 : A[row * ld + j];
                A[row * ld + j] = cur - f * A[k * ld + j];
            }
        }
        __syncthreads();
    }
    if (s_singular) {
        if (t == 0) {
            if (a.status) atomicMax(a.status, h + 1);
            if (a.cand_singular) a.cand_singular[a.cand] = 1;    // (every writer stores the same value)
        }
        return;
    }
    // the elimination inverted P A; A^{-1} = (P A)^{-1} P: undo the interchanges on the columns, last first
    for (int k = n - 1; k >= 0; --k) {
        const int p = piv[k];
        if (p != k) {
            for (int i = t; i < n; i += kPrepThreads) {
                const double x = A[i * ld + k];
                A[i * ld + k] = A[i * ld + p];
                A[i * ld + p] = x;
            }
            __syncthreads();
        }
    }
    __syncthreads();

    // ---- C_h = W_h[Bbar,:] A^{-1} ------------------------------------------------------------------
    const int K = a.d_c - n;
    for (int r0 = 0; r0 < K; r0 += kPrepRows) {
        for (int e = t; e < kPrepRows * n; e += kPrepThreads) {
            const int i = e / n, c = e % n;
            const int r = r0 + i;
            const int src = r < off ? r : r + n;                   // rows outside the window, ascending
            R[i * n + c] = r < K ? load_as_double<WT>(a.W, (int64_t)src * a.ldw + col0 + c) : 0.0;
        }
        __syncthreads();
        if (t < n) {
            double acc[kPrepRows];
#pragma unroll
            for (int m = 0; m < kPrepRows; ++m) acc[m] = 0.0;
#pragma unroll 4
            for (int k = 0; k < n; ++k) {
                const double b = A[k * ld + t];
#pragma unroll
                for (int m = 0; m < kPrepRows; ++m) acc[m] = fma(R[m * n + k], b, acc[m]);
            }
#pragma unroll
            for (int m = 0; m < kPrepRows; ++m) {
                const int r = r0 + m;
                if (r < K) store_rounded<CT>(a.C, (int64_t)r * a.ldC + col0 + t, acc[m]);
            }
        }
        __syncthreads();
    }
}

// Companion block of head blockIdx.x, rows (Q: rows of W_q; O: window rows) blockIdx.y, + gridDim.y, ...
//   Q:  side_out[s][h n + i] = sum_j W_q[s][h n + j] W[off + i][h n + j]        (B_qk^h = W_q^h W_h[B,:]^T)
//   O:  side_out[h n + i][m] = sum_j W[off + i][h n + j] W_o[h n + j][m]        (B_vo^h = W_h[B,:] W_o^h)
template <typename WT, typename CT>
__global__ __launch_bounds__(kPrepThreads) void side_kernel(const PrepArgs a)
{
    // Q: out[s, i] = sum_j W_q[s, col0 + j] W[off + i, col0 + j]      (d_side x d_h per head)
    // O: out[i, m] = sum_j W[off + i, col0 + j] W_o[col0 + j, m]      (d_h x d_side per head)
    // 64 x 64 output tiles, the contraction staged through LDS 16 at a time, 4 x 4 outputs per thread
    // (rows ty + 16 u, columns tx + 16 v); workgroup (head, part) takes tiles part, part + gridDim.y, ...
    // Each output is one sum in ascending j, whatever the grid.
    constexpr int TS = 64, KC = 16;
    __shared__ double As[TS][KC + 1];
    __shared__ double Bs[KC][TS + 1];
    const int n = a.d_h, h = blockIdx.x, t = threadIdx.x;
    const int off = window_start(a);
    if (off < 0) return;
    const int64_t col0 = (int64_t)h * n;
    const bool q = a.side_kind == BDA_SIDE_Q;
    const int R = q ? a.d_side : n, Cn = q ? n : a.d_side;
    auto w = [&](int i, int j) { return load_as_double<WT>(a.W, (int64_t)(off + i) * a.ldw + col0 + j); };
    const int tx = t % 16, ty = t / 16;
    const int tiles_c = (Cn + TS - 1) / TS, n_tiles = ((R + TS - 1) / TS) * tiles_c;
    for (int tile = blockIdx.y; tile < n_tiles; tile += gridDim.y) {
        const int r0 = (tile / tiles_c) * TS, c0 = (tile % tiles_c) * TS;
        double acc[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
        for (int j0 = 0; j0 < n; j0 += KC) {
            for (int e = t; e < TS * KC; e += kPrepThreads) {
                // both operands of Q and the first of O are contiguous along j; W_o is contiguous along m
                const int rr = e / KC, jj = e % KC;
                const bool okj = j0 + jj < n;
                As[rr][jj] = (okj && r0 + rr < R) ? (q ? load_as_double<WT>(a.side, (int64_t)(r0 + rr) * a.ld_side + col0 + j0 + jj)
                                                      : w(r0 + rr, j0 + jj)) : 0.0;
                if (q) Bs[jj][rr] = (okj && c0 + rr < Cn) ? w(c0 + rr, j0 + jj) : 0.0;
            }
            if (!q)
                for (int e = t; e < TS * KC; e += kPrepThreads) {
                    const int jj = e / TS, cc = e % TS;
                    Bs[jj][cc] = (j0 + jj < n && c0 + cc < Cn) ? load_as_double<WT>(a.side, (col0 + j0 + jj) * a.ld_side + c0 + cc) : 0.0;
                }
            __syncthreads();
#pragma unroll
            for (int jj = 0; jj < KC; ++jj) {
                double av[4], bv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) av[u] = As[ty + 16 * u][jj];
#pragma unroll
                for (int v = 0; v < 4; ++v) bv[v] = Bs[jj][tx + 16 * v];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[u][v] = fma(av[u], bv[v], acc[u][v]);
            }
            __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = r0 + ty + 16 * u, c = c0 + tx + 16 * v;
                if (r < R && c < Cn) {
                    if (q) store_rounded<CT>(a.side_out, (int64_t)r * a.ld_side_out + col0 + c, acc[u][v]);
                    else store_rounded<CT>(a.side_out, (col0 + r) * a.ld_side_out + c, acc[u][v]);
                }
            }
    }
}

// Sum of squared reconstruction errors of the stored form of head blockIdx.x (Chat = C as stored, Bhat =
// the companion output as stored, kk = index of row / column k among those outside the window):
//   no companion   W_h[Bbar,:] - Chat A                                       (d_c - d_h) x d_h
//   Q              W_q^h W_h^T - [Bhat at the window columns, Bhat Chat^T]    d_side x d_c
//   O              W_h W_o^h - [Bhat at the window rows; Chat Bhat]           d_c x d_side
// In every case an element is  P1(r, c) - P2(r, c) - S(r, c)  with two products over the head width, of
// which one or the other (or S) is absent for some rows or columns.  The matrix is cut into 64 x 64
// tiles; workgroup (head, part) takes tiles part, part + gridDim.y, ...; the operands of a tile are
// staged through LDS 16 columns of the contraction at a time and every thread owns a 4 x 4 sub-grid
// of the tile (rows ty + 16 u, columns tx + 16 v).  Each thread adds its squares in a fixed order, the
// workgroup adds the 256 sums in thread order: the result does not depend on scheduling.
template <typename WT, typename CT>
__global__ __launch_bounds__(kPrepThreads) void residual_kernel(const PrepArgs a)
{
    constexpr int TS = 64, KC = 16;
    __shared__ double As[TS][KC + 1];
    __shared__ double Bs[KC][TS + 1];
    __shared__ double red[kPrepThreads];
    const int n = a.d_h, h = blockIdx.x, t = threadIdx.x, d_c = a.d_c, K = d_c - n;
    const int off = window_start(a);
    const int64_t col0 = (int64_t)h * n;
    const int kind = a.side_kind;
    const int R = kind == BDA_SIDE_Q ? a.d_side : kind == BDA_SIDE_O ? d_c : K;
    const int Cn = kind == BDA_SIDE_Q ? d_c : kind == BDA_SIDE_O ? a.d_side : n;
    auto w = [&](int k, int j) { return load_as_double<WT>(a.W, (int64_t)k * a.ldw + col0 + j); };
    auto chat = [&](int kk, int i) { return load_as_double<CT>(a.C, (int64_t)kk * a.ldC + col0 + i); };
    auto in_window = [&](int k) { return k >= off && k < off + n; };
    auto outside_index = [&](int k) { return k < off ? k : k - n; };
    // first product: P1(r, c) = sum_j a1(r, j) b1(j, c)
    auto a1 = [&](int r, int j) -> double {
        if (r >= R) return 0.0;
        if (kind == BDA_SIDE_Q) return load_as_double<WT>(a.side, (int64_t)r * a.ld_side + col0 + j);
        if (kind == BDA_SIDE_O) return w(r, j);
        return 0.0;
    };
    auto b1 = [&](int j, int c) -> double {
        if (c >= Cn) return 0.0;
        if (kind == BDA_SIDE_Q) return w(c, j);
        if (kind == BDA_SIDE_O) return load_as_double<WT>(a.side, (col0 + j) * a.ld_side + c);
        return 0.0;
    };
    // second product: P2(r, c) = sum_i a2(r, i) b2(i, c), absent at the window's columns (Q) / rows (O)
    auto a2 = [&](int r, int i) -> double {
        if (r >= R) return 0.0;
        if (kind == BDA_SIDE_Q) return load_as_double<CT>(a.side_out, (int64_t)r * a.ld_side_out + col0 + i);
        if (kind == BDA_SIDE_O) return in_window(r) ? 0.0 : chat(outside_index(r), i);
        return chat(r, i);
    };
    auto b2 = [&](int i, int c) -> double {
        if (c >= Cn) return 0.0;
        if (kind == BDA_SIDE_Q) return in_window(c) ? 0.0 : chat(outside_index(c), i);
        if (kind == BDA_SIDE_O) return load_as_double<CT>(a.side_out, (col0 + i) * a.ld_side_out + c);
        return w(off + i, c);
    };
    // what stands alone: minus Bhat at the window (Q, O); plus the row of W_h itself (no companion)
    auto lone = [&](int r, int c) -> double {
        if (r >= R || c >= Cn) return 0.0;
        if (kind == BDA_SIDE_Q) return in_window(c) ? -load_as_double<CT>(a.side_out, (int64_t)r * a.ld_side_out + col0 + (c - off)) : 0.0;
        if (kind == BDA_SIDE_O) return in_window(r) ? -load_as_double<CT>(a.side_out, (col0 + (r - off)) * a.ld_side_out + c) : 0.0;
        return w(r < off ? r : r + n, c);
    };
    const int tx = t % 16, ty = t / 16;
    const int tiles_c = (Cn + TS - 1) / TS, n_tiles = ((R + TS - 1) / TS) * tiles_c;
    double r2 = 0.0;
    if (off >= 0) {
        for (int tile = blockIdx.y; tile < n_tiles; tile += gridDim.y) {
            const int r0 = (tile / tiles_c) * TS, c0 = (tile % tiles_c) * TS;
            double acc[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
            for (int pass = (kind == BDA_SIDE_NONE ? 1 : 0); pass < 2; ++pass) {
                for (int j0 = 0; j0 < n; j0 += KC) {
                    for (int e = t; e < TS * KC; e += kPrepThreads) {
                        const int rr = e / KC, jj = e % KC;
                        const bool ok = j0 + jj < n;
                        As[rr][jj] = !ok ? 0.0 : pass == 0 ? a1(r0 + rr, j0 + jj) : -a2(r0 + rr, j0 + jj);
                        Bs[jj][rr] = !ok ? 0.0 : pass == 0 ? b1(j0 + jj, c0 + rr) : b2(j0 + jj, c0 + rr);
                    }
                    __syncthreads();
#pragma unroll
                    for (int jj = 0; jj < KC; ++jj) {
                        double av[4], bv[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) av[u] = As[ty + 16 * u][jj];
#pragma unroll
                        for (int v = 0; v < 4; ++v) bv[v] = Bs[jj][tx + 16 * v];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int v = 0; v < 4; ++v) acc[u][v] = fma(av[u], bv[v], acc[u][v]);
                    }
                    __syncthreads();
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double d = acc[u][v] + lone(r0 + ty + 16 * u, c0 + tx + 16 * v);
                    r2 += d * d;
                }
        }
    }
    red[t] = r2;
    __syncthreads();
    if (t == 0) {
        double sum = 0.0;
        for (int i = 0; i < kPrepThreads; ++i) sum += red[i];
        a.partials[((size_t)a.cand * a.H + h) * a.n_parts + blockIdx.y] = sum;
    }
}

// ---------------------------------------------------------------------------------------------
// Companion block and reconstruction error of the stored form with a companion, d_c up to 512.
//
// With S the companion seen as d_side x d_h (W_q^h, or W_o^h transposed) both kinds need P = S W_h^T
// (d_side x d_c): the companion block of ANY window is columns [off, off + d_h) of P, rounded, and the
// error matrix is P - [Phat at the window, Phat_window Chat^T outside it].  A workgroup takes 32 rows of P
// at a time and keeps them while it goes through all candidate windows of the launch: the exact values in
// the matrix cores' result layout in registers (they are the initial accumulators), the rounded ones in
// LDS (any window's columns of them are the row operand).  What a window costs is then only its own product
// 32 x (d_c - d_h) x d_h, whose column operand - the rows of the stored Chat - comes from the L2.
//
// Wave w of nw owns the 16-column tiles w, w + nw, ... of P, both 16-row tiles of each.  Contraction in
// blocks of 32: lane group g takes elements 8 g .. 8 g + 7 of a block (one wide load), element s of each
// group in step s - the same order for both operands, so it is only the order of the sum that changes.
// Each lane adds its squares in a fixed order, the lanes of a wave, the waves and (in select_kernel) the
// parts of a head likewise: the result does not depend on scheduling or on how windows are batched.
// Bound: the double-precision matrix rate.  Against a companion kernel and an error kernel that formed all
// three products per window in vector FMAs fed from LDS (0.05 + 0.35 ms per window for 16 heads of 128,
// d_c 512, d_side 2048): a 25-window search of keys and values 27.5 -> 8.2 ms, two windows for 128 heads
// 5.4 -> 2.2 ms; with a block's row operand read once for all tiles, the column operands fetched a block
// ahead and contiguous for W_o too, 7.0 ms (46 TFLOP/s while a window is measured).
// A wave holds up to 256 registers of tiles, so a compute unit takes eight waves: with narrow latents or
// heads they must be several workgroups, or most of them have no tile (one form of eight waves for all: 120
// heads of 16, d_c 80, d_side 2048, one window, 160 us against 69 with the vector FMAs; 56 now).
// ---------------------------------------------------------------------------------------------
constexpr int kStripThreads = 512, kStripRows = 32, kStripMaxDc = 512, kStripWaves = kStripThreads / 64;

// Wide: measures, 257 .. 512 latent columns; 8 waves, as many tiles each as their registers hold.  Narrow: measures, up to 256.
// Window: no measurement, only the tiles that the window meets (of 256 columns at any start: 17).
enum class StripForm { Wide, Narrow, Window };
constexpr int strip_tiles(StripForm f) { return f == StripForm::Wide ? kStripMaxDc / 16 / kStripWaves : f == StripForm::Narrow ? 2 : 3; }   // 16-column tiles per wave

template <typename T> __device__ __forceinline__ T rounded(double v)
{
    T r;
    store_rounded<T>(&r, 0, v);
    return r;
}
template <typename T> __device__ __forceinline__ double widened(T v) { return load_as_double<T>(&v, 0); }

// widened(rounded<T>(v)) in a few integer operations: the upper word of a double keeps M mantissa bits, to nearest even, and
// below the smallest normal T the distance of neighbours stays 2^-E, which one addition rounds to.  (Written as rounded and
// widened it is some 25 instructions, and vector instructions do not run beside the float64 MFMAs.)
template <typename T>
__device__ __forceinline__ double round_trip(double v)
{
    if constexpr (sizeof(T) != 2) {
        return widened<T>(rounded<T>(v));
    } else {
        constexpr bool kHalf = std::is_same<T, _Float16>::value;
        constexpr int M = kHalf ? 10 : 7;
        constexpr double kMinNormal = kHalf ? 0x1p-14 : 0x1p-126, kUlp = kHalf ? 0x1.8p28 : 0x1.8p-81, kMax = kHalf ? 65520.0 : 0x1.ffp127;
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        constexpr int drop = 52 - M;
        const uint64_t r = (b + ((((uint64_t)1 << (drop - 1)) - 1) + ((b >> drop) & 1))) & ~(((uint64_t)1 << drop) - 1);
        double x = __builtin_bit_cast(double, r);
        const double mag = fabs(v);
        if (mag < kMinNormal) {
            const double s = copysign(kUlp, v);
            x = copysign((v + s) - s, v);
        }
        if (mag >= kMax) x = copysign(__builtin_huge_val(), v);
        return v == v ? x : v;
    }
}

template <typename T>
struct Eight {
    T e[8];
};

// Eight elements; those from `valid` on are zero.  `vec` (uniform): 16-byte aligned, valid either <= 0 or >= 8.
template <typename T>
__device__ __forceinline__ Eight<T> fetch8(const T* p, int valid, bool vec)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int Q = (int)sizeof(T) / 2;      // 16-byte pieces
    u32x4 w[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) w[q] = (u32x4){0, 0, 0, 0};
    if (vec) {
        if (valid >= 8) {
#pragma unroll
            for (int q = 0; q < Q; ++q) w[q] = ((const u32x4*)p)[q];
        }
        return __builtin_bit_cast(Eight<T>, w);
    }
    Eight<T> r = __builtin_bit_cast(Eight<T>, w);
#pragma unroll
    for (int s = 0; s < 8; ++s)
        if (s < valid) r.e[s] = p[s];
    return r;
}

// Columns of P that a strip keeps (a multiple of 16): all of them to measure windows, or the tiles that one window of
// any start meets; LDS rows of doubles for them and for the strip of S.
__host__ __device__ constexpr int strip_width(bool measure, int d_c, int n) { return ((measure ? d_c : n + 15) + 15) / 16 * 16; }
__host__ __device__ constexpr int strip_pitch_p(int width) { return width + 2; }
__host__ __device__ constexpr int strip_pitch_s(int n) { return (n + 31) / 32 * 32 + 2; }
__host__ __device__ constexpr int strip_words(int width, int n)
{
    const int p = strip_pitch_p(width), s = strip_pitch_s(n);
    return kStripRows * (p > s ? p : s);
}

template <typename WT, typename CT, StripForm F>
__global__ __launch_bounds__(kStripThreads) void strip_kernel(const PrepArgs a)
{
    constexpr bool MEASURE = F != StripForm::Window;
    constexpr int TILES = strip_tiles(F);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    double* const ph = (double*)smem_raw;      // first the strip of S, then the rounded strip of P
    const int n = a.d_h, d_c = a.d_c, t = threadIdx.x, lane = t & 63, c = lane & 15, g = lane >> 4;
    const int threads = F == StripForm::Wide ? kStripThreads : blockDim.x, nw = threads >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int h = blockIdx.x;
    const int off0 = window_start(a);
    if (off0 < 0) return;
    const int64_t col0 = (int64_t)h * n;
    const bool q_side = a.side_kind == BDA_SIDE_Q;
    const int n_blk = (n + 31) >> 5, npk = n_blk * 32, lds_s = strip_pitch_s(n);
    const int width = strip_width(MEASURE, d_c, n), lds_p = strip_pitch_p(width);
    const int base = MEASURE ? 0 : off0 & ~15;                              // first column of P that is kept
    const int l_end = MEASURE ? d_c : off0 + n;                             // end of the columns needed
    const int z_lo = MEASURE ? (int)((int64_t)a.n_cand * blockIdx.z / gridDim.z) : 0;
    const int z_hi = MEASURE ? (int)((int64_t)a.n_cand * (blockIdx.z + 1) / gridDim.z) : 0;
    double* const sums = ph + strip_words(width, n);                        // [wave][window - z_lo]
    const int n_z = z_hi - z_lo;
    const WT* const W = (const WT*)a.W;
    const WT* const S = (const WT*)a.side;
    CT* const side_out = (CT*)a.side_out;
    const bool w_vec = n % 8 == 0 && (uintptr_t)W % 16 == 0 && (a.ldw * (int64_t)sizeof(WT)) % 16 == 0;
    for (int z = lane; z < n_z; z += 64) sums[wave * n_z + z] = 0.0;

    const int n_strips = (a.d_side + kStripRows - 1) / kStripRows;
    for (int strip = blockIdx.y; strip < n_strips; strip += gridDim.y) {
        const int s0 = strip * kStripRows;
        __syncthreads();                       // the strip before is no longer read
        if (q_side && npk == 32) {             // several rows per wave and load; zeros beside the narrow ones
            const int shift = n <= 4 ? 2 : n <= 8 ? 3 : n <= 16 ? 4 : 5, kw = 1 << shift, k = t & (kw - 1);
#pragma unroll 4
            for (int r = t >> shift; r < kStripRows; r += threads >> shift)
                ph[r * lds_s + k] = (k < n && s0 + r < a.d_side) ? widened<WT>(S[(int64_t)(s0 + r) * a.ld_side + col0 + k]) : 0.0;
            if (kw < 32)
                for (int r = t >> 5; r < kStripRows; r += 2 * nw)
                    if ((t & 31) >= kw) ph[r * lds_s + (t & 31)] = 0.0;
        } else if (q_side) {
            for (int k = lane; k < npk; k += 64)
#pragma unroll 4
                for (int r = wave; r < kStripRows; r += nw)
                    ph[r * lds_s + k] = (k < n && s0 + r < a.d_side) ? widened<WT>(S[(int64_t)(s0 + r) * a.ld_side + col0 + k]) : 0.0;
        } else {
            const int r = t % kStripRows;
#pragma unroll 4
            for (int k = t / kStripRows; k < npk; k += threads / kStripRows)
                ph[r * lds_s + k] = (k < n && s0 + r < a.d_side) ? widened<WT>(S[(col0 + k) * a.ld_side + s0 + r]) : 0.0;
        }
        __syncthreads();

        // ---- P: rows s0 .. s0 + 31, this wave's column tiles ----
        f64x4 P[TILES][2];
        bool live[TILES];
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            P[j][0] = P[j][1] = (f64x4){0.0, 0.0, 0.0, 0.0};
            live[j] = base + (wave + nw * j) * 16 < l_end;
        }
        Eight<WT> w[TILES];
        auto fetch_w = [&](int b) {
#pragma unroll
            for (int j = 0; j < TILES; ++j) {
                const int l = base + (wave + nw * j) * 16 + c, k0 = 32 * b + 8 * g;
                w[j] = fetch8<WT>(W + (int64_t)l * a.ldw + col0 + k0, live[j] && l < d_c ? n - k0 : 0, w_vec);
            }
        };
        constexpr bool kAheadW = sizeof(WT) <= 4, kAheadC = sizeof(CT) <= 2;   // (as far as the registers go)
        if (kAheadW) fetch_w(0);
        for (int b = 0; b < n_blk; ++b) {
            const int k0 = 32 * b + 8 * g;
            if (!kAheadW) fetch_w(b);
            Eight<WT> now[TILES];
#pragma unroll
            for (int j = 0; j < TILES; ++j) now[j] = w[j];
            if (kAheadW && b + 1 < n_blk) fetch_w(b + 1);
            double av[2][8];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int s = 0; s < 8; ++s) av[rt][s] = ph[(16 * rt + c) * lds_s + k0 + s];
#pragma unroll
            for (int j = 0; j < TILES; ++j)
                if (live[j]) {
#pragma unroll
                    for (int s = 0; s < 8; ++s) {
                        const double bv = widened<WT>(now[j].e[s]);
                        P[j][0] = mfma_f64(av[0][s], bv, P[j][0]);
                        P[j][1] = mfma_f64(av[1][s], bv, P[j][1]);
                    }
                }
        }
        __syncthreads();                       // the strip of S is no longer read
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            const int l = base + (wave + nw * j) * 16 + c;
            if (live[j] && l < d_c) {
#pragma unroll
                for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) ph[(16 * rt + 4 * r + g) * lds_p + l - base] = widened<CT>(rounded<CT>(P[j][rt][r]));
            }
        }
        __syncthreads();

        if (a.write_side) {
            for (int e = t; e < kStripRows * n; e += threads) {
                const int r = q_side ? e / n : e % kStripRows, i = q_side ? e % n : e / kStripRows;
                if (s0 + r < a.d_side) {
                    const CT v = rounded<CT>(ph[r * lds_p + off0 - base + i]);
                    if (q_side) side_out[(int64_t)(s0 + r) * a.ld_side_out + col0 + i] = v;
                    else side_out[(col0 + i) * a.ld_side_out + s0 + r] = v;
                }
            }
        }

        // ---- the windows: blocks of the contraction outside, this wave's tiles inside, so that a block's row operand is
        // read once for all of them; the column operands are fetched one block ahead, across windows ----
        if constexpr (MEASURE) {
            Eight<CT> ct[TILES];
            auto fetch_c = [&](int z, int b) {
                const int off = window_start(a, z), k0 = 32 * b + 8 * g;
                const Slot slot = slot_of(a, z);
                const bool c_vec = n % 8 == 0 && (uintptr_t)slot.p % 16 == 0 && (slot.ld * (int64_t)sizeof(CT)) % 16 == 0;
#pragma unroll
                for (int j = 0; j < TILES; ++j) {
                    const int l = (wave + nw * j) * 16 + c;
                    const bool outside = l < d_c && (l < off || l >= off + n);      // (a lane inside the window adds nothing)
                    ct[j] = fetch8<CT>((const CT*)slot.p + slot_row(slot, l < off ? l : l - n, h, n) + k0, outside ? n - k0 : 0, c_vec);
                }
            };
            if (kAheadC && z_lo < z_hi) fetch_c(z_lo, 0);
            for (int z = z_lo; z < z_hi; ++z) {
                const int off = window_start(a, z);
                f64x4 acc[TILES][2];
#pragma unroll
                for (int j = 0; j < TILES; ++j) { acc[j][0] = -P[j][0]; acc[j][1] = -P[j][1]; }
                for (int b = 0; b < n_blk; ++b) {
                    const int k0 = 32 * b + 8 * g;
                    if (!kAheadC) fetch_c(z, b);
                    Eight<CT> now[TILES];
#pragma unroll
                    for (int j = 0; j < TILES; ++j) now[j] = ct[j];
                    if (kAheadC) {
                        if (b + 1 < n_blk) fetch_c(z, b + 1);
                        else if (z + 1 < z_hi) fetch_c(z + 1, 0);
                    }
#pragma unroll
                    for (int half = 0; half < 8; half += 4) {
                        double av[2][4];
#pragma unroll
                        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                            for (int s = 0; s < 4; ++s) av[rt][s] = k0 + half + s < n ? ph[(16 * rt + c) * lds_p + off + k0 + half + s] : 0.0;
#pragma unroll
                        for (int j = 0; j < TILES; ++j) {
                            const int l0 = (wave + nw * j) * 16;
                            if (l0 < d_c && (l0 < off || l0 + 16 > off + n)) {
#pragma unroll
                                for (int s = 0; s < 4; ++s) {
                                    const double bv = widened<CT>(now[j].e[half + s]);
                                    acc[j][0] = mfma_f64(av[0][s], bv, acc[j][0]);
                                    acc[j][1] = mfma_f64(av[1][s], bv, acc[j][1]);
                                }
                            }
                        }
                    }
                }
                double r2 = 0.0;
#pragma unroll
                for (int j = 0; j < TILES; ++j) {
                    const int l = (wave + nw * j) * 16 + c;
                    const bool in_window = l >= off && l < off + n;
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            double d = acc[j][rt][r];
                            if (in_window) d += ph[(16 * rt + 4 * r + g) * lds_p + l];
                            r2 = fma(d, d, r2);
                        }
                }
                for (int s = 32; s >= 1; s >>= 1) r2 += __shfl_xor(r2, s, 64);
                if (lane == 0) sums[wave * n_z + z - z_lo] += r2;
            }
        }
    }
    if (!MEASURE) return;
    __syncthreads();
    for (int z = z_lo + t; z < z_hi; z += threads) {
        double sum = 0.0;
        for (int w = 0; w < nw; ++w) sum += sums[w * n_z + z - z_lo];
        a.partials[((size_t)(a.cand + z) * a.H + h) * a.n_parts + blockIdx.y] = sum;
    }
}

// ---------------------------------------------------------------------------------------------
// strip_kernel's measuring forms for the shapes that nearly every projection has: head widths 32 NBLK, latents of whole
// 16-column tiles, windows that start on multiples of 16, 16-byte aligned rows, 16-bit results.  A tile then lies inside a
// window or outside it, a lane's operands are always eight elements, and nothing in the loops depends on the lane but
// addresses.  What that buys is exact counts of loads in flight: with a branch per lane the compiler waits for every load
// before it uses any, so that the blocks fetched ahead were waited for at once (MFMA pipes busy 55 %).  Buffer loads return
// zeros past the arrays' ends.  LDS holds the strip of -Phat, and a window's first product starts from P itself.
// Vector instructions do not run beside the float64 MFMAs (one between every two MFMAs of a loop costs 12 cycles, four 19,
// of the MFMA's 64), so conversions come together, addresses are scalar and a lane's squares stay in LDS till the end.
// Same sums as strip_kernel, in the same order but for a lane's squares over the strips.
// The form for 257 .. 512 columns spills 28 to 75 of its 256 registers (offsets of the strip's rows and tiles, which all strips share: stored once,
// fetched once a strip); the loop over the windows has no scratch access.  The form up to 256 columns spills none.
// Against strip_kernel: 25 windows of 16 heads for keys and values 7.05 -> 6.0 ms, two windows of 128 heads 2.15 -> 1.87 (with
// the chosen window copied instead of prepared again; the matrix pipes busy 69 % of the time, 54 before); with the inversion
// in panels 5.77 and 1.85.
// ---------------------------------------------------------------------------------------------
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
constexpr uint32_t kNoOffset = 0x80000000u;   // beyond every range here

__device__ __forceinline__ __amdgpu_buffer_rsrc_t range_of(const void* p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ Eight<T> load8(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    constexpr int Q = (int)sizeof(T) / 2;
    struct { u32x4_t w[Q]; } v;
#pragma unroll
    for (int q = 0; q < Q; ++q) v.w[q] = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff + 16 * q, 0);
    return __builtin_bit_cast(Eight<T>, v);
}

template <typename WT, typename CT, int NBLK, StripForm F>
__global__ __launch_bounds__(kStripThreads) void measure_kernel(const PrepArgs a)
{
    constexpr int TILES = strip_tiles(F), n = 32 * NBLK, lds_s = strip_pitch_s(n);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    double* const ph = (double*)smem_raw;      // first the strip of S, then the rounded strip of -P
    const int d_c = a.d_c, t = threadIdx.x, lane = t & 63, c = lane & 15, g = lane >> 4;
    const int threads = F == StripForm::Wide ? kStripThreads : blockDim.x, nw = threads >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int h = blockIdx.x, n_tiles = d_c / 16;
    const int64_t col0 = (int64_t)h * n;
    const bool q_side = a.side_kind == BDA_SIDE_Q;
    const int lds_p = strip_pitch_p(d_c);
    const int z_lo = (int)((int64_t)a.n_cand * blockIdx.z / gridDim.z), z_hi = (int)((int64_t)a.n_cand * (blockIdx.z + 1) / gridDim.z);
    double* const sums = ph + strip_words(d_c, n);                           // [wave][window - z_lo]
    const int n_z = z_hi - z_lo;
    const WT* const S = (const WT*)a.side;
    CT* const side_out = (CT*)a.side_out;
    const bool lane_sums = a.lane_sums;
    for (int z = lane; z < (lane_sums ? 64 * n_z : n_z); z += 64) sums[wave * n_z * (lane_sums ? 64 : 1) + z] = 0.0;

    const __amdgpu_buffer_rsrc_t rW = range_of((const WT*)a.W + col0, ((int64_t)(d_c - 1) * a.ldw + n) * (int64_t)sizeof(WT));
    const __amdgpu_buffer_rsrc_t rC = range_of(a.C, ((int64_t)(d_c - n - 1) * a.ldC + (int64_t)a.H * n) * (int64_t)sizeof(CT));
    const int64_t out_rows = q_side ? a.d_side : (int64_t)a.H * n, out_cols = q_side ? (int64_t)a.H * n : a.d_side;
    const __amdgpu_buffer_rsrc_t rO = range_of(a.side_out, ((out_rows - 1) * a.ld_side_out + out_cols) * (int64_t)sizeof(CT));
    auto tile = [&](int j) { return wave + nw * j; };
    auto in_window = [&](int off, int j) { return 16 * tile(j) >= off && 16 * tile(j) < off + n; };
    const uint32_t c_lane = (uint32_t)(c * a.ldC + 8 * g) * (uint32_t)sizeof(CT), o_lane = (uint32_t)(c * a.ld_side_out + 8 * g) * (uint32_t)sizeof(CT);
    uint32_t w_off[TILES];
#pragma unroll
    for (int j = 0; j < TILES; ++j)
        w_off[j] = tile(j) < n_tiles ? (uint32_t)((16 * tile(j) + c) * a.ldw + 8 * g) * (uint32_t)sizeof(WT) : kNoOffset;

    // The strip of S.  Eight waves have a fixed share of it, fetched while the windows of the strip before are measured (a
    // compute unit holds one workgroup, so nothing else covers the fetch); fewer waves are several workgroups.
    constexpr bool kAhead = F == StripForm::Wide;
    constexpr int OWN = kAhead ? kStripRows * n / kStripThreads : 1;
    WT own[OWN];
    auto s_place = [&](int e, int& r, int& k) {  // element e of this thread's
        const int i = e * kStripThreads + t;
        r = q_side ? i / n : i % kStripRows;
        k = q_side ? i % n : i / kStripRows;
    };
    auto fetch_s = [&](int s0) {
#pragma unroll
        for (int e = 0; e < OWN; ++e) {
            int r, k;
            s_place(e, r, k);
            own[e] = (WT)0.0f;
            if (s0 + r < a.d_side) own[e] = q_side ? S[(int64_t)(s0 + r) * a.ld_side + col0 + k] : S[(col0 + k) * a.ld_side + s0 + r];
        }
    };
    const int n_strips = (a.d_side + kStripRows - 1) / kStripRows;
    if (kAhead) fetch_s(blockIdx.y * kStripRows);
    for (int strip = blockIdx.y; strip < n_strips; strip += gridDim.y) {
        const int s0 = strip * kStripRows;
        Eight<WT> w[2][TILES];
#pragma unroll
        for (int j = 0; j < TILES; ++j) w[0][j] = load8<WT>(rW, w_off[j], 0);
        __syncthreads();                       // the strip before is no longer read
        if constexpr (kAhead) {
#pragma unroll
            for (int e = 0; e < OWN; ++e) {
                int r, k;
                s_place(e, r, k);
                ph[r * lds_s + k] = widened<WT>(own[e]);
            }
        } else if (q_side) {
            constexpr int PER = n % 64 ? 32 : 64, ROWS = 64 / PER;            // columns and rows of a wave's load
#pragma unroll
            for (int k = 0; k < n; k += PER)
#pragma unroll 4
                for (int r = wave * ROWS + lane / PER; r < kStripRows; r += nw * ROWS) {
                    const int kk = k + lane % PER;
                    ph[r * lds_s + kk] = s0 + r < a.d_side ? widened<WT>(S[(int64_t)(s0 + r) * a.ld_side + col0 + kk]) : 0.0;
                }
        } else {
            const int r = t % kStripRows;
#pragma unroll 4
            for (int k = t / kStripRows; k < n; k += threads / kStripRows)
                ph[r * lds_s + k] = s0 + r < a.d_side ? widened<WT>(S[(col0 + k) * a.ld_side + s0 + r]) : 0.0;
        }
        __syncthreads();

        // ---- P: rows s0 .. s0 + 31, this wave's column tiles ----
        f64x4 P[TILES][2];
#pragma unroll
        for (int j = 0; j < TILES; ++j) P[j][0] = P[j][1] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            if (b + 1 < NBLK) {
#pragma unroll
                for (int j = 0; j < TILES; ++j) w[(b + 1) & 1][j] = load8<WT>(rW, w_off[j], (uint32_t)(32 * (b + 1) * sizeof(WT)));
            }
            f64x2 av[2][4];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int s = 0; s < 4; ++s) av[rt][s] = *(const f64x2*)(ph + (16 * rt + c) * lds_s + 32 * b + 8 * g + 2 * s);
#pragma unroll
            for (int j = 0; j < TILES; ++j) {
                if (tile(j) >= n_tiles) continue;
                double bv[8];
#pragma unroll
                for (int s = 0; s < 8; ++s) bv[s] = widened<WT>(w[b & 1][j].e[s]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    P[j][0] = mfma_f64(av[0][s >> 1][s & 1], bv[s], P[j][0]);
                    P[j][1] = mfma_f64(av[1][s >> 1][s & 1], bv[s], P[j][1]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // Rows of the stored Chat for window z.  Everything that changes with the window is scalar: a tile's 16 rows are
        // consecutive rows of the output (see Slot).  A tile inside the window, or past the last, fetches rows of another.
        Eight<CT> ct[2][TILES];
        int off = 0, next_off = 0;
        bool in_c = false;
        uint32_t c_soff[TILES];
        auto enter_window = [&](int z) {
            next_off = window_start(a, z);
            const Slot slot = slot_of(a, z);
            in_c = !a.search || z < a.c_slots;
#pragma unroll
            for (int j = 0; j < TILES; ++j) {
                const int l0 = 16 * tile(j);
                const int kk0 = l0 < next_off ? l0 : l0 >= next_off + n && l0 < d_c ? l0 - n : 0;
                c_soff[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(slot_row(slot, kk0, h, n) * (int64_t)sizeof(CT)));
            }
        };
        auto fetch = [&](auto set, uint32_t block) {
            const __amdgpu_buffer_rsrc_t r = in_c ? rC : rO;
            const uint32_t voff = in_c ? c_lane : o_lane;
#pragma unroll
            for (int j = 0; j < TILES; ++j) ct[decltype(set)::value][j] = load8<CT>(r, voff, c_soff[j] + block * (uint32_t)(32 * sizeof(CT)));
        };
        if (n_z > 0) {
            enter_window(z_lo);
            fetch(std::integral_constant<int, 0>{}, 0);
        }
        __syncthreads();                       // the strip of S is no longer read
#pragma unroll
        for (int j = 0; j < TILES; ++j)
            if (tile(j) < n_tiles) {
#pragma unroll
                for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) ph[(16 * rt + 4 * r + g) * lds_p + 16 * tile(j) + c] = -round_trip<CT>(P[j][rt][r]);
                __builtin_amdgcn_sched_barrier(0);
            }
        __syncthreads();

        if (a.write_side) {
            const int off0 = window_start(a);
            for (int e = t; e < kStripRows * n; e += threads) {
                const int r = q_side ? e / n : e % kStripRows, i = q_side ? e % n : e / kStripRows;
                if (s0 + r < a.d_side) {
                    const CT v = rounded<CT>(-ph[r * lds_p + off0 + i]);
                    if (q_side) side_out[(int64_t)(s0 + r) * a.ld_side_out + col0 + i] = v;
                    else side_out[(col0 + i) * a.ld_side_out + s0 + r] = v;
                }
            }
        }

        if (kAhead && strip + (int)gridDim.y < n_strips) fetch_s(s0 + (int)gridDim.y * kStripRows);

        // ---- the windows: blocks of the contraction outside, this wave's tiles inside, so that a block's row operand is read
        // once for all of them; the column operands are fetched one block ahead, across windows ----
        auto window = [&](auto set0, int z) {  // set0: where the window's first block has been fetched to
            constexpr int S0 = decltype(set0)::value;
            off = next_off;
            f64x4 acc[TILES][2];
            static_for_blocks<NBLK>([&](auto bc) {
                constexpr int b = decltype(bc)::value, now = (S0 + b) & 1;
                if constexpr (b + 1 == NBLK) {
                    if (z + 1 < z_hi) enter_window(z + 1);   // (past the last window: its own blocks once more)
                    fetch(std::integral_constant<int, 1 - now>{}, 0);
                } else {
                    fetch(std::integral_constant<int, 1 - now>{}, b + 1);
                }
#pragma unroll
                for (int half = 0; half < 8; half += 4) {
                    f64x2 av[2][2];
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                        for (int s = 0; s < 2; ++s) av[rt][s] = *(const f64x2*)(ph + (16 * rt + c) * lds_p + off + 32 * b + 8 * g + half + 2 * s);
#pragma unroll
                    for (int j = 0; j < TILES; ++j)
                        if (tile(j) < n_tiles && !in_window(off, j)) {
                            double bv[4];      // (together, ahead of the MFMAs: vector instructions between them cost three times as much)
#pragma unroll
                            for (int s = 0; s < 4; ++s) bv[s] = widened<CT>(ct[now][j].e[half + s]);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int s = 0; s < 4; ++s) {
                                acc[j][0] = mfma_f64(av[0][s >> 1][s & 1], bv[s], b + half + s == 0 ? P[j][0] : acc[j][0]);
                                acc[j][1] = mfma_f64(av[1][s >> 1][s & 1], bv[s], b + half + s == 0 ? P[j][1] : acc[j][1]);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                }
            });
            double r2 = 0.0;
#pragma unroll
            for (int j = 0; j < TILES; ++j) {
                if (tile(j) >= n_tiles) continue;
                if (in_window(off, j)) {
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const double d = P[j][rt][r] + ph[(16 * rt + 4 * r + g) * lds_p + 16 * tile(j) + c];
                            r2 = fma(d, d, r2);
                        }
                } else {
#pragma unroll
                    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) r2 = fma(acc[j][rt][r], acc[j][rt][r], r2);
                }
            }
            if (lane_sums) {                   // (added over the lanes once, at the end)
                sums[(wave * n_z + z - z_lo) * 64 + lane] += r2;
            } else {
                for (int s = 32; s >= 1; s >>= 1) r2 += __shfl_xor(r2, s, 64);
                if (lane == 0) sums[wave * n_z + z - z_lo] += r2;
            }
        };
        const std::integral_constant<int, 0> set0;
        const std::integral_constant<int, 1> set1;
        if constexpr (NBLK % 2 == 0) {
            for (int z = z_lo; z < z_hi; ++z) window(set0, z);
        } else {
            for (int z = z_lo;;) {
                if (z >= z_hi) break;
                window(set0, z++);
                if (z >= z_hi) break;
                window(set1, z++);
            }
        }
    }
    if (lane_sums)
        for (int z = 0; z < n_z; ++z) {
            double* const at = sums + (wave * n_z + z) * 64;
            double r2 = at[lane];
            for (int s = 32; s >= 1; s >>= 1) r2 += __shfl_xor(r2, s, 64);
            if (lane == 0) at[0] = r2;
        }
    __syncthreads();
    for (int z = z_lo + t; z < z_hi; z += threads) {
        double sum = 0.0;
        for (int w = 0; w < nw; ++w) sum += sums[(w * n_z + z - z_lo) * (lane_sums ? 64 : 1)];
        a.partials[((size_t)(a.cand + z) * a.H + h) * a.n_parts + blockIdx.y] = sum;
    }
}

struct SelectArgs {
    double* partials;           // (a head's first part is overwritten with the root of its sum)
    const int* cand_singular;
    int* basis_offset_out;
    double* resid_out;           // NULL or 3 doubles: first window, last window, chosen window
    int n_cand, H, n_parts, d_c, d_h;
    int offs[kMaxCandidates];
};

// One workgroup.  Every sum is taken by one thread in a fixed order - a head's parts in order, a candidate's
// heads in order, the candidates in order - so the result does not depend on how the work is spread: first
// a thread per (candidate, head) adds that head's parts and leaves the root in the first part's place (the
// partial sums are the call's own workspace), then a thread per candidate takes the mean over the heads,
// then one thread compares the candidates.
constexpr int kSelectThreads = 256;
__global__ __launch_bounds__(kSelectThreads) void select_kernel(const SelectArgs a)
{
    __shared__ double s_mean[kMaxCandidates];
    const int t = threadIdx.x;
    if (a.partials) {
        for (int e = t; e < a.n_cand * a.H; e += kSelectThreads) {
            double* part = a.partials + (size_t)e * a.n_parts;
            double s = 0.0;
            for (int p = 0; p < a.n_parts; ++p) s += part[p];
            part[0] = sqrt(s);
        }
    }
    __syncthreads();
    for (int ci = t; ci < a.n_cand; ci += kSelectThreads) {
        double mean = 0.0;
        if (a.partials) {
            for (int h = 0; h < a.H; ++h) mean += a.partials[((size_t)ci * a.H + h) * a.n_parts];
            mean /= a.H;
        }
        s_mean[ci] = mean;
    }
    __syncthreads();
    if (t != 0) return;
    const double inf = __builtin_huge_val(), nan = __builtin_nan("");
    double best = inf, r_first = nan, r_last = nan;
    int best_off = -1;
    for (int ci = 0; ci < a.n_cand; ++ci) {
        const bool singular = a.cand_singular[ci] != 0;
        double mean = s_mean[ci];
        if (singular || mean != mean) mean = inf;
        if (a.offs[ci] == 0) r_first = mean;
        if (a.offs[ci] == a.d_c - a.d_h) r_last = mean;
        const bool take = best_off < 0 ? !singular : mean < best;
        if (take) { best = mean; best_off = a.offs[ci]; }
    }
    *a.basis_offset_out = best_off;
    if (a.resid_out) { a.resid_out[0] = r_first; a.resid_out[1] = r_last; a.resid_out[2] = best; }
}

// The chosen window's stored C from its slot to C: a wave per piece of d_h elements at a time.
template <typename CT>
__global__ __launch_bounds__(256) void copy_kernel(const PrepArgs a)
{
    const int off = *a.off_ptr, n = a.d_h, K = a.d_c - n;
    if (off < 0) return;
    int z = 0;
    while (z + 1 < a.n_cand && (a.off + z * a.off_step < a.off_last ? a.off + z * a.off_step : a.off_last) != off) ++z;
    const Slot slot = slot_of(a, z);
    const int lane = threadIdx.x & 63;
    for (int64_t e = blockIdx.x * 4 + (threadIdx.x >> 6); e < (int64_t)K * a.H; e += gridDim.x * 4) {
        const int h = (int)(e / K), kk = (int)(e % K);
        const CT* const from = (const CT*)slot.p + slot_row(slot, kk, h, n);
        CT* const to = (CT*)a.C + kk * a.ldC + (int64_t)h * n;
        for (int i = lane; i < n; i += 64) to[i] = from[i];
    }
}

__global__ void fill_int_kernel(int* p, int n, int v)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

int check_launch(const char* what)
{
    const hipError_t err = hipGetLastError();
    return err == hipSuccess ? BDA_OK : fail(BDA_EHIP, "bda_prepare_device: %s: %s", what, hipGetErrorString(err));
}

// Raises a kernel's dynamic LDS limit on the current device (once per device; tried again after a failure).
int raise_lds(const void* kernel, int bytes, LdsLimitState& state)
{
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return fail(BDA_EHIP, "bda_prepare_device: hipGetDevice: %s", hipGetErrorString(err));
    const bool tracked = dev >= 0 && dev < LdsLimitState::kMaxDevices;
    if (tracked && state.done[dev].load(std::memory_order_acquire)) return BDA_OK;
    err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (err != hipSuccess) return fail(BDA_EHIP, "bda_prepare_device: LDS size %d: %s", bytes, hipGetErrorString(err));
    if (tracked) state.done[dev].store(true, std::memory_order_release);
    return BDA_OK;
}

template <int NB>
int launch_invert(const PrepArgs& a, hipStream_t st)
{
    static LdsLimitState once;
    constexpr int lds = invert_lds_bytes<NB>();
    if (int rc = raise_lds((const void*)invert_kernel<NB>, lds, once)) return rc;
    // workgroups per head and window: up to one per compute unit, at most one per row tile.  (They repeat the inversion
    // and share the rows after it: the call alone is faster, and calls on other streams find the chip full.)
    const int row_tiles = (a.d_c - a.d_h + 15) / 16;
    int per_head = 256 / (a.H * a.n_cand);
    per_head = per_head < 1 ? 1 : per_head > row_tiles ? row_tiles : per_head;
    hipLaunchKernelGGL(invert_kernel<NB>, dim3(a.H, per_head, a.n_cand), dim3(kInvertThreads), lds, st, a);
    return check_launch("prepare kernel");
}

template <typename WT, typename CT>
int launch_prepare(PrepArgs a, int batch, hipStream_t st)
{
    const int n = a.d_h;
    if (n <= 32) return launch_invert<1>(a, st);
    if (n <= 64) return launch_invert<2>(a, st);
    if (n <= 96) return launch_invert<3>(a, st);
    if (n <= kPrepLdsDh) return launch_invert<4>(a, st);
    const size_t lds = (size_t)kPrepRows * n * sizeof(double);
    for (int h0 = 0; h0 < a.H; h0 += batch) {
        a.h0 = h0;
        const int heads = a.H - h0 < batch ? a.H - h0 : batch;
        hipLaunchKernelGGL((prepare_wide_kernel<WT, CT>), dim3(heads), dim3(kPrepThreads), lds, st, a);
        if (int rc = check_launch("prepare kernel")) return rc;
    }
    return BDA_OK;
}

// Whether measure_kernel takes the windows of this launch: see there.
template <typename WT, typename CT>
bool regular_windows(const PrepArgs& a)
{
    const int64_t N = (int64_t)a.H * a.d_h, limit = (int64_t)1 << 31;
    const bool q = a.side_kind == BDA_SIDE_Q;
    const int64_t out_rows = q ? a.d_side : N, out_cols = q ? N : a.d_side;
    return a.d_h % 32 == 0 && a.d_h <= kPrepLdsDh && a.d_c % 16 == 0 && a.off % 16 == 0 && a.off_step % 16 == 0 && a.off_last % 16 == 0 && !a.off_ptr &&
           aligned(a.W, 16) && a.ldw * (int64_t)sizeof(WT) % 16 == 0 && aligned(a.C, 16) && a.ldC * (int64_t)sizeof(CT) % 16 == 0 &&
           (a.n_cand == 1 || (aligned(a.side_out, 16) && a.ld_side_out * (int64_t)sizeof(CT) % 16 == 0)) &&
           a.d_c * a.ldw * (int64_t)sizeof(WT) < limit && a.d_c * a.ldC * (int64_t)sizeof(CT) < limit &&
           ((out_rows - 1) * a.ld_side_out + out_cols) * (int64_t)sizeof(CT) < limit;
}

constexpr int kMeasureLds = 160 * 1024;

template <typename WT, typename CT, int NBLK, StripForm F>
int launch_measure(const PrepArgs& a, dim3 grid, int threads, int lds, int max_lds, hipStream_t st)
{
    static LdsLimitState once;
    if (int rc = raise_lds((const void*)measure_kernel<WT, CT, NBLK, F>, max_lds, once)) return rc;
    hipLaunchKernelGGL((measure_kernel<WT, CT, NBLK, F>), grid, dim3(threads), lds, st, a);
    return check_launch("companion kernel");
}

// Waves of a workgroup: as few as hold the strip's column tiles in their registers, so that narrow latents and heads
// leave none idle and a compute unit takes several workgroups; more, up to one per tile, while the launch would not
// give every compute unit eight waves.
template <typename WT, typename CT, StripForm F>
int launch_strip(const PrepArgs& a, hipStream_t st)
{
    static LdsLimitState once;
    constexpr bool measure = F != StripForm::Window;
    constexpr int max_dc = F == StripForm::Narrow ? kStripMaxDc / 2 : kStripMaxDc;
    constexpr int max_lds = (strip_words(strip_width(measure, max_dc, kPrepMaxDh), kPrepMaxDh) + (measure ? kStripWaves * kMaxCandidates : 0)) * (int)sizeof(double);
    if (int rc = raise_lds((const void*)strip_kernel<WT, CT, F>, max_lds, once)) return rc;
    const int64_t n_strips = ((int64_t)a.d_side + kStripRows - 1) / kStripRows;
    const int width = strip_width(measure, a.d_c, a.d_h), tiles = width / 16;
    int nw = F == StripForm::Wide ? kStripWaves : 1;
    while (nw * strip_tiles(F) < tiles || (nw < kStripWaves && nw < tiles && a.H * nw * (measure ? std::min<int64_t>(n_strips, a.n_parts) : n_strips) < 2048)) nw *= 2;
    // a part of a head's error sum is a workgroup; where those leave the chip idle they also share out the windows
    const int64_t parts = measure ? a.n_parts : std::max<int64_t>(1, std::min<int64_t>(n_strips, 16384 / ((int64_t)a.H * nw)));
    const int64_t busy = a.H * std::min(n_strips, parts) * nw;
    const int split = measure ? (int)std::max<int64_t>(1, std::min<int64_t>(4096 / busy, a.n_cand)) : 1;
    const int lds = (strip_words(width, a.d_h) + (measure ? nw * ((a.n_cand + split - 1) / split) : 0)) * (int)sizeof(double);
    if constexpr (measure && sizeof(CT) == 2 && sizeof(WT) <= 4) {
        if (regular_windows<WT, CT>(a)) {
            const dim3 grid(a.H, (unsigned)parts, split);
            // the lanes' sums in LDS where they fit the limit that the kernel was given
            PrepArgs m = a;
            const int most = strip_words(width, a.d_h) * (int)sizeof(double) + nw * ((a.n_cand + split - 1) / split) * 64 * (int)sizeof(double);
            m.lane_sums = most <= kMeasureLds;
            const int lds_m = m.lane_sums ? most : lds;
            switch (a.d_h / 32) {
            case 1: return launch_measure<WT, CT, 1, F>(m, grid, 64 * nw, lds_m, kMeasureLds, st);
            case 2: return launch_measure<WT, CT, 2, F>(m, grid, 64 * nw, lds_m, kMeasureLds, st);
            case 3: return launch_measure<WT, CT, 3, F>(m, grid, 64 * nw, lds_m, kMeasureLds, st);
            default: return launch_measure<WT, CT, 4, F>(m, grid, 64 * nw, lds_m, kMeasureLds, st);
            }
        }
    }
    hipLaunchKernelGGL((strip_kernel<WT, CT, F>), dim3(a.H, (unsigned)parts, split), dim3(64 * nw), lds, st, a);
    return check_launch("companion kernel");
}

// Companion block and (a.measure) reconstruction errors of the windows of this launch.
template <typename WT, typename CT>
int launch_companion(PrepArgs a, hipStream_t st)
{
    if (a.d_c <= kStripMaxDc) {
        if (!a.measure) return launch_strip<WT, CT, StripForm::Window>(a, st);
        return a.d_c > kStripMaxDc / 2 ? launch_strip<WT, CT, StripForm::Wide>(a, st) : launch_strip<WT, CT, StripForm::Narrow>(a, st);
    }
    // wider latents: their strips do not fit the LDS; one window per launch, the companion block first
    const int64_t tiles = (((int64_t)a.d_side + 63) / 64) * ((a.d_h + 63) / 64);   // 64 x 64 tiles of the companion block, at most 64 workgroups a head
    hipLaunchKernelGGL((side_kernel<WT, CT>), dim3(a.H, (unsigned)std::min<int64_t>(tiles, 64)), dim3(kPrepThreads), 0, st, a);
    if (int rc = check_launch("companion kernel")) return rc;
    if (!a.measure) return BDA_OK;
    hipLaunchKernelGGL((residual_kernel<WT, CT>), dim3(a.H, a.n_parts), dim3(kPrepThreads), 0, st, a);
    return check_launch("residual kernel");
}

// What a call needs beyond its inputs and outputs, and where it lies in the workspace.
struct Plan {
    int n_cand, n_parts, batch;
    bool want_resid, big;
    size_t flags_bytes, partial_bytes, mat_bytes_per_head;
    int offs[kMaxCandidates];
};

int make_plan(const char* fn, int d_c, int H, int d_h, int mode, int explicit_offset, bool resid_wanted, Plan& p)
{
    const int last = d_c - d_h;
    p.n_cand = 0;
    switch (mode) {
    case BDA_BASIS_FIRST: p.offs[p.n_cand++] = 0; break;
    case BDA_BASIS_LAST: p.offs[p.n_cand++] = last; break;
    case BDA_BASIS_RESIDUAL_MIN: p.offs[p.n_cand++] = 0; p.offs[p.n_cand++] = last; break;
    case BDA_BASIS_OFFSET_SEARCH:
        if (last / 16 + 2 > kMaxCandidates) return fail(BDA_EINVAL, "%s: more than %d candidate windows", fn, kMaxCandidates);
        for (int o = 0; o <= last; o += 16) p.offs[p.n_cand++] = o;
        if (last % 16) p.offs[p.n_cand++] = last;
        break;
    case BDA_BASIS_EXPLICIT:
        if (explicit_offset < 0 || explicit_offset > last) return fail(BDA_EINVAL, "%s: basis_offset %d outside [0, %d]", fn, explicit_offset, last);
        p.offs[p.n_cand++] = explicit_offset;
        break;
    default: return fail(BDA_EINVAL, "%s: bad basis mode %d", fn, mode);
    }
    p.want_resid = p.n_cand > 1 || resid_wanted;
    p.big = d_h > kPrepLdsDh;
    int parts = 1024 / H;
    p.n_parts = parts < 1 ? 1 : parts > kMaxParts ? kMaxParts : parts;
    p.flags_bytes = kMaxCandidates * sizeof(int);
    p.partial_bytes = p.want_resid ? (((size_t)p.n_cand * H * p.n_parts * sizeof(double) + 255) & ~(size_t)255) : 0;
    p.mat_bytes_per_head = p.big ? (size_t)d_h * d_h * sizeof(double) : 0;
    p.batch = 0;
    return BDA_OK;
}

struct PrepCall {
    const void* W; int64_t ldw; int w_dtype; int d_c, H, d_h;
    const void* side; int64_t ld_side; int d_side; int side_kind;
    int mode, explicit_offset;
    void* C; int64_t ldC; void* side_out; int64_t ld_side_out; int c_dtype;
    int* basis_offset_out; double* resid_out; int* singular_head;
};

template <typename WT, typename CT>
int run_prepare(const PrepCall& c, const Plan& p, unsigned char* ws, hipStream_t st)
{
    int* flags = (int*)ws;
    double* partials = p.want_resid ? (double*)(ws + p.flags_bytes) : nullptr;
    double* mat = p.big ? (double*)(ws + p.flags_bytes + p.partial_bytes) : nullptr;
    PrepArgs a{};
    a.W = c.W; a.side = c.side; a.C = c.C; a.side_out = c.side_out;
    a.status = c.singular_head;
    a.cand_singular = ws ? flags : nullptr;
    a.partials = partials; a.mat = mat;
    a.ldw = c.ldw; a.ld_side = c.ld_side; a.ldC = c.ldC; a.ld_side_out = c.ld_side_out;
    a.d_c = c.d_c; a.H = c.H; a.d_h = c.d_h; a.d_side = c.d_side; a.side_kind = c.side_kind;
    a.n_parts = p.n_parts;
    a.w_type = c.w_dtype; a.c_type = c.c_dtype;
    const bool multi = p.n_cand > 1, companion = c.side_kind != BDA_SIDE_NONE;
    if (ws) {
        hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(kMaxCandidates), 0, st, flags, kMaxCandidates, 0);
        if (int rc = check_launch("fill kernel")) return rc;
    }
    a.off = p.offs[0];
    a.off_step = multi ? p.offs[1] - p.offs[0] : 0;
    a.off_last = p.offs[p.n_cand - 1];
    a.status = multi ? nullptr : c.singular_head;          // during a search a singular window is just a bad candidate
    a.measure = p.want_resid;
    // Candidate windows that one launch prepares and measures: as many stored C's as the outputs have room for
    // until the chosen window is known.
    // A search of a few windows that the companion output can hold alone leaves C out of it: the chosen one is then
    // copied to C, where larger searches prepare it once more (two windows of 128 heads: 178 us).
    int slots = 1;
    const int K = c.d_c - c.d_h;
    a.c_slots = 1;
    if (multi && companion && !p.big && c.d_c <= kStripMaxDc) {
        a.search = 1;
        int beside = c.d_side / K;
        if (c.side_kind == BDA_SIDE_O) {       // (one head width: a multiplication in place of the division; exact to 2^24 pieces)
            a.width_magic = c.d_h > 1 ? (uint32_t)((((uint64_t)1 << 32) + c.d_h - 1) / c.d_h) : 1;
            beside = c.d_h * std::min(c.d_side / c.d_h, 1024) / K;
        }
        a.c_slots = beside >= p.n_cand ? 0 : 1;
        slots = beside + a.c_slots;
    }
    for (int ci = 0; ci < p.n_cand; ci += slots) {
        a.cand = ci;
        a.n_cand = std::min(slots, p.n_cand - ci);
        a.write_side = !multi;
        if (int rc = launch_prepare<WT, CT>(a, p.batch, st)) return rc;
        if (companion) {
            if (int rc = launch_companion<WT, CT>(a, st)) return rc;
        } else if (p.want_resid) {
            hipLaunchKernelGGL((residual_kernel<WT, CT>), dim3(c.H, p.n_parts), dim3(kPrepThreads), 0, st, a);
            if (int rc = check_launch("residual kernel")) return rc;
        }
    }
    if (p.want_resid) {
        SelectArgs s{};
        s.partials = partials; s.cand_singular = flags; s.basis_offset_out = c.basis_offset_out; s.resid_out = c.resid_out;
        s.n_cand = p.n_cand; s.H = c.H; s.n_parts = p.n_parts; s.d_c = c.d_c; s.d_h = c.d_h;
        for (int i = 0; i < p.n_cand; ++i) s.offs[i] = p.offs[i];
        hipLaunchKernelGGL(select_kernel, dim3(1), dim3(kSelectThreads), 0, st, s);
        if (int rc = check_launch("select kernel")) return rc;
    } else if (c.basis_offset_out) {
        hipLaunchKernelGGL(fill_int_kernel, dim3(1), dim3(64), 0, st, c.basis_offset_out, 1, p.offs[0]);
        if (int rc = check_launch("fill kernel")) return rc;
    }
    if (multi) {
        // the chosen window into the outputs for good (its start is read on the device)
        const bool copy = a.search && a.c_slots == 0;
        a.off_ptr = c.basis_offset_out;
        if (copy) {
            const int64_t pieces = (int64_t)K * c.H;
            hipLaunchKernelGGL((copy_kernel<CT>), dim3((unsigned)std::min<int64_t>((pieces + 7) / 8, 2048)), dim3(256), 0, st, a);
            if (int rc = check_launch("copy kernel")) return rc;
        }
        a.search = 0;
        a.cand = 0;
        a.n_cand = 1;
        a.cand_singular = nullptr;
        a.status = c.singular_head;
        a.measure = 0;
        a.write_side = 1;
        if (!copy)
            if (int rc = launch_prepare<WT, CT>(a, p.batch, st)) return rc;
        if (companion) return launch_companion<WT, CT>(a, st);
    }
    return BDA_OK;
}

template <typename WT>
int dispatch_c(const PrepCall& c, const Plan& p, unsigned char* ws, hipStream_t st)
{
    switch (c.c_dtype) {
    case BDA_F64: return run_prepare<WT, double>(c, p, ws, st);
    case BDA_F32: return run_prepare<WT, float>(c, p, ws, st);
    case BDA_F16: return run_prepare<WT, _Float16>(c, p, ws, st);
    case BDA_BF16: return run_prepare<WT, __bf16>(c, p, ws, st);
    default: return fail(BDA_EDTYPE, "bda_prepare_device: bad c_dtype %d", c.c_dtype);
    }
}

int dispatch_w(const PrepCall& c, const Plan& p, unsigned char* ws, hipStream_t st)
{
    switch (c.w_dtype) {
    case BDA_F64: return dispatch_c<double>(c, p, ws, st);
    case BDA_F32: return dispatch_c<float>(c, p, ws, st);
    case BDA_F16: return dispatch_c<_Float16>(c, p, ws, st);
    case BDA_BF16: return dispatch_c<__bf16>(c, p, ws, st);
    default: return fail(BDA_EDTYPE, "bda_prepare_device: bad w_dtype %d", c.w_dtype);
    }
}

// Argument checks shared by the entry points; fills the plan (without the batch size).
int check_call(const char* fn, const PrepCall& c, Plan& p)
{
    if (!c.W || !c.C) return fail(BDA_EINVAL, "%s: NULL W or C", fn);
    if (c.d_h <= 0 || c.d_c <= c.d_h || c.H <= 0) return fail(BDA_EINVAL, "%s: need 0 < d_h < d_c and H > 0", fn);
    if (c.d_h > kPrepMaxDh) return fail(BDA_EINVAL, "%s: d_h = %d exceeds %d (use bda_prepare)", fn, c.d_h, kPrepMaxDh);
    const int64_t N = (int64_t)c.H * c.d_h;
    if (c.ldw < N || c.ldC < N) return fail(BDA_EINVAL, "%s: leading dimension smaller than H d_h = %lld", fn, (long long)N);
    if (c.side_kind != BDA_SIDE_NONE) {
        if (c.side_kind != BDA_SIDE_Q && c.side_kind != BDA_SIDE_O) return fail(BDA_EINVAL, "%s: bad side_kind %d", fn, c.side_kind);
        if (!c.side || !c.side_out || c.d_side <= 0) return fail(BDA_EINVAL, "%s: companion asked for but side or side_out NULL or d_side <= 0", fn);
        const int64_t need = c.side_kind == BDA_SIDE_Q ? N : c.d_side;
        if (c.ld_side < need || c.ld_side_out < need) return fail(BDA_EINVAL, "%s: companion leading dimension too small (need %lld)", fn, (long long)need);
    }
    if (int rc = make_plan(fn, c.d_c, c.H, c.d_h, c.mode, c.explicit_offset, c.resid_out != nullptr, p)) return rc;
    if ((p.n_cand > 1 || c.resid_out) && !c.basis_offset_out) return fail(BDA_EINVAL, "%s: basis_offset_out is NULL", fn);
    return BDA_OK;
}

// Workspace bytes of a call: the flags, the residual partial sums, and (d_h > 128) `batch` basis blocks.
size_t workspace_need(const Plan& p, int batch) { return p.flags_bytes + p.partial_bytes + p.mat_bytes_per_head * (size_t)batch; }

int run_with_workspace(const char* fn, const PrepCall& c, Plan& p, void* workspace, size_t workspace_bytes, hipStream_t st)
{
    const bool needs = p.want_resid || p.big;
    if (!needs) return dispatch_w(c, p, nullptr, st);
    const size_t least = workspace_need(p, p.big ? 1 : 0);
    if (!workspace || workspace_bytes < least)
        return fail(BDA_EINVAL, "%s: workspace of %zu bytes, this call needs at least %zu", fn, workspace ? workspace_bytes : (size_t)0, least);
    if ((uintptr_t)workspace % 16) return fail(BDA_EINVAL, "%s: workspace not 16-byte aligned", fn);
    if (p.big) {
        const size_t heads = (workspace_bytes - p.flags_bytes - p.partial_bytes) / p.mat_bytes_per_head;
        p.batch = (int)(heads < (size_t)c.H ? heads : (size_t)c.H);
    }
    return dispatch_w(c, p, (unsigned char*)workspace, st);
}

// Address of the static scratch array on the current device; looked up once per device.
int static_scratch(const char* fn, unsigned char** out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptrs[kMaxDevices] = {};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return fail(BDA_EHIP, "%s: hipGetDevice: %s", fn, hipGetErrorString(err));
    if (dev < 0 || dev >= kMaxDevices) return fail(BDA_EINVAL, "%s: device index %d beyond %d", fn, dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess || !p) return fail(BDA_EHIP, "%s: hipGetSymbolAddress: %s", fn, hipGetErrorString(err));
        ptrs[dev] = p;
    }
    *out = (unsigned char*)ptrs[dev];
    return BDA_OK;
}

}  // namespace
}  // namespace bda

using namespace bda;

extern "C" size_t bda_prepare_device_workspace_bytes(int d_c, int H, int d_h, bda_basis_mode mode, int want_residuals)
{
    clear_error();
    if (d_h <= 0 || d_c <= d_h || H <= 0 || d_h > kPrepMaxDh) return 0;
    Plan p;
    if (make_plan("bda_prepare_device_workspace_bytes", d_c, H, d_h, (int)mode, 0, want_residuals != 0, p)) return 0;
    if (!p.want_resid && !p.big) return 0;
    return workspace_need(p, p.big ? (H < 32 ? H : 32) : 0);
}

extern "C" int bda_prepare_device_ex(const void* W, int64_t ldw, bda_dtype w_dtype, int d_c, int H, int d_h,
                                     const void* side, int64_t ld_side, int d_side, bda_side side_kind,
                                     bda_basis_mode mode, int explicit_offset,
                                     void* C, int64_t ldC, void* side_out, int64_t ld_side_out, bda_dtype c_dtype,
                                     int* basis_offset_out, double* resid_out, int* singular_head,
                                     void* workspace, size_t workspace_bytes, void* stream)
{
    clear_error();
    const PrepCall c{W, ldw, (int)w_dtype, d_c, H, d_h, side, ld_side, d_side, side ? (int)side_kind : (int)BDA_SIDE_NONE,
                     (int)mode, explicit_offset, C, ldC, side_out, ld_side_out, (int)c_dtype,
                     basis_offset_out, resid_out, singular_head};
    Plan p;
    if (int rc = check_call("bda_prepare_device_ex", c, p)) return rc;
    return run_with_workspace("bda_prepare_device_ex", c, p, workspace, workspace_bytes, (hipStream_t)stream);
}

extern "C" int bda_prepare_device(const void* W, int64_t ldw, bda_dtype w_dtype, int d_c, int H, int d_h,
                                  int basis_offset, void* C, int64_t ldC, bda_dtype c_dtype,
                                  int* singular_head, void* stream)
{
    clear_error();
    if (d_h > kPrepLdsDh) return fail(BDA_EINVAL, "bda_prepare_device: d_h = %d exceeds %d (bda_prepare_device_ex takes a workspace for up to %d)", d_h, kPrepLdsDh, kPrepMaxDh);
    const PrepCall c{W, ldw, (int)w_dtype, d_c, H, d_h, nullptr, 0, 0, (int)BDA_SIDE_NONE, (int)BDA_BASIS_EXPLICIT, basis_offset,
                     C, ldC, nullptr, 0, (int)c_dtype, nullptr, nullptr, singular_head};
    Plan p;
    if (int rc = check_call("bda_prepare_device", c, p)) return rc;
    return dispatch_w(c, p, nullptr, (hipStream_t)stream);
}

extern "C" int bda_prepare_device_static(const void* W, int64_t ldw, bda_dtype w_dtype, int d_c, int H, int d_h,
                                         const void* side, int64_t ld_side, int d_side, bda_side side_kind,
                                         bda_basis_mode mode, int explicit_offset,
                                         void* C, int64_t ldC, void* side_out, int64_t ld_side_out, bda_dtype c_dtype,
                                         int* basis_offset_out, double* resid_out, int* singular_head, void* stream)
{
    clear_error();
    const char* fn = "bda_prepare_device_static";
    const PrepCall c{W, ldw, (int)w_dtype, d_c, H, d_h, side, ld_side, d_side, side ? (int)side_kind : (int)BDA_SIDE_NONE,
                     (int)mode, explicit_offset, C, ldC, side_out, ld_side_out, (int)c_dtype,
                     basis_offset_out, resid_out, singular_head};
    Plan p;
    if (int rc = check_call(fn, c, p)) return rc;
    if (!p.want_resid && !p.big) return dispatch_w(c, p, nullptr, (hipStream_t)stream);
    const size_t least = workspace_need(p, p.big ? 1 : 0);
    if (least > kStaticScratchBytes)
        return fail(BDA_EINVAL, "%s: this call needs %zu bytes of scratch, the built-in scratch holds %zu: use bda_prepare_device_ex with a workspace",
                    fn, least, kStaticScratchBytes);
    unsigned char* ws = nullptr;
    if (int rc = static_scratch(fn, &ws)) return rc;
    return run_with_workspace(fn, c, p, ws, kStaticScratchBytes, (hipStream_t)stream);
}
