"""GPU parity of the K/V projection's gradients (bda_kv_project_backward through the C ABI) against
the fp64 oracle, element by element on the same seeded inputs.

Tolerance: |g - o| <= tol * max(|o|, RMS of o's column) (+ half a bf16 ulp for bf16 storage), with
tol 2e-3 for fp16 / bf16 and 1e-5 for fp32 -- the forward's bar with the per-head floor replaced
by a per-column one: the window columns of grad_c (a sum of a few heads) and its other columns (a
contraction over all output columns) differ in scale by an order of magnitude."""
import numpy as np
import pytest

import bda_workloads as wl
import oracle
from helpers import assert_parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import gpu_harness as gh          # noqa: E402
import paper_2510_01718_amd as bda  # noqa: E402


def _inputs(seed, T, d_c, d_h, H, dtype, c_scale=1.0, C_scale=0.25):
    """Latent rows, upstream gradient and coefficients: independent Gaussians rounded to the
    storage type (the gradient formulas do not care whether C came from a preparation)."""
    rng = np.random.default_rng([seed, T, d_c])
    N = sum(H) * d_h
    c_s, c64 = wl.to_storage(c_scale * rng.standard_normal((T, d_c)), dtype)
    g_s, g64 = wl.to_storage(rng.standard_normal((T, N)), dtype)
    C_s, C64 = wl.to_storage(C_scale * rng.standard_normal((d_c - d_h, N)), dtype)
    return (c_s, c64), (g_s, g64), (C_s, C64)


def _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, grad_dtype=None, pad=0, want=(True, True), fill=None, policy=0):
    grad_dtype = dtype if grad_dtype is None else grad_dtype
    N = sum(H) * d_h
    K = d_c - d_h
    ldc, ldg, ldC, ld_gc, ld_gC = d_c + pad, N + pad, N + 2 * pad, d_c + 3 * pad, N + pad
    c_d = gh.to_device(c_s, dtype, ldc) if T else gh.new_out(1, ldc, dtype)
    g_d = gh.to_device(g_s, dtype, ldg) if T else gh.new_out(1, ldg, dtype)
    C_d = gh.to_device(C_s, dtype, ldC)
    gc_d = gh.new_out(max(T, 1), ld_gc, grad_dtype, fill) if want[0] else None
    gC_d = gh.new_out(K, ld_gC, grad_dtype, fill) if want[1] else None
    if policy:
        bda.bda_kv_project_backward_ex(c_d if want[1] else None, ldc, g_d, ldg, C_d if want[0] else None, ldC,
                                       T, d_c, d_h, H, offs, gc_d, ld_gc, gC_d, ld_gC, dtype, grad_dtype, gh.stream(), policy)
    else:
        bda.bda_kv_project_backward(c_d if want[1] else None, ldc, g_d, ldg, C_d if want[0] else None, ldC,
                                    T, d_c, d_h, H, offs, gc_d, ld_gc, gC_d, ld_gC, dtype, grad_dtype, gh.stream())
    torch.cuda.synchronize()
    gc = gh.to_host64(gc_d[:T], grad_dtype, d_c) if want[0] else None
    gC = gh.to_host64(gC_d, grad_dtype, N) if want[1] else None
    return gc, gC, gc_d, gC_d


def _check(T, d_c, d_h, H, offs, dtype, grad_dtype=None, pad=0, policy=0, seed=5, what=""):
    (c_s, c64), (g_s, g64), (C_s, C64) = _inputs(seed, T, d_c, d_h, H, dtype)
    ref_c, ref_C = oracle.kv_project_backward(c64, g64, C64, d_h, H, offs)
    gc, gC, _, _ = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, grad_dtype, pad, policy=policy)
    gd = dtype if grad_dtype is None else grad_dtype
    tag = f"{what} T={T} d_c={d_c} d_h={d_h} H={H} offs={offs} dtype={dtype}/{gd} policy={policy}"
    if T:
        assert_parity(gc, ref_c, 1, dtype, gd, "grad_c " + tag)
    assert_parity(gC, ref_C, 1, dtype, gd, "grad_C " + tag)


SHAPES = [
    (300, 512, 128, [3, 2], [0, 384]),     # first / last window, ragged token tail
    (130, 256, 64, [2, 3], [64, 192]),     # interior and last window, two groups with different windows
    (77, 192, 32, [5], [40]),              # window start a multiple of 8 only
    (64, 128, 32, [1], [96]),              # a single tile
    (200, 320, 96, [2, 1], [16, 224]),     # d_h not a power of two: chunks of 64 straddle heads
]


@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("T,d_c,d_h,H,offs", SHAPES)
@pytest.mark.parametrize("policy", [0, 1])
def test_backward_mfma_matches_oracle(T, d_c, d_h, H, offs, dtype, policy):
    _check(T, d_c, d_h, H, offs, dtype, policy=policy)


@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
def test_backward_float32_gradients_and_padded_rows(dtype):
    _check(150, 256, 64, [2, 2], [0, 128], dtype, grad_dtype=wl.F32, pad=8)
    _check(150, 256, 64, [2, 2], [192, 64], dtype, grad_dtype=wl.F32, pad=16, policy=1)


@pytest.mark.parametrize("dtype", [wl.F32, wl.F16, wl.BF16])
def test_backward_general_kernels(dtype):
    # fp32 inputs, and 16-bit inputs whose head width / window start / row pitch rule out MFMA tiles
    _check(50, 72, 24, [2, 1], [3, 48], dtype)
    _check(70, 96, 32, [3], [20], dtype, pad=3)
    if dtype != wl.F32:
        _check(33, 64, 16, [2], [8], dtype, grad_dtype=wl.F32)


# The general kernel: each product's remainders in rows, columns and contraction, windows that differ between groups,
# and sizes at which 16-byte pieces do not apply (odd head width or pitch).  (Every tile: test_general_kernel_every_tile.)
GENERAL_SHAPES = [
    (1, 96, 32, [1, 2], [0, 64], 0),            # one token: 32 x 32 tiles, contractions below and above one chunk
    (31, 512, 64, [8, 8], [0, 448], 0),
    (33, 132, 20, [3, 2], [4, 112], 0),         # d_h not a multiple of 32 or 16
    (700, 512, 64, [8, 8], [448, 128], 4),
    (1030, 160, 80, [13, 4], [16, 0], 0),       # 64 x 32 and 32 x 32 tiles, cut
    (2050, 288, 96, [12, 11], [0, 192], 0),
    (4100, 256, 128, [7, 6], [128, 32], 0),     # gradients of 64 x 32 tiles, cut
    (130, 97, 33, [2, 1], [5, 31], 0),          # element by element
    (900, 128, 64, [9, 9], [0, 64], 1),
]


@pytest.mark.parametrize("T,d_c,d_h,H,offs,pad", GENERAL_SHAPES)
def test_float32_general_kernel_tiles(T, d_c, d_h, H, offs, pad):
    """Forward and both gradients.  A float32 sum of n products is off by at most n 2^-24 of the sum of their
    magnitudes, and by about sqrt(n) 2^-24 of the result's own size: 4e-6 at the longest contraction here."""
    _check(T, d_c, d_h, H, offs, wl.F32, pad=pad)
    (c_s, c64), _, (C_s, C64) = _inputs(5, T, d_c, d_h, H, wl.F32)
    N = sum(H) * d_h
    got, raw = gh.kv_project(c_s, C_s, d_c, d_h, H, offs, wl.F32, ldc=d_c + pad, ldC=N + pad, ld_out=N + pad, fill=7.5, extra_rows=1)
    assert_parity(got, oracle.kv_project(c64, C64, d_h, H, offs), d_h, wl.F32, wl.F32, f"forward T={T} d_c={d_c} d_h={d_h}")
    raw = raw.cpu().numpy()
    assert np.all(raw[T:] == 7.5) and np.all(raw[:, N:] == 7.5)


def _general_tile(rows, contraction, H, d_h, dtype, vec):
    """Tile of the general kernel for a product of these extents.  All three products choose by the same rule, so the
    launch plan of a forward with the same output and contraction tells the gradients' tiles (contraction rounded up
    to a multiple of four, which keeps 16-byte pieces possible; an odd pitch rules them out).  (Limits of the latent
    gradient's own: element by element, beyond 256 tiles of 64 x 64 and 80 elements.)"""
    contraction = (contraction + 3) // 4 * 4
    p = bda.bda_kv_project_plan(rows, contraction + d_h, d_h, H, [0] * len(H), dtype,
                                ldC=None if vec else sum(H) * d_h + 1)
    assert p["kernel"] == bda.KERNEL_GENERAL
    return p["tile_tokens"], p["tile_columns"], p["threads"]


T128, T64, T64x32, T32, SHORT = (128, 128, 512), (64, 64, 512), (64, 32, 512), (32, 32, 512), (64, 64, 256)
_VEC = [
    # product, tile, T, d_c, d_h, H, offs: cut rows, columns and contraction, one round of the tile over the compute units
    ("forward", T128, 1990, 136, 64, [15, 15], [0, 72]),
    ("forward", T64, 990, 144, 60, [8, 8], [8, 0]),
    ("forward", T64x32, 990, 144, 60, [3, 5], [8, 84]),
    ("forward", T32, 290, 144, 60, [3, 5], [8, 84]),
    ("latent", T128, 7990, 476, 40, [1, 1], [4, 436]),
    ("latent", T64, 1990, 476, 40, [1, 1], [4, 436]),
    ("latent", T64x32, 990, 476, 40, [1, 1], [0, 100]),
    ("latent", T32, 290, 476, 40, [2, 1], [0, 100]),
    ("weight", T128, 70, 536, 40, [101, 99], [4, 496]),
    ("weight", T64, 70, 536, 40, [26, 24], [4, 496]),
    ("weight", T64x32, 333, 536, 40, [13, 12], [0, 60]),
    ("weight", T32, 333, 536, 40, [5, 6], [0, 60]),
    # short contractions: below, at and above a chunk of 16, up to the limit of 48, and the tile beyond it
    ("forward", SHORT, 130, 60, 40, [3, 2], [0, 20]),
    ("forward", SHORT, 70, 88, 40, [3, 2], [0, 48]),
    ("forward", T32, 70, 92, 40, [3, 2], [0, 48]),
    ("forward", SHORT, 1, 12, 8, [9], [4]),
    ("latent", SHORT, 130, 84, 12, [1, 2], [0, 64]),
    ("latent", SHORT, 300, 512, 48, [1], [128]),
    ("weight", SHORT, 1, 104, 40, [3, 2], [0, 64]),
    ("weight", SHORT, 17, 536, 40, [13, 12], [0, 60]),
    ("weight", SHORT, 48, 200, 72, [5, 2], [12, 100]),
]
# element by element (an odd pitch): 64 x 64, 32 x 32 and the short tile
_ELEM = [
    ("forward", T64, 990, 144, 60, [8, 8], [8, 0]),
    ("forward", T32, 290, 143, 60, [3, 5], [7, 83]),
    ("forward", SHORT, 130, 61, 40, [3, 2], [0, 21]),
    ("forward", SHORT, 66, 34, 33, [3], [1]),
    # beyond 256 tiles of 64 x 64: the short tile for several of its chunks, up to a limit
    ("forward", SHORT, 1400, 172, 60, [8, 8], [8, 0]),
    ("forward", T64, 1400, 176, 60, [8, 8], [8, 0]),
    ("forward", SHORT, 1100, 360, 60, [8, 8], [8, 0]),
    ("latent", SHORT, 2100, 475, 40, [1, 1], [3, 435]),
    ("weight", SHORT, 115, 535, 40, [26, 28], [3, 495]),
    ("latent", T64, 1990, 476, 40, [1, 1], [3, 436]),
    ("latent", T32, 290, 475, 41, [1, 1], [3, 434]),
    ("latent", SHORT, 130, 83, 21, [1, 2], [0, 62]),
    ("weight", T64, 70, 536, 40, [26, 24], [3, 496]),
    ("weight", T32, 333, 535, 41, [5, 6], [0, 60]),
    ("weight", SHORT, 1, 103, 41, [3, 2], [0, 62]),
    ("weight", SHORT, 64, 535, 41, [13, 12], [0, 60]),
]


@pytest.mark.parametrize("product,tile,T,d_c,d_h,H,offs,dtype,grad_dtype,pad",
                         [c + (wl.F32, wl.F32, 4) for c in _VEC] +
                         [c + (d, g, 1) for c in _ELEM for d, g in ((wl.F32, wl.F32), (wl.F16, wl.F16), (wl.BF16, wl.F32))])
def test_general_kernel_every_tile(product, tile, T, d_c, d_h, H, offs, dtype, grad_dtype, pad):
    """Each product with each tile of its rule, in 16-byte pieces and element by element; the rest of the padded rows
    stays as it was.  Tolerance as in test_float32_general_kernel_tiles."""
    N, K, vec = sum(H) * d_h, d_c - d_h, pad % 4 == 0
    (c_s, c64), (g_s, g64), (C_s, C64) = _inputs(7, T, d_c, d_h, H, dtype)
    what = f"{product} tile={tile} T={T} d_c={d_c} d_h={d_h} H={H} dtype={dtype}/{grad_dtype}"
    if product == "forward":
        assert _general_tile(T, K, H, d_h, dtype, vec) == tile, what
        got, raw = gh.kv_project(c_s, C_s, d_c, d_h, H, offs, dtype, grad_dtype, ldc=d_c + pad, ldC=N + pad, ld_out=N + pad, fill=7, extra_rows=1)
        assert_parity(got, oracle.kv_project(c64, C64, d_h, H, offs), d_h, dtype, grad_dtype, what)
        raw = raw.cpu().numpy()
        assert np.all(raw[T:] == 7) and np.all(raw[:, N:] == 7), what
        return
    latent = product == "latent"
    assert _general_tile(T if latent else K, N if latent else T, [1] if latent else H, d_c if latent else d_h, dtype, vec) == tile, what
    ref_c, ref_C = oracle.kv_project_backward(c64, g64, C64, d_h, H, offs)
    gc, gC, gc_d, gC_d = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, grad_dtype, pad, want=(latent, not latent), fill=7)
    assert_parity(gc if latent else gC, ref_c if latent else ref_C, 1, dtype, grad_dtype, what)
    assert torch.all(gc_d[:, d_c:] == 7) if latent else torch.all(gC_d[:, N:] == 7), what


def test_backward_tile_shapes_chosen_by_size():
    # many 64 x 64 tiles (two per compute unit): 65 x 8 for the latent gradient ...
    _check(4100, 512, 128, [1, 1], [0, 384], wl.F16)
    # ... and 6 x 86 for the weight gradient
    _check(100, 512, 128, [22, 21], [384, 0], wl.BF16)
    # 128 x 128 tiles by size: 65 x 4 latent tiles
    _check(8200, 512, 128, [1], [128], wl.BF16)


# Edges of every tile (policies 1 .. 4): outputs of a tile and a few rows or columns, contractions shorter than the ring of stages
# and one element past a stage, windows that cut a 32-column block at either end, groups that end inside a tile and a stage.
EDGES = [
    (193, 448, 64, [5, 1], [16, 376]),
    (129, 576, 192, [1, 2], [40, 344]),
    (65, 136, 96, [1, 1, 1], [0, 24, 40]),
    (1, 200, 32, [9], [88]),
    (33, 264, 256, [1], [8]),
    (257, 328, 128, [3], [200]),
    (520, 64, 32, [17, 8], [0, 32]),
]


@pytest.mark.parametrize("dtype,grad_dtype", [(wl.F16, wl.F32), (wl.BF16, wl.BF16)])
@pytest.mark.parametrize("T,d_c,d_h,H,offs", EDGES)
@pytest.mark.parametrize("policy", [1, 2, 3, 4, 5])
def test_backward_every_tile_edges(T, d_c, d_h, H, offs, dtype, grad_dtype, policy):
    """Tolerance as everywhere here; the longest contraction has 800 terms, whose float32 sums are off by about
    sqrt(800) 2^-24 = 1.7e-6 of the result's size, far below a result's own rounding."""
    _check(T, d_c, d_h, H, offs, dtype, grad_dtype=grad_dtype, pad=8, policy=policy, seed=17)


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("policy", [1, 2, 3, 4])
@pytest.mark.parametrize("T,d_c,d_h,H,offs,head,col", [
    (150, 512, 256, [6], [128], 4, 200),        # four whole blocks of 64; the element's own is the last
    (150, 576, 192, [3, 2], [64, 320], 1, 5),   # two groups with the same blocks of their own; its own is the first
    (70, 512, 256, [5], [136], 3, 55),          # a window that cuts blocks, 16 columns that straddle two
])
def test_backward_non_finite_gradients_stay_in_their_row_and_blocks(T, d_c, d_h, H, offs, head, col, policy, value):
    """grad_c with one infinite or NaN element in d_out against grad_c without: the same bits in all other rows and, where no
    other group adds to them, in the blocks of 64 latent columns inside the window that the element does not belong to."""
    dtype, token = wl.F16, 37
    (c_s, _), (g_s, _), (C_s, _) = _inputs(29, T, d_c, d_h, H, dtype)
    g_s = g_s.copy()
    n = head * d_h + col                          # an element of group 0
    g_s[token, n] = 0
    clean, _, _, _ = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, want=(True, False), policy=policy)
    bad_s, _ = wl.to_storage(np.array([[value]]), dtype)
    g_s[token, n] = bad_s[0, 0]
    got, _, _, _ = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, want=(True, False), policy=policy)
    others = np.arange(T) != token
    assert np.array_equal(got[others], clean[others])
    first = offs[0] + col // 16 * 16
    own = {first // 64, (first + 15) // 64}
    kept = [b for b in range(-(-offs[0] // 64), (offs[0] + d_h) // 64) if b not in own]
    assert kept
    for b in kept:
        assert np.array_equal(got[token, 64 * b:64 * b + 64], clean[token, 64 * b:64 * b + 64]), b
    assert not np.isfinite(got[token, offs[0] + col])
    assert not np.any(np.isfinite(got[token, :offs[0]])) and not np.any(np.isfinite(got[token, offs[0] + d_h:]))


@pytest.mark.parametrize("policy", [0, 1, 2, 3, 4, 5])
def test_backward_short_contractions(policy):
    """Contractions of 1 .. 12 stages of 64 for every tile: shorter than the ring, as long as it, whole turns of it and the
    stages behind them; the last stage whole or in part, in one group or two.  Tolerance as everywhere here."""
    for n in range(1, 13):
        _check(70, 168, 32, [2 * n - 1] if n % 2 else [n, n - 1], [8, 136][: 1 if n % 2 else 2], wl.F16, pad=8, policy=policy, seed=n)
        _check(64 * n - 24 * (n % 2), 168, 64, [n], [40], wl.BF16, grad_dtype=wl.F32, policy=policy, seed=n)


@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("policy", [1, 2, 3, 4, 5])
def test_backward_weight_gradient_sums_are_in_two_parts_at_least(dtype, policy):
    """Error of float32 weight gradients against 64 bits, for every tile.

    A float32 sum of T independent products of unit size that is rounded after every n of them has a size of sqrt(n j) after
    j roundings, so its error is d sqrt(T / 2n) of the result's sqrt(T); in two sums of T / 2 it is d sqrt(T / 4n).  d, the root
    mean square of one rounding's relative error, is 2^-24 / sqrt(3) times the mean of 1 / m over mantissas m in [1, 2),
    about 0.7: 2.4e-8.  With the two roundings of 8 products each that the errors of this card's MFMAs show, T = 8192 gives
    3.8e-7 in two sums and 5.4e-7 in one (measured 4.0e-7 and 5.7e-7); the bound lies between."""
    T, d_c, d_h, H, offs = 8192, 320, 128, [2], [64]
    (c_s, c64), (g_s, g64), (C_s, C64) = _inputs(23, T, d_c, d_h, H, dtype)
    _, ref = oracle.kv_project_backward(c64, g64, C64, d_h, H, offs)
    _, got, _, _ = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, wl.F32, want=(False, True), policy=policy)
    error = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert error <= 4.7e-7, error


def test_backward_gradients_aligned_to_eight_bytes():
    """16-bit gradients may start on any multiple of 8 bytes: a column view of a wider buffer."""
    T, d_c, d_h, H, offs, dtype = 200, 256, 64, [2, 3], [0, 128], wl.F16
    (c_s, c64), (g_s, g64), (C_s, C64) = _inputs(19, T, d_c, d_h, H, dtype)
    ref_c, ref_C = oracle.kv_project_backward(c64, g64, C64, d_h, H, offs)
    N, K = sum(H) * d_h, d_c - d_h
    c_d, g_d, C_d = gh.to_device(c_s, dtype), gh.to_device(g_s, dtype), gh.to_device(C_s, dtype)
    gc_d, gC_d = gh.new_out(T, d_c + 8, dtype, 3.0), gh.new_out(K, N + 8, dtype, 3.0)
    bda.bda_kv_project_backward(c_d, d_c, g_d, N, C_d, N, T, d_c, d_h, H, offs, gc_d.data_ptr() + 8, d_c + 8, gC_d.data_ptr() + 8, N + 8,
                                dtype, dtype, gh.stream())
    torch.cuda.synchronize()
    gc, gC = gh.to_host64(gc_d, dtype), gh.to_host64(gC_d, dtype)
    assert_parity(gc[:, 4:-4], ref_c, 1, dtype, dtype, "grad_c")
    assert_parity(gC[:, 4:-4], ref_C, 1, dtype, dtype, "grad_C")
    assert np.all(gc[:, :4] == 3) and np.all(gc[:, -4:] == 3) and np.all(gC[:, :4] == 3) and np.all(gC[:, -4:] == 3)


def test_backward_each_gradient_alone_and_no_tokens():
    T, d_c, d_h, H, offs, dtype = 90, 256, 64, [2, 1], [0, 192], wl.F16
    (c_s, c64), (g_s, g64), (C_s, C64) = _inputs(9, T, d_c, d_h, H, dtype)
    ref_c, ref_C = oracle.kv_project_backward(c64, g64, C64, d_h, H, offs)
    gc, none, _, _ = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, want=(True, False))
    assert none is None
    assert_parity(gc, ref_c, 1, dtype, dtype, "grad_c alone")
    none, gC, _, _ = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, want=(False, True))
    assert none is None
    assert_parity(gC, ref_C, 1, dtype, dtype, "grad_C alone")
    # no tokens: the weight gradient is an empty sum
    _, gC0, _, _ = _backward(c_s[:0], g_s[:0], C_s, 0, d_c, d_h, H, offs, dtype, fill=7.0)
    assert gC0.shape == ref_C.shape and not gC0.any()
    (c_s, _), (g_s, _), (C_s, _) = _inputs(9, 0, 72, 24, [2, 1], wl.F32)
    _, gC0, _, _ = _backward(c_s, g_s, C_s, 0, 72, 24, [2, 1], [3, 48], wl.F32, fill=7.0)
    assert gC0.shape == (48, 72) and not gC0.any()


def test_backward_writes_nothing_outside_its_matrices():
    T, d_c, d_h, H, offs, dtype, pad = 70, 128, 32, [2, 1], [32, 96], wl.F16, 8
    (c_s, _), (g_s, _), (C_s, _) = _inputs(11, T, d_c, d_h, H, dtype)
    N = sum(H) * d_h
    _, _, gc_d, gC_d = _backward(c_s, g_s, C_s, T, d_c, d_h, H, offs, dtype, pad=pad, fill=3.0)
    assert torch.all(gc_d[:, d_c:] == 3.0) and torch.all(gC_d[:, N:] == 3.0)


def test_backward_benchmark_shape_full():
    """The V2-Lite-shaped training step (T = 4096, 16 + 16 heads, fp16): every element."""
    _check(4096, 512, 128, [16, 16], [0, 0], wl.F16, what="v2lite")


def test_backward_v3_shape_sampled():
    """The V3-shaped training step (T = 8192, 128 + 128 heads, bf16, two different windows), the
    shape the largest forward configuration has: grad_c on 264 sampled token rows (its rows are
    independent, so the oracle computes exactly those), grad_C on 10 sampled heads (all tokens, all
    rows of C; the oracle is given the reduced problem made of those heads' columns).  Gradients
    start as NaN patterns and must be finite everywhere."""
    T, d_c, d_h, H, offs, dtype = 8192, 512, 128, [128, 128], [0, 384], wl.BF16
    N, K = sum(H) * d_h, d_c - d_h
    rng = np.random.default_rng([31, T, d_c])
    c_s, c64 = wl.to_storage(rng.standard_normal((T, d_c)), dtype)
    C_s, C64 = wl.to_storage(0.25 * rng.standard_normal((K, N)), dtype)
    g_s = np.empty((T, N), dtype=np.uint16)
    for r0 in range(0, T, 512):                                   # chunked: the float64 draw of the whole matrix is 2 GiB
        g_s[r0:r0 + 512], _ = wl.to_storage(rng.standard_normal((512, N)), dtype)
    c_d, g_d, C_d = gh.to_device(c_s, dtype), gh.to_device(g_s, dtype), gh.to_device(C_s, dtype)
    gc_d = gh.new_out(T, d_c, dtype, fill=0x7FC0)
    gC_d = gh.new_out(K, N, dtype, fill=0x7FC0)
    bda.bda_kv_project_backward(c_d, d_c, g_d, N, C_d, N, T, d_c, d_h, H, offs, gc_d, d_c, gC_d, N, dtype, dtype, gh.stream())
    torch.cuda.synchronize()
    gc, gC = gh.to_host64(gc_d, dtype), gh.to_host64(gC_d, dtype)
    assert np.all(np.isfinite(gc)) and np.all(np.isfinite(gC))
    # grad_c: first / last rows, one row per 128-token tile, random rows
    rows = set(range(4)) | set(range(T - 4, T)) | {128 * b + (37 * b + 5) % 128 for b in range(T // 128)}
    rows |= set(int(r) for r in rng.integers(0, T, 192))
    rows = np.array(sorted(rows))
    assert len(rows) >= 256
    ref_c, _ = oracle.kv_project_backward(c64[rows], wl.from_storage(g_s[rows], dtype), C64, d_h, H, offs)
    rel_c = assert_parity(gc[rows], ref_c, 1, dtype, dtype, "v3 grad_c, sampled rows")
    # grad_C: sampled heads of both groups
    heads = sorted({0, 1, 127, 128, 129, 255} | set(int(h) for h in rng.integers(0, 256, 4)))
    cols = np.concatenate([np.arange(h * d_h, (h + 1) * d_h) for h in heads])
    H_sub = [sum(1 for h in heads if h < 128), sum(1 for h in heads if h >= 128)]
    g_sub = wl.from_storage(np.ascontiguousarray(g_s[:, cols]), dtype)
    _, ref_C = oracle.kv_project_backward(c64, g_sub, C64[:, cols], d_h, H_sub, offs)
    rel_C = assert_parity(gC[:, cols], ref_C, 1, dtype, dtype, "v3 grad_C, sampled heads")
    print(f"v3 backward: grad_c {len(rows)} rows {rel_c:.2e}; grad_C {len(heads)} heads {rel_C:.2e}")


@pytest.mark.parametrize("seed", [1, 2])
def test_backward_random_shapes(seed):
    """Seeded random shapes (head widths 32 .. 128 incl. 96, contraction 32 .. 448 in steps of 8 with
    windows anywhere on the multiples of 8, one to three groups, 1 .. 700 tokens, padded rows) through
    both tile shapes of the gradient kernels."""
    rng = np.random.default_rng(3000 + seed)
    for case in range(14):
        d_h = int(rng.choice([32, 64, 96, 128]))
        K = 8 * int(rng.integers(4, 57))
        d_c = K + d_h
        G = int(rng.integers(1, 4))
        H = [int(rng.integers(1, 5)) for _ in range(G)]
        offs = [8 * int(rng.integers(0, K // 8 + 1)) for _ in range(G)]
        T = int(rng.choice([1, 33, 64, 100, 129, 256, 300, 700]))
        dtype = wl.F16 if rng.integers(0, 2) else wl.BF16
        grad_dtype = wl.F32 if rng.integers(0, 3) == 0 else None
        pad = 8 * int(rng.integers(0, 3))
        for policy in (0, 1):
            _check(T, d_c, d_h, H, offs, dtype, grad_dtype=grad_dtype, pad=pad, policy=policy, seed=seed * 100 + case,
                   what=f"seed {seed} case {case}")
