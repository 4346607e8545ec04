"""GPU preparation (bda_prepare_device_ex) against the oracle's prepare: every window mode, with and
without companion weights, stored-form residuals, the search's choice, head widths up to 256.

The GPU inverts the basis block by Gauss-Jordan elimination, the oracle solves by LU: the float64
results agree to a multiple of cond * 2^-53, not bit for bit.  Stored (rounded) outputs are therefore
compared with the rounding of the GPU's own float64 result (exact), and that float64 result with the
oracle's (1e-9 of the largest coefficient).  Residuals are compared to 1e-6 relative; window choices
must be equal (the inputs keep the candidates' residuals apart)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import bda_workloads as wl  # noqa: E402
import gpu_harness as gh  # noqa: E402
import oracle  # noqa: E402
import paper_2510_01718_amd as bda  # noqa: E402

pytestmark = pytest.mark.gpu

_TDT = {wl.F64: torch.float64, wl.F32: torch.float32, wl.F16: torch.float16, wl.BF16: torch.int16}
FILL = -7


def _weights(d_c, H, d_h, d_side, seed, weak_first=True):
    """Gaussian projection and companions; in head 0 two rows of the first window are made nearly equal,
    so that the first window reconstructs visibly worse than the others once C is rounded."""
    rng = np.random.default_rng(seed)
    W = rng.standard_normal((d_c, H * d_h)) * 0.05
    if weak_first:
        W[1, :d_h] = W[0, :d_h] + 2e-4 * rng.standard_normal(d_h)
    Wq = rng.standard_normal((d_side, H * d_h)) * 0.05
    Wo = rng.standard_normal((H * d_h, d_side)) * 0.05
    return W, Wq, Wo


def _host(t, dtype):
    if dtype == wl.F64:
        return t.cpu().numpy().astype(np.float64)
    return gh.to_host64(t, dtype)


def _run(W, d_c, H, d_h, c_dtype, side=None, side_kind=oracle.SIDE_NONE, mode=oracle.FIRST, explicit_offset=0,
         want_resid=True, workspace_bytes=None):
    N = H * d_h
    W_d = torch.from_numpy(np.ascontiguousarray(W)).cuda()
    C_d = torch.full((d_c - d_h, N), FILL, dtype=_TDT[c_dtype], device="cuda")
    side_d = side_out_d = None
    ld_side = d_side = 0
    if side is not None:
        side_d = torch.from_numpy(np.ascontiguousarray(side)).cuda()
        side_out_d = torch.full(side.shape, FILL, dtype=_TDT[c_dtype], device="cuda")
        ld_side = side.shape[1]
        d_side = side.shape[0] if side_kind == oracle.SIDE_Q else side.shape[1]
    off_d = torch.full((1,), -99, dtype=torch.int32, device="cuda")
    resid_d = torch.zeros(3, dtype=torch.float64, device="cuda") if want_resid else None
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    need = bda.bda_prepare_device_workspace_bytes(d_c, H, d_h, mode, want_resid)
    nbytes = need if workspace_bytes is None else workspace_bytes
    ws = torch.full((max(nbytes, 16),), 0x5A, dtype=torch.uint8, device="cuda") if nbytes else None   # (stale contents must not matter)
    bda.bda_prepare_device_ex(W_d, N, wl.F64, d_c, H, d_h, C_d, N, c_dtype, side=side_d, ld_side=ld_side, d_side=d_side,
                              side_kind=side_kind, side_out=side_out_d, ld_side_out=ld_side, mode=mode,
                              explicit_offset=explicit_offset, basis_offset_out=off_d, resid_out=resid_d,
                              singular_head=flag, workspace=ws, workspace_bytes=nbytes, stream=gh.stream())
    torch.cuda.synchronize()
    return dict(C=_host(C_d, c_dtype), side=None if side is None else _host(side_out_d, c_dtype), off=int(off_d.item()),
                resid=None if resid_d is None else resid_d.cpu().numpy(), flag=int(flag.item()), need=need)


def _check_against_oracle(W, d_c, H, d_h, store, side, side_kind, mode, explicit_offset=0, **kw):
    C_ref, side_ref, off_ref, resid_ref = oracle.prepare(W, d_c, H, d_h, side=side, side_kind=side_kind, mode=mode,
                                                         explicit_offset=explicit_offset, store_dtype=store)
    exact = _run(W, d_c, H, d_h, wl.F64, side, side_kind, oracle.EXPLICIT, off_ref, **kw)      # float64 outputs, the oracle's window
    assert exact["flag"] == 0 and exact["off"] == off_ref
    assert np.max(np.abs(exact["C"] - C_ref)) <= 1e-9 * np.max(np.abs(C_ref))
    if side is not None:
        assert np.max(np.abs(exact["side"] - side_ref)) <= 1e-12 * np.max(np.abs(side_ref))
    got = _run(W, d_c, H, d_h, store, side, side_kind, mode, explicit_offset, **kw)             # stored outputs, the mode under test
    what = f"mode {mode} side {side_kind} store {store}: oracle window {off_ref}, residuals {resid_ref}, GPU {got['off']} {got['resid']}"
    assert got["flag"] == 0, what
    assert got["off"] == off_ref, what
    assert np.array_equal(got["C"], wl.to_storage(exact["C"], store)[1]), what
    if side is not None:
        assert np.array_equal(got["side"], wl.to_storage(exact["side"], store)[1]), what
    last = d_c - d_h
    want = [resid_ref.get(0, np.nan), resid_ref.get(last, np.nan), resid_ref[off_ref]]
    for g, r in zip(got["resid"], want):
        assert (np.isnan(g) and np.isnan(r)) or abs(g - r) <= 1e-6 * abs(r), what
    return got, resid_ref


@pytest.mark.parametrize("store", [wl.F16, wl.BF16])
@pytest.mark.parametrize("side_kind", [oracle.SIDE_NONE, oracle.SIDE_Q, oracle.SIDE_O])
@pytest.mark.parametrize("mode,explicit_offset", [(oracle.FIRST, 0), (oracle.LAST, 0), (oracle.RESIDUAL_MIN, 0),
                                                  (oracle.OFFSET_SEARCH, 0), (oracle.EXPLICIT, 40)])
def test_prepare_device_ex_modes_and_companions(store, side_kind, mode, explicit_offset):
    """Algorithm "BD Attention Preparation (QK)" / Appendix "BD for VO in MHA" / "Residual-Min with Offset
    Search" on the GPU: outputs, residuals of the stored form and the chosen window against the oracle."""
    d_c, H, d_h, d_side = 128, 3, 32, 40
    W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=300 + 10 * mode + side_kind)
    side = None if side_kind == oracle.SIDE_NONE else Wq if side_kind == oracle.SIDE_Q else Wo
    got, resid_ref = _check_against_oracle(W, d_c, H, d_h, store, side, side_kind, mode, explicit_offset)
    if mode == oracle.RESIDUAL_MIN:
        assert got["off"] == d_c - d_h and resid_ref[0] > 1.5 * resid_ref[d_c - d_h]     # the weak first window lost
    if mode == oracle.OFFSET_SEARCH:
        assert len(resid_ref) == 7 and got["off"] != 0


def test_prepare_device_ex_search_keeps_first_on_ties_and_reports_nan_for_windows_not_tried():
    """Float64 storage: every window reconstructs to rounding noise; explicit window: first / last not evaluated."""
    d_c, H, d_h = 96, 2, 32
    W, _, _ = _weights(d_c, H, d_h, 8, seed=77, weak_first=False)
    got = _run(W, d_c, H, d_h, wl.F16, mode=oracle.EXPLICIT, explicit_offset=16)
    assert got["off"] == 16 and np.isnan(got["resid"][0]) and np.isnan(got["resid"][1]) and got["resid"][2] > 0
    # no residuals asked for and one window: no workspace at all
    plain = _run(W, d_c, H, d_h, wl.F16, mode=oracle.LAST, want_resid=False)
    assert plain["need"] == 0 and plain["off"] == d_c - d_h
    C_ref, _, _, _ = oracle.prepare(W, d_c, H, d_h, mode=oracle.LAST)
    assert np.max(np.abs(plain["C"] - wl.to_storage(C_ref, wl.F16)[1])) <= 2.0 ** -10 * np.max(np.abs(C_ref))


@pytest.mark.parametrize("d_c,H,d_h,blocks", [(512, 3, 256, 1), (512, 3, 256, 2), (448, 2, 192, None), (320, 5, 160, None)])
def test_prepare_device_ex_wide_heads(d_c, H, d_h, blocks):
    """Head widths above 128: the basis block is inverted in the workspace, `blocks` heads per launch
    (None: the size bda_prepare_device_workspace_bytes suggests)."""
    W, Wq, _ = _weights(d_c, H, d_h, 24, seed=500 + d_h)
    ws = None
    if blocks is not None:
        ws = 1024 + 256 * ((2 * H * (1024 // H if 1024 // H < 64 else 64) * 8 + 255) // 256) + blocks * d_h * d_h * 8
    _check_against_oracle(W, d_c, H, d_h, wl.BF16, Wq, oracle.SIDE_Q, oracle.RESIDUAL_MIN, workspace_bytes=ws)


def test_prepare_device_ex_singular_windows():
    """A head of rank below d_h makes every window singular: the search reports -1.  One singular
    candidate among good ones is passed over; an explicit singular window is flagged and its C not written."""
    d_c, H, d_h = 96, 3, 32
    W, _, _ = _weights(d_c, H, d_h, 8, seed=91, weak_first=False)
    Wbad = W.copy()
    Wbad[:, d_h + 5] = Wbad[:, d_h + 9]                # head 1: two equal columns in every window
    got = _run(Wbad, d_c, H, d_h, wl.F16, mode=oracle.OFFSET_SEARCH)
    assert got["off"] == -1 and np.isinf(got["resid"][0]) and np.isinf(got["resid"][2])
    W1 = W.copy()
    W1[3, 2 * d_h:3 * d_h] = W1[7, 2 * d_h:3 * d_h]    # head 2: two equal rows inside the first window only
    got = _run(W1, d_c, H, d_h, wl.F16, mode=oracle.RESIDUAL_MIN)
    assert got["off"] == d_c - d_h and np.isinf(got["resid"][0]) and got["flag"] == 0
    C_ref, _, _, _ = oracle.prepare(W1, d_c, H, d_h, mode=oracle.LAST)
    assert np.max(np.abs(got["C"] - wl.to_storage(C_ref, wl.F16)[1])) <= 2.0 ** -10 * np.max(np.abs(C_ref))
    got = _run(W1, d_c, H, d_h, wl.F16, mode=oracle.FIRST)
    assert got["flag"] == 3 and np.all(got["C"][:, 2 * d_h:] == FILL) and not np.any(got["C"][:, :2 * d_h] == FILL)


def test_prepare_device_ex_calls_overlapping_on_several_streams():
    """Searches for different projections issued on four streams at once, each with a workspace and outputs of
    its own (the calls share nothing else): every one gives what it gives alone on one stream, bit for bit."""
    d_c, H, d_h, d_side = 192, 4, 64, 96
    jobs = []
    for j in range(8):
        W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=700 + j, weak_first=(j % 2 == 0))
        kind = oracle.SIDE_Q if j % 2 == 0 else oracle.SIDE_O
        jobs.append((W, Wq if kind == oracle.SIDE_Q else Wo, kind))
    alone = [_run(W, d_c, H, d_h, wl.F16, side, kind, oracle.OFFSET_SEARCH) for W, side, kind in jobs]
    N = H * d_h
    need = bda.bda_prepare_device_workspace_bytes(d_c, H, d_h, oracle.OFFSET_SEARCH, True)
    streams = [torch.cuda.Stream() for _ in range(4)]
    bufs = []
    for W, side, kind in jobs:
        bufs.append(dict(W=torch.from_numpy(np.ascontiguousarray(W)).cuda(), side=torch.from_numpy(np.ascontiguousarray(side)).cuda(),
                         C=torch.full((d_c - d_h, N), FILL, dtype=torch.float16, device="cuda"),
                         side_out=torch.full(side.shape, FILL, dtype=torch.float16, device="cuda"),
                         off=torch.full((1,), -99, dtype=torch.int32, device="cuda"), resid=torch.zeros(3, dtype=torch.float64, device="cuda"),
                         flag=torch.zeros(1, dtype=torch.int32, device="cuda"), ws=torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")))
    torch.cuda.synchronize()
    for rep in range(3):                                   # three waves of eight calls, two per stream, nothing waits in between
        for j, ((W, side, kind), b) in enumerate(zip(jobs, bufs)):
            bda.bda_prepare_device_ex(b["W"], N, wl.F64, d_c, H, d_h, b["C"], N, wl.F16, side=b["side"], ld_side=side.shape[1], d_side=d_side,
                                      side_kind=kind, side_out=b["side_out"], ld_side_out=side.shape[1], mode=oracle.OFFSET_SEARCH,
                                      basis_offset_out=b["off"], resid_out=b["resid"], singular_head=b["flag"], workspace=b["ws"],
                                      workspace_bytes=need, stream=int(streams[j % 4].cuda_stream))
    torch.cuda.synchronize()
    for j, (b, ref) in enumerate(zip(bufs, alone)):
        assert int(b["flag"].item()) == 0 and int(b["off"].item()) == ref["off"], j
        assert np.array_equal(_host(b["C"], wl.F16), ref["C"]) and np.array_equal(_host(b["side_out"], wl.F16), ref["side"]), j
        assert np.array_equal(b["resid"].cpu().numpy(), ref["resid"]), j


@pytest.mark.parametrize("d_c,H,d_h,d_side", [(9, 2, 1, 3), (50, 1, 31, 33), (66, 3, 33, 5), (97, 70, 64, 7), (130, 2, 65, 40),
                                              (200, 2, 97, 16), (145, 2, 127, 31), (131, 3, 128, 65)])
def test_prepare_device_ex_head_widths_at_the_edges_of_the_register_tiles(d_c, H, d_h, d_side):
    """Head widths around the multiples of 32 that the inversion's register tiles are made for, row counts outside the
    window that are no multiple of 16, more heads than workgroups share; zero pivots, so rows have to be taken out of order."""
    W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=40 + d_h, weak_first=False)
    last = d_c - d_h
    if d_h > 2:
        W[last, :d_h // 2] = 0.0                      # the last window's first pivot is zero, and no row is its own pivot
    side, kind = (Wq, oracle.SIDE_Q) if d_h % 2 else (Wo, oracle.SIDE_O)
    _check_against_oracle(W, d_c, H, d_h, wl.F16, side, kind, oracle.LAST)


@pytest.mark.parametrize("d_c,H,d_h,d_side,side_kind,store,mode", [
    (80, 2, 33, 30, oracle.SIDE_Q, wl.F16, oracle.OFFSET_SEARCH),      # one window per launch, columns read one by one
    (80, 2, 33, 150, oracle.SIDE_O, wl.BF16, oracle.OFFSET_SEARCH),    # four per launch, the last with one; last window off the grid of 16
    (512, 1, 128, 1000, oracle.SIDE_Q, wl.F32, oracle.RESIDUAL_MIN),   # largest strip, rows that end inside one
    (496, 3, 96, 405, oracle.SIDE_O, wl.F16, oracle.OFFSET_SEARCH),    # second window of a launch fills the companion output to its edge
    (513, 1, 96, 70, oracle.SIDE_Q, wl.F16, oracle.RESIDUAL_MIN),      # just past the strips
    (64, 40, 16, 33, oracle.SIDE_Q, wl.BF16, oracle.RESIDUAL_MIN),
    (97, 3, 1, 300, oracle.SIDE_O, wl.F16, oracle.OFFSET_SEARCH),      # heads of one column: pieces of one element, four windows per launch
    (97, 3, 1, 192, oracle.SIDE_O, wl.BF16, oracle.RESIDUAL_MIN)])     # the same, both in the companion output
def test_prepare_device_ex_windows_prepared_together(d_c, H, d_h, d_side, side_kind, store, mode):
    """Several candidate windows in one launch, their stored C's in the companion output meanwhile: strips, column
    tiles and windows that end on and off the kernels' tile sizes."""
    W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=60 + d_c + d_side)
    _check_against_oracle(W, d_c, H, d_h, store, Wq if side_kind == oracle.SIDE_Q else Wo, side_kind, mode)


def _padded(stored, dtype, ld, shift=0):
    """Device matrix of row pitch ld whose first element lies `shift` elements into its allocation; the rest is FILL."""
    a = np.ascontiguousarray(stored)
    a = a.view(np.int16) if dtype == wl.BF16 else a
    buf = torch.full((a.shape[0] * ld + shift,), FILL, dtype=_TDT[dtype], device="cuda")
    view = buf[shift:].view(a.shape[0], ld)
    view[:, :a.shape[1]] = torch.from_numpy(a.copy()).cuda()
    return buf, view


def _run_stored(W_s, w_dtype, d_c, H, d_h, c_dtype, side_s, side_kind, mode, explicit_offset=0, want_resid=True, pad_in=0, pad_out=0, shift=0):
    """bda_prepare_device_ex on weights as stored (any type, padded rows, any base); everything beyond the outputs'
    columns must stay FILL."""
    N, K = H * d_h, d_c - d_h
    d_side = side_s.shape[0 if side_kind == oracle.SIDE_Q else 1]
    W_b, W_d = _padded(W_s, w_dtype, N + pad_in, shift)
    s_b, s_d = _padded(side_s, w_dtype, side_s.shape[1] + pad_in, shift)
    fill = lambda rows, cols: _padded(np.full((rows, 0), 0, dtype=np.uint16 if c_dtype == wl.BF16 else np.float32), c_dtype, cols, shift)
    C_b, C_d = fill(K, N + pad_out)
    o_b, o_d = fill(side_s.shape[0], side_s.shape[1] + pad_out)
    off_d = torch.full((1,), -99, dtype=torch.int32, device="cuda")
    resid_d = torch.zeros(3, dtype=torch.float64, device="cuda") if want_resid else None
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    need = bda.bda_prepare_device_workspace_bytes(d_c, H, d_h, mode, want_resid)
    ws = torch.full((max(need, 16),), 0x5A, dtype=torch.uint8, device="cuda")
    bda.bda_prepare_device_ex(W_d, N + pad_in, w_dtype, d_c, H, d_h, C_d, N + pad_out, c_dtype, side=s_d, ld_side=side_s.shape[1] + pad_in,
                              d_side=d_side, side_kind=side_kind, side_out=o_d, ld_side_out=side_s.shape[1] + pad_out, mode=mode,
                              explicit_offset=explicit_offset, basis_offset_out=off_d, resid_out=resid_d, singular_head=flag,
                              workspace=ws, workspace_bytes=need, stream=gh.stream())
    torch.cuda.synchronize()
    assert torch.all(C_d[:, N:] == FILL) and torch.all(o_d[:, side_s.shape[1]:] == FILL)
    assert torch.all(C_b[:shift] == FILL) and torch.all(o_b[:shift] == FILL)
    return dict(C=_host(C_d[:, :N].contiguous(), c_dtype), side=_host(o_d[:, :side_s.shape[1]].contiguous(), c_dtype), off=int(off_d.item()),
                resid=None if resid_d is None else resid_d.cpu().numpy(), flag=int(flag.item()))


@pytest.mark.parametrize("w_dtype,store", [(wl.F32, wl.F16), (wl.F16, wl.F16), (wl.BF16, wl.BF16), (wl.F16, wl.F32), (wl.F32, wl.BF16)])
@pytest.mark.parametrize("side_kind", [oracle.SIDE_Q, oracle.SIDE_O])
@pytest.mark.parametrize("pad_in,pad_out,shift", [(0, 0, 0), (8, 8, 0), (3, 5, 0), (8, 8, 1)])     # wide fetches; pitches and bases that rule them out
@pytest.mark.parametrize("d_c,H,d_h,d_side,mode", [
    (128, 3, 32, 200, oracle.OFFSET_SEARCH),       # three windows per launch with W_q, more with W_o; narrow strips
    (400, 2, 64, 700, oracle.RESIDUAL_MIN),        # wide strips, both windows in one launch
    (120, 5, 24, 70, oracle.LAST),                 # one window, measured; it starts inside a column tile (96 = 6 x 16, of 24)
])
def test_prepare_device_ex_weights_as_stored(w_dtype, store, side_kind, pad_in, pad_out, shift, d_c, H, d_h, d_side, mode):
    """Weights in the types they are shipped in, with rows and bases that allow 16-byte fetches and that do not; stored
    C's of several windows in a padded companion output."""
    W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=900 + d_c)
    W_s, W64 = wl.to_storage(W, w_dtype)
    side_s, side64 = wl.to_storage(Wq if side_kind == oracle.SIDE_Q else Wo, w_dtype)
    C_ref, side_ref, off_ref, resid_ref = oracle.prepare(W64, d_c, H, d_h, side=side64, side_kind=side_kind, mode=mode, store_dtype=store)
    exact = _run_stored(W_s, w_dtype, d_c, H, d_h, wl.F64, side_s, side_kind, oracle.EXPLICIT, off_ref, False)
    assert np.max(np.abs(exact["C"] - C_ref)) <= 1e-9 * np.max(np.abs(C_ref))
    assert np.max(np.abs(exact["side"] - side_ref)) <= 1e-12 * np.max(np.abs(side_ref))
    got = _run_stored(W_s, w_dtype, d_c, H, d_h, store, side_s, side_kind, mode, 0, True, pad_in, pad_out, shift)
    assert got["flag"] == 0 and got["off"] == off_ref, (got["off"], got["resid"], resid_ref)
    assert np.array_equal(got["C"], wl.to_storage(exact["C"], store)[1])
    assert np.array_equal(got["side"], wl.to_storage(exact["side"], store)[1])
    for g, r in zip(got["resid"], [resid_ref.get(0, np.nan), resid_ref.get(d_c - d_h, np.nan), resid_ref[off_ref]]):
        assert (np.isnan(g) and np.isnan(r)) or abs(g - r) <= 1e-6 * abs(r), (got["resid"], resid_ref)


@pytest.mark.parametrize("w_dtype,store", [(wl.F32, wl.F16), (wl.BF16, wl.BF16)])
@pytest.mark.parametrize("side_kind", [oracle.SIDE_Q, oracle.SIDE_O])
@pytest.mark.parametrize("d_c,H,d_h,d_side,mode", [
    (48, 2, 32, 97, oracle.OFFSET_SEARCH),         # three column tiles, the least; strips that end inside one
    (272, 1, 96, 33, oracle.OFFSET_SEARCH),        # the fewest tiles of the eight-wave form, an odd number of blocks, windows one by one
    (512, 2, 128, 500, oracle.OFFSET_SEARCH),      # the most; several batches of windows, the last one short
    (256, 3, 128, 1030, oracle.RESIDUAL_MIN),      # both windows beside C, which the chosen one is copied to
    (320, 2, 64, 300, oracle.LAST),                # one window, measured and written at once
])
def test_prepare_device_ex_regular_windows(w_dtype, store, side_kind, d_c, H, d_h, d_side, mode):
    """The form for head widths of whole blocks of 32 and windows on whole column tiles."""
    test_prepare_device_ex_weights_as_stored(w_dtype, store, side_kind, 0, 0, 0, d_c, H, d_h, d_side, mode)


@pytest.mark.parametrize("store,scale", [(wl.F16, 1e-5), (wl.F16, 1e-8), (wl.F16, 3e7), (wl.BF16, 1e-37), (wl.BF16, 1.0)])
def test_prepare_device_ex_companion_below_and_beyond_the_stored_range(store, scale):
    """Companions that are stored as subnormal numbers, as zeros of either sign and as infinities."""
    d_c, H, d_h, d_side = 96, 2, 32, 70
    W, Wq, _ = _weights(d_c, H, d_h, d_side, seed=77, weak_first=False)
    W_s, W64 = wl.to_storage(W, wl.F32)
    side_s, side64 = wl.to_storage(Wq * scale, wl.F32)
    exact = _run_stored(W_s, wl.F32, d_c, H, d_h, wl.F64, side_s, oracle.SIDE_Q, oracle.EXPLICIT, d_c - d_h, False)
    got = _run_stored(W_s, wl.F32, d_c, H, d_h, store, side_s, oracle.SIDE_Q, oracle.LAST)
    with np.errstate(over="ignore"):
        assert np.array_equal(got["side"], wl.to_storage(exact["side"], store)[1])
    assert got["off"] == d_c - d_h


@pytest.mark.parametrize("d_c,H,d_h,d_side,off", [(20, 3, 4, 70, 16), (24, 70, 8, 33, 9), (64, 40, 16, 300, 17), (90, 3, 33, 40, 57), (144, 2, 48, 65, 41),
                                                   (300, 2, 113, 31, 187), (260, 1, 128, 100, 0), (512, 2, 250, 33, 262), (512, 1, 256, 40, 255)])
@pytest.mark.parametrize("side_kind", [oracle.SIDE_Q, oracle.SIDE_O])
def test_prepare_device_ex_companion_of_one_window(d_c, H, d_h, d_side, off, side_kind):
    """The companion alone (no residuals): windows at any start, of widths that meet one to seventeen column tiles,
    workgroups of one to eight waves."""
    W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=1300 + d_c, weak_first=False)
    W_s, W64 = wl.to_storage(W, wl.F32)
    side_s, side64 = wl.to_storage(Wq if side_kind == oracle.SIDE_Q else Wo, wl.F32)
    C_ref, side_ref, _, _ = oracle.prepare(W64, d_c, H, d_h, side=side64, side_kind=side_kind, mode=oracle.EXPLICIT, explicit_offset=off)
    got = _run_stored(W_s, wl.F32, d_c, H, d_h, wl.F64, side_s, side_kind, oracle.EXPLICIT, off, False, 1, 2)
    assert got["flag"] == 0 and got["off"] == off
    assert np.max(np.abs(got["C"] - C_ref)) <= 1e-9 * np.max(np.abs(C_ref))
    assert np.max(np.abs(got["side"] - side_ref)) <= 1e-12 * np.max(np.abs(side_ref))


@pytest.mark.parametrize("side_kind", [oracle.SIDE_Q, oracle.SIDE_O])
@pytest.mark.parametrize("bad", [0, 16, 48, 80, 96])
def test_prepare_device_ex_singular_window_in_a_batch(side_kind, bad):
    """One singular candidate in one head of a search that prepares several windows per launch (seven windows, three
    per launch with W_q: first and middle of a launch, last of one, alone in the last): passed over, +inf where its
    residual is asked for, no flag."""
    d_c, H, d_h, d_side, store = 128, 3, 32, 200, wl.F16
    W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=640, weak_first=False)
    W[bad + d_h - 1, d_h:2 * d_h] = W[bad, d_h:2 * d_h]       # head 1: the window's first and last row equal, both in no other candidate
    side = Wq if side_kind == oracle.SIDE_Q else Wo
    refs = {o: oracle.prepare(W, d_c, H, d_h, side=side, side_kind=side_kind, mode=oracle.EXPLICIT, explicit_offset=o, store_dtype=store)
            for o in range(0, d_c - d_h + 1, 16) if o != bad}
    resid = {o: r[3][o] for o, r in refs.items()}
    best = min(resid, key=lambda o: (resid[o], o))
    got = _run(W, d_c, H, d_h, store, side, side_kind, oracle.OFFSET_SEARCH)
    assert got["off"] == best and got["flag"] == 0, (got["off"], got["resid"], resid)
    for g, r in zip(got["resid"], [resid.get(0, np.inf), resid.get(d_c - d_h, np.inf), resid[best]]):
        assert (np.isinf(g) and np.isinf(r)) or abs(g - r) <= 1e-6 * abs(r), (got["resid"], resid)
    exact = _run(W, d_c, H, d_h, wl.F64, side, side_kind, oracle.EXPLICIT, best)
    assert np.max(np.abs(exact["C"] - refs[best][0])) <= 1e-9 * np.max(np.abs(refs[best][0]))
    assert np.array_equal(got["C"], wl.to_storage(exact["C"], store)[1])
    assert np.array_equal(got["side"], wl.to_storage(exact["side"], store)[1])


@pytest.mark.parametrize("side_kind", [oracle.SIDE_Q, oracle.SIDE_O])
@pytest.mark.parametrize("mode", [oracle.RESIDUAL_MIN, oracle.OFFSET_SEARCH])
def test_prepare_device_ex_every_window_singular_with_a_companion(side_kind, mode):
    """A head of rank below d_h: no window is chosen, and the pass for the chosen window leaves C and the flag alone."""
    d_c, H, d_h, d_side = 128, 3, 32, 200
    W, Wq, Wo = _weights(d_c, H, d_h, d_side, seed=650, weak_first=False)
    W[:, 2 * d_h + 5] = W[:, 2 * d_h + 9]                     # head 2: two equal columns
    got = _run(W, d_c, H, d_h, wl.F16, Wq if side_kind == oracle.SIDE_Q else Wo, side_kind, mode)
    assert got["off"] == -1 and got["flag"] == 0 and np.all(np.isinf(got["resid"]))
    assert np.all(got["C"][:, 2 * d_h:] == FILL)              # (a head that was singular in every window has no C)
