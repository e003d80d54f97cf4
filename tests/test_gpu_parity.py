"""Parity of the HIP path (through the C ABI) with the fp64 oracle.

Every case draws seeded inputs from paper_2402_09900_amd.tapes, runs the
library on the GPU and the oracle on the CPU on the same bytes, and compares
element by element:
  * floats: max over elements of |y - r| / max(|r|, m), with m the oracle's
    magnitude companion, at most 1e-4 for fp32/complex64 arithmetic and 2e-2
    for bf16 inputs (fp32 state);
  * integers (episode indices): bit-exact.
Full-size workloads run at their real shape in the launch configuration the
benchmark times, and are compared on every element: the oracle runs on one
tape, or one block of 32 feature columns, at a time (every tape and feature
is its own scan), so host memory stays bounded.
"""
import numpy as np
import pytest

import oracle
from conftest import announce, cond_err
from paper_2402_09900_amd import tapes

torch = pytest.importorskip("torch")
from paper_2402_09900_amd import binding as mb  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = {"f32": 1e-4, "c64": 1e-4, "bf16": 2e-2}


def to_dev(arr, kind):
    arr = np.ascontiguousarray(arr)
    if kind == "bf16":
        return torch.from_numpy(arr.view(np.int16)).view(torch.bfloat16).to(DEV)
    return torch.from_numpy(arr).to(DEV)


def from_dev(t):
    if t.dtype == torch.bfloat16:
        bits = t.view(torch.int16).cpu().numpy().view(np.uint16)
        return tapes.bf16_bits_to_f32(bits).astype(np.float64)
    return t.cpu().numpy()


def run_fwd(w, out_kind=None, idx=False):
    out_kind = out_kind or w.out_dtype
    out_t = {"f32": torch.float32, "bf16": torch.bfloat16, "c64": torch.complex64}[out_kind]
    a, x, s = to_dev(w.a, w.dtype), to_dev(w.x, w.dtype), to_dev(w.start, "u8")
    ws = torch.empty(max(mb.memoroid_scan_diag_workspace_bytes(
        w.B, w.T, w.d, {"f32": 0, "bf16": 1, "c64": 2}[w.dtype], {"f32": 0, "bf16": 1, "c64": 2}[out_kind]), 256),
        dtype=torch.uint8, device=DEV)
    res = mb.scan_diag(a, x, s, out_dtype=out_t, episode_idx=idx, workspace=ws)
    assert mb.workspace_status(ws) == mb.OK
    return res


def dec(arr, kind):
    """Exact float64 / complex128 decode of a stored input."""
    if kind == "bf16":
        return tapes.bf16_bits_to_f32(arr).astype(np.float64)
    return arr.astype(np.complex128 if kind == "c64" else np.float64)


def select(w, name, tapes_sel=None, cols=None):
    """Decoded slice [tapes][:, cols] of a tape input (a time-invariant a is
    [d] and only takes the column selection)."""
    arr = getattr(w, name)
    if name == "a" and w.a_invariant:
        return dec(arr if cols is None else arr[cols], w.dtype)
    if tapes_sel is not None:
        arr = arr[tapes_sel]
    if cols is not None:
        arr = arr[:, :, cols]
    return dec(arr, w.dtype)


def check_fwd(w, out_kind=None, cols=None, tapes_sel=None, label=""):
    announce("fwd %s B=%d T=%d d=%d %s inv=%s %s" % (label, w.B, w.T, w.d, w.dtype, w.a_invariant, out_kind))
    h, idx = run_fwd(w, out_kind, idx=True)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.episode_idx(w.start))
    if tapes_sel is not None:
        h = h[tapes_sel]
    if cols is not None:
        h = h[:, :, cols]
    h = from_dev(h.contiguous())
    s = w.start if tapes_sel is None else w.start[tapes_sel]
    ref, mag = oracle.diag_fwd(select(w, "a", tapes_sel, cols), select(w, "x", tapes_sel, cols), s)
    err = cond_err(h, ref, mag)
    tol = TOL[w.dtype if (out_kind or w.out_dtype) != "bf16" else "bf16"]
    assert err <= tol, (label, err)
    return err


def check_bwd(w, cols=None, label=""):
    announce("bwd %s B=%d T=%d d=%d %s inv=%s" % (label, w.B, w.T, w.d, w.dtype, w.a_invariant))
    s = w.start
    a_s, x_s, g_s = select(w, "a", None, cols), select(w, "x", None, cols), select(w, "g", None, cols)
    h_ref, _ = oracle.diag_fwd(a_s, x_s, s)
    # both sides consume the same h: the oracle's forward, stored in the
    # tape's dtype
    store = np.complex64 if w.dtype == "c64" else np.float32
    if cols is None:
        h_in = h_ref.astype(store)
    else:
        # sampled columns of a full-size tape: only the sampled columns are
        # compared, so the others may hold any finite h
        h_in = w.x.copy()
        h_in[:, :, cols] = h_ref.astype(store)
    ws = torch.empty(max(mb.memoroid_scan_diag_bwd_workspace_bytes(
        w.B, w.T, w.d, 2 if w.dtype == "c64" else 0, 0 if w.a_invariant else w.d), 256),
        dtype=torch.uint8, device=DEV)
    gx, ga = mb.scan_diag_bwd(to_dev(w.a, w.dtype), to_dev(s, "u8"), to_dev(h_in, w.dtype),
                              to_dev(w.g, w.dtype), workspace=ws)
    assert mb.workspace_status(ws) == mb.OK
    if cols is not None:
        gx = gx[:, :, cols]
        ga = ga if w.a_invariant else ga[:, :, cols]
    gx, ga = from_dev(gx.contiguous()), from_dev(ga.contiguous())
    h_used = dec(h_in if cols is None else h_in[:, :, cols], w.dtype)
    dx, da, m_dx, m_da = oracle.diag_bwd(a_s, s, h_used, g_s)
    assert not (w.a_invariant and cols is not None), "a time-invariant da sums every column"
    e_dx = cond_err(gx, dx, m_dx)
    e_da = cond_err(ga, da, m_da)
    assert e_dx <= TOL[w.dtype], (label, "dx", e_dx)
    assert e_da <= TOL[w.dtype], (label, "da", e_da)
    return e_dx, e_da


# ------------------------------------------------------- the five workloads


def test_workload1_full():
    w = tapes.make_diag(1)
    check_fwd(w, label="workload1")


@pytest.fixture(scope="module")
def w2():
    return tapes.make_diag(2)


def test_workload2_full_fwd(w2):
    check_fwd(w2, label="workload2")


def test_workload2_full_bwd(w2):
    check_bwd(w2, label="workload2")


def test_workload2_reduced_ragged():
    w = tapes.make_diag(2, T=4096 + 37, d=256, seed=102)
    check_fwd(w, label="workload2-small")
    check_bwd(w, label="workload2-small")


def check_linattn(la, label):
    announce("linattn %s T=%d H=%d" % (label, la.T, la.H))
    q, k, v = (to_dev(t, "f32") for t in (la.q, la.k, la.v))
    st = to_dev(la.start, "u8")
    ws = torch.empty(mb.memoroid_scan_linattn_workspace_bytes(la.T, la.H, 64, 64, 64), dtype=torch.uint8,
                     device=DEV)
    out, idx = mb.scan_linattn(q, k, v, st, episode_idx=True, workspace=ws)
    assert mb.workspace_status(ws) == mb.OK
    ref, mag = oracle.linattn(la.q.astype(np.float64), la.k.astype(np.float64), la.v.astype(np.float64),
                              la.start)
    err = cond_err(out.cpu().numpy(), ref, mag)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.episode_idx(la.start))
    assert err <= TOL["f32"], (label, err)
    return err


def test_workload3_reduced_ragged():
    check_linattn(tapes.make_linattn(T=2048 + 13, seed=103), "workload3-small")


def test_workload3_full():
    check_linattn(tapes.make_linattn(), "workload3")


def test_workload3_short_episodes():
    la = tapes.make_linattn(T=777, seed=104)
    la.start[:] = 0
    la.start[::3] = 1
    la.start[100:140] = 1       # single-step episodes
    check_linattn(la, "workload3-short-episodes")


@pytest.mark.parametrize("T,H", [(2048 - 13, 32), (2048 + 17, 64), (1024 - 5, 64)])
def test_linattn_segments_of_several_chunks(T, H):
    """16 segments of two chunks and eleven of three, scanned, and eight of two,
    added up by their readers; the last segment short, its last chunk partial."""
    check_linattn(tapes.make_linattn(T=T, H=H, seed=105 + H), "several chunks a segment")


@pytest.fixture(scope="module")
def w4():
    return tapes.make_diag(4)


def test_workload4_full_every_tape(w4):
    """All 64 tapes x 16384 steps x 512 features, bf16 out, against the
    oracle tape by tape."""
    announce("fwd workload4 full B=%d T=%d d=%d (every element)" % (w4.B, w4.T, w4.d))
    h, idx = run_fwd(w4, idx=True)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.episode_idx(w4.start))
    bits = h.view(torch.int16).cpu().numpy().view(np.uint16)
    del h
    worst = 0.0
    for b in range(w4.B):
        got = tapes.bf16_bits_to_f32(bits[b:b + 1]).astype(np.float64)
        ref, mag = oracle.diag_fwd(select(w4, "a", [b]), select(w4, "x", [b]), w4.start[b:b + 1])
        worst = max(worst, cond_err(got, ref, mag))
        assert worst <= TOL["bf16"], (b, worst)


def test_workload4_reduced_both_outputs():
    w = tapes.make_diag(4, B=3, T=3000, d=512, seed=104)
    check_fwd(w, label="workload4-small")
    check_fwd(w, out_kind="f32", label="workload4-small-f32out")


@pytest.fixture(scope="module")
def w5():
    return tapes.make_diag(5)


BLOCK = 32                      # feature columns the oracle takes at a time


def test_workload5_full_fwd_every_element(w5):
    """T = 2^20 steps x 256 features, forward with episode indices, against
    the oracle one block of 32 columns at a time."""
    announce("fwd workload5 full T=%d d=%d (every element)" % (w5.T, w5.d))
    h, idx = run_fwd(w5, idx=True)
    np.testing.assert_array_equal(idx.cpu().numpy(), oracle.episode_idx(w5.start))
    h = h.cpu().numpy()
    for c0 in range(0, w5.d, BLOCK):
        cols = list(range(c0, min(c0 + BLOCK, w5.d)))
        ref, mag = oracle.diag_fwd(select(w5, "a", None, cols), select(w5, "x", None, cols), w5.start)
        err = cond_err(h[:, :, cols].astype(np.float64), ref, mag)
        assert err <= TOL["f32"], (c0, err)


def test_workload5_full_bwd_every_element(w5):
    """The reverse scan of workload 5 on every element: the saved state h is
    the oracle's forward in float32, built block by block, and dx, da are
    compared block by block."""
    announce("bwd workload5 full T=%d d=%d (every element)" % (w5.T, w5.d))
    h_in = np.empty(w5.x.shape, dtype=np.float32)
    blocks = [list(range(c0, min(c0 + BLOCK, w5.d))) for c0 in range(0, w5.d, BLOCK)]
    for cols in blocks:
        ref, _ = oracle.diag_fwd(select(w5, "a", None, cols), select(w5, "x", None, cols), w5.start)
        h_in[:, :, cols] = ref.astype(np.float32)
    ws = torch.empty(mb.memoroid_scan_diag_bwd_workspace_bytes(w5.B, w5.T, w5.d, mb.F32, w5.d),
                     dtype=torch.uint8, device=DEV)
    gx, ga = mb.scan_diag_bwd(to_dev(w5.a, "f32"), to_dev(w5.start, "u8"), to_dev(h_in, "f32"),
                              to_dev(w5.g, "f32"), workspace=ws)
    assert mb.workspace_status(ws) == mb.OK
    gx, ga = gx.cpu().numpy(), ga.cpu().numpy()
    for cols in blocks:
        dx, da, m_dx, m_da = oracle.diag_bwd(select(w5, "a", None, cols), w5.start,
                                             h_in[:, :, cols].astype(np.float64), select(w5, "g", None, cols))
        e_dx = cond_err(gx[:, :, cols], dx, m_dx)
        e_da = cond_err(ga[:, :, cols], da, m_da)
        assert e_dx <= TOL["f32"] and e_da <= TOL["f32"], (cols[0], e_dx, e_da)


def test_workload5_reduced_ragged():
    w = tapes.make_diag(5, T=20000 + 5, d=256, seed=105)
    check_fwd(w, label="workload5-small")
    check_bwd(w, label="workload5-small")


# ------------------------------------------------------------------ edges

SHAPES = [(1, 1, 1), (1, 2, 3), (2, 63, 4), (1, 64, 32), (3, 65, 33), (1, 129, 256), (2, 1000, 260),
          (1, 257, 512), (1, 5000, 8), (2, 300, 1024)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "c64"])
@pytest.mark.parametrize("inv", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%dT%dd%d" % s)
def test_edge_shapes(dtype, inv, shape):
    B, T, d = shape
    w = tapes.make_custom_diag(dtype, B, T, d, inv, seed=1000 + T + d, mean_episode=40.0)
    check_fwd(w, label="edge")
    if dtype != "bf16":
        check_bwd(w, label="edge")


def _tile_lengths(dtype, inv, d):
    """Forward and reverse tile lengths (steps) of the plans these tapes get
    (torch allocations are 256-byte aligned, so vectorisation follows d)."""
    code = {"f32": mb.F32, "bf16": mb.BF16, "c64": mb.C64}[dtype]
    vec = d % {"c64": 2, "f32": 4, "bf16": 8}[dtype] == 0
    stride = 0 if inv else d
    Ls = {mb.memoroid_testing_tile_steps(0, 2, 1 << 16, d, code, stride, vec)}
    if dtype != "bf16":
        Ls.add(mb.memoroid_testing_tile_steps(1, 2, 1 << 16, d, code, stride, vec))
    assert all(L > 0 for L in Ls)
    return sorted(Ls)


# d = 36: a multiple of 4 but not of 8, so bf16 (8 features per vector lane)
# takes the scalar kernel while f32 stays vectorised
BOUNDARY_CASES = [(dt, inv, d) for dt in ("f32", "bf16", "c64") for inv in (False, True) for d in (256, 7)] + \
    [("bf16", False, 36), ("bf16", True, 36), ("f32", False, 36)]


@pytest.mark.parametrize("dtype,inv,d", BOUNDARY_CASES, ids=lambda v: str(v))
def test_tile_boundary_lengths(dtype, inv, d):
    """T at L - 1, L, L + 1 and 2L + 1 for every tile length L of the
    forward and reverse plans (a tape ending one step before, at and after a
    tile edge; a last tile of a single step)."""
    Ls = _tile_lengths(dtype, inv, d)
    if dtype == "f32" and d == 256:
        # forward / reverse: 16 / 8 steps per lane with a time-invariant a,
        # 18 / 12 with a per-step a (8 groups of 4 wavefronts per tile)
        assert Ls == (sorted({512, 256}) if inv else sorted({576, 384})), Ls
    Ts = sorted({t for L in Ls for t in (L - 1, L, L + 1, 2 * L + 1)})
    for T in Ts:
        w = tapes.make_custom_diag(dtype, 2, T, d, inv, seed=3000 + T + d, mean_episode=150.0)
        check_fwd(w, label="tile edge L=%s" % Ls)
        if dtype != "bf16":
            check_bwd(w, label="tile edge L=%s" % Ls)


# whole chains of vector-wide lanes on rows that are not whole 128-byte lines
# (cached access), and the same rows one line wide or more (outputs streamed)
@pytest.mark.parametrize("inv", [False, True])
@pytest.mark.parametrize("dtype,d", [("f32", 100), ("f32", 96), ("c64", 50), ("c64", 48), ("bf16", 72), ("bf16", 128)])
def test_cache_policies_at_tile_edges(dtype, d, inv):
    for T in (_tile_lengths(dtype, inv, d)[-1] + 1, 2 * _tile_lengths(dtype, inv, d)[0] - 1):
        w = tapes.make_custom_diag(dtype, 2, T, d, inv, seed=5000 + T + d, mean_episode=90.0)
        check_fwd(w, label="cache policy")
        if dtype != "bf16":
            check_bwd(w, label="cache policy")


@pytest.mark.parametrize("dtype,inv", [(dt, inv) for dt in ("f32", "bf16", "c64") for inv in (False, True)])
def test_flags_at_word_and_lane_edges(dtype, inv):
    """Full-width rows read a wavefront's begin flags as 64-bit words: begins
    on and beside every multiple of 64 and of the lanes' 8, 12, 16 and 18
    steps (first tape), and on a third of all steps (second tape), on a tape
    that ends inside its third tile."""
    Ls = _tile_lengths(dtype, inv, 256)
    for T in sorted({2 * L + 5 for L in Ls}):
        w = tapes.make_custom_diag(dtype, 2, T, 256, inv, seed=4000 + T)
        rng = np.random.default_rng(T)
        w.start[:] = 0
        for m in (64, 8 * 9, 12 * 7, 16 * 5, 18 * 11):
            for o in (-1, 0, 1):
                at = np.arange(m, T, m) + o
                w.start[0, at[(at > 0) & (at < T) & (rng.random(at.size) < 0.5)]] = 1
        w.start[1, rng.random(T) < 0.33] = 1
        w.start[:, 0] = 1
        check_fwd(w, label="flag words")
        if dtype != "bf16":
            check_bwd(w, label="flag words")


@pytest.mark.parametrize("pattern", ["all_begins", "single_episode", "begin_at_end", "flag_bytes"])
@pytest.mark.parametrize("dtype", ["f32", "c64"])
def test_flag_patterns(pattern, dtype):
    T = 20000 if pattern == "single_episode" else 3001
    w = tapes.make_custom_diag(dtype, 2, T, 256, False, seed=7, a_range=(0.9, 0.9999))
    if pattern == "all_begins":
        w.start[:] = 1
    elif pattern == "single_episode":
        w.start[:] = 0
    elif pattern == "begin_at_end":
        w.start[:] = 0
        w.start[:, -1] = 1
    else:
        rng = np.random.default_rng(3)
        nz = w.start != 0
        w.start[nz] = rng.integers(2, 256, size=int(nz.sum())).astype(np.uint8)
        w.start[0, 0] = 0      # a zero byte at t = 0 still begins an episode
    check_fwd(w, label=pattern)
    check_bwd(w, label=pattern)


def test_bf16_a_rounding_to_one():
    """a drawn near 1 rounds to exactly 1.0 in bf16: no decay, a running sum."""
    w = tapes.make_custom_diag("bf16", 1, 4000, 64, False, seed=8, a_range=(0.9985, 0.9999))
    assert np.all(tapes.bf16_bits_to_f32(w.a) == 1.0)
    check_fwd(w, out_kind="f32", label="bf16-a-one")


def test_scalar_path_on_misaligned_rows():
    """Base pointers off 16-byte alignment take the scalar kernels."""
    w = tapes.make_custom_diag("f32", 1, 777, 64, False, seed=9)
    B, T, d = w.B, w.T, w.d
    buf_a = torch.zeros(B * T * d + 1, device=DEV)
    buf_x = torch.zeros(B * T * d + 1, device=DEV)
    buf_a[1:] = to_dev(w.a.reshape(-1), "f32")
    buf_x[1:] = to_dev(w.x.reshape(-1), "f32")
    a = buf_a[1:].view(B, T, d)
    x = buf_x[1:].view(B, T, d)
    h = mb.scan_diag(a, x, to_dev(w.start, "u8"))
    ref, mag = oracle.diag_fwd(w.decoded("a"), w.decoded("x"), w.start)
    assert cond_err(from_dev(h), ref, mag) <= 1e-4


def test_nan_stays_in_its_episode():
    w = tapes.make_custom_diag("f32", 1, 3000, 32, False, seed=10)
    w.start[:] = 0
    w.start[0, [0, 700, 1500, 2200]] = 1
    w.x[0, 800, 3] = np.nan
    w.a[0, 1600, 5] = np.inf
    h = from_dev(run_fwd(w))
    assert np.isnan(h[0, 800:1500, 3]).all()
    assert np.isfinite(h[0, :800]).all() and np.isfinite(h[0, 1500:, 3]).all()
    assert np.isfinite(h[0, 2200:]).all()
    g = w.g.copy()
    g[0, 1000, 7] = np.nan
    gx, _ = mb.scan_diag_bwd(to_dev(w.a, "f32"), to_dev(w.start, "u8"), to_dev(np.ones_like(w.x), "f32"),
                             to_dev(g, "f32"))
    gx = from_dev(gx)
    assert np.isnan(gx[0, 700:1001, 7]).all()
    assert np.isfinite(gx[0, :700, 7]).all() and np.isfinite(gx[0, 1001:, 7]).all()


@pytest.mark.parametrize("dtype", ["f32", "c64"])
@pytest.mark.parametrize("B", [1, 2])
def test_time_invariant_da_ignores_the_state_after_the_tape_end(dtype, B):
    """With a time-invariant a the reverse scan sums da over the tape; the
    saved state of the last step, h_{T-1}, enters no term of that sum.  A NaN
    there (x NaN at the last step) must leave da finite, also when T is not
    a multiple of the tile length (one tape: da summed in the kernel; two:
    through the partial rows)."""
    T, d = 1000 + 3, 16
    w = tapes.make_custom_diag(dtype, B, T, d, True, seed=12 + B)
    assert T % mb.memoroid_testing_tile_steps(1, B, T, d, mb.F32 if dtype == "f32" else mb.C64, 0, 1) != 0
    w.x[:, T - 1, :] = np.nan
    announce("bwd invariant-a da with NaN at h_{T-1} %s B=%d" % (dtype, B))
    e_dx, e_da = check_bwd(w, label="NaN h at tape end")
    assert e_dx <= TOL[dtype] and e_da <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "c64"])
def test_invariant_a_nonfinite_adjoint_at_a_begin(dtype):
    """A non-finite upstream gradient at a begin step makes that step's
    adjoint non-finite, but no earlier step's (the step before ends an
    episode) and no term of the time-invariant da (begin steps take none):
    da stays finite and equal to the oracle's.  One begin opens a lane's
    steps (704: a multiple of the lane's 8 or 16 steps), the other falls
    inside a lane (1500)."""
    T, d = 3000, 16
    w = tapes.make_custom_diag(dtype, 1, T, d, True, seed=31)
    w.start[:] = 0
    w.start[0, [0, 704, 1500, 2200]] = 1
    g = w.g.copy()
    g[0, 704, 3] = np.nan
    g[0, 1500, 5] = np.nan
    announce("bwd invariant-a NaN adjoint at begins %s" % dtype)
    store = np.complex64 if dtype == "c64" else np.float32
    h_ref, _ = oracle.diag_fwd(dec(w.a, dtype), dec(w.x, dtype), w.start)
    h_in = h_ref.astype(store)
    gx, ga = mb.scan_diag_bwd(to_dev(w.a, dtype), to_dev(w.start, "u8"), to_dev(h_in, dtype), to_dev(g, dtype))
    gx, ga = from_dev(gx), from_dev(ga)
    dx, da, m_dx, m_da = oracle.diag_bwd(dec(w.a, dtype), w.start, dec(h_in, dtype), dec(g, dtype))
    bad = np.isnan(dx)
    assert bad[0, 704, 3] and bad[0, 1500, 5] and bad.sum() == 2
    assert np.array_equal(np.isnan(gx), bad)
    assert cond_err(gx[~bad], dx[~bad], m_dx[~bad]) <= TOL[dtype]
    assert np.isfinite(da).all() and np.isfinite(ga).all()
    assert cond_err(ga, da, m_da) <= TOL[dtype]


def test_linattn_nan_stays_in_its_episode():
    la = tapes.make_linattn(T=640, seed=11)
    la.start[:] = 0
    la.start[[0, 100, 130, 300]] = 1
    la.v[120, 2, 5] = np.nan
    q, k, v = (to_dev(t, "f32") for t in (la.q, la.k, la.v))
    out = mb.scan_linattn(q, k, v, to_dev(la.start, "u8")).cpu().numpy()
    assert np.isnan(out[120:130, 2, 5]).all()
    assert np.isfinite(out[:120]).all() and np.isfinite(out[130:]).all()
    assert np.isfinite(out[:, [0, 1, 3]]).all()


def test_repeated_runs_agree():
    w = tapes.make_diag(5, T=200000, d=256, seed=12)
    ref, mag = oracle.diag_fwd(w.decoded("a"), w.decoded("x"), w.start)
    for rep in range(4):
        announce("repeat %d" % rep)
        assert cond_err(from_dev(run_fwd(w)), ref, mag) <= 1e-4


def test_autograd_function():
    w = tapes.make_custom_diag("c64", 2, 1500, 64, True, seed=13)
    a = to_dev(w.a, "c64").requires_grad_(True)
    x = to_dev(w.x, "c64").requires_grad_(True)
    h = mb.diag_scan(a, x, to_dev(w.start, "u8"))
    h.backward(to_dev(w.g, "c64"))
    h_ref, m_h = oracle.diag_fwd(w.decoded("a"), w.decoded("x"), w.start)
    assert cond_err(from_dev(h.detach()), h_ref, m_h) <= 1e-4
    dx, da, m_dx, _ = oracle.diag_bwd(w.decoded("a"), w.start, h_ref, w.decoded("g"))
    assert cond_err(from_dev(x.grad), dx, m_dx) <= 1e-4
    # da here uses the GPU's own h, whose error scales with the forward
    # companion m_h: bound da's error by sum_t m_lam,t * m_h,t-1
    nb = (w.start == 0)
    nb[:, 0] = False
    mh_prev = np.concatenate([np.zeros_like(m_h[:, :1]), m_h[:, :-1]], axis=1)
    loose = (m_dx * mh_prev * nb[..., None]).sum(axis=(0, 1))
    err = np.abs(from_dev(a.grad) - da) / np.maximum(np.abs(da), loose)
    assert err.max() <= 1e-4


def test_invariant_da_long_tape_uses_column_sum_kernels():
    """More partial rows than the in-kernel da reduction takes: the column-sum
    kernels add them up instead."""
    w = tapes.make_custom_diag("c64", 1, 600_000, 32, True, seed=14, a_range=(0.9, 0.999), mean_episode=300.0)
    check_bwd(w, label="long-invariant")
