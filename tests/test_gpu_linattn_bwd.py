"""Parity of the linear-attention gradient kernels (through the C ABI) with
the fp64 oracle: conditioned relative error (|y - r| / max(|r|, m), m the
oracle's magnitude companion) at most 1e-4 for dq, dk and dv, and for the
forward output they are taken at (fp32 arithmetic).  The full workload is compared on every element."""
import numpy as np
import pytest

import oracle
from conftest import announce, cond_err
from paper_2402_09900_amd import tapes

torch = pytest.importorskip("torch")
from paper_2402_09900_amd import binding as mb  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = 1e-4


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def grad_input(la, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return rng.standard_normal(la.v.shape, dtype=np.float32)


def check(la, label, seed=1):
    announce("linattn bwd %s T=%d H=%d" % (label, la.T, la.H))
    g = grad_input(la, seed)
    q, k, v, s = dev(la.q), dev(la.k), dev(la.v), dev(la.start)
    out = mb.scan_linattn(q, k, v, s)
    gq, gk, gv = mb.scan_linattn_bwd(q, k, v, s, out, dev(g))
    torch.cuda.synchronize()
    # the forward output these gradients are taken at, on the same flag
    # patterns, lengths and head counts
    ro, mo = oracle.linattn(la.q.astype(np.float64), la.k.astype(np.float64), la.v.astype(np.float64), la.start)
    e = cond_err(out.cpu().numpy(), ro, mo)
    assert e <= TOL, (label, "out", e)
    rq, rk, rv, mq, mk, mv = oracle.linattn_bwd(la.q.astype(np.float64), la.k.astype(np.float64),
                                                la.v.astype(np.float64), la.start, g.astype(np.float64))
    for name, got, ref, m in (("dq", gq, rq, mq), ("dk", gk, rk, mk), ("dv", gv, rv, mv)):
        e = cond_err(got.cpu().numpy(), ref, m)
        assert e <= TOL, (label, name, e)


def test_workload3_full():
    check(tapes.make_linattn(3), "workload3")


@pytest.mark.parametrize("T", [1, 63, 64, 65, 1000, 4097])
def test_ragged_lengths(T):
    check(tapes.make_linattn(3, seed=300 + T, T=T, H=2), "ragged")


@pytest.mark.parametrize("H", [1, 3, 5])
def test_head_counts(H):
    """Odd head counts: the grid is (chunks, heads) and each head's rows are
    a 256-byte slice of every [T][H][64] row."""
    check(tapes.make_linattn(3, seed=400 + H, T=1000 + 13 * H, H=H), "heads")


@pytest.mark.parametrize("T,H", [(64 * 65, 1), (64 * 129, 1), (64 * 257 - 3, 1), (64 * 1026, 1), (64 * 1026 + 13, 4),
                                 (64 * 513, 1), (64 * 1021 - 51, 4), (64 * 4100 - 3, 1)])
def test_segment_lengths_and_scan_rounds(T, H):
    """Segments of one chunk in numbers just past what 2, 4 and 8 segments per
    thread of the state scan take at once (65, 129, 257), 206 segments of five
    chunks and 172 of six, the last of them short, 513 of one chunk (two rounds
    of the scan, carried over), 128 of eight chunks and 684 of six (two
    rounds), the last short."""
    check(tapes.make_linattn(3, seed=500 + H, T=T, H=H), "segments")


@pytest.mark.parametrize("T", [64 * 2, 64 * 8 - 5, 64 * 8, 64 * 8 + 1])
@pytest.mark.parametrize("begins", [(), (70,), (0, 63, 64, 65, 400)])
def test_few_segments_add_up_states(T, begins):
    """Up to eight segments: every workgroup adds up the summaries back (and,
    in reverse, ahead) to the nearest segment with a begin step -- one episode
    over all of them, one begin step early, begins at segment edges; one
    segment more takes the scan."""
    la = tapes.make_linattn(3, seed=600 + T, T=T, H=2)
    f = np.zeros(T, np.uint8)
    f[[b for b in begins if b < T]] = 1
    check(_with_flags(la, f), "few segments")


def _with_flags(la, flags):
    la.start = flags.astype(np.uint8)
    return la


@pytest.mark.parametrize("kind", ["short", "all_begins", "single_episode", "chunk_starts", "chunk_second_rows",
                                  "flag_bytes"])
def test_flag_patterns(kind):
    rng = np.random.default_rng(17)
    T = 3 * 1024 + 17
    la = tapes.make_linattn(3, seed=77, T=T, H=2)
    f = np.zeros(T, np.uint8)
    if kind == "short":
        f = tapes.flags_from_lengths(rng.integers(1, 40, size=T), T)
    elif kind == "all_begins":
        f[:] = 1
    elif kind == "chunk_starts":
        f[::64] = 1
    elif kind == "chunk_second_rows":
        f[1::64] = 1
    elif kind == "flag_bytes":
        f = (rng.random(T) < 0.01).astype(np.uint8) * rng.integers(1, 256, size=T).astype(np.uint8)
    check(_with_flags(la, f), kind)


def test_autograd_function():
    la = tapes.make_linattn(3, seed=88, T=700, H=2)
    announce("linattn autograd T=700")
    q, k, v = (dev(a).requires_grad_(True) for a in (la.q, la.k, la.v))
    g = grad_input(la, 5)
    out = mb.linattn(q, k, v, dev(la.start))
    (out * dev(g)).sum().backward()
    rq, rk, rv, mq, mk, mv = oracle.linattn_bwd(la.q.astype(np.float64), la.k.astype(np.float64),
                                                la.v.astype(np.float64), la.start, g.astype(np.float64))
    assert cond_err(q.grad.cpu().numpy(), rq, mq) <= TOL
    assert cond_err(k.grad.cpu().numpy(), rk, mk) <= TOL
    assert cond_err(v.grad.cpu().numpy(), rv, mv) <= TOL


def test_nonfinite_values_stay_in_their_episode():
    """NaN in k, q, v and the upstream gradient, each inside one episode of a
    chunk that holds other episodes: every element the oracle computes as
    finite (the other episodes, and the steps of the same episode that do
    not depend on the planted value) is finite on the GPU and within the
    tolerance, and every element the oracle leaves non-finite is non-finite
    (the reset theorem's barrier, carried by selects, for the gradient)."""
    T, H = 5 * 64 + 9, 2
    la = tapes.make_linattn(3, seed=91, T=T, H=H)
    f = np.zeros(T, np.uint8)
    f[[0, 70, 90, 100, 140, 200, 230, 260, 300]] = 1       # several episodes per chunk
    la.start = f
    g = grad_input(la, 9)
    la.k[95, 0, 3] = np.nan        # episode [90, 100), chunk 1, head 0
    la.q[150, 1, 5] = np.nan       # episode [140, 200), chunks 2-3, head 1
    la.v[210, 0, 7] = np.nan       # episode [200, 230), chunk 3, head 0
    g[245, 1, 11] = np.nan         # episode [230, 260), chunk 3, head 1
    announce("linattn bwd non-finite T=%d H=%d" % (T, H))
    q, k, v, s = dev(la.q), dev(la.k), dev(la.v), dev(la.start)
    out = mb.scan_linattn(q, k, v, s)
    gq, gk, gv = mb.scan_linattn_bwd(q, k, v, s, out, dev(g))
    torch.cuda.synchronize()
    ro, mo = oracle.linattn(la.q.astype(np.float64), la.k.astype(np.float64), la.v.astype(np.float64), la.start)
    rq, rk, rv, mq, mk, mv = oracle.linattn_bwd(la.q.astype(np.float64), la.k.astype(np.float64),
                                                la.v.astype(np.float64), la.start, g.astype(np.float64))
    for name, got, ref, m in (("out", out, ro, mo), ("dq", gq, rq, mq), ("dk", gk, rk, mk), ("dv", gv, rv, mv)):
        got = got.cpu().numpy()
        fin = np.isfinite(ref)
        assert (~fin).any(), name                       # the planted values reach their episodes
        assert np.isfinite(got[fin]).all(), (name, np.argwhere(fin & ~np.isfinite(got))[:5])
        assert not np.isfinite(got[~fin]).any(), name
        e = cond_err(got[fin], ref[fin], m[fin])
        assert e <= TOL, (name, e)


# (T, H, rows of a segment): 13 segments of one chunk and 16 of two, scanned,
# eleven of three, scanned, and eight of two, added up by their readers
SEGMENTED = [(64 * 12 + 9, 2, 64), (2048 - 13, 32, 128), (2048 + 17, 64, 192), (1024 - 5, 64, 128)]


@pytest.mark.parametrize("T,H,rows", SEGMENTED)
def test_nonfinite_values_beside_segment_edges(T, H, rows):
    """Values that are not finite in the last and the first row of segments and
    of chunks inside them, in episodes that cross the edges: they reach the
    rest of their episode, over the states of the scan and of the walk, and
    nothing else (as the test above)."""
    la = tapes.make_linattn(3, seed=92 + H, T=T, H=H)
    f = np.zeros(T, np.uint8)
    f[[0, rows - 10, rows + 7, 2 * rows, 3 * rows - 1, 3 * rows + 33, 5 * rows + 3, T - 12]] = 1
    la.start = f
    g = grad_input(la, 10)
    la.k[rows - 1, 0, 3] = np.nan          # last row of a segment, episode over its edge
    la.v[2 * rows, H - 1, 7] = np.inf      # begin step on an edge
    la.q[3 * rows, 0, 5] = np.nan          # first row of a segment, episode from the row before
    la.k[4 * rows - 1, 0, 9] = np.nan      # an episode over two edges, from the first on
    g[4 * rows + 1, H - 1, 11] = np.nan    # the same episode in another head, and back over its first edge
    la.v[T - 1, 0, 2] = np.nan             # last step of the tape
    announce("linattn bwd non-finite beside segment edges T=%d H=%d" % (T, H))
    q, k, v, s = dev(la.q), dev(la.k), dev(la.v), dev(la.start)
    out = mb.scan_linattn(q, k, v, s)
    gq, gk, gv = mb.scan_linattn_bwd(q, k, v, s, out, dev(g))
    torch.cuda.synchronize()
    wide = [a.astype(np.float64) for a in (la.q, la.k, la.v)]
    ro, mo = oracle.linattn(*wide, la.start)
    rq, rk, rv, mq, mk, mv = oracle.linattn_bwd(*wide, la.start, g.astype(np.float64))
    for name, got, ref, m in (("out", out, ro, mo), ("dq", gq, rq, mq), ("dk", gk, rk, mk), ("dv", gv, rv, mv)):
        got = got.cpu().numpy()
        fin = np.isfinite(ref)
        assert (~fin).any(), name
        assert np.isfinite(got[fin]).all(), (name, np.argwhere(fin & ~np.isfinite(got))[:5])
        assert not np.isfinite(got[~fin]).any(), (name, np.argwhere(~fin & np.isfinite(got))[:5])
        e = cond_err(got[fin], ref[fin], m[fin])
        assert e <= TOL, (name, e)


@pytest.mark.parametrize("kind", ["short", "all_begins", "single_episode", "chunk_starts", "chunk_second_rows",
                                  "segment_starts", "flag_bytes"])
def test_flag_patterns_in_segments_of_two_chunks(kind):
    T, H, rows = SEGMENTED[1]
    rng = np.random.default_rng(18)
    la = tapes.make_linattn(3, seed=78, T=T, H=H)
    f = np.zeros(T, np.uint8)
    if kind == "short":
        f = tapes.flags_from_lengths(rng.integers(1, 40, size=T), T)
    elif kind == "all_begins":
        f[:] = 1
    elif kind == "chunk_starts":
        f[::64] = 1
    elif kind == "chunk_second_rows":
        f[1::64] = 1
    elif kind == "segment_starts":
        f[::rows] = 1
    elif kind == "flag_bytes":
        f = (rng.random(T) < 0.01).astype(np.uint8) * rng.integers(1, 256, size=T).astype(np.uint8)
    check(_with_flags(la, f), kind + ", two chunks a segment")


@pytest.mark.parametrize("T,H", [(2048 + 17, 64), (1024, 64), (1024 - 5, 64)])
def test_segments_of_several_chunks(T, H):
    """Eleven segments of three chunks, scanned, the last partial; eight of two,
    added up by their readers, whole and with a partial last chunk."""
    check(tapes.make_linattn(3, seed=600 + T, T=T, H=H), "several chunks a segment")


def test_errors_do_not_grow_with_the_episode():
    """One episode over the whole tape, in segments of eight chunks: the
    2-norm errors of 262144 steps stay within 1.5 times those of 1024.  What
    grows is the rounding of states that the episode has made large; with one
    per 16-row block and one per segment of the scan the ratios are 1.12 (dq)
    and 1.04 (dk), with one per row they were 1.97 and 1.95."""
    errors = []
    for T, H in ((1024, 4), (262144, 1)):
        la = tapes.make_linattn(3, seed=700, T=T, H=H)
        la.start = np.zeros(T, np.uint8)
        announce("linattn bwd one episode T=%d H=%d" % (T, H))
        g = grad_input(la, 3)
        q, k, v, s = dev(la.q), dev(la.k), dev(la.v), dev(la.start)
        out = mb.scan_linattn(q, k, v, s)
        got = (out,) + mb.scan_linattn_bwd(q, k, v, s, out, dev(g))
        wide = [a.astype(np.float64) for a in (la.q, la.k, la.v)]
        ref = (oracle.linattn(*wide, la.start)[0],) + oracle.linattn_bwd(*wide, la.start, g.astype(np.float64))[:3]
        errors.append([float(np.linalg.norm(a.cpu().numpy() - r) / np.linalg.norm(r)) for a, r in zip(got, ref)])
    for name, short, long in zip(("out", "dq", "dk", "dv"), *errors):
        assert long <= 1.5 * short, (name, short, long)
