"""Row locks where many sources want one row: vertices that are drawn far more often than their
own degree says, because edges lead to them and none (or few) lead away.  Such rows take atomic
adds; under a lock their holders would queue up."""
import numpy as np
import pytest
import torch

import paper_2008_12336_amd as G
from oracle import gosh_oracle as O
from tests.test_gpu_hot_mode import ring
from tests.test_gpu_layout import DEV, SEQ_LAYOUT, TOL, say, start_matrix, upload
from tests.util import HOT_ALL, HOT_LOCKED, SEAM_LOCK_TRIES, SEAM_LOCKS_HELD, last_hot_mode, rel_err, seam

pytestmark = pytest.mark.gpu


def sink_graph(n, sinks, per_vertex, seed):
    """Directed: every vertex but the `sinks` first ones has one edge to a sink and per_vertex - 1
    to anywhere; the sinks have none."""
    rng = np.random.default_rng(seed)
    rows = np.sort(np.concatenate((rng.integers(0, sinks, (n - sinks, 1)),
                                   rng.integers(sinks, n, (n - sinks, per_vertex - 1))), 1), 1)
    xadj = np.concatenate((np.zeros(sinks, dtype=np.int64), np.arange(n - sinks + 1, dtype=np.int64) * per_vertex))
    return xadj, rows.ravel().astype(np.int32)


def milliseconds(run):
    times = []
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def assert_first_order(M, before, want, g, k, epoch):
    """Every row within 2 % of its own movement of the sequential result, and what the roundings of
    that many updates of a row can add up to."""
    step = np.abs(want.astype(np.float64) - before).max(axis=1)
    err = np.abs(M.cpu().numpy().astype(np.float64) - want).max(axis=1)
    say(f"[contended] d={M.shape[1]}: worst err/step {np.max(err / np.maximum(step, 1e-30)):.3e}")
    ids = torch.empty(g.n * (k + 1), dtype=torch.int32, device=DEV)
    G.gosh_sample_epoch(g, k, 77, epoch, 1, ids)
    ids = ids.cpu().numpy()
    updates = np.bincount(ids[ids >= 0], minlength=g.n) + k + 2
    assert (err <= 0.02 * step + updates * 2.0 ** -23 * np.abs(before).max()).all()


@pytest.mark.parametrize("sinks", [1, 40])
@pytest.mark.parametrize("d,k", [(128, 3), (64, 9)])
def test_epoch_does_not_queue_up_at_a_sink(d, k, sinks):
    """As atomic adds a fifth of all positive samples on one row cost a few times an ordinary epoch;
    one holder after another they cost a thousand times one.  The bar lies between: four times
    the all-atomic epoch."""
    n = 80_000
    xadj, adj = sink_graph(n, sinks, 5, 3)
    g, keep = upload(n, xadj, adj, True)
    M0 = torch.from_numpy(start_matrix(n, d, 5, 0.5)).to(DEV)
    ms = {}
    for flags in (G.GOSH_FLAG_ATOMIC_ADDS, 0):
        M = M0.clone()
        ms[flags] = milliseconds(lambda: G.gosh_train_epoch(g, M, k, 1e-4, 7, 0, 0, flags))
    say(f"[contended] d={d} k={k} sinks={sinks}: default {ms[0]:.3f} ms, adds {ms[G.GOSH_FLAG_ATOMIC_ADDS]:.3f} ms")
    assert ms[0] <= 4 * ms[G.GOSH_FLAG_ATOMIC_ADDS]


def test_rotation_does_not_queue_up_at_a_sink():
    n, d, k, K = 400_000, 128, 3, 4
    xadj, adj = sink_graph(n, 10, 5, 4)
    xt, at = torch.from_numpy(xadj).to(DEV), torch.from_numpy(adj).to(DEV)
    M0 = torch.from_numpy(start_matrix(n, d, 5, 0.5)).to(DEV)
    ms = {}
    for flags in (G.GOSH_FLAG_ATOMIC_ADDS, 0):
        M = M0.clone()
        ms[flags] = min(G.gosh_train_parts(n, xt, at, M, k, 1, 1e-5, 7, force_K=K, B=5, flags=flags)["kernel_ms"]
                        for _ in range(2))
    say(f"[contended] rotation: default {ms[0]:.2f} ms, adds {ms[G.GOSH_FLAG_ATOMIC_ADDS]:.2f} ms")
    assert ms[0] <= 4 * ms[G.GOSH_FLAG_ATOMIC_ADDS]


@pytest.mark.parametrize("d,n,k", [(36, 140_000, 10), (128, 40_000, 3)])
def test_rows_drawn_often_lose_no_update(d, n, k):
    """Sinks that thousands of sources draw, beside rows under locks: in sequential order the
    sequential result; concurrent, to first order (the bar of the all-atomic epoch, see
    test_locked_rows), twice, so that the counts of the first launch must have been cleared."""
    xadj, adj = sink_graph(n, 30, 4, 9)
    g, keep = upload(n, xadj, adj, False)
    M0 = start_matrix(n, d, 5, 0.5)
    want = M0.copy()
    O.train_epoch(xadj, adj, want, k, 0.02, 77, 0, 1)
    M = torch.from_numpy(M0).to(DEV)
    G.gosh_train_epoch(g, M, k, 0.02, 77, 0, 1, SEQ_LAYOUT)
    torch.cuda.synchronize()
    assert rel_err(M.cpu().numpy(), want) <= TOL
    M = torch.from_numpy(M0).to(DEV)
    for epoch in range(2):
        before = M.cpu().numpy()
        want = before.copy()
        O.train_epoch(xadj, adj, want, k, 1e-5, 77, epoch, 1)
        G.gosh_train_epoch(g, M, k, 1e-5, 77, epoch, 1)
        torch.cuda.synchronize()
        assert_first_order(M, before, want, g, k, epoch)


@pytest.mark.parametrize("d,n,k", [(64, 50_000, 11), (100, 37_000, 11), (128, 40_000, 3), (260, 20_000, 6)])
def test_updates_whose_lock_cannot_be_had_are_added(d, n, k):
    """Every lock held when the launch begins and nobody to let go: the tries end and every update is
    added, the source's own change too.  As nothing is stored then, nothing is lost: the sequential
    result in sequential order and, concurrent, the bar of the all-atomic epoch."""
    xadj, adj = sink_graph(n, 30, 4, 9)
    g, keep = upload(n, xadj, adj, False)
    M0 = start_matrix(n, d, 5, 0.5)
    try:
        with seam(SEAM_LOCK_TRIES, 2), seam(SEAM_LOCKS_HELD, 1):
            for lr, flags in ((0.02, SEQ_LAYOUT), (1e-5, 0)):
                want = M0.copy()
                O.train_epoch(xadj, adj, want, k, lr, 77, 0, 1)
                M = torch.from_numpy(M0).to(DEV)
                G.gosh_train_epoch(g, M, k, lr, 77, 0, 1, flags)
                torch.cuda.synchronize()
                assert last_hot_mode() == HOT_LOCKED
                if flags:
                    assert rel_err(M.cpu().numpy(), want) <= TOL
                else:
                    assert_first_order(M, M0, want, g, k, 0)
    finally:
        with seam(SEAM_LOCKS_HELD, 2):
            G.gosh_train_epoch(g, M, k, 1e-5, 77, 0, 1)
            torch.cuda.synchronize()


@pytest.mark.parametrize("d,n", [(64, 240_000), (100, 220_000), (128, 92_000), (512, 22_000)])
def test_infinities_and_nan_under_locks(d, n):
    """Rows that hold what is no number spread it as they do with adds, in sequential order entry by
    entry: the same entries finite, and those the same numbers.  No negatives and a ring, so that it
    does not reach everywhere."""
    rng = np.random.default_rng(2)
    xadj, adj = ring(n)
    g, keep = upload(n, xadj, adj, False)
    M0 = start_matrix(n, d, 5, 0.5)
    for v, x in zip(rng.choice(n, 40, replace=False), [np.nan, np.inf, -np.inf, 3e38] * 10):
        M0[v, rng.integers(0, d)] = x
    got = []
    G.gosh_set_tuning(hot_all_inv_eps=64)  # every row is hot also without negatives
    try:
        for flags in (SEQ_LAYOUT, SEQ_LAYOUT | G.GOSH_FLAG_ATOMIC_ADDS):
            M = torch.from_numpy(M0.copy()).to(DEV)
            G.gosh_train_epoch(g, M, 0, 1e-3, 77, 0, 1, flags)
            torch.cuda.synchronize()
            assert last_hot_mode() == (HOT_LOCKED if flags == SEQ_LAYOUT else HOT_ALL)
            got.append(M.cpu().numpy())
    finally:
        G.gosh_set_tuning()
    finite = [np.isfinite(x) for x in got]
    hit = (~finite[0]).any(axis=1).sum()
    say(f"[contended] d={d}: {hit} rows with entries that are no numbers")
    assert np.array_equal(*finite) and 40 <= hit < n / 2
    ok = finite[0] & (np.abs(got[1]) < 1e3)
    assert rel_err(np.where(ok, got[0], 0), np.where(ok, got[1], 0)) <= TOL


@pytest.mark.parametrize("d,n,k", [(64, 45_000, 15), (36, 140_000, 15), (100, 37_000, 15)])
def test_locked_epoch_with_as_many_samples_as_lanes_or_more(d, n, k):
    """A source's samples are taken in chunks of a lane group's size (16 for d <= 64, 32 for d <= 128):
    chunks that are just full, and half empty.  The sequential result; concurrent, to first order."""
    xadj, adj = sink_graph(n, 30, 4, 9)
    g, keep = upload(n, xadj, adj, True)
    M0 = start_matrix(n, d, 5, 0.5)
    for lr, flags in ((0.02, SEQ_LAYOUT), (1e-5, 0)):
        want = M0.copy()
        O.train_epoch(xadj, adj, want, k, lr, 77, 0, 1)
        M = torch.from_numpy(M0).to(DEV)
        G.gosh_train_epoch(g, M, k, lr, 77, 0, 1, flags)
        torch.cuda.synchronize()
        assert last_hot_mode() == HOT_LOCKED
        if flags:
            assert rel_err(M.cpu().numpy(), want) <= TOL
        else:
            assert_first_order(M, M0, want, g, k, 0)


@pytest.mark.parametrize("d,n,k,B", [(64, 20_000, 3, 5), (64, 20_000, 15, 1), (100, 16_000, 3, 8), (128, 9_000, 3, 9),
                                     (260, 7_500, 12, 5)])
def test_locked_visits_of_several_chunks(d, n, k, B):
    """Visits whose sources take more samples than a lane group has lanes: a last chunk of 4 of 16, one
    full, one full of 32, 4 of 32 and 1 of 64.  Sequential order against the oracle."""
    xadj, adj = sink_graph(n, 30, 4, 9)
    xt, at = torch.from_numpy(xadj).to(DEV), torch.from_numpy(adj).to(DEV)
    M0 = start_matrix(n, d, 5, 0.5)
    want = M0.copy()
    O.train_parts(xadj, adj, want, k, B, 0.02, 77, 0, K=1, B=B)
    M = torch.from_numpy(M0).to(DEV)
    G.gosh_train_parts(n, xt, at, M, k, B, 0.02, 77, force_K=1, B=B, flags=SEQ_LAYOUT)
    torch.cuda.synchronize()
    assert last_hot_mode() == HOT_LOCKED
    assert rel_err(M.cpu().numpy(), want) <= TOL


@pytest.mark.parametrize("d,n,k,B", [(64, 40_000, 3, 5), (64, 40_000, 15, 2), (36, 125_000, 3, 5), (100, 32_000, 3, 9), (128, 18_000, 3, 9),
                                     (200, 16_000, 6, 10), (260, 15_000, 12, 5)])
def test_concurrent_visits_of_several_chunks(d, n, k, B):
    """All groups of all wavefronts at work, each with a lock, the next chunk's ids and its counts of draws
    carried over a chunk's border at its own pace (20 or 32 samples of 16 lanes, 36 of 32, 65 or 70 of 64):
    two parts, two rotations in one call, so that locks and counts left behind would show.  To first order,
    as in assert_first_order.  (An epoch has at most 16 samples and, under locks, at least 16 lanes.)"""
    K, lr = 2, 1e-5
    xadj, adj = sink_graph(n, 30, 4, 9)
    xt, at = torch.from_numpy(xadj).to(DEV), torch.from_numpy(adj).to(DEV)
    M0 = start_matrix(n, d, 5, 0.5)
    want = M0.copy()
    O.train_parts(xadj, adj, want, k, 2 * B * K, lr, 77, 0, K, B)
    M = torch.from_numpy(M0).to(DEV)
    st = G.gosh_train_parts(n, xt, at, M, k, 2 * B * K, lr, 77, force_K=K, B=B)
    torch.cuda.synchronize()
    assert last_hot_mode() == HOT_LOCKED and st["rotations"] == 2
    updates = np.full(n, 2.0 * K)  # a source's own change is added once a visit
    narrow = np.zeros((n, 4), dtype=np.float32)
    for rotation in range(2):
        for q, (pa, pb) in enumerate(O.pair_order(K)):
            ids = O.train_pair(xadj, adj, narrow, k, B, K, pa, pb, 0.0, 77, rotation, 0, q, want_stream=True)
            updates += np.bincount(ids[ids >= 0], minlength=n)
    updates += 2 * K * B * (k + 1)  # the roundings of the copy that the source works on
    step = np.abs(want.astype(np.float64) - M0).max(axis=1)
    err = np.abs(M.cpu().numpy().astype(np.float64) - want).max(axis=1)
    say(f"[contended] visits d={d} k={k} B={B}: worst err/step {np.max(err / np.maximum(step, 1e-30)):.3e}")
    assert (err <= 0.02 * step + updates * 2.0 ** -23 * np.abs(M0).max()).all()
