"""Triangle counting, pushing and pulling forms, against the oracle (exact)."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import graphgen as gg
import oracle
import paper_2010_16012_amd as pp
from tests import helpers as H
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

DIRS = [pp.PP_PULL, pp.PP_PUSH]


def _tc(host, d):
    g = pp.Graph(host, relabel=False)
    out = pp.triangles(g, d)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _same(host):
    want = oracle.triangles(host.off, host.idx)
    for d in DIRS:
        announce(f"tc {host.name} n={host.n} nnz={host.nnz} dir={d}")
        got = _tc(host, d)
        np.testing.assert_array_equal(got, want)
    return want


def test_closed_forms():
    k = H.complete(40)
    np.testing.assert_array_equal(_same(k), np.full(40, 39 * 38 // 2))
    assert _same(H.star(500)).sum() == 0
    assert _same(H.cycle(3)).tolist() == [1, 1, 1]
    assert _same(H.cycle(50)).sum() == 0
    assert _same(H.full_grid(20, 30)).sum() == 0


def test_random_graphs_and_rmat14():
    for s, (n, m) in enumerate([(10, 30), (300, 3000), (5000, 60000)]):
        _same(H.random_graph(n, m, 40 + s, symmetric=True))
    _same(gg.workload("rmat14"))


def test_rows_across_many_slices_and_heavy_pairs():
    # a hub adjacent to everything plus a dense core: the hub row spans many
    # 256-edge slices, hub-core pairs need the wavefront-wide intersection
    n = 6000
    src = list(range(1, n))
    dst = [0] * (n - 1)
    rng = np.random.default_rng(3)
    core = rng.choice(np.arange(1, n), size=120, replace=False)
    for i in range(len(core)):
        for j in range(i + 1, len(core)):
            src.append(int(core[i]))
            dst.append(int(core[j]))
    extra = rng.integers(1, n, size=(20000, 2))
    src += extra[:, 0].tolist()
    dst += extra[:, 1].tolist()
    _same(gg.from_edges(n, src, dst, True, name="hub+core"))


def test_empty_and_isolated():
    _same(gg.from_edges(7, [], [], True, name="empty"))
    _same(gg.from_edges(9, [0, 1, 2], [1, 2, 0], True, name="triangle+isolated"))


def test_push_equals_pull_on_rmat16():
    host = gg.rmat(16, 16, seed=2)
    g = pp.Graph(host, relabel=False)
    a = pp.triangles(g, pp.PP_PULL)
    b = pp.triangles(g, pp.PP_PUSH)
    assert torch.equal(a, b)
    want = oracle.triangles(host.off, host.idx)
    np.testing.assert_array_equal(a.cpu().numpy(), want)


def test_unsorted_rows_are_rejected():
    host = gg.from_edges(6, [0, 0, 0, 1, 2], [1, 2, 3, 2, 3], True)
    idx = host.idx.copy()
    r0, r1 = int(host.off[0]), int(host.off[1])
    idx[r0:r1] = idx[r0:r1][::-1].copy()  # row 0 descending
    bad = gg.HostGraph(host.n, host.off.copy(), idx, True, name="unsorted")
    g = pp.Graph(bad, relabel=False)
    with pytest.raises(pp.PPError):
        pp.triangles(g, pp.PP_PULL)


@pytest.mark.parametrize("n,directed", [(300, False), (300, True), ((1 << 20) + 77, False), ((1 << 20) + 77, True)])
def test_owner_rows_at_the_class_edges(n, directed):
    # dense blobs whose row lengths straddle the lane (16), wavefront (64) and
    # bitmap classes, on ids that reach past one bitmap window (2^20) when n
    # does; directed: about half the edges have no edge back
    rng = np.random.default_rng(n + directed)
    src, dst = [], []
    at = np.sort(rng.choice(n, size=280, replace=False))
    at[:2], at[-2:] = (0, 1), (n - 2, n - 1)
    for size in (15, 16, 17, 18, 33, 64, 65, 66, 67, 130, 270):
        ids = rng.choice(at, size=size, replace=False)
        a, b = np.meshgrid(ids, ids)
        keep = (a < b) if not directed else (a != b) & (rng.random(a.shape) < 0.7)
        src += a[keep].tolist()
        dst += b[keep].tolist()
    host = gg.from_edges(n, src, dst, not directed, name=f"blobs{n}{'d' if directed else ''}")
    if not directed:
        _same(host)
        return
    host.ensure_transpose()
    A = sp.csr_matrix((np.ones(host.nnz, dtype=np.int64), host.idx, host.off), shape=(n, n))
    C = A.multiply(A @ A.T)  # common out-neighbours of the ends of every edge
    np.testing.assert_array_equal(_tc(host, pp.PP_PULL), np.asarray(C.sum(1)).ravel() // 2)
    np.testing.assert_array_equal(_tc(host, pp.PP_PUSH), np.asarray(C.sum(0)).ravel() // 2)


def test_self_loops_count_as_before():
    # a stored self-loop (v, v) meets v's whole row
    off = np.array([0, 3, 5, 7], dtype=np.int64)
    idx = np.array([0, 1, 2, 0, 2, 0, 1], dtype=np.int32)
    host = gg.HostGraph(3, off, idx, True, name="loop")
    host.in_off, host.in_idx = off, idx
    rows = [set(idx[off[v]:off[v + 1]].tolist()) for v in range(3)]
    pull = [sum(len(rows[v] & rows[w]) for w in rows[v]) // 2 for v in range(3)]
    push = [sum(len(rows[v] & rows[w]) for v in range(3) if w in rows[v]) // 2 for w in range(3)]
    assert _tc(host, pp.PP_PULL).tolist() == pull
    assert _tc(host, pp.PP_PUSH).tolist() == push


@pytest.mark.parametrize("n,m", [(200_000, 0), (200_000, 900_000), (600_000, 0), (600_000, 3_000_000), (5_000, 0)])
def test_owner_rows_searched_or_in_a_bitmap(n, m):
    # blobs whose rows straddle the lengths at which a row's pairs are counted in the
    # lane (16), by a search of the row (64, or 512 where a bitmap is large) and by
    # bitmap, in sparse (m = 0) and denser graphs, whose forms differ
    rng = np.random.default_rng(n + m)
    at = np.sort(rng.choice(n, size=620, replace=False))
    src, dst = [rng.integers(0, n, m)], [rng.integers(0, n, m)]
    for size in (17, 64, 66, 512, 513, 515, 610):
        ids = rng.choice(at, size=size, replace=False)
        a, b = np.meshgrid(ids, ids)
        keep = a < b
        src.append(a[keep])
        dst.append(b[keep])
    _same(gg.from_edges(n, np.concatenate(src), np.concatenate(dst), True, name=f"blobs{n}_{m}"))


@pytest.mark.parametrize("d", [2, 15, 17, 40, 64])
def test_no_row_needs_a_bitmap(d):
    # rows of at most 64 entries: summed without counts beforehand, or by searches alone
    n = 30_000
    k = np.arange(n)
    ring = [(k + s) % n for s in range(1, d // 2 + 1)]
    _same(gg.from_edges(n, np.tile(k, len(ring)), np.concatenate(ring), True, name=f"ring{d}"))


@pytest.mark.parametrize("n,d", [(1, 0), (3, 2), (100, 40), (5_000, 2), (5_000, 16), (5_000, 18), (5_000, 64),
                                 (20_481, 16), (20_479, 16), (49_152, 18), (49_151, 18)])
def test_few_slices_have_a_workgroup_each(n, d):
    # small graphs without rows for a bitmap, to both sides of the edge counts from
    # which they are summed without counts (327,680 edges) or searched alone (786,432;
    # with 256 compute units), and a directed graph whose pairs are met one way
    k = np.arange(n)
    ring = [(k + s) % n for s in range(1, d // 2 + 1)]
    src, dst = np.tile(k, len(ring)), np.concatenate(ring) if ring else np.zeros(0, int)
    _same(gg.from_edges(n, src, dst, True, name=f"ring{n}_{d}"))
    if 100 < n <= 20_000:
        _same(gg.from_edges(n, src, dst, False, name=f"arcs{n}_{d}").ensure_transpose())


def test_sparse_graphs_are_not_charged_for_bitmaps():
    # a grid of a million vertices has no row for a bitmap: counting its triangles
    # (134 us) is less work than 20 PageRank steps (350 us), and was more (504 us)
    # when every slice was looked through beside a bitmap of 128 KB
    g = pp.Graph(gg.grid(1000, 1031, 0.05, seed=1), relabel=False)

    def best(fn):
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fn()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert best(lambda: pp.triangles(g, pp.PP_PULL)) < best(lambda: pp.pagerank(g, 20, 0.85, pp.PP_PULL))
