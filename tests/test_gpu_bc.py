"""Betweenness centrality (Brandes on the BFS step), pushing and pulling
phases in every combination, against the FP64 oracle."""
import itertools

import numpy as np
import pytest
import torch

import graphgen as gg
import oracle
import paper_2010_16012_amd as pp
from tests import helpers as H
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

COMBOS = list(itertools.product([pp.PP_PUSH, pp.PP_PULL], repeat=2))
RTOL = 1e-9  # FP64 sums in another order (push: atomics)


def _check(host, sources, combos=COMBOS):
    want = oracle.bc(host.off, host.idx, sources)
    g = pp.Graph(host)
    for fd, bd in combos:
        announce(f"bc {host.name} n={host.n} sources={len(sources)} fwd={fd} bwd={bd}")
        got = pp.betweenness(g, sources, fd, bd)
        torch.cuda.synchronize()
        np.testing.assert_allclose(got.cpu().numpy(), want, rtol=RTOL, atol=1e-9 * max(1.0, np.abs(want).max()))
    return want


def test_closed_forms():
    n = 33
    i = np.arange(n)
    np.testing.assert_allclose(_check(H.path(n), i), 2.0 * i * (n - 1 - i))
    want = np.zeros(n)
    want[0] = (n - 1) * (n - 2)
    np.testing.assert_allclose(_check(H.star(n), i), want)
    _check(H.complete(20), np.arange(20))
    _check(H.full_grid(12, 17), np.arange(0, 204, 7))


def test_random_undirected_and_directed():
    for sym in (True, False):
        for seed, (n, m) in enumerate([(50, 150), (700, 4000)]):
            h = H.random_graph(n, m, 80 + seed, symmetric=sym)
            if not sym:
                h.ensure_transpose()
            _check(h, np.arange(0, n, max(1, n // 40)))


def test_rmat14_sources_with_hubs_and_isolated():
    host = gg.workload("rmat14")
    src = np.concatenate([[0], gg.pick_vertices(host, 15, seed=3)])
    deg = np.diff(host.off)
    isolated = np.nonzero(deg == 0)[0][:2]
    _check(host, np.concatenate([src, isolated]))


def test_long_rows_both_phases():
    # hub rows (walked by a whole wave) and long in-rows summed by the wave
    n = 3000
    src = np.concatenate([np.zeros(n - 1, np.int64), np.arange(1, n - 1)])
    dst = np.concatenate([np.arange(1, n), np.arange(2, n)])
    _check(gg.from_edges(n, src, dst, True, "star+path"), [0, 1, 1500, 2999])


def test_errors():
    g = pp.Graph(H.path(5))
    with pytest.raises(pp.PPError):
        pp.betweenness(g, [5])
    with pytest.raises(pp.PPError):
        pp.betweenness(g, [0], pp.PP_SWITCH, pp.PP_PULL)
    z = pp.betweenness(g, np.zeros(0, np.int32))
    assert torch.count_nonzero(z).item() == 0


def test_source_batches_and_small_workspace():
    # 70 sources run as batches of 32, 32 and 6; a workspace for a few
    # sources at a time gives smaller batches and the same scores
    from paper_2010_16012_amd import _lib

    host = gg.workload("rmat14")
    src = gg.pick_vertices(host, 70, seed=5)
    want = oracle.bc(host.off, host.idx, src)
    g = pp.Graph(host)
    tol = dict(rtol=RTOL, atol=1e-9 * max(1.0, np.abs(want).max()))
    for fd, bd in [(pp.PP_PULL, pp.PP_PULL), (pp.PP_PUSH, pp.PP_PUSH)]:
        announce(f"bc rmat14 70 sources fwd={fd} bwd={bd}")
        got = pp.betweenness(g, src, fd, bd)
        torch.cuda.synchronize()
        np.testing.assert_allclose(got.cpu().numpy(), want, **tol)
    full = _lib.pp_bc_workspace_bytes(g.handle)
    ws = torch.empty(full // 8, dtype=torch.uint8, device=g.device)
    bc = torch.empty(g.n, dtype=torch.float64, device=g.device)
    announce("bc rmat14 9 sources, workspace for four at a time")
    _lib.pp_bc_run(g.handle, pp.PP_PULL, pp.PP_PUSH, src[:9], bc, ws)
    torch.cuda.synchronize()
    want9 = oracle.bc(host.off, host.idx, src[:9])
    np.testing.assert_allclose(bc.cpu().numpy(), want9, rtol=RTOL, atol=1e-9 * max(1.0, np.abs(want9).max()))
    with pytest.raises(pp.PPError):
        _lib.pp_bc_run(g.handle, pp.PP_PULL, pp.PP_PULL, src[:2], bc, torch.empty(1024, dtype=torch.uint8,
                                                                                   device=g.device))


@pytest.mark.parametrize("count", [1, 4, 5, 8, 9, 16, 17, 32, 33])
def test_sources_that_share_their_levels(count):
    # both passes pulling: every width of the batch, full and not, with a source
    # given twice; rows cut into several pieces, groups of rows at and past the
    # edge count that a wavefront takes together, more than 32 levels, vertices
    # that no source reaches, and a workspace that holds a single source's slab
    hosts = [H.star(1500), H.complete(260), H.path(75), gg.rmat(11, 8, seed=2),
             gg.from_edges(70, [1, 2, 3, 3], [2, 3, 4, 68], True)]
    hosts.append(H.random_graph(300, 9000, 7, symmetric=False))
    hosts[-1].ensure_transpose()
    # eight rows of 32 edges each (a group of exactly 256), then of 33
    for d in (32, 33):
        hosts.append(gg.from_edges(8 + d, np.repeat(np.arange(8), d), np.tile(8 + np.arange(d), 8), True))
    for h in hosts:
        src = np.random.default_rng(count).integers(0, h.n, count)
        src[-1] = src[0]
        want = _check(h, src, [(pp.PP_PULL, pp.PP_PULL)])
        g = pp.Graph(h)
        bc = torch.empty(h.n, dtype=torch.float64, device="cuda")
        slab = (pp.pp_bc_workspace_bytes(g.handle) - 1024) // 32
        pp.pp_bc_run(g.handle, pp.PP_PULL, pp.PP_PULL, src, bc,
                     torch.empty(1024 + slab, dtype=torch.uint8, device="cuda"), None)
        np.testing.assert_allclose(bc.cpu().numpy(), want, rtol=RTOL, atol=1e-9 * max(1.0, np.abs(want).max()))


@pytest.mark.parametrize("leaves", [63, 64, 65, 127, 128, 129, 5000])
def test_pushed_levels_of_one_vertex(leaves):
    # a wavefront's appends collect 128 vertices before they go to the order: a
    # hub's row that ends short of that, at it and past it, with a second level
    # that all of them share, hot ids and others
    h = gg.from_edges(2 + leaves, np.concatenate([np.zeros(leaves, np.int64), np.ones(leaves, np.int64)]),
                      np.concatenate([2 + np.arange(leaves)] * 2), True)
    _check(h, [0, 1, 2, leaves + 1], [(pp.PP_PUSH, pp.PP_PUSH), (pp.PP_PUSH, pp.PP_PULL)])
