"""The core path (block words of the last ranks) against the oracle and against the bucket kernels.

Graphs of at least 2^17 samples, built with default flags, are laid out for the core path, and counted
by it when owners with much 2-hop work dominate; any flag (here TC_F_NO_MID, which moves no count)
leaves them to the bucket kernels.  Sizes sit around the path's limits: the ranks that 22, 21 and 20 ids
per word reach (22528, 43008, 81920), out-degrees of 64 and 128 (a launch's threads), 1024 and 2048, and
graphs whose triangles lie inside, outside and across the core.
"""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TC_F_NO_MID = 0x2000


def _thin(g, every, seed=3):
    """g without about one edge in `every`."""
    keep = np.random.default_rng(seed).integers(0, every, g.m_in) != 0
    return gg.EdgeList(g.n, g.src[keep], g.dst[keep], g.name + "+thin")


def _cliques(k, size):
    i, j = np.triu_indices(size, 1)
    base = (np.arange(k) * size)[:, None]
    return gg.EdgeList(k * size, (base + i).ravel().astype(np.uint32), (base + j).ravel().astype(np.uint32),
                       f"{k}xK{size}")


CASES = [
    gg.complete(513),                                          # just above 2^17 samples, one window
    gg.with_isolated(_thin(gg.complete(700), 3), 22528 - 700),      # every rank in 22-id words, exactly
    gg.with_isolated(_thin(gg.complete(700), 3), 22529 - 700),      # one rank more: 21 ids
    gg.with_isolated(_thin(gg.complete(1100), 2), 43009 - 1100),    # 20 ids
    gg.with_isolated(_thin(gg.complete(1500), 2), 81921 - 1500),    # outside: one isolated rank; bin 1
    gg.complete(2100),                                         # out-degrees up to 2099: both parts of bin 1
    _cliques(1000, 100),                                       # 57% of the cliques outside the core
    _thin(_cliques(400, 260), 4),                              # workgroup-bin owners outside the core
    _cliques(700, 65), _cliques(700, 130),                     # out-degrees at 64 and 128
    gg.rmat(13, 32, seed=5), gg.rmat(15, 16, seed=6), gg.rmat(17, 12, seed=7), gg.rmat(18, 10, seed=8),
    gg.erdos_renyi(1 << 15, 1 << 18, seed=9),                  # light owners only: the path stays off
    gg.erdos_renyi(3000, 1 << 19, seed=10),                    # dense and uniform
    gg.with_isolated(gg.star(140000), 3),                      # no triangles, one hub
]


@pytest.mark.parametrize("g", CASES, ids=[g.name for g in CASES])
def test_core_path_against_oracle_and_bucket_kernels(g):
    from paper_2103_08053_amd import Context, Params
    print(f"[gpu] core {g.name} n={g.n} m_in={g.m_in}", flush=True)
    d = gg.dirty(g, seed=2, dup_frac=0.1)
    want = oracle.count(d.n, d.src, d.dst, per_vertex=True)
    for flags in (0, TC_F_NO_MID):
        ctx = Context(0, Params(flags=flags))
        gr = ctx.build(d.src, d.dst, d.n)
        total, pv = gr.count(per_vertex=True)
        assert total == want.total
        assert (pv.cpu().numpy().astype(np.uint64) == want.per_vertex).all()
        assert gr.count()[0] == want.total
    one, _ = Context(0).count(d.src, d.dst, d.n)
    assert one == want.total


@pytest.mark.parametrize("g", [gg.rmat(16, 16, seed=4), _cliques(800, 110)], ids=["rmat16", "cliques"])
def test_core_path_shards_replay_static_and_small_grids(g):
    import ctypes

    import torch

    from paper_2103_08053_amd import Context, Params
    print(f"[gpu] core {g.name} n={g.n} m_in={g.m_in}", flush=True)
    want = oracle.count(g.n, g.src, g.dst, per_vertex=True)
    ref = want.per_vertex.astype(np.int64)
    ctx = Context(0)
    gr = ctx.build(g.src, g.dst, g.n)
    parts = [gr.count(per_vertex=True, shard=(r, 3)) for r in range(3)]
    assert sum(t for t, _ in parts) == want.total
    assert (sum(p.cpu().numpy() for _, p in parts) == ref).all()
    out = torch.empty(g.n, dtype=torch.int64, device="cuda")
    for _ in range(3):  # the captured launches, with eager work between
        out.fill_(-1)
        gr.count_async(out, replay=True)
        assert int(gr.total_dev.item()) == want.total
        assert (out.cpu().numpy() == ref).all()
        assert gr.count()[0] == want.total
    tot = torch.full((1,), 7, dtype=torch.int64, device="cuda")
    assert ctx.lib.tc_graph_count_static(ctx.h, gr.h, tot.data_ptr(), out.data_ptr(),
                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert int(tot.item()) == want.total and (out.cpu().numpy() == ref).all()
    totals, pvs = ctx.count_graphs([gr, gr], per_vertex=True)  # many-graph launches: bucket kernels, same lists
    assert totals == [want.total] * 2 and (pvs[1].cpu().numpy() == ref).all()
    for grid in (1, 3):
        c1 = Context(0, Params(grid_wgs=grid))
        t1, p1 = c1.build(g.src, g.dst, g.n).count(per_vertex=True)
        assert t1 == want.total and (p1.cpu().numpy() == ref).all()


@pytest.mark.parametrize("n,m", [(1 << 22, 1 << 26), (1 << 20, 16_777_003), (70_000, 1 << 18)])
def test_core_path_shares_the_edge_list_bounds_memory(n, m):
    """A graph uses the list bounds per edge or the core path's layout, so its storage holds the larger of them."""
    import ctypes

    from paper_2103_08053_amd import Context
    ctx = Context(0)
    storage, temp = ctypes.c_uint64(), ctypes.c_uint64()
    assert ctx.lib.tc_graph_footprint(ctx.h, n, m, ctypes.byref(storage), ctypes.byref(temp)) == 0
    csr = 8 * (n + 1) + 4 * (n + 1) + 4 * m + 4 * n + 4 * n
    assert storage.value <= csr + max(8 * m, 4 * m + 28 * n) + 4096


def test_core_path_keeps_a_grid_of_the_callers():
    """A small grid given in workgroups of wg_waves wavefronts is about as many wavefronts on the core path, whose
    workgroups are smaller for owners of little work: no slower than the bucket kernels with that grid (with as
    many workgroups instead it took 1.45 times as long)."""
    import time

    import torch

    from paper_2103_08053_amd import Context, Params
    g = gg.rmat(18, 16, seed=12)
    print(f"[gpu] core grid {g.name}", flush=True)
    ms, seen = [], []
    for flags in (0, TC_F_NO_MID):
        gr = Context(0, Params(flags=flags, grid_wgs=64)).build(g.src, g.dst, g.n)
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            total, pv = gr.count(per_vertex=True)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        ms.append(best * 1e3)
        seen.append((total, pv))
    assert seen[0][0] == seen[1][0] and bool((seen[0][1] == seen[1][1]).all())
    assert ms[0] < 1.1 * ms[1], ms


def test_core_path_is_off_where_few_ids_per_edge_are_in_the_core():
    """Uniform, 2^18 vertices of degree 128: a third of the edges end in the core, 43 probes per edge; counting
    there took 1.4 times as long as the bucket kernels."""
    import time

    import torch

    from paper_2103_08053_amd import Context, Params
    n, m = 1 << 18, 1 << 24
    gen = torch.Generator(device="cuda").manual_seed(5)
    src, dst = (torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2))
    print(f"[gpu] core uniform n={n} m_in={m}", flush=True)
    ms, seen = [], []
    for flags in (0, TC_F_NO_MID):
        gr = Context(0, Params(flags=flags)).build(src, dst, n)
        best = 1e9
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            total, _ = gr.count()
            best = min(best, time.perf_counter() - t0)
        ms.append(best * 1e3)
        seen.append(total)
    assert seen[0] == seen[1]
    assert ms[0] < 1.2 * ms[1], ms


@pytest.mark.parametrize("k,size", [(330, 130), (150, 600)])
def test_core_path_on_cliques(k, size):
    """Cliques inside the core (out-degrees around 128) and half outside it, with enough ids per edge for the path."""
    from math import comb

    from paper_2103_08053_amd import Context
    g = _cliques(k, size)
    print(f"[gpu] core {g.name}", flush=True)
    total, pv = Context(0).build(g.src, g.dst, g.n).count(per_vertex=True)
    assert total == k * comb(size, 3)
    assert (pv.cpu().numpy() == comb(size - 1, 2)).all()
