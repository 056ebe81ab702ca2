"""The build (canonical sort, distinct edges, degrees, rank, CSR, schedule) against the oracle.

Sizes sit at the edges of its tiles (4096 keys of the distinct-edge pass, 2048, 4096 and 18432 elements of a
sort pass, 28672 of the upper-id partition), at the id widths where the number of passes or the
treatment of the upper ids changes (2^9, 2^12, 2^15, 2^16, 2^24, 2^25 ids), and at inputs made of
duplicates or of self-loops, whose groups of equal keys run over many tiles.
"""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu


def _check(g):
    from paper_2103_08053_amd import Context
    print(f"[gpu] build {g.name} n={g.n} m_in={g.m_in}", flush=True)
    want = oracle.count(g.n, g.src, g.dst, per_vertex=True)
    gr = Context(0).build(g.src, g.dst, g.n)
    info = gr.info()
    assert (info.m, info.wedges_plus, info.max_dplus) == (want.m, want.wedges_plus, want.max_dplus)
    assert sum(gr.bin_work()) == want.wedges_plus
    total, pv = gr.count(per_vertex=True)
    assert total == want.total
    assert (pv.cpu().numpy().astype(np.uint64) == want.per_vertex).all()


def _pairs(n, m, seed, distinct=None):
    """m random pairs on n ids; with `distinct`, drawn from that many pairs."""
    rng = np.random.default_rng(seed)
    s = rng.integers(0, n, distinct or m, dtype=np.uint32)
    d = rng.integers(0, n, distinct or m, dtype=np.uint32)
    if distinct:
        pick = rng.integers(0, distinct, m)
        s, d = s[pick], d[pick]
        flip = rng.random(m) < 0.5
        s, d = np.where(flip, d, s), np.where(flip, s, d)
    return gg.EdgeList(n, s, d, f"pairs{n}_{m}_{distinct}")


@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 2047, 2048, 2049, 4096, 4097, 7168, 7169, 14337])
@pytest.mark.parametrize("n", [3, 60, 700])
def test_build_tile_edges(n, m):
    _check(_pairs(n, m, seed=m + n))


@pytest.mark.parametrize("n", [511, 512, 513, 4096, 4097, 32768, 32769, 65536, 65537, 131073, 1 << 24, (1 << 24) + 1,
                               (1 << 25) + 1, (1 << 27) + 3])
def test_build_id_widths(n):
    g = gg.rmat(12, 16, seed=n % 97)
    spread = np.sort(np.random.default_rng(n % 89).choice(n, min(n, g.n), replace=False)).astype(np.uint32)
    keep = (g.src < len(spread)) & (g.dst < len(spread))
    _check(gg.EdgeList(n, spread[g.src[keep]], spread[g.dst[keep]], f"rmat12 on {n} ids"))


@pytest.mark.parametrize("n,distinct", [(2, 1), (5, 4), (900, 1), (900, 3000), (70000, 50), (70000, 30000),
                                        (1 << 20, 2), (1 << 20, 90000)])
def test_build_duplicates(n, distinct):
    _check(_pairs(n, 150_001, seed=n + distinct, distinct=distinct))


@pytest.mark.parametrize("n", [3, 4096, 100_000])
def test_build_self_loops_and_a_few_edges(n):
    rng = np.random.default_rng(n)
    s = np.full(60_000, n - 1, np.uint32)
    d = s.copy()
    s[::3] = rng.integers(0, n, len(s[::3]))
    d[::3] = s[::3]
    s[:300], d[:300] = rng.integers(0, n, 300), rng.integers(0, n, 300)
    _check(gg.EdgeList(n, s, d, f"loops{n}"))


@pytest.mark.parametrize("m", [(1 << 19) - 1, 1 << 19, 3_499_999, 3_500_000, 190 * 18432 + 1])  # tile sizes
def test_build_tile_sizes(m):
    _check(_pairs(300_000, m, seed=m))
    _check(gg.dirty(gg.rmat(17, 12, seed=m % 31), seed=3))


@pytest.mark.parametrize("flags", [0x8, 0x40, 0x80, 0x4000, 0x1000])
def test_build_variants(flags):
    from paper_2103_08053_amd import Context, Params
    g = gg.dirty(gg.rmat(14, 16, seed=11), seed=5)
    print(f"[gpu] build flags {flags:#x} n={g.n} m_in={g.m_in}", flush=True)
    want = oracle.count(g.n, g.src, g.dst, per_vertex=True)
    gr = Context(0, Params(flags=flags)).build(g.src, g.dst, g.n)
    assert gr.info().wedges_plus == want.wedges_plus
    total, pv = gr.count(per_vertex=True)
    assert total == want.total and (pv.cpu().numpy().astype(np.uint64) == want.per_vertex).all()


@pytest.mark.parametrize("m", [40_000, 3_600_000])  # tile sizes
@pytest.mark.parametrize("n", [(1 << 21), (1 << 21) + 1, 1 << 22, (1 << 23) - 5, 1 << 25, (1 << 25) + 1])
def test_build_upper_partitions(n, m):
    """Upper ids in every partition, and all of them within two neighbouring ones (many units of each)."""
    rng = np.random.default_rng(n + m)
    _check(_pairs(n, m, seed=m + n % 83))
    at = n - 1 - (1 << 16) - 1000  # across a multiple of 2^16, the ids of a partition at most
    at += (1 << 16) - (at & 0xFFFF) - 1000
    ids = np.concatenate([at + np.arange(2000), [n - 1, 0, 1]]).astype(np.uint32)
    s, d = ids[rng.integers(0, len(ids), m)], ids[rng.integers(0, len(ids), m)]
    _check(gg.EdgeList(n, s, d, f"narrow{n}_{m}"))


@pytest.mark.parametrize("n,spread", [(60, 8), (700, 300), (4096, 4000), (70000, 4000), (70000, 1), (1 << 20, 8000),
                                      ((1 << 24) + 1, 16000)])
def test_build_long_groups(n, spread):
    """Groups of equal top bits that hold the first keys of three, four or more tiles of 4096, begin or end at a
    tile, or follow one another within one, of few or many distinct pairs (`spread` upper ids)."""
    sizes = [1000, 3096, 16384, 12288, 12289, 16383, 16385, 20000, 100, 3, 20001, 4095, 8200, 40000, 28671, 2]
    rng = np.random.default_rng(n + spread)
    s, d = [], []
    for i, size in enumerate(sizes):
        s.append(np.full(size, i, np.uint32))
        d.append((i + 1 + rng.integers(0, min(spread, n - i - 1), size)).astype(np.uint32))
    s, d = np.concatenate(s), np.concatenate(d)
    order = rng.permutation(len(s))
    flip = rng.random(len(s)) < 0.5
    s, d = s[order], d[order]
    _check(gg.EdgeList(n, np.where(flip, d, s), np.where(flip, s, d), f"groups{n}_{spread}"))


@pytest.mark.parametrize("n", [4, 700, 4096, 1 << 20])
@pytest.mark.parametrize("pairs", [1, 4])
def test_build_repeated_samples_are_not_read_by_one_workgroup(n, pairs):
    """2^24 samples of few pairs, a third of them self-loops, are built in the time of distinct ones (0.5-0.9 ms);
    read to their end by one workgroup they took 13-26."""
    import time

    import torch

    from paper_2103_08053_amd import Context
    rng = np.random.default_rng(n + pairs)
    m = 1 << 24
    e = rng.choice(n, (2, pairs)).astype(np.uint32)
    e[:, 0] = 0, n - 1
    at = rng.integers(0, pairs, m)
    s, d = e[0][at], e[1][at]
    s[: m // 3] = d[: m // 3]
    print(f"[gpu] build repeats n={n} m={m} pairs={pairs}", flush=True)
    ctx = Context(0)
    s, d = (torch.as_tensor(x.astype(np.int32)).to("cuda") for x in (s, d))
    ms = []
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        gr = ctx.build(s, d, n)
        torch.cuda.synchronize()
        ms.append((time.perf_counter() - t0) * 1e3)
    want = {(min(int(a), int(b)), max(int(a), int(b))) for a, b in e.T if a != b}
    assert gr.info().m == len(want)
    assert min(ms) < 5, ms


@pytest.mark.parametrize("flags", [0x80, 0x80 | 0x8, 0x40, 0])
def test_build_order_does_not_depend_on_the_samples_order(flags):
    """Hash ids are the graph's own: builds from reordered, repeated and flipped samples get tables of the same
    collisions, also where ids are handed out neighbour by neighbour (0x80)."""
    from paper_2103_08053_amd import Context, Params
    g = gg.rmat(15, 12, seed=21)
    ctx = Context(0, Params(flags=flags))
    rng = np.random.default_rng(4)
    seen = []
    for i in range(4):
        at = rng.permutation(np.concatenate([np.arange(g.m_in), rng.integers(0, g.m_in, 1000 * i)]))
        flip = rng.random(len(at)) < 0.5
        s, d = np.where(flip, g.dst[at], g.src[at]), np.where(flip, g.src[at], g.dst[at])
        print(f"[gpu] build order flags {flags:#x} m={len(at)}", flush=True)
        seen.append(ctx.build(s, d, g.n).collisions())
    assert all(x == seen[0] for x in seen), seen


def test_build_dense_rows_in_rank_order():
    """A complete graph whose owners need tables in memory (more than 4096 out-neighbours) beside a ring is counted
    from samples in random order as fast as from sorted ones (lists in the samples' order took 1.4-1.6 times as
    long)."""
    import time

    import torch

    from paper_2103_08053_amd import Context
    k, n = 5000, 100_000
    i, j = torch.triu_indices(k, k, 1, device="cuda")
    gen = torch.Generator("cuda").manual_seed(1)
    ids = torch.randperm(n, device="cuda", generator=gen)
    clique, ring = ids[:k].sort().values, ids[k:]
    s, d = torch.cat([clique[i], ring]), torch.cat([clique[j], ring.roll(1)])
    order = torch.randperm(s.numel(), device="cuda", generator=gen)
    each = torch.zeros(n, dtype=torch.int64, device="cuda")
    each[clique] = (k - 1) * (k - 2) // 2
    ctx, ms = Context(0), []
    print(f"[gpu] build dense n={n} m_in={s.numel()}", flush=True)
    for at in (slice(None), order):
        gr = ctx.build(s[at], d[at], n)
        assert gr.info().n_hub > 0
        best = 1e9
        for _ in range(2):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            total, pv = gr.count(per_vertex=True)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        ms.append(best * 1e3)
        assert total == k * (k - 1) * (k - 2) // 6 and bool((pv == each).all())
    assert ms[1] < 1.15 * ms[0], ms


def test_build_largest_id_range():
    """2^32 - 1 vertices, the most that ids allow: loops over vertices end, and every vertex is scheduled once."""
    import torch

    from paper_2103_08053_amd import Context
    n = (1 << 32) - 1
    ids = np.array([0, 1, 2, 77, 1 << 16, 1 << 31, n - 1025, n - 1024, n - 3, n - 2, n - 1], np.uint32)
    i, j = np.triu_indices(len(ids), 1)
    ctx = Context(0)
    torch.cuda.empty_cache()
    need = ctx.workspace_bytes(n, len(i))
    if torch.cuda.mem_get_info()[0] < need + (2 << 30):
        pytest.skip(f"{need >> 30} GiB of device memory needed")
    print(f"[gpu] build n={n} workspace {need >> 30} GiB", flush=True)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    try:
        k = len(ids)
        assert ctx.count(ids[i].astype(np.int64), ids[j].astype(np.int64), n, workspace=ws)[0] == k * (k - 1) * (k - 2) // 6
    finally:
        del ws
        torch.cuda.empty_cache()
