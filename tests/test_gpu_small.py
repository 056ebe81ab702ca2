"""One-shot counts by the adjacency bit matrix (up to 8192 vertices) against the oracle and the general path.

Sizes sit at the row widths (128 vertices per 16-byte word; the lanes per edge double at 1, 2, 4, ... words),
at the sample counts of a wavefront, and around the rule's lines (8192 vertices; samples x vertices 2^32).
TC_F_NO_MID moves no count and keeps a call on the general path.
"""
import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

TC_F_NO_MID = 0x2000


def _pairs(n, m, seed):
    rng = np.random.default_rng(seed)
    u = rng.random((2, m))
    e = (u * u * n).astype(np.uint32)
    return gg.EdgeList(n, e[0], e[1], f"pairs{n}_{m}")


@pytest.mark.parametrize("n,m", [(1, 1), (2, 5), (3, 64), (127, 1000), (128, 1001), (129, 63), (256, 65), (257, 3000),
                                 (511, 4096), (513, 4097), (1000, 4000), (1024, 20000), (1025, 20001), (2049, 9999),
                                 (4096, 65536), (4097, 30011), (8191, 70001), (8192, 524288), (8192, 524289),
                                 (8193, 40000), (300, 300_000)])
def test_small_against_oracle_and_general_path(n, m):
    from paper_2103_08053_amd import Context, Params
    g = _pairs(n, m, seed=n + m)
    print(f"[gpu] small {g.name}", flush=True)
    want = oracle.count(g.n, g.src, g.dst, per_vertex=True)
    for flags in (0, TC_F_NO_MID):
        ctx = Context(0, Params(flags=flags))
        for pv in (False, True, True):  # twice: the workspace holds the first call's rows
            total, got = ctx.count(g.src, g.dst, g.n, per_vertex=pv)
            assert total == want.total
            if pv:
                assert (got.cpu().numpy().astype(np.uint64) == want.per_vertex).all()


def test_small_workspace_reused_unaligned_and_checked():
    import torch

    from paper_2103_08053_amd import Context, TCError
    g = gg.dirty(gg.rmat(10, 8, seed=3), seed=1)
    want = oracle.count(g.n, g.src, g.dst, per_vertex=True)
    ctx = Context(0)
    print(f"[gpu] small {g.name} n={g.n} m_in={g.m_in}", flush=True)
    need = ctx.workspace_bytes(g.n, g.m_in)
    s, d = (torch.as_tensor(x.astype(np.int64)).to("cuda").to(torch.int32) for x in (g.src, g.dst))
    for shift in (0, 256, 4096 + 8):
        ws = torch.full((need + shift,), 0xA5, dtype=torch.uint8, device="cuda")
        total, pv = ctx.count(s, d, g.n, per_vertex=True, workspace=ws[shift:])
        assert total == want.total and (pv.cpu().numpy().astype(np.uint64) == want.per_vertex).all()
        assert bool((ws[:shift] == 0xA5).all())
    import ctypes
    tot = ctypes.c_uint64()
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert ctx.lib.tc_count(ctx.h, g.n, g.m_in, s.data_ptr(), d.data_ptr(), None, ws.data_ptr(), need - 1, st,
                            ctypes.byref(tot)) == 3
    bad = s.clone()
    bad[7] = g.n
    with pytest.raises(TCError):
        ctx.count(bad, d, g.n)
    assert ctx.count(s, d, g.n)[0] == want.total


def test_small_timing_and_stream():
    import torch

    from paper_2103_08053_amd import Context
    g = gg.complete(300)
    ctx = Context(0)
    ctx.timing(True)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        total, pv = ctx.count(g.src, g.dst, g.n, per_vertex=True, stream=side)
    side.synchronize()
    assert total == 300 * 299 * 298 // 6 and bool((pv == 299 * 298 // 2).all())
    b, c = ctx.last_times_ms()
    assert b >= 0 and c >= 0


def _repeats(n, m, pairs, seed):
    """m samples drawn from `pairs` pairs of n vertices."""
    rng = np.random.default_rng(seed)
    e = rng.integers(0, n, (2, pairs), dtype=np.uint32)
    e[:, 0] = 0, n - 1
    at = rng.integers(0, pairs, m)
    return gg.EdgeList(n, e[0][at], e[1][at], f"repeats{n}_{m}_{pairs}")


@pytest.mark.parametrize("n,m,pairs", [(2, 4096, 1), (2, 4097, 1), (16, 1 << 18, 120), (16, (1 << 18) + 1, 120),
                                       (100, 600_000, 30), (1000, 600_000, 3000), (8191, 300_000, 5000)])
def test_small_repeated_samples_against_oracle(n, m, pairs):
    """Sample counts around the workgroup sizes and the table of pairs just seen."""
    from paper_2103_08053_amd import Context
    g = _repeats(n, m, pairs, seed=m + pairs)
    print(f"[gpu] small {g.name}", flush=True)
    want = oracle.count(g.n, g.src, g.dst, per_vertex=True)
    ctx = Context(0)
    total, got = ctx.count(g.src, g.dst, g.n, per_vertex=True)
    assert total == want.total and (got.cpu().numpy().astype(np.uint64) == want.per_vertex).all()
    assert ctx.count(g.src, g.dst, g.n)[0] == want.total


@pytest.mark.parametrize("n,pairs", [(2, 1), (16, 120), (100, 100)])
def test_small_repeated_samples_are_not_bound_by_their_atomics(n, pairs):
    """2^24 samples of few pairs take about what reading them takes (0.03 ms), 0.2-0.5 ms, as the general path
    takes 1; an atomic per sample took 13 (100 pairs of 100 vertices) to 190 ms."""
    import time

    import torch

    from paper_2103_08053_amd import Context
    g = _repeats(n, 1 << 24, pairs, seed=n)
    print(f"[gpu] small {g.name}", flush=True)
    ctx = Context(0)
    s, d = (torch.as_tensor(x.astype(np.int32)).to("cuda") for x in (g.src, g.dst))
    ws = torch.empty(ctx.workspace_bytes(n, g.m_in), dtype=torch.uint8, device="cuda")
    ms = []
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ctx.count(s, d, n, workspace=ws)
        ms.append((time.perf_counter() - t0) * 1e3)
    assert min(ms) < 5, ms


def test_small_answers_of_calls_at_the_same_time():
    """One-shot counts that run at the same time, in threads of their own, each get their own answer: on contexts of
    their own, and through one context that has been warmed up."""
    import threading

    import torch

    from paper_2103_08053_amd import Context
    shared = Context(0)
    graphs = [gg.complete(20 + 7 * i) for i in range(8)] + [gg.with_isolated(gg.complete(30 + i), 9000) for i in range(8)]
    wrong, ready = [], threading.Barrier(len(graphs))

    def work(i, ctx):
        g, k = graphs[i], [20 + 7 * i, 30 + i - 8][i >= 8]
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            s, d = (torch.as_tensor(x.astype(np.int32)).to("cuda") for x in (g.src, g.dst))
            ws = torch.empty(ctx.workspace_bytes(g.n, g.m_in), dtype=torch.uint8, device="cuda")
            stream.synchronize()
            ready.wait()
            for _ in range(200):
                total, _ = ctx.count(s, d, g.n, workspace=ws, stream=stream)
                if total != k * (k - 1) * (k - 2) // 6:
                    wrong.append((i, k, total))

    for g in graphs:
        shared.count(g.src, g.dst, g.n)
    for ctxs in ([Context(0) for _ in graphs], [shared] * len(graphs)):
        print(f"[gpu] small {len(graphs)} threads", flush=True)
        threads = [threading.Thread(target=work, args=(i, c)) for i, c in enumerate(ctxs)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not wrong, wrong[:5]


@pytest.mark.parametrize("g", [gg.complete(3), gg.complete(150), gg.star(2000), gg.rmat(8, 8, seed=1), gg.rmat(12, 16, seed=2),
                               gg.erdos_renyi(500, 3000, seed=3), gg.erdos_renyi(8000, 20_000, seed=4)],
                         ids=lambda g: g.name)
def test_general_one_shot_path_on_small_graphs(g):
    """The default one-shot count of the same graphs with isolated vertices beyond the bit matrix's 8192: the build
    and the hash kernels, total and per vertex."""
    from paper_2103_08053_amd import Context
    d = gg.dirty(gg.with_isolated(g, 8200), seed=5)
    print(f"[gpu] one-shot {d.name} n={d.n} m_in={d.m_in}", flush=True)
    assert d.n > 8192
    want = oracle.count(d.n, d.src, d.dst, per_vertex=True)
    ctx = Context(0)
    total, pv = ctx.count(d.src, d.dst, d.n, per_vertex=True)
    assert total == want.total and (pv.cpu().numpy().astype(np.uint64) == want.per_vertex).all()
    assert ctx.count(d.src, d.dst, d.n)[0] == want.total
