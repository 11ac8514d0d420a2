"""Kernels whose workgroup size or launch count follows the problem's size, at
the sizes where that changes: the compaction of masks at the limit below which
it takes one launch (lists, table and slot pairs), group norm and max-pool over
many short bodies (their smaller workgroups, bodies of more rows than stay in
registers), and the transposed table at the edges of its 64-row blocks.
Against the oracle or its definition written out; every input is seeded.
"""
import numpy as np
import pytest
import torch

from oracle import shc_oracle as O
from paper_2608_09388_amd import binding as shc
from paper_2608_09388_amd import synth
from paper_2608_09388_amd.pipeline import SparseStack
from tests.gpu_util import (TORCH, Compaction, assert_gn_close, down, gn_floor, require_gpu, up)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def table_of(m, nbr):
    B, V = m.shape
    coords, inv, _, n = O.compact(m)
    t = np.full((nbr.shape[1], n), -1, np.int64)
    for j in range(nbr.shape[1]):
        u = nbr[coords[:, 1], j].astype(np.int64)
        ok = (u >= 0) & (u < V)
        r = inv[coords[:, 0] * V + np.where(ok, u, 0)]
        t[j] = np.where(ok, r, -1)
    return t


# the one-launch limit is 64 KB of mask: totals at and one past it, totals
# that leave 1 to 15 bytes past a 16-byte group, bodies that start at any byte;
# with the table, at and past 256 bodies
@pytest.mark.parametrize("B,V,p", [(1, 1, 1.0), (3, 5, 0.5), (4, 655, 0.1), (1, 65535, 0.3),
                                   (1, 65536, 0.3), (1, 65537, 0.3), (16, 4096, 1.0),
                                   (5, 13107, 0.05), (13, 5041, 0.0), (13, 5042, 0.2),
                                   (100, 655, 0.4), (101, 655, 0.4), (256, 255, 0.2),
                                   (257, 37, 0.5), (16384, 4, 0.3)])
def test_compaction_launches(dev, B, V, p):
    rng = np.random.default_rng(B * 977 + V)
    m = (rng.random((B, V)) < p).astype(np.uint8)
    m[m != 0] = rng.integers(1, 256, size=int(m.sum()))
    ref_c, ref_inv, ref_rp, ref_n = O.compact(m)
    c = Compaction(m)
    c.ws.fill_(0xAB)
    assert c.run() == ref_n
    assert np.array_equal(down(c.inv), ref_inv) and np.array_equal(down(c.row_ptr), ref_rp)
    assert np.array_equal(down(c.coords)[:ref_n], ref_c)
    if V > shc.COMPACT_TABLE_MAX_V:
        return
    K = 3
    nbr = rng.integers(-1, V + 1, size=(V, K)).astype(np.int32)
    nbr[:, 0] = np.arange(V)
    c = Compaction(m)
    table = torch.full((K * max(c.cap, 1),), -7, dtype=torch.int32, device=dev)
    pc = shc.PreparedCompact(c.mask, B, V, c.coords, c.inv, c.row_ptr, c.n_dev, c.ws,
                             nbr=up(nbr), table=table)
    pc.start()
    n = pc.wait()
    torch.cuda.synchronize()
    assert n == ref_n
    assert np.array_equal(down(c.inv), ref_inv) and np.array_equal(down(c.row_ptr), ref_rp)
    assert np.array_equal(down(c.coords)[:n], ref_c)
    assert np.array_equal(down(table)[: K * n].reshape(K, n), table_of(m, nbr))


@pytest.mark.parametrize("K,n", [(1, 1), (3, 5), (9, 1820), (9, 1821), (1, 16384), (1, 16385),
                                 (32, 700)])
def test_slot_pairs_launches(dev, K, n):
    rng = np.random.default_rng(K * 31 + n)
    t = rng.integers(0, n, size=(K, n)).astype(np.int32)
    t[rng.random((K, n)) < 0.6] = -1
    pairs = torch.full((K * n, 2), -7, dtype=torch.int32, device=dev)
    ptr = torch.full((K + 1,), -7, dtype=torch.int32, device=dev)
    shc.build_slot_pairs(up(t), n, K, pairs, ptr)
    j, i = np.nonzero(t >= 0)
    got = down(pairs)
    assert np.array_equal(got[: len(j)], np.stack([j, i], 1)) and np.all(got[len(j):] == -7)
    assert np.array_equal(down(ptr), np.concatenate([[0], np.cumsum((t >= 0).sum(1))]))


# B above the CU count: workgroups of 256, 512 or 1024 threads by the mean row
# count; body 3 is full (more rows than stay in registers), 1 and B - 1 empty
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,V,C,G,p", [(300, 400, 32, 8, 0.12), (600, 655, 256, 32, 0.1),
                                       (280, 300, 96, 4, 0.5), (270, 700, 256, 1, 0.4)])
def test_short_bodies_norm_and_pool(dev, dtype, B, V, C, G, p):
    rng = np.random.default_rng(B + V + C)
    m = (rng.random((B, V)) < p).astype(np.uint8)
    m[[1, B - 1]] = 0
    m[3] = 1
    m[4] = 0
    m[4, 7] = 1
    coords, inv, rp, n = O.compact(m)
    S = (rng.standard_normal((n, C)) * 2.0 + rng.standard_normal(C) * 3.0).astype(np.float32)
    S = synth.as_dtype(S, dtype)[1]
    Sd = up(S, dtype)
    out = torch.full((n + 3, C), float("nan"), dtype=TORCH[dtype], device=dev)
    shc.segment_group_norm(Sd, up(rp), n, B, G, out)
    got = down(out)
    assert np.all(np.isnan(got[n:]))
    assert_gn_close(got[:n], O.group_norm(S.astype(np.float64), rp, G), dtype,
                    gn_floor(S, rp, G), f"group norm B={B} C={C} G={G}")
    P = torch.full((B, C), float("nan"), dtype=TORCH[dtype], device=dev)
    shc.segment_maxpool(Sd, up(rp), n, B, P, -2.0)
    assert np.array_equal(down(P), O.segment_max(S.astype(np.float64), rp, -2.0))


# a few bodies longer than the workgroup's registers hold (64 rows of 256 fp32
# channels, 128 of bf16, 256-thread workgroups), streamed in batches of that
# many rows: at and beside whole batches, and many of them
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_norm_streams_long_bodies(dev, dtype):
    B, C, G = 600, 256, 32
    rng = np.random.default_rng(9)
    rows = rng.integers(0, 12, size=B)
    rows[:12] = [63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 2500]
    rp = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    n = int(rp[-1])
    S = (rng.standard_normal((n, C)) * 2.0 + rng.standard_normal(C) * 3.0).astype(np.float32)
    S = synth.as_dtype(S, dtype)[1]
    out = torch.full((n + 3, C), float("nan"), dtype=TORCH[dtype], device=dev)
    shc.segment_group_norm(up(S, dtype), up(rp), n, B, G, out)
    got = down(out)
    assert np.all(np.isnan(got[n:]))
    assert_gn_close(got[:n], O.group_norm(S.astype(np.float64), rp, G), dtype,
                    gn_floor(S, rp, G), "group norm of long bodies")


# bodies longer than a small workgroup's registers hold, shared by the
# workgroups of their grid column: 256 threads and four ranges of 16 (C 256),
# 8 (128) and 6 vectors (96), two where groups (G 2) or 64 bytes a row (C 32)
# allow no more, none (G 1), and 512 threads with two (mean of 65 rows); at and
# beside the rows that one workgroup and all of them hold
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("C,G,mean", [(256, 32, 6), (128, 32, 6), (96, 4, 6), (128, 2, 6),
                                      (32, 8, 6), (256, 1, 6), (256, 32, 65)])
def test_norm_long_bodies_share_channels(dev, dtype, C, G, mean):
    B = 600
    rng = np.random.default_rng(C + G + mean)
    rows = rng.integers(0, 2 * mean, size=B)
    tx = C * (2 if dtype == "bf16" else 4) // 16
    held = 16 * ((256 if mean == 6 else 512) // tx)
    lens = [held - 1, held, held + 1, held + 17]
    lens += [k * held + d for k in (2, 4) for d in (-1, 0, 1)]
    at = rng.permutation(B)[:len(lens)]
    rows[at] = lens
    rp = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    n = int(rp[-1])
    S = (rng.standard_normal((n, C)) * 2.0 + rng.standard_normal(C) * 3.0).astype(np.float32)
    S = synth.as_dtype(S, dtype)[1]
    out = torch.full((n + 3, C), float("nan"), dtype=TORCH[dtype], device=dev)
    shc.segment_group_norm(up(S, dtype), up(rp), n, B, G, out)
    got = down(out)
    assert np.all(np.isnan(got[n:]))
    assert_gn_close(got[:n], O.group_norm(S.astype(np.float64), rp, G), dtype,
                    gn_floor(S, rp, G), f"long bodies C={C} G={G} mean={mean}")


@pytest.mark.parametrize("V,n,K", [(40, 1, 1), (200, 63, 9), (200, 64, 9), (300, 65, 5),
                                   (655, 1300, 9)])
def test_transposed_table_blocks(dev, V, n, K):
    rng = np.random.default_rng(V + n + K)
    B = 2
    nbr = np.stack([rng.permutation(V) for _ in range(K)], 1).astype(np.int32)
    if K > 1:
        nbr[rng.random((V, K)) < 0.2] = -1
        nbr[:, 1] = rng.integers(0, V // 2, size=V)      # several senders through one slot
    m = np.zeros(B * V, np.uint8)
    m[rng.permutation(B * V)[:n]] = 1
    m = m.reshape(B, V)
    c = Compaction(m)
    assert c.run() == n
    nbr_t, slot_of, Kt = shc.transpose_neighbors(up(nbr))
    tt = torch.full((Kt * n + 5,), -7, dtype=torch.int32, device=dev)
    rs = torch.full((n + 1,), -7, dtype=torch.int64, device=dev)
    shc.build_transposed_table(c.coords, c.inv, n, B, V, nbr_t, Kt, tt, rs)
    coords, inv, _, _ = O.compact(m)
    tv = down(nbr_t).reshape(-1)[: V * Kt].reshape(V, Kt)
    u = tv[coords[:, 1]]
    r = np.where(u >= 0, inv[coords[:, 0][:, None] * V + np.maximum(u, 0)], -1)
    got = down(tt)
    assert np.array_equal(got[: Kt * n].reshape(Kt, n), r.T) and np.all(got[Kt * n:] == -7)
    bits = ((r >= 0).astype(object) << np.arange(Kt).astype(object)).sum(1)
    have = down(rs)
    assert [int(x) & (2 ** 64 - 1) for x in have[:n]] == [int(b) for b in bits] and have[n] == -7


@pytest.mark.parametrize("incremental", [False, True])
def test_stack_schedules(dev, incremental):
    """The native loop's three-stream schedule (9 batches of 314 K entries, no
    feed) against a serial stack's and the Python loop's, bit for bit, after a
    run short enough for one stream and before one with a feed; step() on a
    serial stack."""
    B, V, K, C = 30, 10475, 9, 32
    rng = np.random.default_rng(5)
    _, nbr = synth.mesh("ellipsoid", V, K, 4)
    masks = [(rng.random((B, V)) < p).astype(np.uint8) for p in (0.05, 0.04)]
    x = synth.as_dtype(rng.standard_normal((B * V, C)).astype(np.float32), "bf16")[1]

    def values(*shape):
        w = rng.standard_normal(shape) / np.sqrt(np.prod(shape[:-1]))
        return synth.as_dtype(w.astype(np.float32).reshape(-1), "bf16")[1].reshape(shape)

    w = synth.Workload("schedules", B, V, K, "bf16", np.zeros((0, 3)), nbr, masks[0], x,
                       [synth.Layer("linear", C, C, values(C, C), None, True),
                        synth.Layer("conv", C, C, values(K, C, C), None, True)],
                       pool=True, scatter=True)
    dm = [up(m.reshape(-1)) for m in masks]

    def drive(st):
        out = []
        for steps, feed in ((2, None), (9, None), (3, lambda k: st.mask.copy_(dm[k % 2])),
                            (8, None), (1, None)):
            n = st.run(steps, feed=feed)
            torch.cuda.synchronize()
            out += [n, st.dense_out.clone(), st.pooled.clone(), st.acts[-1][:n].clone()]
        if st.side is None:
            n = st.step()
            torch.cuda.synchronize()
            assert n == out[-4] and torch.equal(st.dense_out, out[-3])
        return out

    runs = [drive(SparseStack(w, side_stream=side, executor=ex, incremental_scatter=incremental))
            for side, ex in ((True, "native"), (False, "native"), (True, "python"))]
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert a == b if isinstance(a, int) else torch.equal(a, b)


def test_fed_runs_use_the_side_stream_where_it_pays(dev):
    """Fed batches of a stack whose zero-fill scatter writes 257 MB: from 8
    batches a run on, batch k + 1 is fed and compacted on the side stream; a
    shorter run, one with the incremental scatter and one of a small stack stay
    on the stack's own stream.  Outputs equal a serial stack's, batch by batch
    different masks and features."""
    rng = np.random.default_rng(8)

    def workload(B, V, C):
        _, nbr = synth.mesh("ellipsoid", V, 9, 4)
        W = (rng.standard_normal((C, C)) / C ** 0.5).astype(np.float32)
        Wc = (rng.standard_normal((9, C, C)) / (9 * C) ** 0.5).astype(np.float32)
        x = synth.as_dtype(rng.standard_normal((B * V, C)).astype(np.float32), "bf16")[1]
        return synth.Workload("fed", B, V, 9, "bf16", np.zeros((0, 3)), nbr,
                              (rng.random((B, V)) < 0.03).astype(np.uint8), x,
                              [synth.Layer("linear", C, C, synth.as_dtype(W, "bf16")[1], None, True),
                               synth.Layer("conv", C, C, synth.as_dtype(Wc, "bf16")[1], None, True)],
                              pool=True, scatter=True)

    big, small = workload(192, 10475, 64), workload(4, 10475, 64)

    def drive(w, side, incremental, steps):
        st = SparseStack(w, device=dev, side_stream=side, incremental_scatter=incremental)
        masks = [up((np.random.default_rng(k).random(w.B * w.V) < 0.02 + 0.004 * k)
                    .astype(np.uint8)) for k in range(steps)]
        streams = []

        def feed(k):
            streams.append(torch.cuda.current_stream() == st.side)
            st.mask.copy_(masks[k])
            st.x.mul_(-1.0 if k % 3 else 1.0)

        n = st.run(steps, feed=feed)
        torch.cuda.synchronize()
        return streams, (n, st.dense_out, st.pooled, st.acts[-1][:n])

    for w, incremental, steps, on_side in ((big, False, 8, True), (big, False, 9, True),
                                           (big, False, 7, False), (big, True, 9, False),
                                           (small, False, 9, False)):
        streams, got = drive(w, True, incremental, steps)
        assert streams == [False] + [on_side] * (steps - 1)
        _, ref = drive(w, False, incremental, steps)
        assert got[0] == ref[0] and all(torch.equal(a, b) for a, b in zip(got[1:], ref[1:]))
