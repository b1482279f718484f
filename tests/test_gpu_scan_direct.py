"""The direct matrix-core scan (several queries on one bank, small and medium
products): edges of its row, query and reduction tiles and of every rule that
picks a tile, both element types, and operands whose three-way bf16 split is not
defined. Every score is checked (k = n) where n allows it. The filtered scan of
larger products follows with the row-sample cases that need many queries."""
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2607_27090_amd import (InferScaleError, is_ann_build, is_ann_build_workspace_size,
                                  is_retrieve, is_retrieve_workspace_size)
from paper_2607_27090_amd.pipeline import RequestBuffers
from tests import parity
from tests.gpu_harness import filtered, host_emb, log, sample_most

pytestmark = pytest.mark.gpu


def _unit(rows, d, g):
    x = torch.randn(rows, d, generator=g, device="cuda")
    return x / x.norm(dim=1, keepdim=True)


def _retrieve(q, bank, k):
    n, d = bank.shape
    buf = RequestBuffers(n=n, d=d, k=k, nq=q.shape[0], emb_dtype=bank.dtype, max_tokens=1)
    buf.retrieve(q, bank)
    torch.cuda.synchronize()
    return buf.ids.cpu().numpy(), buf.scores.cpu().numpy()


def _check(q, bank, k):
    n, d = bank.shape
    gids, gsc = _retrieve(q, bank, k)
    qh, odt = host_emb(q)
    bh, _ = host_emb(bank)
    ids_o, _, s_all = oracle.retrieve(qh, bh, n, d, k, q.shape[0], 0, odt)
    dec = oracle.bf16_to_f64 if odt == oracle.BF16 else (lambda x: x.astype(np.float64))
    near = 0
    for r in range(q.shape[0]):
        near += parity.check_ids(gids[r], ids_o[r], s_all[r], n)
        parity.check_scores(gsc[r], s_all[r][gids[r]],
                            np.abs(dec(bh[gids[r]]) * dec(qh[r])).sum(axis=1))
    return gids, near


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,d,nq", [
    (1, 8, 9), (15, 24, 9), (16, 1032, 16), (17, 1152, 17),   # one fragment and its edges
    (127, 128, 33), (129, 136, 32), (1000, 520, 31),          # ragged steps, ragged queries
    (1023, 64, 257),                                          # several query tiles, 16 x 16
    (6145, 72, 40),                                           # 32 x 16
    (6200, 40, 100),                                          # 32 x 32
    (12289, 104, 65),                                         # 64 x 32, a ragged last tile of one row
    (2049, 1024, 5), (300, 4104, 3),                          # second pass of the row scan
])
def test_direct_scan_shapes(n, d, nq, dt):
    g = torch.Generator(device="cuda").manual_seed(n + d + nq)
    bank, q = _unit(n, d, g).to(dt), _unit(nq, d, g).to(dt)
    _, near = _check(q, bank, min(n, 1024))
    log(f"direct scan n={n} d={d} nq={nq} {dt}: near-tie swaps {near}")


def test_direct_scan_scores_are_no_further_off_than_row_sums():
    # fp32 scores against 64 bits: one rounding of the sum (2^-24) and a little
    g = torch.Generator(device="cuda").manual_seed(5)
    bank, q = _unit(900, 1536, g), _unit(64, 1536, g)
    gids, gsc = _retrieve(q, bank, 900)
    ex = (q.double() @ bank.double().t()).cpu().numpy()
    ex = np.take_along_axis(ex, gids.astype(np.int64), axis=1)
    assert np.linalg.norm(gsc - ex) / np.linalg.norm(ex) < 2.0 ** -24


@pytest.mark.parametrize("n", [40_001, 40_002, 40_003])
def test_dense_tiles_write_rows_of_any_length(n):
    # score rows that are no multiples of 16 bytes, the last one up to its end
    g = torch.Generator(device="cuda").manual_seed(n)
    bank, q = _unit(n, 64, g).bfloat16(), _unit(160, 64, g).bfloat16()
    q[-1] = bank[-1]
    _check(q, bank, 10)


def test_dense_tiles_rows_of_any_length_take_no_longer():
    # 256 queries over 40,000 and 40,001 rows: 29 and 31 us (55 score by score)
    g = torch.Generator(device="cuda").manual_seed(4)
    us = []
    for n in (40_000, 40_001):
        bank, q = _unit(n, 64, g).bfloat16(), _unit(256, 64, g).bfloat16()
        buf = RequestBuffers(n=n, d=64, k=10, nq=256, emb_dtype=bank.dtype, max_tokens=1)
        buf.retrieve(q, bank)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                buf.retrieve(q, bank)
        us.append(_us(graph.replay) / 20)
    log(f"256 x 40,000 / 40,001: {us[0]:.1f} / {us[1]:.1f} us")
    assert us[1] < 1.4 * us[0]


@pytest.mark.parametrize("d", [40, 64, 72, 88, 128])
def test_short_rows_are_no_further_off_than_row_sums(d):
    # one or two steps of few matrix ops; a single query takes the row scan
    g = torch.Generator(device="cuda").manual_seed(d)
    n, nq, k, off = 20_000, 13, 512, [0.0, 0.0]
    for _ in range(4):
        bank, q = _unit(n, d, g).bfloat16(), _unit(nq, d, g).bfloat16()
        ex = (q.double() @ bank.double().t()).cpu().numpy()
        batch = _retrieve(q, bank, k)
        for r in range(nq):
            single = _retrieve(q[r:r + 1], bank, k)
            for i, (ids, sc) in enumerate(((batch[0][r], batch[1][r]), (single[0][0], single[1][0]))):
                off[i] += np.square(sc - ex[r][ids]).sum()
    log(f"d = {d}: {off[0] ** 0.5:.3e}, row sums {off[1] ** 0.5:.3e}")
    assert off[0] <= off[1]


@pytest.mark.parametrize("n,d,nq,dt", [
    (249, 776, 10, torch.float32), (250, 520, 32, torch.float32),     # 4 loads per lane
    (888, 1024, 9, torch.float32),
    (301, 1032, 3, torch.float32), (130, 2048, 9, torch.float32),     # 8
    (90, 2096, 6, torch.float32), (257, 4096, 2, torch.float32),      # 16
    (70, 4104, 5, torch.float32), (208, 8192, 12, torch.float32),     # 32
    (200, 2056, 9, torch.bfloat16), (301, 4096, 2, torch.bfloat16),   # 8 loads per lane
    (90, 4104, 6, torch.bfloat16), (1, 8192, 16, torch.bfloat16),     # 16
])
def test_few_scores_of_long_rows(n, d, nq, dt):
    # one query per block; the 4 (bf16: 8) products of a unit are added in fp32,
    # units in binary64
    g = torch.Generator(device="cuda").manual_seed(n + d)
    bank, q = _unit(n, d, g).to(dt), _unit(nq, d, g).to(dt)
    gids, gsc = _retrieve(q, bank, n)
    a, b = q.double(), bank.double()
    ex, mag = (a @ b.t()).cpu().numpy(), (a.abs() @ b.abs().t()).cpu().numpy()
    off = size = 0.0
    for r in range(nq):
        assert sorted(gids[r].tolist()) == list(range(n)) and (np.diff(gsc[r]) <= 0).all()
        e = ex[r][gids[r]]
        assert (np.abs(gsc[r] - e) <= 2.0 ** -24 * (np.abs(e) + 8 * mag[r][gids[r]])).all()
        off, size = off + np.square(gsc[r] - e).sum(), size + np.square(e).sum()
    # no further off than one rounding of the sum (2^-24) would be at most
    assert np.sqrt(off / size) < 2.0 ** -24


def test_few_scores_of_long_rows_take_no_longer_than_a_step_chain():
    # 250 rows of 8,192 fp32 values, two queries: 28 us on the matrix cores, one
    # step after another over each row, against 9
    g = torch.Generator(device="cuda").manual_seed(3)
    long_rows, short_rows = _unit(250, 8192, g), _unit(250, 512, g)
    us = []
    for bank in (long_rows, short_rows):
        q = bank[:2].contiguous()
        buf = RequestBuffers(n=250, d=bank.shape[1], k=10, nq=2, emb_dtype=bank.dtype, max_tokens=1)
        buf.retrieve(q, bank)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                buf.retrieve(q, bank)
        us.append(_us(graph.replay) / 20)
    log(f"250 x 2, d = 8,192 / 512: {us[0]:.1f} / {us[1]:.1f} us")
    assert us[0] < 2.2 * us[1]


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_direct_scan_non_finite_operands(dt):
    g = torch.Generator(device="cuda").manual_seed(8)
    n, d, nq = 70, 136, 19
    bank, q = _unit(n, d, g), _unit(nq, d, g)
    bank[3, 5] = float("inf")
    bank[4] = float("nan")
    bank[6, 7], bank[6, 100] = -float("inf"), float("inf")
    bank[9, 3] = 3.0e38
    bank[20] *= 1e-36       # the lower parts fall below the smallest bf16
    q[1, 5] = 0.0            # 0 * inf
    q[2, 9] = float("inf")
    q[4, 3] = 1.0            # an operand whose lower parts are zero
    q[5, 3] = 100.0          # overflows with row 9
    bank, q = bank.to(dt), q.to(dt)
    gids, gsc = _retrieve(q, bank, n)
    ex = (q.double() @ bank.double().t()).float().cpu().numpy()
    for r in range(nq):
        assert sorted(gids[r].tolist()) == list(range(n))
        e, s = ex[r][gids[r]], gsc[r]
        np.testing.assert_array_equal(np.isnan(s), np.isnan(e))
        inf = np.isinf(e)
        np.testing.assert_array_equal(s[inf], e[inf])
        fin = np.isfinite(e)
        mag = (q[r].double().abs() * bank.double().abs()).sum(1).cpu().numpy()[gids[r]]
        assert (np.abs(s[fin].astype(np.float64) - e[fin]) <= 2.0 ** -20 * mag[fin]).all()


@pytest.mark.parametrize("small,large", [
    (1.2345e-36, 1e35), (1.2e-38, 1e35), (3e-41, 1e38), (1e-36, 1.0), (1e-31, 1e30), (1e-29, 1e28)])
@pytest.mark.parametrize("swap", [False, True])
def test_direct_scan_tiny_operands(small, large, swap):
    # operands whose lower bf16 parts are cut short or lost, against large ones:
    # what is lost then counts. Rows 0 to 9 hold tiny values only, 10 to 19 a few
    # among ordinary ones, 20 is zero. fp32 products of d terms: d roundings.
    g = torch.Generator(device="cuda").manual_seed(9)
    n, d, nq = 70, 72, 19
    a, b = torch.rand(n, d, generator=g, device="cuda") + 1, torch.rand(nq, d, generator=g, device="cuda") + 1
    a[:10] *= small
    a[10:20, 3:7] *= small
    a[10:20, 7:] = 0
    a[20] = 0
    b *= large
    if swap:
        a, b, n, nq = b, a, nq, n
    gids, gsc = _retrieve(b, a, n)
    p = b.double().cpu().numpy()[:, None, :] * a.double().cpu().numpy()[None, :, :]
    ids = gids.astype(np.int64)
    e = np.take_along_axis(p.sum(-1), ids, axis=1)
    mag = np.take_along_axis(np.abs(p).sum(-1), ids, axis=1)
    fin = e <= 3.4e38
    assert (np.abs(gsc[fin].astype(np.float64) - e[fin]) <= d * 2.0 ** -24 * mag[fin] + d * 2.0 ** -149).all()


@pytest.mark.parametrize("n,d,nq,k", [
    (16_385, 16, 9, 100),       # 32-row tiles: 513 maxima, one per thread; a last tile of one row
    (20_011, 72, 64, 50),       # 64-row tiles
    (100_003, 16, 8, 1024),     # 3,126 maxima, four per thread; the largest k
    (300_001, 8, 5, 64),        # 9,376 maxima, sixteen per thread
    (16_500, 8, 9, 515),        # tiles two per result: 516 x 32 rows
    (600_000, 8, 3, 7),         # more tiles than one block takes: chunk winners
    (40_000, 16, 5, 520),       # more results than are ranked pairwise
    (300_001, 16, 5, 1000),     # nearly one result per thread: the tiles are ranked first
])
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_select_from_tile_maxima(n, d, nq, k, dt):
    # small-integer operands: scores are exact, with many ties, so the ids must
    # equal a stable sort's
    g = torch.Generator(device="cuda").manual_seed(n + k)
    bank = torch.randint(-8, 9, (n, d), generator=g, device="cuda").to(dt)
    q = torch.randint(-8, 9, (nq, d), generator=g, device="cuda").to(dt)
    q[0] = 0                                    # every score ties
    q[1] = -q[1].abs()
    bank[:, 0] = bank[:, 0].abs() + 20          # query 2: one sign only
    q[2] = 0
    q[2, 0] = -1
    bank[n // 2, :] = 64                        # a tile with the best row of many queries
    gids, gsc = _retrieve(q, bank, k)
    s = q.double() @ bank.double().t()
    o = torch.sort(s, dim=1, descending=True, stable=True)
    np.testing.assert_array_equal(gids, o.indices[:, :k].cpu().numpy())
    np.testing.assert_array_equal(gsc, o.values[:, :k].float().cpu().numpy())


def test_select_from_tile_maxima_with_nan_scores():
    # NaN ranks lowest: tiles that hold nothing else have the lowest maximum,
    # and with fewer than k numbers the NaN rows fill up in id order
    g = torch.Generator(device="cuda").manual_seed(12)
    n, d, nq, k = 17_000, 136, 12, 60
    bank, q = _unit(n, d, g), _unit(nq, d, g)
    bank[40:] = float("nan")
    gids, gsc = _retrieve(q, bank, k)
    s = (q.double() @ bank[:40].double().t()).cpu().numpy()
    for r in range(nq):
        assert set(gids[r, :40].tolist()) == set(range(40))
        assert (np.diff(s[r][gids[r, :40]]) <= 1e-6).all()
        assert gids[r, 40:].tolist() == list(range(40, 60)) and np.isnan(gsc[r, 40:]).all()


def _us(call):
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 100)
    return min(times)


def test_ranking_does_not_walk_whole_rows():
    # one workgroup ranks a query: with more results than it ranks pairwise, or
    # more equal scores, it must not go through all 300,000 scores by itself
    # (1,800 and 360 us against 33 where it did)
    g = torch.Generator(device="cuda").manual_seed(31)
    n, d, nq = 300_000, 64, 8
    bank, q = _unit(n, d, g).to(torch.bfloat16), _unit(nq, d, g).to(torch.bfloat16)

    def us(k, q):
        buf = RequestBuffers(n=n, d=d, k=k, nq=nq, emb_dtype=bank.dtype, max_tokens=1)
        return _us(lambda: buf.retrieve(q, bank))

    plain = us(100, q)
    tied = q.clone()
    tied[3] = 0
    times = {"600 results": us(600, q), "1,024 results": us(1024, q), "a zero query": us(100, tied)}
    log(f"100 results {plain:.1f} us, " + ", ".join(f"{a} {b:.1f}" for a, b in times.items()))
    assert times["a zero query"] < 3 * plain
    assert times["600 results"] < 4 * plain and times["1,024 results"] < 8 * plain


@pytest.mark.parametrize("n,nq", [(70_000, 300), (140_000, 200)])
def test_filtered_scan_every_row_survives_many_queries(n, nq):
    # row sample (of one or two select chunks), then the filter; the rows after
    # the sample all equal query 0, so its survivor regions fill to capacity and
    # its ties go to the lower ids
    g = torch.Generator(device="cuda").manual_seed(n)
    d, k, S = 72, 50, sample_most(n)
    assert filtered(n, nq)
    bank, q = _unit(n, d, g).to(torch.bfloat16), _unit(nq, d, g).to(torch.bfloat16)
    v = bank[7].clone()
    bank[S:] = v
    q[0] = v
    gids, near = _check(q, bank, k)
    assert gids[0][0] == 7 and list(gids[0][1:]) == list(range(S, S + k - 1))
    log(f"filtered scan n={n}, all rows survive for one query: near-tie swaps {near}")


def _integers(rows, d, g, dt):
    return torch.randint(-8, 9, (rows, d), generator=g, device="cuda").to(dt)


def _asked(call):
    """Workspace bytes a call asks for at least, from its refusal."""
    with pytest.raises(InferScaleError) as e:
        call(torch.empty(256, dtype=torch.uint8, device="cuda"))
    return int(re.search(r"needs (\d+) bytes", str(e.value))[1])


@pytest.mark.parametrize("n,d,nq,k,dt", [
    (20_000, 72, 40, 30, torch.float32),       # chunk winners instead of tile maxima
    (30_000, 72, 300, 50, torch.bfloat16),     # the same after the block-staged scan
    (40_000, 72, 2000, 20, torch.bfloat16),    # filtered: the larger row sample; small ranking blocks
    (140_000, 72, 100, 700, torch.bfloat16),   # filtered, a sample ranked by its chunks' winners
    (400_000, 72, 40, 100, torch.bfloat16),    # filtered
])
def test_smaller_workspaces_give_the_same(n, d, nq, k, dt):
    # small-integer operands: exact scores with many ties, so any path must rank
    # as a stable sort does
    g = torch.Generator(device="cuda").manual_seed(n)
    bank, q = _integers(n, d, g, dt), _integers(nq, d, g, dt)
    ids = torch.empty(nq, k, dtype=torch.int32, device="cuda")
    sc = torch.empty(nq, k, device="cuda")

    def call(ws):
        is_retrieve(q, bank, n, d, k, ids, sc, nq=nq, workspace=ws)
        torch.cuda.synchronize()

    want = is_retrieve_workspace_size(n, d, k, nq, 0 if dt == torch.float32 else 1)
    least = _asked(call)
    assert least <= want
    s = q.double() @ bank.double().t()
    o = torch.sort(s, dim=1, descending=True, stable=True)
    for size in (want, least):
        ids.fill_(-1)
        call(torch.empty(size, dtype=torch.uint8, device="cuda"))
        assert torch.equal(ids.long(), o.indices[:, :k]), size
        assert torch.equal(sc.double(), o.values[:, :k])


@pytest.mark.parametrize("n,d,nq", [(70_000, 768, 300), (140_000, 1024, 100), (400_000, 768, 40)])
def test_filtered_scan_scores_equal_rows_equally(n, d, nq):
    # each of 40 queries is a row of the sample that also stands among the rows
    # after it: both copies score the same bits and the lower id comes first,
    # also with k = 1, where the copy is dropped, and with the least workspace
    g = torch.Generator(device="cuda").manual_seed(d + nq)
    bank, q = _unit(n, d, g).to(torch.bfloat16), _unit(nq, d, g).to(torch.bfloat16)
    first = torch.arange(40, device="cuda")
    bank[n - 50 + first] = bank[first]
    q[:40] = bank[first]
    assert filtered(n, nq)
    for k in (50, 1):
        ids = torch.empty(nq, k, dtype=torch.int32, device="cuda")
        sc = torch.empty(nq, k, device="cuda")

        def call(ws):
            is_retrieve(q, bank, n, d, k, ids, sc, nq=nq, workspace=ws)
            torch.cuda.synchronize()

        results = []
        for size in (is_retrieve_workspace_size(n, d, k, nq, 1), _asked(call)):
            call(torch.empty(size, dtype=torch.uint8, device="cuda"))
            results.append((ids.clone(), sc.clone()))
            assert torch.equal(ids[:40, 0].long(), first)
            if k > 1:
                assert torch.equal(ids[:40, 1].long(), n - 50 + first)
                assert torch.equal(sc[:40, 0], sc[:40, 1])
        assert torch.equal(results[0][0], results[1][0])
        assert torch.equal(results[0][1], results[1][1])


@pytest.mark.parametrize("n,R", [(1500, 20), (7000, 64), (40_000, 64)])
def test_build_batches_give_the_same_graph(n, R):
    # batches of 1,024, of 512 and (the least workspace) of 256 rows; the last
    # batch is ragged in each
    g = torch.Generator(device="cuda").manual_seed(n)
    d = 64
    bank = _integers(n, d, g, torch.bfloat16)

    def call(ws):
        out = torch.full((n, R), -1, dtype=torch.int32, device="cuda")
        is_ann_build(bank, n, d, R, out, workspace=ws)
        torch.cuda.synchronize()
        return out

    want = is_ann_build_workspace_size(n, d, R, 1)
    least = _asked(call)
    first = call(torch.empty(want, dtype=torch.uint8, device="cuda"))
    for size in (want - 256, least):
        assert torch.equal(call(torch.empty(size, dtype=torch.uint8, device="cuda")), first)
    s = (bank[:3].double() @ bank.double().t())
    for i in range(3):
        s[i, i] = -float("inf")
        f = torch.sort(s[i], descending=True, stable=True).indices[:R // 2]
        assert torch.equal(first[i, :R // 2].long(), f)


@pytest.mark.parametrize("n,d,dt", [
    (700, 768, torch.bfloat16),      # 256 rows: tiles of 16 x 16, their sums in eight parts
    (1300, 200, torch.float32),      # last batches of 20 and 276 rows
    (7000, 768, torch.bfloat16),     # 1,024 rows would be past the direct scan's bound
    (33_044, 264, torch.bfloat16),   # filtered; last batches of 20 and 276 rows
])
def test_build_does_not_depend_on_the_workspace(n, d, dt):
    # real-valued rows: every batch size scores a row in the same order of sums,
    # so the graph is the same bit for bit; rows that stand twice tie exactly
    g = torch.Generator(device="cuda").manual_seed(n)
    R = 48
    bank = _unit(n, d, g).to(dt)
    bank[n // 2:n // 2 + 200] = bank[:200]

    def call(ws):
        out = torch.full((n, R), -1, dtype=torch.int32, device="cuda")
        is_ann_build(bank, n, d, R, out, workspace=ws)
        torch.cuda.synchronize()
        return out

    want = is_ann_build_workspace_size(n, d, R, 0 if dt == torch.float32 else 1)
    first = call(torch.empty(want, dtype=torch.uint8, device="cuda"))
    for size in (want - 256, _asked(call)):
        assert torch.equal(call(torch.empty(size, dtype=torch.uint8, device="cuda")), first)
    assert torch.equal(first[:200, 0].long(), n // 2 + torch.arange(200, device="cuda"))


@pytest.mark.parametrize("n,d,nq,dt", [(60, 4104, 1, torch.float32), (60, 8192, 1, torch.float32),
                                       (60, 8192, 3, torch.float32), (60, 8192, 1, torch.bfloat16)])
def test_longest_rows(n, d, nq, dt):
    # one query: the row scan's longest rows (32 loads per lane); a result is
    # off by more than half of its size if a row's second half is left out
    g = torch.Generator(device="cuda").manual_seed(d)
    _check(_unit(nq, d, g).to(dt), _unit(n, d, g).to(dt), n)
