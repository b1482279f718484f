"""Paged logits at the edges of the kernel's tiles: every head dimension and
group size it takes, token counts around 16, one and several blocks per request,
heads shared out over blocks, skipped tokens, and non-finite operands. The
reference is the same sum in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2607_27090_amd import (IS_DEV_BAD_BLOCK, IS_DEV_SLOT_RANGE, IS_ROPE_HALF_SPLIT,
                                  IS_ROPE_INTERLEAVED, is_paged_scores)

pytestmark = pytest.mark.gpu

THETA = 10000.0


def _setup(nq, Hq, H, D, tokens, P, start, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    blocks = -(-(start + tokens) // P)
    bt = torch.randperm(nq * blocks + 3, generator=torch.Generator().manual_seed(seed))
    bt = bt[:nq * blocks].to(torch.int32).view(nq, blocks).cuda()
    pk = torch.randn(2, (nq * blocks + 3) * P, H, D, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(nq, Hq, D, generator=g, device="cuda").to(torch.bfloat16)
    m = torch.randint(max(0, tokens - 20), tokens + 1, (nq,), generator=g, device="cuda").to(torch.int32)
    m[0] = tokens
    return bt, pk, q, m


def _run(bt, pk, q, m, tokens, P, start, layer, interleaved, num_slots=None):
    nq, Hq, D = q.shape
    sc = torch.full((nq, Hq, tokens), -7.0, device="cuda")
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    qpos = m + start
    is_paged_scores(q, qpos, pk, layer, bt, P, start, m, sc, nq=nq, Hq=Hq, H=pk.shape[2], D=D, L=2,
                    num_slots=pk.shape[1] if num_slots is None else num_slots,
                    max_blocks=bt.shape[1], max_tokens=tokens, rope_theta=THETA,
                    pairing=IS_ROPE_INTERLEAVED if interleaved else IS_ROPE_HALF_SPLIT, status=st)
    torch.cuda.synchronize()
    return sc, int(st)


def _reference(bt, pk, q, m, P, start, layer, interleaved, r):
    nq, Hq, D = q.shape
    H, n = pk.shape[2], int(m[r])
    f = THETA ** (-torch.arange(0, D, 2, dtype=torch.float64, device="cuda") / D)
    a = float(start + n) * f
    c, s = torch.cos(a), torch.sin(a)
    x = q[r].double()
    y = torch.empty_like(x)
    i0 = slice(0, None, 2) if interleaved else slice(0, D // 2)
    i1 = slice(1, None, 2) if interleaved else slice(D // 2, None)
    y[:, i0], y[:, i1] = x[:, i0] * c - x[:, i1] * s, x[:, i1] * c + x[:, i0] * s
    pos = start + torch.arange(n, device="cuda")
    slot = bt[r].long()[pos // P] * P + pos % P
    k = pk[layer][slot].double().repeat_interleave(Hq // H, dim=1)
    return (k * y).sum(-1).t(), (k.abs() * y.abs()).sum(-1).t(), slot


@pytest.mark.parametrize("D,Hq,H", [(16, 6, 2), (32, 5, 1), (32, 8, 8), (64, 24, 3), (64, 40, 5),
                                    (128, 32, 8), (128, 28, 4), (128, 15, 3), (256, 16, 2),
                                    (256, 2, 2), (512, 16, 2), (512, 3, 1)])
@pytest.mark.parametrize("nq,tokens", [(1, 1), (2, 16), (3, 49), (1, 700), (40, 333)])
def test_paged_scores_shapes(D, Hq, H, nq, tokens):
    P, start, interleaved = (16, 5, False) if tokens != 49 else (3, 0, True)
    bt, pk, q, m = _setup(nq, Hq, H, D, tokens, P, start, seed=D + Hq + tokens)
    sc, st = _run(bt, pk, q, m, tokens, P, start, 1, interleaved)
    assert st == 0
    for r in range(nq):
        ref, mag, _ = _reference(bt, pk, q, m, P, start, 1, interleaved, r)
        n = int(m[r])
        # the query's rotation rounds once or twice (2^-23 of the magnitudes),
        # the sum at most D / 32 + 6 times
        tol = (3 + D / 32 + 6) * 2.0 ** -24 * mag
        assert ((sc[r, :, :n].double() - ref).abs() <= tol).all()
        assert (sc[r, :, n:] == -7.0).all()


def test_paged_scores_many_tokens_per_block():
    # more (request, 16 tokens) groups than blocks: several groups per block
    bt, pk, q, m = _setup(64, 8, 2, 64, 2000, 16, 9, seed=3)
    sc, st = _run(bt, pk, q, m, 2000, 16, 9, 0, False)
    assert st == 0
    for r in (0, 31, 63):
        ref, mag, _ = _reference(bt, pk, q, m, 16, 9, 0, False, r)
        assert ((sc[r, :, :int(m[r])].double() - ref).abs() <= 11 * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("nq,tokens,capacity", [
    (200, 2700, 2700),              # past 512 tokens per block: mapped in two parts
    (3, 50, 131_072), (3, 1, 5000), (70, 333, 9000),   # far below the capacity
])
def test_paged_scores_shares(nq, tokens, capacity):
    P, start = 16, 7
    bt, pk, q, m = _setup(nq, 6, 2, 32, tokens, P, start, seed=nq)
    wide = torch.full((nq, -(-(start + capacity) // P)), -1, dtype=torch.int32, device="cuda")
    wide[:, :bt.shape[1]] = bt
    sc, st = _run(wide, pk, q, m, capacity, P, start, 1, False)
    assert st == 0
    for r in {0, 1, nq // 2, nq - 1}:
        ref, mag, _ = _reference(bt, pk, q, m, P, start, 1, False, r)
        n = int(m[r])
        assert ((sc[r, :, :n].double() - ref).abs() <= 10 * 2.0 ** -24 * mag).all()
        assert (sc[r, :, n:] == -7.0).all()


@pytest.mark.parametrize("tokens,capacity,limit", [
    (2560, 131_072, 3.0),  # 10 and 209 us where a block's share followed the capacity
    # 10.7 us and 4.1 in a tight buffer, 2.6 times, where the number of heads per
    # block followed it; 5.8, 1.4 times, now (the blocks of a longer request
    # start and find nothing): half way between the two
    (100, 4096, 2.0),
])
def test_paged_scores_capacity_costs_nothing(tokens, capacity, limit):
    # 4 requests in a buffer for their tokens and in a larger one
    bt, pk, q, m = _setup(4, 32, 32, 32, tokens, 16, 0, seed=5)
    wide = torch.full((4, capacity // 16), -1, dtype=torch.int32, device="cuda")
    wide[:, :bt.shape[1]] = bt

    def us(bt, tokens):
        sc = torch.empty(4, 32, tokens, device="cuda")

        def call():
            is_paged_scores(q, m, pk, 0, bt, 16, 0, m, sc, nq=4, Hq=32, H=32, D=32, L=2,
                            num_slots=pk.shape[1], max_blocks=bt.shape[1], max_tokens=tokens,
                            rope_theta=THETA)

        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                call()
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    tight, loose = us(bt, tokens), us(wide, capacity)
    assert loose < limit * tight, (tight, loose)


def test_paged_scores_skips_bad_tokens_only():
    bt, pk, q, m = _setup(2, 8, 2, 128, 100, 16, 3, seed=4)
    bt[0, 2] = -1
    bt[1, 4] = bt.max() + 50
    sc, st = _run(bt, pk, q, m, 100, 16, 3, 1, False)
    assert st == IS_DEV_BAD_BLOCK | IS_DEV_SLOT_RANGE
    pos = 3 + np.arange(100)
    for r, blk in ((0, 2), (1, 4)):
        bad = torch.from_numpy(pos // 16 == blk).cuda()
        n = int(m[r])
        assert (sc[r][:, bad] == -7.0).all()
        good = ~bad
        good[n:] = False
        safe = bt.clone()
        safe[r, blk] = 0
        ref, mag, _ = _reference(safe, pk, q, m, 16, 3, 1, False, r)
        err = (sc[r, :, :n].double() - ref).abs()
        assert (err <= 13 * 2.0 ** -24 * mag)[:, good[:n]].all()


def test_paged_scores_non_finite_operands():
    # position 0 leaves the query as it is: its lower parts are zero, and a
    # zero part times an infinite key must not turn the logit into NaN
    bt, pk, q, m = _setup(1, 8, 2, 64, 20, 16, 0, seed=6)
    q = q.abs() + 1
    slot = int(bt[0, 0]) * 16
    pk[0, slot + 2, 0, 5] = float("inf")
    pk[0, slot + 3, 1, 6] = float("nan")
    pk[0, slot + 4, 0] = torch.full((64,), 1e-36, dtype=torch.bfloat16)
    q[0, 7, 3] = float("inf")
    sc = torch.zeros(1, 8, 20, device="cuda")
    is_paged_scores(q, torch.zeros(1, dtype=torch.int32, device="cuda"), pk, 0, bt, 16, 0, m, sc,
                    nq=1, Hq=8, H=2, D=64, L=2, num_slots=pk.shape[1], max_blocks=bt.shape[1],
                    max_tokens=20, rope_theta=THETA)
    torch.cuda.synchronize()
    assert torch.isposinf(sc[0, :4, 2]).all()
    assert torch.isnan(sc[0, 4:, 3]).all()
    e = (q[0, :4].double() * pk[0, slot + 4, 0].double()).sum(-1)
    assert ((sc[0, :4, 4].double() - e).abs() <= 64 * 2.0 ** -24 * e).all()
    assert not torch.isfinite(sc[0, 7]).any()
    assert torch.isfinite(sc[0, :4, 5:]).all()


@pytest.mark.parametrize("scale", [1e-38, 1e-36, 1e-33, 1e-29])
@pytest.mark.parametrize("interleaved", [False, True])
def test_paged_scores_tiny_queries(scale, interleaved):
    # a rotated query below 2^-110 does not fit three bf16 parts; keys that make
    # its logits large, ordinary and small, and heads with a few tiny elements
    bt, pk, q, m = _setup(2, 8, 2, 64, 60, 16, 3, seed=11)
    pk[:, :, :, ::5] = (pk[:, :, :, ::5].float() * 1e30).to(torch.bfloat16)
    pk[:, ::3] = (pk[:, ::3].float() * 1e-6).to(torch.bfloat16)
    q[:, :6] = (q[:, :6].float() * scale).to(torch.bfloat16)
    q[:, 6, 5:40] = (q[:, 6, 5:40].float() * scale).to(torch.bfloat16)
    q[:, 7, 9] = 0
    q[:, 5] = 0
    sc, st = _run(bt, pk, q, m, 60, 16, 3, 1, interleaved)
    assert st == 0
    for r in range(2):
        ref, mag, _ = _reference(bt, pk, q, m, 16, 3, 1, interleaved, r)
        err = (sc[r, :, :int(m[r])].double() - ref).abs()
        # (a rotated element below 2^-126 rounds to a multiple of 2^-149)
        kmag = pk.double().abs().max()
        assert (err <= 11 * 2.0 ** -24 * mag + 64 * 2.0 ** -149 * (1 + kmag)).all()


def test_paged_scores_rotated_past_the_largest_bf16():
    # an element between the largest bf16 and the largest fp32 after the rotation
    bt, pk, q, m = _setup(1, 2, 1, 16, 4, 16, 0, seed=12)
    q[:] = 0
    q[0, :, 0], q[0, :, 8] = 2.8e38, 2.0e38
    pk[:] = 0
    pk[0, :, 0, 0], pk[0, :, 0, 8] = 1e-3, 1e-3
    x0, x1 = float(q[0, 0, 0]), float(q[0, 0, 8])
    rotated = {p: (x0 * np.cos(p) - x1 * np.sin(p), x1 * np.cos(p) + x0 * np.sin(p))
               for p in range(1, 4000)}
    best = next(p for p, y in rotated.items() if 3.398e38 < max(abs(y[0]), abs(y[1])) < 3.4026e38)
    qp = torch.tensor([best], dtype=torch.int32, device="cuda")
    sc = torch.zeros(1, 2, 4, device="cuda")
    is_paged_scores(q, qp, pk, 0, bt, 16, 0, m, sc, nq=1, Hq=2, H=1, D=16, L=2,
                    num_slots=pk.shape[1], max_blocks=bt.shape[1], max_tokens=4, rope_theta=THETA)
    torch.cuda.synchronize()
    e = sum(rotated[best]) * float(pk[0, 0, 0, 0])
    got = sc[0, :, :int(m[0])].double()
    assert torch.isfinite(got).all() and ((got - e).abs() <= 2.0 ** -20 * 4e35).all()


@pytest.mark.parametrize("D", [16, 32, 64, 128, 256, 512])
def test_paged_scores_precision(D):
    # against 64 bits no further off than fp32 multiply-adds over eight elements,
    # added pairwise (emulated; the query's rotation rounds in both)
    bt, pk, q, m = _setup(6, 8, 2, D, 640, 16, 0, seed=D)
    sc, st = _run(bt, pk, q, m, 640, 16, 0, 0, False)
    assert st == 0
    off = [0.0, 0.0, 0.0]
    f = THETA ** (-torch.arange(0, D, 2, dtype=torch.float64, device="cuda") / D)
    for r in range(6):
        ref, _, slot = _reference(bt, pk, q, m, 16, 0, 0, False, r)
        n = int(m[r])
        a = (float(n) * f).remainder(2 * np.pi).float()
        c, s, x, h = a.cos(), a.sin(), q[r].float(), D // 2
        y = torch.cat([x[:, :h] * c - x[:, h:] * s, x[:, h:] * c + x[:, :h] * s], -1)
        p = y.view(1, 8, D // 8, 8) * pk[0][slot].float().repeat_interleave(4, 1).view(n, 8, D // 8, 8)
        t = p[..., 0]
        for e in range(1, 8):
            t = t + p[..., e]
        while t.shape[-1] > 1:
            t = t[..., ::2] + t[..., 1::2]
        off[0] += float((sc[r, :, :n].double() - ref).square().sum())
        off[1] += float((t[..., 0].t().double() - ref).square().sum())
        off[2] += float(ref.square().sum())
    ours, theirs = (off[0] / off[2]) ** 0.5, (off[1] / off[2]) ** 0.5
    assert ours <= theirs, (ours, theirs)
