"""Ranges of buckets that begin at any 16 bytes: launches step back to whole cache lines there, and what stands in
front of the range in its first tile belongs to somebody else.  One call per bucket, the last bucket first, in every
form of a round; against the oracle over ALL buckets, so that a store in front of a range shows up."""
import numpy as np
import pytest
import torch

from harness import Pair
from oracle import eager_oracle as eo
from workloads import grads as wg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_04207_amd import binding
    return binding


def _layout(numel, align):
    off, cur = [], 0
    for n in numel:
        off.append(cur)
        cur = (cur + n + align - 1) // align * align
    return off, cur


# shorter and longer than what is stepped back for; ends in the first tile, at the end of one, behind it; the buckets
# between begin at every multiple of 4 (8) elements in turn
SMALL = [1024, 12, 1023, 1028, 8, 1080, 20, 1025, 60, 3001, 4, 1276, 44, 20_003, 40, 70_007, 36, 1024, 133_001, 5]


def _check_sums(raw, pair, w_before):
    got = raw.cpu().numpy().reshape(-1, 4)
    want = eo.bucket_stats(pair.oracle_recv, w_before, pair.offset, pair.numel)
    # 64-bit sums in another order: 1e-10 is what the statistics promise
    np.testing.assert_allclose(got[:, 0], [x[0] for x in want], rtol=1e-10)
    np.testing.assert_allclose(got[:, 1], [x[1] for x in want], rtol=1e-10)
    assert got[:, 2].copy().view(np.uint64).tolist() == [x[2] for x in want]


def _by_layer(eb, pair, masks, raw=None):
    host = pair.set_grads([wg.fill(torch.empty(pair.arena, dtype=pair.dtype), pair.seed, 0, p, pair.gs)
                           for p in range(pair.P)])
    nb = len(pair.numel)
    for t, mask in enumerate(masks):
        plan = eb.make_plan(eb.MAJORITY, pair.P, t, mask)
        w_before = pair.oracle.w.copy()
        for b in range(nb - 1, -1, -1):
            pair.round(plan, host, b, b + 1, fused=t % 3 != 2, want_recv=True)
            if b == nb // 2:                      # those in front have not been touched
                pair.compare(exact=True, check_recv=t > 0, what=f"round {t}, from bucket {b}")
        if raw is not None:
            _check_sums(raw, pair, w_before if t % 3 != 2 else None)
        if t % 3 == 2:
            for b in range(nb):
                pair.sgd(b, b + 1)
        pair.compare(exact=True, check_recv=True, what=f"round {t}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P,chunk,stats", [(3, 0, False), (9, 0, False), (9, 16, False), (20, 0, False), (3, 0, True),
                                           (12, 0, True)])
def test_small_ranges(eb, dtype, P, chunk, stats):
    off, n = _layout(SMALL, 8 if dtype == "bf16" else 4)
    pair = Pair(eb, P, off, SMALL, n, dtype, 0, seed=P)
    pair.ctx.eager_set_launch("chunk", chunk)
    raw = None
    if stats:
        raw = torch.full((len(SMALL) * 4,), -1.0, dtype=torch.float64, device="cuda")
        need = pair.ctx.eager_stats_workspace_bytes()
        ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
        pair.ctx.eager_stats_attach(raw, ws, need)
    everyone = (1 << P) - 1
    _by_layer(eb, pair, [1, everyone & ~2, 0b101, everyone], raw)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("split", [1, 2])
@pytest.mark.parametrize("stats", [False, True])
def test_streamed_ranges(eb, dtype, split, stats):
    """Runs that move more than 112 MiB (bursts), with the copies inside and as a launch of their own."""
    numel = [12, 2_600_003, 100, 2_600_012, 20, 2_599_999]
    off, n = _layout(numel, 8 if dtype == "bf16" else 4)
    pair = Pair(eb, 9, off, numel, n, dtype, 0, seed=4)
    pair.ctx.eager_set_launch("split", split)
    raw = None
    if stats:
        raw = torch.full((len(numel) * 4,), -1.0, dtype=torch.float64, device="cuda")
        need = pair.ctx.eager_stats_workspace_bytes()
        ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
        pair.ctx.eager_stats_attach(raw, ws, need)
    _by_layer(eb, pair, [0b000000111, 0b111000000, 0b101010101], raw)


def test_runs_of_buckets_with_norms(eb):
    """Several buckets to a run that begins inside a tile, so that the run's first bucket is not the one in front."""
    numel = [1000, 300, 24, 77, 5000, 260, 8, 40_001]
    off, n = _layout(numel, 4)
    pair = Pair(eb, 4, off, numel, n, "f32", 0, seed=8)
    raw = torch.zeros(len(numel) * 4, dtype=torch.float64, device="cuda")
    need = pair.ctx.eager_stats_workspace_bytes()
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device="cuda")
    pair.ctx.eager_stats_attach(raw, ws, need)
    host = pair.set_grads([wg.fill(torch.empty(n), 8, 0, p, 1e-3) for p in range(4)])
    w_before = pair.oracle.w.copy()
    for b0, b1 in ((2, 8), (1, 2), (0, 1)):
        pair.round(eb.make_plan(eb.SOLO, 4, 0, 0b0110), host, b0, b1, want_recv=True)
        pair.compare(exact=True, what=f"buckets {b0}..{b1}")
    _check_sums(raw, pair, w_before)
