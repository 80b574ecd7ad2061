"""The two forms of a round - everything at once for small runs, bursts for large ones - at the
sizes where each can go wrong: edges of tiles, ragged tails, one element, both sides of the line
between them, slot lists of odd length and without any slot; against the oracle, bit for bit in
fixed order.  (The line: a run that moves 96 MiB, 4 bytes per slot and copy side and 16 for w, v.)
"""
import numpy as np
import pytest
import torch

from harness import Pair
from workloads import grads as wg

pytestmark = pytest.mark.gpu

LINE = 96 << 20


@pytest.fixture(scope="module")
def eb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_04207_amd import binding
    return binding


def _rounds(eb, pair, masks, order, n):
    """Rounds with the given masks, fused and unfused, then a flush of what is pending."""
    grads = [wg.fill(torch.empty(pair.arena, dtype=pair.dtype), pair.seed, 0, p, pair.gs)
             for p in range(pair.P)]
    host = pair.set_grads(grads)
    for t, mask in enumerate(masks):
        plan = eb.make_plan(eb.MAJORITY, pair.P, t, mask)
        fused = t % 3 != 2
        pair.round(plan, host, fused=fused, want_recv=True)
        if not fused:
            pair.sgd()
    pair.flush()
    pair.compare(exact=order == eb.ORDER_FIXED, check_recv=True, what=f"{n} elements")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("order", [0, 1])
def test_small_runs_at_tile_edges(eb, dtype, order):
    align = 8 if dtype == "bf16" else 4
    for n in (1, 3, 4, 5, 7, 8, 9, 252, 255, 256, 257, 263, 264, 511, 512, 517, 16389):
        pair = Pair(eb, 5, [0], [n], (n + align - 1) // align * align, dtype, order, seed=n)
        # 5 slots; 4 slots and 1 copy; everybody late but one with 8 slots; pairs; all on time
        _rounds(eb, pair, [0b11111, 0b01111, 0b00001, 0b10110, 0b01001, 0b11111], order, n)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("off", [-1, 0, 1, 3, 255, 258])
def test_both_sides_of_the_line_between_the_forms(eb, dtype, off):
    align = 8 if dtype == "bf16" else 4
    # mask 0b011 of 3 with nothing pending: 2 slots, 1 copy, w and v read and written
    n = LINE // (4 * (2 + 2 + 4)) + off
    pair = Pair(eb, 3, [0], [n], (n + align - 1) // align * align, dtype, 0, seed=5)
    _rounds(eb, pair, [0b011, 0b110, 0b111], 0, n)


@pytest.mark.parametrize("P,n", [(64, 70_003), (33, 400_009), (9, 1_500_007)])
def test_many_slots_and_copies(eb, P, n):
    """Long slot lists in both forms: 64 pairs, 63 copies, odd counts, nobody pending."""
    pair = Pair(eb, P, [0], [n], (n + 3) // 4 * 4, "f32", 0, seed=P)
    everyone = (1 << P) - 1
    _rounds(eb, pair, [1, everyone, 1 << (P - 1), everyone & ~2, everyone], 0, n)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_statistics_of_a_streamed_round(eb, dtype):
    """By-products in the burst form, buckets that begin and end anywhere in a tile."""
    num = [1, 255, 7, 1_000_003, 64, 4096, 2_000_001, 129, 300_000]
    off, cur = [], 0
    for m in num:
        off.append(cur)
        cur = (cur + m + 7) // 8 * 8
    P = 4
    pair = Pair(eb, P, off, num, cur, dtype, 0, seed=8)
    stats = torch.zeros(len(num) * 32, dtype=torch.uint8, device="cuda:0")
    need = pair.ctx.eager_stats_workspace_bytes()
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    pair.ctx.eager_stats_attach(stats, ws, need)
    grads = [wg.fill(torch.empty(cur, dtype=pair.dtype), 8, 0, p, pair.gs) for p in range(P)]
    grads[1][off[3] + 777] = float("inf")
    host = pair.set_grads(grads)
    for t, mask in enumerate((0b0111, 0b1110)):
        w_before = pair.oracle.w.copy()
        pair.round(eb.make_plan(eb.MAJORITY, P, t, mask), host, want_recv=True)
        torch.cuda.synchronize()
        got = stats.view(torch.float64).view(-1, 4)[:, :2].cpu().numpy()
        bad = stats.view(torch.int64).view(-1, 4)[:, 2].cpu().numpy()
        for b, (o, m) in enumerate(zip(off, num)):
            u = pair.oracle_recv[o:o + m].astype(np.float64)
            w = w_before[o:o + m].astype(np.float64)
            fine = np.isfinite(u)
            assert bad[b] == np.count_nonzero(~fine), (t, b)
            # 64-bit sums in another order: 1e-10 is what the statistics promise
            assert np.isclose(got[b, 0], np.sum(u[fine] ** 2), rtol=1e-10, atol=0), (t, b)
            assert np.isclose(got[b, 1], np.sum(w[np.isfinite(w)] ** 2), rtol=1e-10, atol=0), (t, b)
