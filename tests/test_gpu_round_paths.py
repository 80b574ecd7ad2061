"""The two forms of a round - everything at once for small runs, bursts for large ones - at the
sizes where each can go wrong: edges of tiles, ragged tails, one element, both sides of the line
between them, slot lists of odd length and without any slot; against the oracle, bit for bit in
fixed order.  (The line: a run that moves 112 MiB, gradients counted by their type, 4 bytes for a send
buffer read or written, 16 for w and v.)
"""
import numpy as np
import pytest
import torch

from harness import Pair
from workloads import grads as wg

pytestmark = pytest.mark.gpu

LINE = 112 << 20


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
    n = LINE // (26 if dtype == "bf16" else 32) + off
    pair = Pair(eb, 3, [0], [n], (n + align - 1) // align * align, dtype, 0, seed=5)
    _rounds(eb, pair, [0b011, 0b110, 0b111], 0, n)


@pytest.mark.parametrize("P,n", [(64, 70_003), (33, 400_009), (9, 1_500_007)])
def test_many_slots_and_copies(eb, P, n):
    """Long slot lists in both forms: 64 pairs, 63 copies, odd counts, nobody pending."""
    pair = Pair(eb, P, [0], [n], (n + 3) // 4 * 4, "f32", 0, seed=P)
    everyone = (1 << P) - 1
    _rounds(eb, pair, [1, everyone, 1 << (P - 1), everyone & ~2, everyone], 0, n)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P,n", [(9, 1), (9, 63), (17, 65), (17, 4099), (40, 257), (9, 131_072), (12, 131_073)])
def test_one_element_to_a_lane(eb, dtype, P, n):
    """Very small runs of many slots, up to 131072 elements one to a lane; pairs across the 8, 16 and 32 slots
    that are in flight together (process 0 is on time with nothing pending, then everybody is late but it)."""
    pair = Pair(eb, P, [0], [n], (n + 7) // 8 * 8, dtype, 0, seed=P + n)
    everyone = (1 << P) - 1
    _rounds(eb, pair, [1, everyone, 0b101, everyone & ~1, everyone], 0, n)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("n", [3, 64, 257, 4099, 131_072, 131_081, 262_147])
def test_short_lists_of_every_length(eb, dtype, order, n):
    """1 to 16 streams, one element to a lane and four: 16 as 8 pairs, 15 with 7 copies, copies behind a sum of one slot
    and behind one of nine, exactly 8."""
    pair = Pair(eb, 8, [0], [n], (n + 7) // 8 * 8, dtype, order, seed=n % 89)
    _rounds(eb, pair, [1, 255, 1, 2, 255, 0b1111, 255 & ~0b11, 0b10101010, 255, 0b11111110], order, n)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("form,P,n", [
    ("short, 8 streams", 4, 523), ("short, 16 streams, one element to a lane", 9, 523),
    ("short, 16 streams, four", 8, 131_072 + 523), ("long, one element to a lane", 17, 523),
    ("chunks of 8", 9, 523), ("chunks of 16", 9, 523), ("bursts", 4, 0)])
def test_signed_zeros_and_infinities_in_every_form(eb, dtype, form, P, n):
    """Late, late again with a pending buffer, on time with one (a pair), everybody on time: gradients, pending
    buffers, parameters and momentum of -0.0, and infinities and NaN that meet in a sum, a pair or not at all, bit
    for bit in fixed order - with branches (short_kernel with up to 8 and up to 16 streams, chunk_kernel with longer
    lists and where a launch option asks for it, one element to a lane and four) and with the masks of burst_kernel,
    where what is masked out is +0.0.  In the ragged tail too."""
    # every mask moves at least all gradients, w and v, the latter two read and written
    per = P * (2 if dtype == "bf16" else 4) + 16
    n = n or LINE // per + 303
    assert (n * per > LINE) == (form == "bursts")
    pair = Pair(eb, P, [0], [n], (n + 7) // 8 * 8, dtype, 0, seed=6)
    if form.startswith("chunks"):
        pair.ctx.eager_set_launch("chunk", int(form.split()[-1]))
    neg = torch.full((pair.arena,), -0.0, dtype=pair.dtype)
    mixed = neg.clone()
    mixed[::3] = 0.0
    mixed[1::7] = -1e-3
    mixed[5::11] = 1e-3
    for t, start in ((pair.w, 0), (pair.v, 32)):
        t[start:start + 64] = -0.0
        t[n - 40:] = -0.0
    pair.oracle.w[:] = pair.w.cpu().numpy()
    pair.oracle.v[:] = pair.v.cpu().numpy()
    inf, everyone = float("inf"), (1 << P) - 1
    at = [200, 257, n - 2]                               # first tile, second tile, ragged tail
    for t, mask in enumerate([everyone & ~2, everyone & ~6, 0b1010, everyone, 1, everyone & ~1, everyone]):
        g = [(neg if (t + p) % 2 == 0 else mixed).clone() for p in range(P)]
        for k in at:
            g[t % P][k] = inf                            # alone; it may be pending for a while
            g[1][k + 1], g[2][k + 1] = inf, -inf         # two that meet, in one round or in two
        g[0][210 + t] = float("nan")
        pair.round(eb.make_plan(eb.SOLO, P, t, mask), pair.set_grads(g), want_recv=True)
        pair.compare(exact=True, check_recv=True, what=f"{form}, round {t}, mask {mask:#b}")
    assert np.signbit(pair.oracle_recv[pair.oracle_recv == 0.0]).sum() == 0
    assert np.isnan(pair.oracle.w[[210, at[1] + 1]]).all() and np.isfinite(pair.oracle.w[:200]).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [700_003, 1_048_576, 16 * 65536 + 5, 20 * 65536, 20 * 65536 + 1])
def test_stores_of_copies_one_at_a_time(eb, dtype, n):
    """Runs of 56 to 112 MiB with many copies, on both sides of the number of elements up to which all wavefronts are
    resident (16 or 20 tiles per CU): 7, 6 and 5 of 8 late, fused and into the receive buffer."""
    pair = Pair(eb, 8, [0], [n], (n + 7) // 8 * 8, dtype, 0, seed=n % 97)
    _rounds(eb, pair, [0b00000001, 0b00010000, 0b01000001, 0b10000000, 0b00110001, 0b00000010], 0, n)


def test_a_run_longer_than_one_launch_of_chunks(eb):
    """Beyond 2^29 elements chunk_kernel goes over a run in several launches: element by element against torch,
    and the statistics of both."""
    n = (1 << 29) + 1027
    if torch.cuda.mem_get_info()[0] < 30 * n:
        pytest.skip("needs 16 GB of free device memory")
    dev = torch.device("cuda:0")
    ctx = eb.Context(2, [0], [n])
    ctx.eager_set_launch("chunk", 16)
    G = [torch.empty(n, device=dev).normal_() for _ in range(2)]
    unread = torch.zeros(4, device=dev)
    recv = torch.full((n + 1,), -1.0, device=dev)
    stats = torch.zeros(32, dtype=torch.uint8, device=dev)
    need = ctx.eager_stats_workspace_bytes()
    workspace = torch.empty(need, dtype=torch.uint8, device=dev)     # (the caller's as long as it is attached)
    ctx.eager_stats_attach(stats, workspace, need)
    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, 2, 0, 0b11), G, [unread, unread], recv=recv)
    torch.cuda.synchronize()
    want = G[0].add_(G[1]).mul_(0.5)
    assert torch.equal(recv[:n], want) and recv[n].item() == -1.0
    total = sum(float((x.double() ** 2).sum()) for x in want.split(1 << 27))
    assert abs(float(stats.view(torch.float64)[0]) - total) <= 1e-10 * total
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P,n", [(3, 90_003), (4, 300_003), (6, 60_001), (8, 300_007), (32, 50_001), (64, 140_001)])
@pytest.mark.parametrize("pending", ["every second", "all but one", "first half"])
def test_any_order_is_no_further_from_the_sum(eb, dtype, P, n, pending):
    """A small round in fast order with pending buffers: no further from the sum in 64 bits than two sums in 32 bits
    that take the streams in turn, send buffer before gradient, nor than one sum of pairs of neighbours.  (With fp32
    gradients the three differ by up to 0.7 % either way, and that of n elements by less than 1 %: 2 %.)"""
    dev, tdt = torch.device("cuda:0"), torch.bfloat16 if dtype == "bf16" else torch.float32
    G = [wg.fill(torch.empty(n, dtype=tdt), 9, 0, p, 1e-3).to(dev) for p in range(P)]
    R = [wg.fill(torch.empty(n), 9, 1, p, 1e-3).to(dev) for p in range(P)]
    ctx = eb.Context(P, [0], [n], eb.BF16 if dtype == "bf16" else eb.F32, eb.ORDER_FAST)
    late = [p for p in range(P) if {"every second": p % 2 == 0, "all but one": p != 1, "first half": p < P // 2}[pending]]
    ctx.eager_set_valid(0, sum(1 << p for p in late))
    recv = torch.empty(n, device=dev)
    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, P, 0, (1 << P) - 1), G, R, recv=recv)
    streams = [x for p in range(P) for x in ([R[p]] if p in late else []) + [G[p]]]
    part = [torch.zeros(n, device=dev) for _ in range(3)]
    for k, x in enumerate(streams):
        part[k % 2] += x.float()
    for k in range(0, len(streams), 2):
        part[2] += streams[k].float() + streams[k + 1].float() if k + 1 < len(streams) else streams[k].float()
    exact = sum(x.double() for x in streams) / P
    error = lambda x: float((x.double() - exact).square().mean().sqrt())          # noqa: E731
    inv = torch.tensor(1.0 / P, device=dev)
    assert error(recv) <= 1.02 * min(error((part[0] + part[1]) * inv), error(part[2] * inv))
    ctx.close()


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


@pytest.mark.parametrize("num", [
    [2048 * 3, 100, 2047, 2049, 5, 256, 2048],            # groups of 8 tiles begin and end everywhere
    [3], [255, 4096, 1], [2048 * 40 + 3, 1_400_001, 9],
    [13_000_001, 40, 2_000_000]])                         # enough records for slices
def test_layerwise_norms_by_groups_of_tiles(eb, num):
    """Norms, rates and the layer-wise step over buckets that begin and end anywhere in groups of 8
    tiles (the norms pass itself works in groups from 50 M elements only), in a workspace that a round
    with statistics has used before."""
    off, cur = [], 0
    for m in num:
        off.append(cur)
        cur = (cur + m + 3) // 4 * 4
    dev = torch.device("cuda:0")
    P, trust, eps, lr, mu, wd = 2, 0.02, 1e-9, 0.1, 0.9, 1e-3
    ctx = eb.Context(P, off, num)
    ctx.eager_set_update_rule(wd, False)
    fill = lambda rank, sigma: wg.fill(torch.empty(cur), 3, 0, rank, sigma)   # noqa: E731
    w, v, u = fill(wg.PARAM_RANK, 0.02), fill(9, 1e-3), fill(8, 1e-3)
    u[off[0]] = float("nan")
    stats = torch.zeros(len(num) * 32, dtype=torch.uint8, device=dev)
    need = ctx.eager_stats_workspace_bytes()
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    ctx.eager_stats_attach(stats, ws, need)
    wd_, vd, ud = w.to(dev), v.to(dev), u.to(dev)
    G = [torch.zeros(cur, device=dev) for _ in range(P)]
    R = [torch.zeros(cur, device=dev) for _ in range(P)]
    recv = torch.empty(cur, device=dev)
    for t, (b0, b1) in enumerate(((0, len(num)), (len(num) - 1, len(num)), (0, 1))):
        ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, P, t, 0b11), G, R, recv=recv)
        before_w, before_v = wd_.cpu(), vd.cpu()
        ctx.eager_sgd_step_lars(ud, (wd_, vd, lr, mu), trust, eps, b0=b0, b1=b1)
        torch.cuda.synchronize()
        norms = stats.view(torch.float64).view(-1, 4)[:, :2].cpu()
        bad = stats.view(torch.int64).view(-1, 4)[:, 2].cpu()
        rates = stats.view(torch.float32).view(-1, 8)[:, 6].cpu()
        for b in range(b0, b1):
            sl = slice(off[b], off[b] + num[b])
            x, y, z = u[sl].double(), before_w[sl].double(), before_v[sl].double()
            ok = torch.isfinite(x)
            oky = torch.isfinite(y)
            su, sw = float((x[ok] ** 2).sum()), float((y[oky] ** 2).sum())
            assert int(bad[b]) == int((~ok).sum())
            assert abs(float(norms[b, 0]) - su) <= 1e-10 * su and abs(float(norms[b, 1]) - sw) <= 1e-10 * sw
            rate = trust * sw ** 0.5 / (su ** 0.5 + wd * sw ** 0.5 + eps) if su and sw else 1.0
            assert abs(float(rates[b]) - rate) <= 1.2e-7 * rate      # one rounding to fp32
            g = rate * (x + wd * y)
            vn = mu * z + g
            wn = y - lr * vn
            # a handful of fp32 roundings per element
            for got, want in ((vd.cpu()[sl], vn), (wd_.cpu()[sl], wn)):
                fine = torch.isfinite(want)
                assert torch.equal(torch.isfinite(got), fine)
                if bool(fine.any()):
                    scale = float(want[fine].abs().max())
                    assert float((got.double() - want)[fine].abs().max()) <= 1e-6 * scale
    ctx.close()


@pytest.mark.parametrize("n", [4, 255, 256, 1027, 16389])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_statistics_where_elements_are_not_finite(eb, n, bad):
    """A tile whose sums are taken without a look at its elements beside tiles that hold one that is not
    finite, in the update and in the parameters: counted and left out."""
    dev = torch.device("cuda:0")
    arena = (n + 3) // 4 * 4
    ctx = eb.Context(2, [0], [n])
    stats = torch.zeros(32, dtype=torch.uint8, device=dev)
    need = ctx.eager_stats_workspace_bytes()
    workspace = torch.empty(need, dtype=torch.uint8, device=dev)     # (the caller's as long as it is attached)
    ctx.eager_stats_attach(stats, workspace, need)
    G = [wg.fill(torch.empty(arena), 4, 0, p, 1.0).to(dev) for p in range(2)]
    w = wg.fill(torch.empty(arena), 4, 0, wg.PARAM_RANK, 1.0).to(dev)
    G[1][n // 2] = bad
    G[0][n - 1] = bad
    w[n // 3] = bad
    u, w0 = ((G[0].double() + G[1].double()) / 2)[:n], w[:n].double()
    R = [torch.zeros(arena, device=dev) for _ in range(2)]
    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, 2, 0, 0b11), G, R, opt=(w, torch.zeros_like(w), 0.1, 0.9))
    torch.cuda.synchronize()
    got = stats.view(torch.float64)[:2].tolist()
    assert int(stats.view(torch.int64)[2]) == int((~torch.isfinite(u)).sum())
    for value, x in zip(got, (u, w0)):
        want = float((x[torch.isfinite(x)] ** 2).sum())
        # the sum of two fp32 values rounds once (2^-24 relative, its square 2^-23)
        assert abs(value - want) <= 1.3e-7 * want
    ctx.close()


@pytest.mark.parametrize("size", [1, 30, 63, 255, 258, 513])
def test_statistics_beside_padding(eb, size):
    """Buckets whose last lane is part padding, which holds infinities and NaN: what lies in it is neither added
    nor counted, by a round (plain and into the receive buffer) and by the layer-wise rule."""
    nb, dev = 7, torch.device("cuda:0")
    stride = (size + 3) // 4 * 4 + (0 if size % 4 else 4)
    off, n = [b * stride for b in range(nb)], nb * stride
    inside = torch.zeros(n, dtype=torch.bool, device=dev)
    for o in off:
        inside[o:o + size] = True
    ctx = eb.Context(2, off, [size] * nb)
    stats = torch.zeros(nb * 32, dtype=torch.uint8, device=dev)
    need = ctx.eager_stats_workspace_bytes()
    workspace = torch.empty(need, dtype=torch.uint8, device=dev)
    ctx.eager_stats_attach(stats, workspace, need)
    bad = torch.tensor([float("nan"), float("inf"), float("-inf")], device=dev).repeat(n)[:n]

    def values(rank):
        x = wg.fill(torch.empty(n), 4, 0, rank, 1.0).to(dev)
        return torch.where(inside, x, bad)

    def check(u, w, what):
        torch.cuda.synchronize()
        got = stats.view(torch.float64).view(nb, 4)[:, :2]
        assert int(stats.view(torch.int64).view(nb, 4)[:, 2].abs().max()) == 0, what
        for k, x in enumerate((u, w)):
            for b, o in enumerate(off):
                want = float((x[o:o + size].double() ** 2).sum()) if x is not None else 0.0
                # sums in 64 bits of the exact squares of what is stored
                assert abs(float(got[b, k]) - want) <= 1e-12 * want, (what, b, k)

    G = [values(0), values(1)]
    R = [torch.zeros(n, device=dev) for _ in range(2)]
    w, v, recv = values(wg.PARAM_RANK), torch.zeros(n, device=dev), torch.zeros(n, device=dev)
    w0 = w.clone()
    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, 2, 0, 0b11), G, R, recv=recv, opt=(w, v, 0.1, 0.9))
    check(recv, w0, "fused")
    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, 2, 1, 0b11), G, R, recv=recv)
    check(recv, None, "into the receive buffer")
    u, w0 = values(5), w.clone()
    ctx.eager_sgd_step_lars(u, (w, v, 0.1, 0.9), 0.02, 1e-9)
    check(u, w0, "layer-wise")
    ctx.close()
