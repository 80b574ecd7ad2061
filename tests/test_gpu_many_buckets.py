"""Per-bucket statistics and the layer-wise rule of models with many buckets: both sizes of the
finishing workgroup, with and without slices, next to buckets of one element; and of a model
large enough for the norms pass in groups of tiles.  Against plain 64-bit sums."""
import numpy as np
import pytest
import torch

from workloads import grads as wg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_04207_amd import binding
    return binding


def _layout(count, large):
    """`count` buckets of 1 to 700 elements, one of `large` elements among them."""
    num = [1 + (37 * k) % 700 for k in range(count)]
    num[count // 2] = large
    off, cur = [], 0
    for m in num:
        off.append(cur)
        cur = (cur + m + 3) // 4 * 4
    return off, num, cur


@pytest.mark.parametrize("count,large", [(768, 5), (769, 5), (3000, 900), (768, 3_400_001), (769, 3_400_001)])
def test_sums_and_rates(eb, count, large):
    off, num, n = _layout(count, large)
    P, trust, eps, lr, mu = 2, 0.02, 1e-9, 0.1, 0.9
    dev = torch.device("cuda:0")
    ctx = eb.Context(P, off, num)
    stats = torch.zeros(count * 32, dtype=torch.uint8, device=dev)
    need = ctx.eager_stats_workspace_bytes()
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    ctx.eager_stats_attach(stats, ws, need)
    inside = torch.zeros(n + 1, dtype=torch.int32)
    inside[torch.tensor(off)] += 1
    inside.index_add_(0, torch.tensor(off) + torch.tensor(num), torch.full((count,), -1, dtype=torch.int32))
    inside = inside.cumsum(0)[:n] > 0
    G = [wg.fill(torch.empty(n), 3, 0, p, 1e-3) * inside for p in range(P)]
    w0 = wg.fill(torch.empty(n), 3, 0, wg.PARAM_RANK, 0.02) * inside
    G[1][off[count - 1]] = float("inf")
    w, v, recv = w0.to(dev), torch.zeros(n, device=dev), torch.zeros(n, device=dev)
    grads, resid = [g.to(dev) for g in G], [torch.zeros(n, device=dev) for _ in range(P)]
    u = ((G[0] + G[1]) * 0.5).numpy()
    finite = np.isfinite(u)
    sums = lambda x: np.add.reduceat(x, off)                                # noqa: E731
    su = sums(np.where(finite, u, 0).astype(np.float64) ** 2)
    sw = sums(w0.numpy().astype(np.float64) ** 2)

    def check(with_w):
        torch.cuda.synchronize()
        got = stats.view(torch.float64).view(-1, 4)[:, :2].cpu().numpy()
        # 64-bit sums in another order: 1e-10 is what the statistics promise
        np.testing.assert_allclose(got[:, 0], su, rtol=1e-10)
        np.testing.assert_allclose(got[:, 1], sw if with_w else 0 * sw, rtol=1e-10)
        assert np.array_equal(stats.view(torch.int64).view(-1, 4)[:, 2].cpu().numpy(), sums((~finite).astype(np.int64)))

    ctx.eager_partial_allreduce(eb.make_plan(eb.MAJORITY, P, 0, 0b11), grads, resid, recv=recv)
    check(False)
    ctx.eager_sgd_step_lars(recv, (w, v, lr, mu), trust, eps)
    check(True)
    rate = np.where((su > 0) & (sw > 0), trust * np.sqrt(sw) / (np.sqrt(su) + eps), 1.0)
    got = stats.view(torch.float32).view(-1, 8)[:, 6].cpu().numpy()
    np.testing.assert_allclose(got, rate, rtol=1.2e-7)                       # one rounding to fp32
    # lars_kernel: two fp32 roundings of an element, plus the rate's
    each = np.repeat(rate, num)
    want = (w0.numpy()[inside.numpy()] - lr * each * u[inside.numpy()].astype(np.float64))
    have = w.cpu().numpy()[inside.numpy()]
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(have), ok)
    assert np.max(np.abs(have[ok] - want[ok])) <= 1e-6 * np.max(np.abs(want[ok]))
    ctx.close()


@pytest.mark.parametrize("num", [
    [2048 * 3, 100, 2047, 2049, 5, 256, 2048, 50_400_001, 1, 1_300_003, 30_000, 2048 * 8, 77, 250_000],
    [2048 * 3, 100, 2047, 2049, 5, 256, 2048, 50_400_001, 1, 1_300_003, 30_000, 2048 * 8, 77, 250_003],
    [52_001, 60_000, 2048 * 20, 7, 90_002] * 240])
def test_norms_in_groups_of_tiles(eb, num):
    """More than 50 M elements: groups of 8 tiles that lie inside one bucket, that buckets share, that
    end with the run; enough records for slices; a range of buckets for which groups are too
    few; more buckets than the large finishing workgroups are for."""
    off, n = [], 0
    for m in num:
        off.append(n)
        n = (n + m + 3) // 4 * 4
    dev = torch.device("cuda:0")
    trust, eps, lr, mu = 0.02, 1e-9, 0.1, 0.9
    ctx = eb.Context(1, off, num)
    stats = torch.zeros(len(num) * 32, dtype=torch.uint8, device=dev)
    need = ctx.eager_stats_workspace_bytes()
    ws = torch.full((need,), 0x5A, dtype=torch.uint8, device=dev)            # stale records
    ctx.eager_stats_attach(stats, ws, need)
    gen = torch.Generator(device=dev).manual_seed(11)
    u = torch.empty(n, device=dev).normal_(0.0, 1e-3, generator=gen)
    w0 = torch.empty(n, device=dev).normal_(0.0, 0.02, generator=gen)
    u[off[1]], u[off[7] + 4_000_000], u[off[-1] + num[-1] - 1] = float("nan"), float("inf"), float("-inf")
    w0[off[9] + 17] = float("nan")
    for b0, b1 in ((0, len(num)), (8, len(num)), (0, len(num))):
        w, v = w0.clone(), torch.zeros(n, device=dev)
        stats.zero_()
        ctx.eager_sgd_step_lars(u, (w, v, lr, mu), trust, eps, b0=b0, b1=b1)
        torch.cuda.synchronize()
        norms = stats.view(torch.float64).view(-1, 4)[:, :2].cpu()
        bad = stats.view(torch.int64).view(-1, 4)[:, 2].cpu()
        rates = stats.view(torch.float32).view(-1, 8)[:, 6].cpu()
        for b in range(b0, b1):
            sl = slice(off[b], off[b] + num[b])
            x, y = u[sl].double(), w0[sl].double()
            fine = torch.isfinite(x)
            su, sw = float(x[fine].square().sum()), float(y[torch.isfinite(y)].square().sum())
            assert int(bad[b]) == int((~fine).sum()), b
            assert abs(float(norms[b, 0]) - su) <= 1e-10 * su and abs(float(norms[b, 1]) - sw) <= 1e-10 * sw, b
            rate = trust * sw ** 0.5 / (su ** 0.5 + eps)
            assert abs(float(rates[b]) - rate) <= 1.2e-7 * rate, b           # one rounding to fp32
            want = y - lr * (rate * x)
            ok = torch.isfinite(want)
            assert torch.equal(torch.isfinite(w[sl]), ok)
            # a handful of fp32 roundings per element
            assert float((w[sl].double() - want)[ok].abs().max()) <= 1e-6 * float(want[ok].abs().max())
    ctx.close()
