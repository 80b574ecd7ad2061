"""The layer-wise rule where every bucket is small enough for a workgroup of its own, at the sizes where its three forms
begin and end, next to empty buckets, ragged ends and padding - which between buckets of the range takes the rate of the
bucket before it, and elsewhere stays as it is; and just beyond, with large buckets or long padding.  Against plain 64-bit
arithmetic, every element."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_04207_amd import binding
    return binding


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("num,gap", [
    ([1], 8), ([0, 3, 4, 5, 0], 8), ([1024, 1, 1023, 255, 256, 257, 0, 7], 8), ([1025, 4, 1021, 2], 8),
    ([1016, 3, 1013, 1024], 8), ([4096, 4095, 4093, 1, 0, 64], 8), ([4088, 4087, 4096], 8), ([4097, 12, 4099], 8),
    ([16384, 16383, 16381, 5, 1027], 8), ([16376, 16375, 16384], 8), ([16385, 100, 3], 8), ([300] * 600 + [16384], 8),
    ([2000] * 600 + [16001], 8), ([1000, 5, 0, 2000, 7], 252), ([4096, 5, 16384], 256), ([16384, 5, 2000], 256), ([1004, 6, 2000], 256), ([3, 4096, 9], 50_000)])
def test_norms_rates_and_update(eb, num, gap, order):
    off, n = [], 64                                             # (nobody's elements in front)
    for m in num:
        off.append(n)
        n = (n + m + 3) // 4 * 4 + gap                          # padding behind every bucket
    dev = torch.device("cuda:0")
    trust, eps, lr, mu, wd = 0.02, 1e-9, 0.1, 0.9, 1e-3
    gen = torch.Generator(device=dev).manual_seed(len(num))
    u = torch.empty(n, device=dev).normal_(0.0, 1e-3, generator=gen)
    w0 = torch.empty(n, device=dev).normal_(0.0, 0.02, generator=gen)
    v0 = torch.empty(n, device=dev).normal_(0.0, 1e-3, generator=gen)
    last = max(b for b, m in enumerate(num) if m)
    u[off[last] + num[last] - 1] = float("inf")                 # the last element of the last bucket that has any
    w0[off[len(num) // 2]:off[len(num) // 2] + num[len(num) // 2]] = 0.0
    raw = torch.empty(len(num) * 32, dtype=torch.uint8, device=dev)
    starts, sizes = torch.tensor(off, device=dev), torch.tensor(num, device=dev)
    at = torch.arange(n, device=dev)
    of = (torch.searchsorted(starts, at, right=True) - 1).clamp_(min=0)
    data = (at >= starts[of]) & (at < starts[of] + sizes[of])
    x, y, z = u.double(), w0.double(), v0.double()
    fine = torch.isfinite(x)
    add = lambda what: torch.zeros(len(num), dtype=torch.float64, device=dev).index_add_(0, of[data], what[data])  # noqa: E731
    su, sw, bad = add(torch.where(fine, x, 0.0).square()), add(y.square()), add((~fine).double())
    assert int(bad.sum()) == 1
    norms = trust * sw.sqrt() / (su.sqrt() + wd * sw.sqrt() + eps)
    rate = torch.where((su > 0) & (sw > 0), norms, torch.ones_like(norms))
    for nesterov, (b0, b1) in ((False, (0, len(num))), (True, (len(num) // 3, len(num))), (False, (0, (len(num) + 1) // 2))):
        ctx = eb.Context(1, off, num, order=order)
        ctx.eager_set_update_rule(wd, nesterov)
        need = ctx.eager_stats_workspace_bytes()
        ws = torch.full((need,), 0x5A, dtype=torch.uint8, device=dev)
        raw.fill_(0x5A)
        ctx.eager_stats_attach(raw, ws, need)
        w, v = w0.clone(), v0.clone()
        ctx.eager_sgd_step_lars(u, (w, v, lr, mu), trust, eps, b0=b0, b1=b1)
        torch.cuda.synchronize()
        mine = slice(b0, b1)
        sums, count = raw.view(torch.float64).view(-1, 4)[mine], raw.view(torch.int64).view(-1, 4)[mine, 2]
        rates = raw.view(torch.float32).view(-1, 8)[mine, 6].double()
        assert ((sums[:, 0] - su[mine]).abs() <= 1e-10 * su[mine]).all()
        assert ((sums[:, 1] - sw[mine]).abs() <= 1e-10 * sw[mine]).all()
        assert torch.equal(count.double(), bad[mine])
        assert ((rates - rate[mine]).abs() <= 1.2e-7 * rate[mine]).all()                # one rounding to fp32
        # from the first bucket of the range to the end of the last, padding between them too
        touched = (at >= off[b0]) & (at < off[b1 - 1] + num[b1 - 1])
        assert torch.equal(w[~touched], w0[~touched]) and torch.equal(v[~touched], v0[~touched])
        g = rate[of] * (x + wd * y)
        vn = mu * z + g
        wn = y - lr * (g + mu * vn if nesterov else vn)
        for got, want in ((w, wn), (v, vn)):
            ok = torch.isfinite(want)
            assert torch.equal(torch.isfinite(got)[touched], ok[touched])
            # a handful of fp32 roundings per element: 1e-6 of the largest of its bucket (and the padding behind)
            want = torch.where(ok, want, 0.0)
            most = torch.zeros(len(num), dtype=torch.float64, device=dev).scatter_reduce_(0, of, want.abs(), "amax")
            off_by = torch.where(touched & ok, (got.double() - want).abs() - 1e-6 * most[of], -1.0)
            assert float(off_by.max()) <= 0.0, int(off_by.argmax())
        ctx.close()
