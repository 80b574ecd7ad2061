"""The layer-wise rule where every bucket is small enough for a workgroup of its own, at the sizes where its three forms
begin and end, next to empty buckets, ragged ends and padding that must stay as it is; and just beyond.  Against plain
64-bit arithmetic."""
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
@pytest.mark.parametrize("num", [
    [1], [0, 3, 4, 5, 0], [1024, 1, 1023, 255, 256, 257, 0, 7], [1025, 4, 1021, 2], [4096, 4095, 4093, 1, 0, 64],
    [4097, 12, 4099], [16384, 16383, 16381, 5, 1027], [16385, 100, 3], [300] * 600 + [16384], [2000] * 600 + [16001]])
def test_norms_rates_and_update(eb, num, order):
    off, n = [], 0
    for m in num:
        off.append(n)
        n = (n + m + 3) // 4 * 4 + 8                            # padding behind every bucket
    dev = torch.device("cuda:0")
    trust, eps, lr, mu, wd = 0.02, 1e-9, 0.1, 0.9, 1e-3
    gen = torch.Generator(device=dev).manual_seed(len(num))
    u = torch.empty(n, device=dev).normal_(0.0, 1e-3, generator=gen)
    w0 = torch.empty(n, device=dev).normal_(0.0, 0.02, generator=gen)
    v0 = torch.empty(n, device=dev).normal_(0.0, 1e-3, generator=gen)
    u[off[-1] + num[-1] - 1] = float("inf")                     # the last element of the last bucket
    w0[off[len(num) // 2]:off[len(num) // 2] + num[len(num) // 2]] = 0.0
    raw = torch.full((len(num) * 32,), 0x5A, dtype=torch.uint8, device=dev)
    for nesterov, (b0, b1) in ((False, (0, len(num))), (True, (len(num) // 3, len(num)))):
        ctx = eb.Context(1, off, num, order=order)
        ctx.eager_set_update_rule(wd, nesterov)
        need = ctx.eager_stats_workspace_bytes()
        ws = torch.full((need,), 0x5A, dtype=torch.uint8, device=dev)
        ctx.eager_stats_attach(raw, ws, need)
        w, v = w0.clone(), v0.clone()
        ctx.eager_sgd_step_lars(u, (w, v, lr, mu), trust, eps, b0=b0, b1=b1)
        torch.cuda.synchronize()
        sums = raw.view(torch.float64).view(-1, 4)[:, :2].cpu().tolist()
        bad = raw.view(torch.int64).view(-1, 4)[:, 2].cpu().tolist()
        rates = raw.view(torch.float32).view(-1, 8)[:, 6].cpu().tolist()
        touched = torch.zeros(n, dtype=torch.bool, device=dev)
        for b in range(b0, b1):
            sl = slice(off[b], off[b] + num[b])
            touched[sl] = True
            if b > 8 and b < len(num) - 8:
                continue
            x, y, z = u[sl].double(), w0[sl].double(), v0[sl].double()
            fine = torch.isfinite(x)
            su, sw = float(x[fine].square().sum()), float(y.square().sum())
            assert abs(sums[b][0] - su) <= 1e-10 * su and abs(sums[b][1] - sw) <= 1e-10 * sw, b
            assert bad[b] == int((~fine).sum()), b
            rate = trust * sw ** 0.5 / (su ** 0.5 + wd * sw ** 0.5 + eps) if su > 0 and sw > 0 else 1.0
            assert abs(rates[b] - rate) <= 1.2e-7 * rate, b      # one rounding to fp32
            g = rate * (x + wd * y)
            vn = mu * z + g
            wn = y - lr * (g + mu * vn if nesterov else vn)
            for got, want in ((w[sl], wn), (v[sl], vn)):
                ok = torch.isfinite(want)
                assert torch.equal(torch.isfinite(got), ok), b
                if ok.any():                                     # a handful of fp32 roundings per element
                    assert float((got.double() - want)[ok].abs().max()) <= 1e-6 * float(want[ok].abs().max()), b
        # other buckets stay as they are (padding may be overwritten)
        for b in range(b0):
            sl = slice(off[b], off[b] + num[b])
            assert torch.equal(w[sl], w0[sl]) and torch.equal(v[sl], v0[sl]), b
        ctx.close()
