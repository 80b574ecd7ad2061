"""A receive buffer that is also a process's gradient buffer: every element of the gradient is read,
and carried where its process is late, before the result is stored over it.  Against the oracle, bit
for bit, at sizes of both forms of a round."""
import pytest
import torch

from harness import Pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1908_04207_amd import binding
    return binding


@pytest.mark.parametrize("n", [5, 20_003, 6_000_005])
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("late", [True, False])
def test_recv_in_a_gradient_buffer(eb, n, fused, late):
    pair = Pair(eb, 3, [0], [n], (n + 3) // 4 * 4, "f32", 0, seed=n)
    for t, mask in enumerate((0b011, 0b101, 0b110)):
        host = pair.fresh_grads(t)
        here = next(p for p in range(3) if bool((mask >> p) & 1) != late)
        pair.recv = pair.G[here]
        pair.round(eb.make_plan(eb.MAJORITY, 3, t, mask), host, fused=fused, want_recv=True)
        pair.compare(exact=True, check_recv=True, what=f"{n} elements, step {t}")
        pair.recv = torch.empty_like(pair.recv)
