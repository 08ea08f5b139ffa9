"""Block summaries (sva_pool_blocks) at the edges of blocks and of a workgroup's
rows, against the same means in float64.

The inputs are multiples of 2^-8 below 2^4, so a block's float64 sum is exact in
any order and the float32 result is the correctly rounded mean.
"""
import pytest

import paper_2606_23743_amd as sva

from .gpu_cases import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("S", [64, 128])
@pytest.mark.parametrize("D", [64, 112, 128])
@pytest.mark.parametrize("N", [1, 15, 33, 64, 129, 1000])
def test_pool_is_the_rounded_mean(N, D, S):
    say(f"[pool N={N} D={D} S={S}]")
    g = torch.Generator(device="cuda").manual_seed(N + D + S)
    # multiples of 2^-8 keep every sum exact
    q, k = ((torch.randn((2, 3, N, D), generator=g, device="cuda") * 256).round().div(256).bfloat16() for _ in "qk")
    got = sva.pool_blocks(sva.problem(2, 3, N, D, (1, 1, N), S), q, k)
    for x, y in zip((q, k), got):
        for i in range(-(-N // S)):
            rows = x[:, :, i * S:(i + 1) * S].double()
            count = torch.tensor(float(rows.shape[2]), dtype=torch.float64, device="cuda")
            assert torch.equal(y[:, :, i], (rows.sum(2) / count).float()), i
