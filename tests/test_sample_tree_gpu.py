"""Samples at the edges of the search tree and of the launch.

For r, the sample is the first output whose cumulative P exceeds r * sum P: the
cumulative sum below it is at most that and the one through it exceeds it, but for
the rounding of the two FP64 sums that are compared, M additions of 2^-53 of the
total each.  A drawn output has P > 0.  Sizes: one block, one state past a block, one and
two levels, a level past the part kept in LDS, two runs of block sums; counts around
a lane group, a wave and the whole chip's waves.
"""
import numpy as np
import pytest

from paper_2204_00602_amd import slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # m, n, dtype, samples
    (3, 2, "c64", 1),             # 6 states
    (2, 31, "c128", 5),           # 32 states
    (44, 2, "c128", 16),          # 990: one block
    (45, 2, "c64", 17),           # 1,035: two
    (12, 6, "c64", 63),           # 13 blocks
    (14, 6, "c128", 65),          # 27: a second level
    (16, 7, "c64", 4097),         # 167
    (18, 8, "c128", 64 * 8192 + 5),   # 1,057 blocks: two runs, the tree's first level above the LDS's
    (20, 10, "c64", 64 * 8192 + 77),  # 19,561
]


@pytest.mark.parametrize("m,n,dtype,count", CASES)
def test_samples_cross_the_cumulative_sum(m, n, dtype, count):
    print(f"[sample] m={m} n={n} {dtype} count={count}", flush=True)
    plan = slos.Plan([n] + [0] * (m - 1), dtype)
    M = plan.num_outputs
    g = torch.Generator(device="cuda").manual_seed(m * 100 + n)
    P = torch.rand(M, generator=g, device="cuda", dtype=torch.float64)
    P[torch.rand(M, generator=g, device="cuda") < 0.3] = 0.0  # outputs that are never drawn
    P[M // 3:M // 2] = 0.0                                    # whole chunks and blocks of them
    P[0] = 0.5
    P = (P / P.sum()).to(torch.float32 if dtype == "c64" else torch.float64)
    r = torch.rand(count, generator=g, device="cuda", dtype=torch.float64)
    r[0] = 0.0
    r[-1] = 1.0 - 2.0 ** -53
    plan.cdf(P)
    ranks = plan.sample(P, r)
    torch.cuda.synchronize()
    cum = torch.cumsum(P.to(torch.float64), 0)
    eps = M * 2.0 ** -52 * float(cum[-1])
    t = r * cum[-1]
    assert bool(((ranks >= 0) & (ranks < M)).all())
    assert bool((P[ranks] > 0).all())
    assert bool((cum[ranks] >= t - eps).all())
    below = torch.where(ranks > 0, cum[(ranks - 1).clamp(min=0)], torch.zeros_like(t))
    assert bool((below <= t + eps).all())
