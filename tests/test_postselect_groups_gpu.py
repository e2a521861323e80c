"""Group counts of single outputs against the enumerated occupations.

The table is P(S) / kept sum for a kept rank and zero otherwise, one FP64 division;
the kept sum of M non-negative terms is within M roundings of 2^-53.  Sizes: one
mode, many photons, 255 modes, more photons than the walk reads ahead, one group, as many
as a word holds and one more, sixteen; photons outside every group; ranks outside
the distribution.
"""
import numpy as np
import pytest

from paper_2204_00602_amd import slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(1, 5), (2, 32), (255, 2), (20, 4), (9, 7), (5, 0)])
@pytest.mark.parametrize("groups", [1, 4, 5, 16])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_table_and_sum(m, n, groups, dtype):
    print(f"[postselect] m={m} n={n} groups={groups} {dtype}", flush=True)
    rng = np.random.default_rng(m * 100 + n * 10 + groups)
    plan = slos.Plan([n] + [0] * (m - 1), dtype)
    M = plan.num_outputs
    states = np.stack([slos.fock_unrank(m, n, r) for r in range(M)])
    group = rng.integers(-1, groups, m).astype(np.int32)
    counts = np.stack([states[:, group == g].sum(axis=1) for g in range(groups)])
    low = np.array([int(rng.integers(0, 2)) if n > 1 and c.max() > 0 else 0 for c in counts], np.int32)
    high = np.array([max(int(l), int(rng.integers(0, n + 1))) for l in low], np.int32)
    ok = ((counts >= low[:, None]) & (counts <= high[:, None])).all(axis=0)
    P = torch.from_numpy(rng.random(M)).to(torch.float32 if dtype == "c64" else torch.float64).cuda()
    P /= P.sum()
    p = P.cpu().numpy().astype(np.float64)
    ranks = np.concatenate([rng.integers(0, M, 200), [0, M - 1, -1, M]]).astype(np.int64)
    kept, masked, table = plan.postselect(P, group, low, high, masked=True, ranks=torch.from_numpy(ranks).cuda())
    want = p[ok].sum()
    assert abs(float(kept) - want) <= 2 * M * 2.0 ** -53 * max(want, 0.0)
    assert np.array_equal(masked.cpu().numpy(), np.where(ok, P.cpu().numpy(), 0))
    inside = (ranks >= 0) & (ranks < M)
    at = np.where(inside, ranks, 0)
    keep = inside & ok[at]
    got = table.cpu().numpy()
    assert np.all(got[~keep] == 0.0)
    assert np.allclose(got[keep], p[at][keep] / float(kept), rtol=4 * 2.0 ** -53, atol=0.0)
