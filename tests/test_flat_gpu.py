"""The table-driven layers against the tiled kernels, bit for bit.

A plan made with a tiling option runs the tiled kernels on every layer; the
default plan runs its small layers from tables in the same order of
summation, so the amplitudes are equal in every bit, and each sum of P is
within the rounding of its own fixed-order FP64 sum.  Sizes at the edges: one
state per layer, single-photon passes, more than eight occupied modes, m = 255,
a first launch of one and of several workgroups, layers just below and above
the first launch's and the tables' limits, several instances.
"""
import math

import numpy as np
import pytest

from paper_2204_00602_amd import inputs, slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # m, input, dtype, compensated
    (1, [5], "c128", False),                        # one state in every layer
    (2, [16, 16], "c128", False),                   # 32 photons, 33 states
    (3, [0, 1, 0], "c64", True),                    # a single photon
    (255, [1] + [0] * 254, "c64", False),           # 255 states from one photon
    (255, [1, 0, 1] + [0] * 252, "c64", True),      # 32,640: the tables past a 255-state first layer
    (6, [1, 1, 1, 0, 0, 0], "c128", False),         # one workgroup
    (9, [1] * 9, "c64", True),                      # nine occupied modes: a second chunk of terms
    (12, [1] * 6 + [0] * 6, "c64", False),          # several workgroups in one launch
    (12, [2, 2, 1, 0, 0, 1] + [0] * 6, "c64", "knuth"),
    (13, [1] * 6 + [0] * 7, "c64", "fp64"),         # 6,188 states kept in LDS
    (11, [1] * 9 + [0] * 2, "c128", False),
    (18, [1] * 8 + [0] * 10, "c64", True),          # 1,081,575: the tables' leaf size of larger layers
    (19, [1] * 9 + [0] * 10, "c64", True),          # 4,686,825: a tiled layer after the tables
]


@pytest.mark.parametrize("m,T,dtype,comp", CASES)
def test_equal_to_the_tiled_layers(m, T, dtype, comp):
    print(f"[flat] m={m} T={T[:12]} {dtype} comp={comp}", flush=True)
    T = np.array(T, np.int32)
    cdt = torch.complex64 if dtype == "c64" else torch.complex128
    U = torch.from_numpy(inputs.haar_unitary(m, 31) if m > 1 else np.ones((1, 1), complex)).to(cdt).cuda()
    default = slos.Plan(T, dtype, compensated=comp)
    tiled = slos.Plan(T, dtype, compensated=comp, options={"block_threads": 256})
    s1 = torch.full((1,), math.nan, dtype=torch.float64, device="cuda")
    s2 = torch.full((1,), math.nan, dtype=torch.float64, device="cuda")
    for _ in range(2):  # the counters of a pass are left ready for the next
        a, b = default.amplitudes(U, sum_p=s1), tiled.amplitudes(U, sum_p=s2)
        assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
        # both are sums of the same M non-negative FP64 terms
        assert abs(float(s1) - float(s2)) <= 2 * a.numel() * 2.0 ** -53 * float(s2)
    assert torch.equal(default.probs(U), tiled.probs(U))


@pytest.mark.parametrize("m,n,dtype,comp,keep", [(12, 6, "c64", True, False), (15, 6, "c128", False, False),
                                                 (10, 5, "c64", False, True), (3, 1, "c128", False, True)])
def test_instances_of_one_call(m, n, dtype, comp, keep):
    print(f"[flat] many m={m} n={n} {dtype} comp={comp} keep={keep}", flush=True)
    B = 70  # more instances than workgroups a single one would take
    cdt = torch.complex64 if dtype == "c64" else torch.complex128
    U = torch.stack([torch.from_numpy(inputs.haar_unitary(m, 60 + b)) for b in range(B)]).to(cdt).cuda()
    T = inputs.first_modes_input(m, n)
    many = slos.Plan(T, dtype, compensated=comp, keep_layers=keep, options={"max_batch": B})
    tiled = slos.Plan(T, dtype, compensated=comp, options={"max_batch": B, "block_threads": 256})
    s1 = torch.empty(B, dtype=torch.float64, device="cuda")
    s2 = torch.empty(B, dtype=torch.float64, device="cuda")
    a, b = many.amplitudes_many(U, sum_p=s1), tiled.amplitudes_many(U, sum_p=s2)
    assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
    assert float((s1 - s2).abs().max()) <= 2 * a.shape[1] * 2.0 ** -53 * float(s2.max())


def test_non_finite_coefficients_stay_in_their_outputs():
    """A padded term adds nothing: an infinite coefficient of the last mode
    reaches only the outputs with a photon there."""
    m, T = 8, [1, 1, 1, 0, 0, 0, 0, 0]
    U = torch.from_numpy(inputs.haar_unitary(m, 5)).cuda()
    U[m - 1, 0] = complex(math.inf, 0.0)
    p = slos.Plan(T, "c128")
    a = torch.view_as_real(p.amplitudes(U))
    below = slos.fock_count(m - 1, 3)  # the outputs without a photon in the last mode
    assert bool(torch.isfinite(a[:below]).all()) and not bool(torch.isfinite(a[below:]).any(dim=1).all())
