"""The table-driven adjoint against the unit kernels and the tail's edges.

A plan made with a tiling option runs the adjoint's unit kernels; the default
plan runs it from successor tables.  Both form the same sums in other orders,
so each element of G_U agrees within the rounding of its terms, whose magnitudes
are bounded by the same adjoint on absolute values (of U and of dL/da): n
forward and n reverse layers, each a sum of at most m products stored in the
plan's type.
"""
import numpy as np
import pytest

from paper_2204_00602_amd import inputs, slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # m, n, dtype, batch
    (1, 3, "c128", 1),      # one state per layer
    (2, 30, "c128", 1),     # 30 reverse layers in the tail
    (5, 1, "c64", 1),       # one layer, one state below it
    (12, 6, "c64", 3),      # the whole adjoint in the tail
    (13, 4, "c128", 1),     # more modes than a thread's turn of the tail
    (37, 3, "c128", 2),     # three turns; a layer above the tail
    (16, 7, "c128", 1),     # four layers above the tail
    (18, 7, "c64", 40),     # several states per thread
    (255, 2, "c64", 1),     # the most modes
]


@pytest.mark.parametrize("m,n,dtype,batch", CASES)
def test_equal_to_the_unit_kernels(m, n, dtype, batch):
    print(f"[flat adjoint] m={m} n={n} {dtype} batch={batch}", flush=True)
    cdt = torch.complex64 if dtype == "c64" else torch.complex128
    T = inputs.random_input(m, n, np.random.default_rng(m), max_per_mode=max(2, -(-n // m)))
    Us = [inputs.haar_unitary(m, 90 + b) if m > 1 else np.ones((1, 1), complex) for b in range(batch)]
    U = torch.stack([torch.from_numpy(u) for u in Us]).to(cdt).cuda()
    default = slos.Plan(T, dtype, keep_layers=True, options={"max_batch": batch})
    units = slos.Plan(T, dtype, keep_layers=True, options={"max_batch": batch, "block_threads": 128})
    gen = torch.Generator(device="cuda").manual_seed(m * 100 + n)
    M = default.num_outputs
    ga = torch.randn((batch, M), dtype=torch.complex128, device="cuda", generator=gen).to(cdt)
    got, ref = [], []
    for plan, to in ((default, got), (units, ref)):
        for _ in range(2):
            plan.amplitudes_many(U)
            to.append(plan.backward_many(U, ga).to(torch.complex128))
    assert torch.equal(torch.view_as_real(got[0]), torch.view_as_real(got[1]))  # fixed order
    # the adjoint of the absolute values bounds every term's magnitude
    absU = U.abs().to(cdt)
    units.amplitudes_many(absU)
    bound = units.backward_many(absU, ga.abs().to(cdt)).real.to(torch.float64)
    eps = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53
    # n layers of forward and reverse sums of up to m terms each, stored in the plan's type
    tol = 2 * n * (m + 4) * eps * bound
    assert bool(((got[0] - ref[0]).abs() <= tol).all()), float(((got[0] - ref[0]).abs() / bound.clamp_min(1e-300)).max())
