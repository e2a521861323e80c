"""An infinite or undefined dL/da through the table-driven adjoint, against the unit kernels.

Both form exactly the products of dL/da with U and with the kept layers that the adjoint
has, so an element of G_U is infinite, undefined or finite in both, and the finite ones
(none of whose terms is anything else) agree within the rounding of test_flat_bwd_gpu.
Sizes: mode counts that are no multiple of the modes taken together and layers that are
no multiple of the states taken together, in the tail launch and above it; the infinite
element is the last output, the only successor of the last state by the last mode.
"""
import numpy as np
import pytest

from paper_2204_00602_amd import inputs, slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["last", "middle"])
@pytest.mark.parametrize("m,n,dtype,batch", [
    (5, 2, "c64", 1),       # four lanes a state
    (13, 5, "c128", 1),     # a state per thread, thirteen modes
    (16, 7, "c128", 1),     # layers above the tail
    (18, 7, "c64", 40),     # several states per thread
])
def test_other_elements_stay_as_they_are(m, n, dtype, batch, where):
    print(f"[non-finite adjoint] m={m} n={n} {dtype} batch={batch} {where}", flush=True)
    cdt = torch.complex64 if dtype == "c64" else torch.complex128
    T = inputs.random_input(m, n, np.random.default_rng(m), max_per_mode=2)
    U = torch.stack([torch.from_numpy(inputs.haar_unitary(m, 40 + b)) for b in range(batch)]).to(cdt).cuda()
    default = slos.Plan(T, dtype, keep_layers=True, options={"max_batch": batch})
    units = slos.Plan(T, dtype, keep_layers=True, options={"max_batch": batch, "block_threads": 128})
    gen = torch.Generator(device="cuda").manual_seed(m * 100 + n)
    M = default.num_outputs
    ga = torch.randn((batch, M), dtype=torch.complex128, device="cuda", generator=gen).to(cdt)
    at = M - 1 if where == "last" else M // 2
    finite = ga.clone()
    finite[:, at] = 0
    for value in (complex(float("inf"), 1.0), complex(-2.0, float("-inf")), complex(float("nan"), 1.0)):
        ga[:, at] = value
        got, ref = [], []
        for plan, to in ((default, got), (units, ref)):
            plan.amplitudes_many(U)
            to.append(torch.view_as_real(plan.backward_many(U, ga).to(torch.complex128)))
        got, ref = got[0], ref[0]
        absU = U.abs().to(cdt)
        units.amplitudes_many(absU)
        bound = units.backward_many(absU, finite.abs().to(cdt)).real.to(torch.float64)
        eps = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53
        tol = (2 * n * (m + 4) * eps * bound)[..., None]
        assert torch.equal(got.isnan(), ref.isnan()), (value, int((got.isnan() != ref.isnan()).sum()))
        inf = ref.isinf()
        assert torch.equal(got.isinf(), inf) and torch.equal(got[inf], ref[inf]), value
        ok = ref.isfinite()
        assert bool(((got - ref).abs() <= tol)[ok].all()), value
        assert not bool(ok.all())
