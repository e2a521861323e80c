"""The mesh kernels in their shape for many phase sets: one, two or four waves to a set,
phase factors alone prepared, an adjoint whose sums are per wave.  The oracle and the
tolerances are those of test_mesh_gpu.py."""
import numpy as np
import pytest

import oracle
from paper_2204_00602_amd import inputs, slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [3, 10, 13, 18, 21, 24, 40, 41, 50])
def test_many_sets_match_oracle(m):
    print(f"[mesh, many] m={m}", flush=True)
    batch = 2049
    ph = inputs.mesh_phases(batch, slos.mesh_mzi_count(m), 800 + m)
    d = torch.from_numpy(ph).cuda()
    gen = torch.Generator(device="cuda").manual_seed(m)
    G = torch.view_as_complex(torch.randn((batch, m, m, 2), dtype=torch.float64, device="cuda", generator=gen))
    U = slos.mesh_unitary(d, m, "c128")
    g = slos.mesh_backward(d, G)
    for b in (0, 1024, batch - 1):
        Gb = G[b].cpu().numpy()
        assert np.abs(U[b].cpu().numpy() - oracle.clements_unitary(m, ph[b])).max() <= 8 * m * 2.0 ** -53
        tol = 32 * m * 2.0 ** -53 * np.abs(Gb).sum(axis=0).max() * np.sqrt(m)
        assert np.abs(g[b].cpu().numpy() - oracle.mesh_vjp(ph[b], m, Gb)).max() <= tol
