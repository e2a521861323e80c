"""Source mixtures from predecessor tables against those from leaves.

An explicit leaf size of 256, the default's, asks for the leaves; the sums are taken
in the same order, so every probability has the same bits.  Sizes: one source,
photon numbers below and above the eight terms of a chunk and above the modes,
no pair emission, fewer photon numbers than the sources emit, one mode, two photons
in a mode of the input.
"""
import numpy as np
import pytest

from paper_2204_00602_amd import inputs, slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # input, emission, g2, indistinguishability, nmax
    ([1], 0.7, 0.1, 0.5, None),
    ([2], 0.7, 0.1, 0.5, None),
    ([1, 0, 0, 1], 0.462, 0.149, 0.443, None),
    ([1, 0, 1, 0, 1, 0], 0.9, 0.0, 0.9, None),
    ([1] * 5 + [0] * 7, 0.9, 0.05, 0.95, None),   # ten photons in twelve modes: two chunks
    ([2, 1, 1, 0], 0.8, 0.2, 0.3, None),
    ([1] * 4 + [0] * 5, 0.9, 0.1, 0.9, 3),
    ([1] * 3 + [0] * 3, 0.9, 0.1, 0.9, 0),
    ([0, 0], 0.9, 0.1, 0.9, None),                # no sources
    ([1, 1] + [0] * 98, 0.9, 0.1, 0.9, None),     # one hundred modes
]


@pytest.mark.parametrize("T,emission,g2,indist,nmax", CASES)
def test_equal_to_the_leaves(T, emission, g2, indist, nmax):
    print(f"[source] T={T[:12]} m={len(T)} nmax={nmax}", flush=True)
    T = np.array(T, np.int32)
    m = len(T)
    U = inputs.haar_unitary(m, 7) if m > 1 else np.ones((1, 1), complex)
    kw = {} if nmax is None else {"nmax": nmax}
    flat = slos.Source(T, emission, g2, indist, **kw)
    leaves = slos.Source(T, emission, g2, indist, options={"leaf_max": 256}, **kw)
    Ud = torch.from_numpy(np.ascontiguousarray(U)).to(torch.complex128).cuda()
    for _ in range(2):
        got = flat.probs(Ud, out=torch.full((flat.num_outputs,), float("nan"), dtype=torch.float64, device="cuda"))
        want = leaves.probs(Ud)
        assert torch.equal(got, want)
