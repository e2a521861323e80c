"""The table-driven batch against the tiled batch kernel.

A batch made with a tiling option runs the tiled kernel; the default runs from
tables in the same order of summation, so the unnormalised sums have equal bits
and an amplitude differs by the rounding of its FP64 normalisation (one product
more) and, in c64, of the conversion after it: four units in the last place
bound both.  A sum of P differs by the order of its FP64 additions: an output's
rounding each, within 1e-10 for the sizes here.  The sizes are those at which
the kernel changes its way: instances on waves and on whole workgroups, layers
that fit the LDS, that are staged in blocks and that are read from memory,
instances cut into parts, one state per layer, no photons, more than eight
occupied modes.
"""
import numpy as np
import pytest

from paper_2204_00602_amd import inputs, slos

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def single(m, n):
    """n photons in m modes, one a mode and round again."""
    return [n // m + (i < n % m) for i in range(m)]


BATCHES = {
    "waves": [single(m, n) for m, n in [(6, 3), (8, 4), (10, 4), (9, 5), (6, 2)]] * 13,
    "wave and workgroup": [single(9, 5), single(10, 5), single(8, 6)] * 100,
    "one state, no photons": [[7], [0, 0, 0], [0], [0, 1], [1, 0], [8, 8], [16, 0, 0]],
    "more than eight modes": [single(10, 9), single(12, 6), single(9, 9), single(20, 4)],
    "edge of the LDS": [single(12, 7), single(13, 7), single(11, 7)],
    "parts": [single(14, 7)] + [single(6, 3)] * 5,
    "no parts": [single(14, 7)] * 300,
    "long blocks": [single(50, 5), single(40, 5), single(6, 3)],
    "several mode counts": [single(m, n) for m in range(6, 15) for n in range(2, min(m, 7) + 1)],
}


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("name", BATCHES)
def test_equal_to_the_tiled_batch(name, dtype):
    print(f"[flat batch] {name} {dtype}", flush=True)
    states = BATCHES[name]
    cdt = np.complex64 if dtype == "c64" else np.complex128
    eps = 4.0 * np.finfo(cdt).eps
    flat, tiled = slos.Batch(states, dtype), slos.Batch(states, dtype, options={"block_threads": 256})
    for turn in range(2):  # the second launch finds the counters of the first
        us = {}  # one unitary per mode count
        U = [us.setdefault(len(t), inputs.haar_unitary(len(t), 3 + turn + 10 * len(t)) if len(t) > 1 else np.ones((1, 1))) for t in states]
        got, want = [], []
        for b, res in ((flat, got), (tiled, want)):
            sum_p = torch.full((len(states),), -1.0, dtype=torch.float64, device="cuda")
            a = b.amplitudes(b.pack_u(U), sum_p=sum_p)
            torch.cuda.synchronize()
            res += [torch.view_as_real(a), sum_p]
        assert bool((torch.abs(got[0] - want[0]) <= eps * torch.abs(want[0])).all())
        assert bool((torch.abs(got[1] - want[1]) <= 1e-10).all())
