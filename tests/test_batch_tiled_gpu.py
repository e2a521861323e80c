"""The tiled batch kernel at the scale of the 4,096-instance workload: large instances or
tables select it, and so does any tiling option, as here."""
import math

import numpy as np
import pytest

from paper_2204_00602_amd import inputs, slos
from test_batch_gpu import check_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,options", [
    ("c64", {"block_threads": 256, "grid_blocks": 4096, "leaf_max": 6144, "low_block_max": 2048, "outputs_per_lane": 4}),
    ("c128", {"leaf_max": 1024}),
])
def test_tiled_batch_of_4096_instances(dtype, options):
    """sum P = 1 for every instance, and every output of a seeded subset of 32 instances
    (and the largest) against the oracle."""
    print(f"[tiled batch] {dtype} {options}", flush=True)
    inst = inputs.batch_instances(4096, seed=4)
    b = slos.Batch([t for (_, _, t, _) in inst], dtype, options=options)
    U = b.pack_u([u for (_, _, _, u) in inst])
    s = torch.zeros(b.count, dtype=torch.float64, device="cuda")
    out = b.amplitudes(U, sum_p=s)
    torch.cuda.synchronize()
    assert np.abs(s.cpu().numpy() - 1.0).max() <= (1e-6 if dtype == "c64" else 1e-12)
    sizes = [math.comb(m + n - 1, n) for (m, n, _, _) in inst]
    pick = set(int(i) for i in np.random.default_rng(405).choice(4096, 32, replace=False)) | {int(np.argmax(sizes))}
    for i in sorted(pick):
        check_instance(b, out, i, inst[i][2], inst[i][3], dtype)
