"""Selected outputs whose largest sub-lattice needs more of a workgroup's LDS than the
usual 32 KiB by an amount that does not divide by its parts, beside small targets that run
in those parts.  The oracle and the tolerance are those of test_select_classes_gpu."""
import numpy as np
import pytest

from paper_2204_00602_amd import inputs
from test_select_classes_gpu import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,dtype", [
    (12, 11, "c128"),  # 36,640 bytes: eighths of 4,580
    (13, 13, "c64"),   # 68,240 bytes: eighths of 8,530
])
def test_small_targets_beside_a_large_one(m, n, dtype):
    print(f"[select parts] m={m} n={n} {dtype}", flush=True)
    targets = inputs.uniform_fock_states(m, n, 600, 3)
    targets[0] = np.arange(m) < n
    targets[1] = [n] + [0] * (m - 1)
    targets[2] = [0, n - 1, 1] + [0] * (m - 3)
    check(m, n, dtype, targets)
