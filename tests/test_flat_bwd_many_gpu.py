"""The adjoint's tail launch for more instances than compute units, where a workgroup
has 64 or 256 threads instead of 1024.  References and tolerances are those of
test_flat_bwd_gpu.py (the unit kernels) and test_backward_gpu.py (the loss in two calls).
"""
import pytest

import test_backward_gpu
import test_flat_bwd_gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # m, n, dtype, instances
    (2, 7, "c128", 300),   # 64 threads, seven layers
    (8, 3, "c64", 257),    # 64 threads, more states than a turn of them
    (9, 4, "c64", 300),    # 256 threads, four lanes a state
    (13, 5, "c64", 260),   # 256 threads do not fit four times: 1024
    (10, 5, "c64", 300),   # 256 threads, a state per thread
    (64, 3, "c64", 257),   # 256 threads, a layer above the tail
]


@pytest.mark.parametrize("m,n,dtype,batch", CASES)
def test_many_instances(m, n, dtype, batch):
    test_flat_bwd_gpu.test_equal_to_the_unit_kernels(m, n, dtype, batch)


@pytest.mark.parametrize("m,n,dtype,batch", CASES[1:5])
def test_fused_loss_of_many_instances(m, n, dtype, batch):
    print(f"[fused loss] m={m} n={n} {dtype} batch={batch}", flush=True)
    test_backward_gpu.test_fused_loss_backward_equals_two_calls(dtype, m, [1] * n + [0] * (m - n), batch)
