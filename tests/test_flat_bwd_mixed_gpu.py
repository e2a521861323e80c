"""The adjoint where its layers change from one kind of kernel to another.

Reverse layers run from successor tables up to a size, above it in unit kernels, and the
last layer's forward may be tiled where its reverse is not: then the seed kernel fills
g_n and the table-driven layers take it as it is.  The reference and the tolerance are those of
test_flat_bwd_gpu.  The squared-error loss is compared, bit for bit, with its two
calls (the loss's gradient, then the adjoint) at sizes whose top layers are above
the tail launch.
"""
import pytest

from paper_2204_00602_amd import inputs
import test_backward_gpu
import test_flat_bwd_gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,dtype", [
    (16, 10, "c128"),  # layer 10 tiled forward, table-driven in reverse
    (13, 15, "c64"),   # reverse layers 15 and 14 in unit kernels, 13..1 from tables
    (80, 5, "c64"),    # layer 5's successor table would be over the limit of all tables
])
def test_hand_over_between_kernels(m, n, dtype):
    test_flat_bwd_gpu.test_equal_to_the_unit_kernels(m, n, dtype, 1)


@pytest.mark.parametrize("m,n,batch,dtype", [
    (13, 7, 3, "c64"),    # above the tail, the whole adjoint from tables
    (16, 8, 1, "c128"),
    (16, 10, 1, "c128"),  # a tiled last layer
])
def test_fused_loss_above_the_tail(m, n, batch, dtype):
    print(f"[fused loss] m={m} n={n} {dtype} batch={batch}", flush=True)
    test_backward_gpu.test_fused_loss_backward_equals_two_calls(dtype, m, [int(v) for v in inputs.first_modes_input(m, n)], batch)
