"""The gate network's training passes where their tilings change: one and
several samples per workgroup, a ragged last row of partial sums, ragged
sample groups, and lattices on both sides of the one-batch staging of a
weight-gradient sample.  Every layer is checked against the fp64 reference
with the layer tests' own bounds."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import test_gpu_cnn as cnn_tests  # noqa: E402

# L, batch: smallest lattice and batches; 9 samples per row, the last row with
# 3, and 5 per forward workgroup; staging in one batch (up to L = 13) and in
# two to four; L = 25
CASES = [(2, 1), (2, 2), (3, 1101), (16, 9), (17, 9), (24, 3), (25, 5)]


@pytest.mark.parametrize("L,B", CASES)
def test_training_pass(L, B):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    cnn_tests.say(f"training pass L={L} B={B}")
    layers = cnn_tests.run_layers(L, B, cnn_tests.SEED + 1000 * L + B)
    cnn_tests.test_input_planes_exact(layers)
    cnn_tests.test_forward_layers(layers)
    cnn_tests.test_backward_layers(layers)
