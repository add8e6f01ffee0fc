"""The gate network's fused inference against the oracle's own layers (training
and inference forward share a kernel, so comparing them with each other pins
neither), and a training pass whose weight-gradient workgroups take several
samples of a lattice that is staged in more than one batch."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import test_gpu_cnn as cnn_tests  # noqa: E402
from oracle import cnn  # noqa: E402
from paper_1302_2669_amd import gate  # noqa: E402
from paper_1302_2669_amd.inputs import cnn_init, uniform_rates, uniform_syndromes  # noqa: E402

SEED = 0x1302266900000A90


def setup_module(module):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")


# one sample; full and partial groups and 16-pixel tiles; one sample per group
@pytest.mark.parametrize("L,B", [(2, 1), (2, 17), (3, 37), (8, 50), (13, 23), (17, 9), (25, 3)])
def test_inference_matches_oracle(L, B):
    # the oracle rounds at the kernel's own points, so only roundings of values at
    # a tie differ: 1% of the logit scale, as for the training forward
    syn = uniform_syndromes(L, B, SEED + 31 * L + B, density=0.15)
    p = uniform_rates(B, SEED + B)
    prm = cnn_init(L, SEED + 6)
    prm += np.random.default_rng(SEED + 7).normal(0.0, 0.05, size=prm.size).astype(np.float32)
    got, _ = gate.infer(L, torch.from_numpy(prm).cuda(), torch.from_numpy(syn).cuda(),
                        torch.from_numpy(p).cuda())
    torch.cuda.synchronize()
    ref, _ = cnn.forward(L, cnn.unflatten(L, prm.astype(np.float64)), syn, p.astype(np.float64))
    got = got.cpu().numpy().astype(np.float64)[:, :7]
    scale = np.abs(ref).max() + 1.0
    assert np.abs(got - ref).max() <= 0.01 * scale
    # and no sample has another's logits
    if B > 1:
        assert np.abs(got[0] - got[1]).max() > 0.01 * np.abs(ref[0] - ref[1]).max() > 0


def test_training_pass_of_several_samples_per_workgroup():
    layers = cnn_tests.run_layers(17, 140, SEED)
    cnn_tests.test_forward_layers(layers)
    cnn_tests.test_backward_layers(layers)
