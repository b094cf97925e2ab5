"""The loss of large batches: squared errors are formed in float32 (three
roundings of 2^-24 each) and added in double, so the mean agrees with the same
float32 squares added exactly to a few 2^-53, and with float64 squares to
4 x 2^-24 = 2.4e-7.  Equal targets make a float32 chain's roundings add up
instead of averaging out."""
import numpy as np
import pytest

from paper_2606_08039_amd import md

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 4096, 100000, 1 << 20])
def test_loss_is_summed_in_double(B):
    import torch
    print("batch %d" % B, flush=True)
    m = md.md_mlp_create(B)
    try:
        md.md_mlp_set_params(m, np.zeros(md.MLP_NPARAMS, np.float32))  # every output 0, identity scales
        t = np.float32(0.3173)
        X = torch.zeros((B, 64), device="cuda")
        T = torch.full((B, 6), float(t), device="cuda")
        md.md_mlp_forward(m, X)
        md.md_mlp_backward(m, T)
        assert md.md_mlp_loss(m) == pytest.approx(float(t) ** 2, rel=2.4e-7)
    finally:
        md.md_mlp_destroy(m)
