"""Gradients of one batch, formed again and again, bit for bit: every element
of the data gradients' on-chip operands has one writer between two barriers, so
no order of the waves shows in the result.  At one sample, one tile, the
training batch and with a second tile per workgroup, beside work on another
stream that shifts the waves against one another."""
import numpy as np
import pytest

from paper_2606_08039_amd import md
from test_gpu_mlp import _data, _init, _norm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 16, 4096, 16400])
def test_repeated_backward_is_bitwise_equal(B):
    import torch
    rng = np.random.default_rng(B)
    X, T = _data(rng, B)
    m = md.md_mlp_create(B)
    other, busy = torch.cuda.Stream(), torch.ones((512, 512), device="cuda")
    try:
        md.md_mlp_set_params(m, _init(rng))
        md.md_mlp_set_norm(m, _norm(rng))
        Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
        md.md_mlp_forward(m, Xd)
        md.md_mlp_backward(m, Td)
        ref, loss = md.md_mlp_get_grads(m), md.md_mlp_loss(m)
        assert np.isfinite(ref).all() and np.abs(ref).max() > 0
        for rep in range(40):
            if rep % 2:
                with torch.cuda.stream(other):
                    busy.mul_(1.0)
            md.md_mlp_backward(m, Td)
            got = md.md_mlp_get_grads(m)
            np.testing.assert_array_equal(got, ref, err_msg="batch %d, pass %d" % (B, rep))
            assert md.md_mlp_loss(m) == loss
    finally:
        md.md_mlp_destroy(m)
