"""The network's outputs written over its inputs: the workgroups read and write
different rows at different times, so outputs that overlap the inputs are put
in place after all of them have read.  Bitwise the outputs of separate buffers,
at the start of the inputs, inside them, across their end and before them, and
the gradients of the kept pass with them."""
import numpy as np
import pytest

from paper_2606_08039_amd import md
from test_gpu_mlp import _data, _init, _norm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 17, 1000, 4096, 20000])
def test_outputs_over_inputs(B):
    import torch
    rng = np.random.default_rng(B)
    X, T = _data(rng, B)
    m = md.md_mlp_create(B)
    try:
        md.md_mlp_set_params(m, _init(rng))
        md.md_mlp_set_norm(m, _norm(rng))
        Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
        ref = torch.empty((B, 6), device="cuda")
        md.md_mlp_forward(m, Xd, Y=ref)
        md.md_mlp_backward(m, Td)
        grads = md.md_mlp_get_grads(m)
        pad = 6 * B  # room before and after the inputs
        for at in (-6 * B + 5, -3, 0, 29 * B, 64 * B - 7, 64 * B):  # of the outputs, from the inputs' start
            for noalloc in ([False, True] if B <= md.MD_MLP_NOALLOC_MAX_BATCH else [False]):
                print("batch %d, outputs at %d, %s" % (B, at, "noalloc" if noalloc else "kept"), flush=True)
                buf = torch.zeros(2 * pad + 64 * B, device="cuda")
                x = buf[pad:pad + 64 * B].view(B, 64)
                x.copy_(Xd)
                y = buf[pad + at:pad + at + 6 * B].view(B, 6)
                if noalloc:
                    md.md_mlp_forward_noalloc(m, x, y)
                else:
                    md.md_mlp_forward(m, x, Y=y)
                    md.md_mlp_backward(m, Td)
                    np.testing.assert_array_equal(md.md_mlp_get_grads(m), grads)
                assert torch.equal(y, ref)
    finally:
        md.md_mlp_destroy(m)
