"""The network's fused kernels at the sizes where a tile, a pass or a slice
ends: one sample, around the 16-sample tile and the 32-sample chunk, around the
256-sample slice, more tiles than workgroups (a second pass of the chain
kernels) and slices longer than eight chunks; and an input that is not
16-byte aligned.

Tolerances: activations and gradients are rounded to bfloat16 (relative
2^-9) in front of every product, with the oracle rounding the forward operands
alike; an fp32 sum that ends on the other side of a rounding boundary moves
one operand by 2^-8, averaged over 64-128 terms, so outputs agree to 2e-3 in
the norm, and the gradients, whose backward operands the oracle does not
round, to 2e-2 per block."""
import numpy as np
import pytest

import oracle as orc
from paper_2606_08039_amd import md
from test_gpu_mlp import _data, _init, _norm, _oracle_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 32, 33, 255, 257, 8209, 33000])
def test_step_matches_oracle(B):
    import torch
    print("batch %d" % B, flush=True)
    rng = np.random.default_rng(B)
    flat, norm = _init(rng), _norm(rng)
    X, T = _data(rng, B)
    m = md.md_mlp_create(B + 40)  # the kept rows' stride follows the batch, not the largest one
    try:
        md.md_mlp_set_params(m, flat)
        md.md_mlp_set_norm(m, norm)
        Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
        # a larger call first: what it leaves behind must not be read
        md.md_mlp_forward(m, torch.ones((B + 40, 64), device="cuda"))
        md.md_mlp_backward(m, torch.ones((B + 40, 6), device="cuda"))
        Yd = torch.full((B, 6), float("nan"), device="cuda")
        md.md_mlp_forward(m, Xd, Y=Yd)
        md.md_mlp_backward(m, Td)
        grads, loss = md.md_mlp_get_grads(m).astype(np.float64), md.md_mlp_loss(m)
        got = Yd.cpu().numpy()
    finally:
        md.md_mlp_destroy(m)
    Y, Ystd, acts, Ws, bs, Xused = _oracle_forward(flat, norm, X)
    assert np.linalg.norm((got - Y) / norm[134:140]) < 2e-3 * np.linalg.norm(Ystd)
    Tstd = (T.astype(np.float64) - norm[128:134]) / norm[134:140]
    dWs, dbs, _ = orc.mlp_backward(Ws, bs, Xused, acts, 2.0 * (Ystd - Tstd) / (B * 6))
    for i, (a, b) in enumerate(zip(md.mlp_unflatten(grads), [x for pair in zip(dWs, dbs) for x in pair])):
        assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b), i
    assert loss == pytest.approx(np.mean((Ystd - Tstd) ** 2), rel=1e-2)


def test_unaligned_input():
    import torch
    rng = np.random.default_rng(7)
    m = md.md_mlp_create(100)
    try:
        md.md_mlp_set_params(m, _init(rng))
        md.md_mlp_set_norm(m, _norm(rng))
        X = torch.from_numpy(_data(rng, 100)[0]).cuda()
        shifted = torch.empty(100 * 64 + 1, device="cuda")[1:].view(100, 64)
        shifted.copy_(X)
        assert shifted.data_ptr() % 16 == 4
        Y = [torch.empty((100, 6), device="cuda") for _ in range(3)]
        md.md_mlp_forward(m, X, Y=Y[0])
        md.md_mlp_forward(m, shifted, Y=Y[1])
        md.md_mlp_forward_noalloc(m, shifted, Y[2])
        assert torch.equal(Y[0], Y[1]) and torch.equal(Y[0], Y[2])
    finally:
        md.md_mlp_destroy(m)
