"""The policy's passes at the edges of their row blocks of 16 and where the launch changes
(2048 rows): the forward pass with the output apart from the input and over it, the gradient and
loss with one batch split of the weight gradients and with two.

Tolerances: the network rounds the operands of its products to BF16 as the oracle does and sums
in FP32 where the oracle sums in FP64; a sum near a rounding boundary can flip a BF16 value by
2^-9 of it, rare enough for 1e-3 in the relative L2 norm, and for 1e-2 in each tensor of the gradient,
whose errors are rounded to BF16 in every layer on the way back as well.  The output over the
input is the same kernel: the same bits.
"""

import ctypes

import numpy as np
import pytest

from oracle import oracle as O
from tests.parity_utils import f32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 63, 65, 2031, 2033, 2048, 2049])
def test_forward_at_row_block_edges(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_10469_amd import binding as B

    pol = B.Policy(max_batch=2112, seed=rows)
    X = np.random.default_rng(rows).normal(size=(rows, 40)).astype(np.float32)
    out = pol.forward(torch.as_tensor(X).cuda())
    ref = O.mlp_forward(pol.get_params().cpu().numpy().astype(np.float64), f32(X), bf16=True)
    got = out.cpu().numpy()
    assert np.linalg.norm(got - ref) <= 1e-3 * np.linalg.norm(ref)
    # the output written over the input
    buf = torch.zeros(rows * 144, device="cuda")
    buf[: rows * 40] = torch.as_tensor(X).cuda().reshape(-1)
    ptr = ctypes.c_void_p(buf.data_ptr())
    assert B.lib().mppi_policy_forward(pol.h, ptr, rows, ptr) == 0
    torch.cuda.synchronize()
    assert torch.equal(buf.reshape(rows, 144), out)


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 63, 65, 128, 129, 192, 257])
def test_gradient_and_loss_at_row_block_edges(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_10469_amd import binding as B

    pol = B.Policy(max_batch=320, seed=rows)
    rng = np.random.default_rng(rows)
    X, Y = (rng.normal(size=(rows, n)).astype(np.float32) for n in (40, 72))
    loss, grad = pol.grad(torch.as_tensor(X).cuda(), torch.as_tensor(Y).cuda())
    P = pol.get_params().cpu().numpy().astype(np.float64)
    want, ref = O.mlp_grad(P, f32(X), f32(Y), bf16=True)
    got = grad.cpu().numpy().astype(np.float64)
    assert abs(float(loss) - want) <= 1e-3 * abs(want)
    off = 0
    for fi, fo in zip(O.MLP_DIMS[:-1], O.MLP_DIMS[1:]):
        for n in (fi * fo, fo):
            assert np.linalg.norm(got[off:off + n] - ref[off:off + n]) <= 1e-2 * np.linalg.norm(ref[off:off + n])
            off += n
    assert torch.equal(loss, pol.nll(torch.as_tensor(X).cuda(), torch.as_tensor(Y).cuda()))
