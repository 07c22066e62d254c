"""The policy's forward pass at the edges of its row blocks of 16 and where its launch changes
(2048 rows), with the output apart from the input and over it.

Tolerance: the network rounds the operands of its products to BF16 as the oracle does and sums
in FP32 where the oracle sums in FP64; a sum near a rounding boundary can flip a BF16 value by
2^-9 of it, rare enough for 1e-3 in the relative L2 norm.  The launches per layer run the same
products in the same order: the same bits.
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
