"""Kernels that only several tokens reach, at the sizes where they can go wrong."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_15779_amd as rcp
import rcp_synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,n,m,dtype", [
    (4, 64, 172, torch.float16),    # the fewest tokens of the 7B down input that take the matrix-core form; ragged last block
    (16, 64, 100, torch.bfloat16),  # last block of four columns, last group of four j
    (2, 64, 256, torch.float32),    # the largest m: whole blocks, two rounds of loads per wavefront
    (16, 128, 92, torch.float16),   # two row-tile sets
    (9, 128, 100, torch.float32),
])
def test_kronecker_rotation_of_several_tokens_on_the_matrix_cores(M, n, m, dtype):
    print(f"kron mfma M={M} {n}x{m} {dtype}", flush=True)
    K = n * m
    x = torch.from_numpy(rcp_synth.activation(21, f"kt{M}x{K}", M, K)).to(DEV).to(dtype)
    Q = rcp_synth.orthogonal(3, m)
    y = rcp.rotate_act(x, rcp.Rotation.kron(n, torch.from_numpy(Q).to(DEV))).cpu().numpy().astype(np.float64)
    x64 = x.double().cpu().numpy()
    ref = oracle.rotate(x64, oracle.ROT_KRON, n, m, Q.astype(np.float64))
    # binary32 sums of m products, then log2(n) butterfly levels and the norm: each rounds relative to the token's norm
    bound = (m + np.log2(n) + 2) * 2.0 ** -24 * np.linalg.norm(x64, axis=1, keepdims=True)
    assert np.all(np.abs(y - ref) <= bound)
