"""The native argument checks of the Python binding (csrc/binding.cpp), as far as they need no GPU: what does not fit is a
ValueError before any call into the library, and the public signatures keep their defaults."""
import inspect

import pytest
import torch

import paper_2502_15779_amd as rcp

N, K = 8, 128
P, C = torch.zeros(N * K // 4, dtype=torch.uint8), torch.zeros((N, 4), dtype=torch.float16)
X, XQ, S = torch.zeros(K), torch.zeros(K // 2, dtype=torch.uint8), torch.zeros(1, dtype=torch.float16)
OUT = torch.zeros((1, N), dtype=torch.float16)


@pytest.mark.parametrize("call, message", [
    (lambda: rcp.w2a4_gemv(P, C, N, K, XQ, S, out=OUT), "packed must be a contiguous CUDA tensor"),
    (lambda: rcp.w2a4_gemv(P[1:], C, N, K, XQ, S, out=OUT), "packed / codebook buffers do not match N, K"),
    (lambda: rcp.w2a4_gemv(P, C, N, K, XQ, S, out=OUT.to(torch.bfloat16)), "out must be float16 or float32"),
    (lambda: rcp.w2a4_gemv(P, C, N, K, XQ, S, out=None, out_dtype=torch.int8), "out must be float16 or float32"),
    (lambda: rcp.quant_w2a4_gemv(P, C, N, K, X[1:], out=OUT), "x must hold K values"),
    (lambda: rcp.quant_w2a4_gemv("P", C, N, K, X, out=OUT), "packed must be a contiguous CUDA tensor"),
    (lambda: rcp.quant_w3a4_gemv(P, C, N, K, X, out=OUT), "packed / codebook buffers do not match N, K"),
    (lambda: rcp.quant_w2a4_gemv_grouped(P, C, N, K, X.double(), out=OUT), "x must hold K values"),
    (lambda: rcp.w2a4_gemm_grouped(P, C, N, K, XQ, S, 2, out=OUT), "out must be float16 or float32 with M"),
    (lambda: rcp.rotate_act(X.double()), "x must be float16, bfloat16 or float32"),
    (lambda: rcp.pack_weights(torch.zeros(N, K), X[:N], X[:N], X[:N]), "clip_lo must be a contiguous CUDA tensor"),
    (lambda: rcp.kv4_append(X.view(1, 1, K)[..., :64], 0, P, P), "x must be contiguous"),
    (lambda: rcp.kv4_append(X.view(1, 1, K), 0, P, P), "codes must be uint8"),
    (lambda: rcp.kv4_attn_decode_batched(X.view(1, 1, K), [1, 2], *[torch.zeros((2, 4, n), dtype=torch.uint8) for n in (64, 4, 64, 4)],
                                         1.0), "must be a contiguous CUDA tensor|one length per sequence"),
])
def test_arguments_that_do_not_fit_are_value_errors(call, message):
    with pytest.raises(ValueError, match=message):
        call()


BIG = 2 ** 32   # a multiple of what 32 bits hold: the low half of BIG + n is n
Q, CODES, PARAMS = torch.zeros((1, 1, K)), torch.zeros((1, 4, 64), dtype=torch.uint8), torch.zeros((1, 4, 4), dtype=torch.uint8)


@pytest.mark.parametrize("call", [
    lambda: rcp.w2a4_gemv(P, C, BIG + N, K, XQ, S, out=OUT),
    lambda: rcp.w2a4_gemv(P, C, N, BIG + K, XQ, S, out=OUT),
    lambda: rcp.w2a4_gemv(P, C, N, K, XQ, S, BIG + 1, out=OUT),
    lambda: rcp.w2a4_gemv(P, C, N - BIG, K, XQ, S, out=OUT),
    lambda: rcp.w2a4_gemv(P, C, 2 ** 70 + N, K, XQ, S, out=OUT),
    lambda: rcp.w2a4_gemm_grouped(P, C, N, K, XQ, S, 1, group=BIG + 128, out=OUT),
    lambda: rcp.pack_weights_grouped(torch.zeros(N, K), X[:N], X[:N], X[:3 * N], group=BIG + 128),
    lambda: rcp.kv4_append_batched(Q, [BIG], CODES, PARAMS),
    lambda: rcp.kv4_attn_decode_batched(Q, [-BIG + 1], CODES, PARAMS, CODES, PARAMS, 1.0),
    lambda: rcp.kv4_attn_decode_batched(Q, [2 ** 70], CODES, PARAMS, CODES, PARAMS, 1.0),
])
def test_numbers_beyond_32_bits_are_not_cut(call):
    with pytest.raises(ValueError, match="32-bit"):
        call()


def test_public_signatures_keep_their_defaults():
    p = inspect.signature(rcp.quant_w2a4_gemv).parameters
    assert list(p)[:6] == ["packed", "codebook", "N", "K", "x", "clip_ratio"] and p["out_dtype"].default is torch.float16
    assert inspect.signature(rcp.kv4_append).parameters["clip_ratio"].default == 0.95
