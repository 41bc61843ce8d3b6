"""The native argument checks of the Python binding (csrc/binding.cpp), as far as they need no GPU: what does not fit is a
ValueError before any call into the library, and the public signatures keep their defaults."""
import inspect

import numpy as np
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
                                         1.0), "one length per sequence"),
    (lambda: rcp.kv4_append_batched(X.view(1, 1, K), [1, 2], P, P), "one position per sequence"),
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


def test_lengths_have_a_length():
    with pytest.raises(TypeError):
        rcp.kv4_append_batched(Q, iter([1]), CODES, PARAMS)


def test_public_signatures_keep_their_defaults():
    p = inspect.signature(rcp.quant_w2a4_gemv).parameters
    assert list(p)[:6] == ["packed", "codebook", "N", "K", "x", "clip_ratio"] and p["out_dtype"].default is torch.float16
    assert inspect.signature(rcp.kv4_append).parameters["clip_ratio"].default == 0.95


def test_an_output_type_left_to_torch():
    """out_dtype=None is torch's default type: float32 is an output type (the next check is the one that fires), float64 is not."""
    call = lambda: rcp.quant_w2a4_gemv(P, C, N, K, X, out_dtype=None)
    with pytest.raises(ValueError, match="must be a contiguous CUDA tensor"):
        call()
    torch.set_default_dtype(torch.float64)
    try:
        with pytest.raises(ValueError, match="out must be float16 or float32"):
            call()
    finally:
        torch.set_default_dtype(torch.float32)


@pytest.mark.gpu
@pytest.mark.parametrize("as_position", [float, np.int64, np.float32, lambda n: torch.tensor(n)])
def test_positions_are_whatever_int_takes(as_position):
    S, H = 3, 2
    x = torch.randn((S, H, 128), generator=torch.Generator().manual_seed(1)).cuda()
    a, b = (rcp.kv4_new_cache(H, S + 2, "cuda") + rcp.kv4_new_cache(H, S + 2, "cuda") for _ in range(2))
    rcp.kv4_append(x, 2, a[0], a[1])
    rcp.kv4_append_kv(x, x, 1, *a)
    want = rcp.kv4_attn_decode(x[0], S, *a, 0.1)
    rcp.kv4_append(x, as_position(2), b[0], b[1])
    rcp.kv4_append_kv(x, x, as_position(1), *b)
    got = rcp.kv4_attn_decode(x[0], as_position(S), *b, 0.1)
    assert all(torch.equal(u, v) for u, v in zip(a, b)) and torch.equal(want, got)
    rcp.kv4_append_batched(x[:1], [as_position(0)], a[0], a[1])
    many = rcp.kv4_attn_decode_batched(x[:1], [as_position(S)], *a, 0.1)
    assert torch.equal(many[0], rcp.kv4_attn_decode(x[0], S, *a, 0.1))
    with pytest.raises((TypeError, ValueError)):
        rcp.kv4_append(x, "two", a[0], a[1])


def _layer(seed):
    """Weights of one small layer (two calls with its output in between) and a key / value cache with some tokens."""
    g = torch.Generator().manual_seed(seed)
    n, k, h = 512, 512, 4
    part = torch.full((n, 3), 1 / 3).cuda()
    packed, codebook = rcp.pack_weights((torch.randn((n, k), generator=g) * 0.02).cuda().half(), torch.full((n,), -0.04).cuda(),
                                        torch.full((n,), 0.04).cuda(), part)
    caches = rcp.kv4_new_cache(h, 40, "cuda") + rcp.kv4_new_cache(h, 40, "cuda")
    for i in (0, 2):
        rcp.kv4_append(torch.randn((30, h, 128), generator=g).cuda(), 0, caches[i], caches[i + 1])
    return packed, codebook, n, k, caches


def _step(layer, x, out):
    """x -> product -> as key, value and query of one more token -> attention output, all on the current stream."""
    packed, codebook, n, k, caches = layer
    rcp.quant_w2a4_gemv(packed, codebook, n, k, x, 0.9, out=out[0])
    token = out[0].view(1, 4, 128)
    rcp.kv4_append_kv(token, token, 30, *caches, rotate_k=True)
    rcp.kv4_rotate_attn_decode(token[0], 31, *caches, 0.1, out=out[1], workspace=out[2])


def _buffers():
    return [torch.zeros((1, 512), dtype=torch.float16, device="cuda"), torch.zeros((4, 128), device="cuda"),
            torch.zeros(rcp.kv4_workspace_bytes(4, 40), dtype=torch.uint8, device="cuda")]


@pytest.mark.gpu
def test_calls_run_on_the_current_stream():
    """On a side stream that first keeps the GPU busy and then writes the input: a call on any other stream would read the
    old input (the default stream is idle meanwhile)."""
    layer, x, new = _layer(3), torch.zeros(512, device="cuda"), torch.randn(512, generator=torch.Generator().manual_seed(4)).cuda()
    want, got = _buffers(), _buffers()
    _step(layer, new, want)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)   # some 10 ms
        x.copy_(new)
        _step(layer, x, got)
    side.synchronize()
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1]) and got[1].abs().max() > 0


@pytest.mark.gpu
def test_calls_can_be_captured():
    """One captured step, replayed on new inputs with eager work between the replays."""
    layer, x, out = _layer(5), torch.zeros(512, device="cuda"), _buffers()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        _step(layer, x, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        _step(layer, x, out)
    g = torch.Generator().manual_seed(6)
    for _ in range(4):
        new, want = torch.randn(512, generator=g).cuda(), _buffers()
        x.copy_(new)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in out[:2]]
        _step(layer, new, want)
        torch.cuda.synchronize()
        assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1]) and got[1].abs().max() > 0
