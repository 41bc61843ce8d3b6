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


@pytest.mark.parametrize("M,n,m", [(16, 128, 88), (16, 128, 100), (16, 64, 172)])
def test_kronecker_rotation_of_several_tokens_is_as_precise_as_of_one(M, n, m):
    """Sums as long as the one-token kernel's leave the same rounding error (5 % for the order of the additions; with half
    as many sums, twice as long, it is 20 % larger)."""
    print(f"kron mfma precision M={M} {n}x{m}", flush=True)
    x = torch.from_numpy(rcp_synth.activation(25, f"kp{M}x{n}x{m}", M, n * m)).to(DEV).float()
    Q = rcp_synth.orthogonal(5, m)
    rot = rcp.Rotation.kron(n, torch.from_numpy(Q).to(DEV))
    ref = oracle.rotate(x.double().cpu().numpy(), oracle.ROT_KRON, n, m, Q.astype(np.float64))
    together = rcp.rotate_act(x, rot).double().cpu().numpy()
    apart = np.stack([rcp.rotate_act(x[i], rot)[0].double().cpu().numpy() for i in range(M)])
    assert np.linalg.norm(together - ref) <= 1.05 * np.linalg.norm(apart - ref)


@pytest.mark.parametrize("H_q,H_kv,S,tokens", [
    (2, 2, 1, 512),        # one token: three wavefronts without work
    (4, 2, 63, 512), (6, 2, 64, 512), (8, 2, 65, 512),   # 2, 3 and 4 query heads per cache head around one chunk
    (10, 2, 255, 512), (16, 2, 257, 512),                # 5 and 8 heads, around one chunk of each wavefront
    (12, 1, 513, 512), (16, 1, 1100, 512),               # 9 to 16 heads, several splits
    (20, 1, 300, 1024), (36, 2, 700, 2048),              # more than sixteen query heads: several workgroups per cache head
    (64, 4, 2100, 0), (32, 8, 5000, 0), (8, 8, 20000, 0),  # automatic split length: 256, 512, 512
])
@pytest.mark.parametrize("q_dtype", [torch.float16, torch.float32, torch.bfloat16])
def test_attention_of_grouped_heads_on_the_matrix_cores(H_q, H_kv, S, tokens, q_dtype):
    """Query and weights enter the matrix cores as pairs of binary16 numbers, codes exactly: the result is held to a few
    binary32 roundings of the largest term a row of the sum can hold (2^-20), far inside the stated 1e-3.  (What a large value
    without attention leaves of the small ones: test_a_large_value_without_attention_leaves_the_rest_precise.)"""
    print(f"kv4 mfma H_q={H_q} H_kv={H_kv} S={S} tokens={tokens} {q_dtype}", flush=True)
    cache = []
    for name, rotate in (("k", True), ("v", False)):
        c, p = rcp.kv4_new_cache(H_kv, S + 3, DEV)
        x = rcp_synth.kv_vectors(31, name, S, H_kv)
        if name == "v":  # value steps over twelve powers of two, growing and shrinking along the sequence
            x = (x * np.exp2(6 * np.sin(np.arange(S) / 40.0))[:, None, None]).astype(np.float16)
        rcp.kv4_append(torch.from_numpy(x).to(DEV), 0, c, p, rotate=rotate)
        cache += [c, p]
    q = torch.from_numpy(rcp_synth.query_vectors(31, f"q{H_q}", H_q)).to(DEV).to(q_dtype)
    rcp.set_option("kv_tokens", tokens)
    try:
        out = rcp.kv4_attn_decode(q, S, *cache, 0.3)   # sharp scores: the reference of the exponentials moves
    finally:
        rcp.set_option("reset", 0)
    host = [a.cpu().numpy() for a in cache]
    q64 = q.double().cpu().numpy()
    ref = oracle.kv4_attn_decode(q64, S, *host, 0.3)
    K, V = (np.abs(oracle.kv4_dequant(host[i], host[i + 1], 0, S)) for i in (0, 2))
    rep = H_q // H_kv
    for h in range(H_q):
        score = 0.3 * np.abs(q64[h]) @ (np.abs(K[:, h // rep]).max(axis=0))   # bound of |score|: relative error of a weight
        bound = (2.0 ** -20 * (1 + score)) * V[:, h // rep].max()
        assert np.abs(out[h].double().cpu().numpy() - ref[h]).max() <= bound, h


@pytest.mark.parametrize("H_q,H_kv", [(2, 2), (8, 2), (16, 2), (16, 1)])
@pytest.mark.parametrize("loud", [5, 900])
@pytest.mark.parametrize("ramp", [0.0, 40.0])   # scores that rise by about 32 along the sequence: the references move in every chunk
def test_a_large_value_without_attention_leaves_the_rest_precise(H_q, H_kv, loud, ramp):
    """One cached value 2^24 times as large as the others, at a token whose weight is below 1e-22: the error stays within a few
    binary32 roundings of the values that are attended to."""
    print(f"kv4 loud value H_q={H_q} H_kv={H_kv} loud={loud} ramp={ramp}", flush=True)
    S, scale = 2048, 0.05
    K, V = (rcp_synth.kv_vectors(71, n, S, H_kv).astype(np.float32) for n in "kv")
    K[..., 0], V = 0.0, V * 2.0 ** -10
    K[..., 1] += np.linspace(0, ramp, S)[:, None]
    K[loud], K[loud, :, 0], V[loud] = 0.0, -20.0, 3e4 * np.sign(V[loud])
    q = rcp_synth.query_vectors(71, f"q{H_q}", H_q).astype(np.float32)
    q[:, 0], q[:, 1] = 64.0, 16.0
    cache = []
    for x in (K, V):
        c, p = rcp.kv4_new_cache(H_kv, S, DEV)
        rcp.kv4_append(torch.from_numpy(x).to(DEV), 0, c, p)
        cache += [c, p]
    rcp.set_option("kv_tokens", 2048)
    try:
        out = rcp.kv4_attn_decode(torch.from_numpy(q).to(DEV), S, *cache, scale)
    finally:
        rcp.set_option("reset", 0)
    host = [a.cpu().numpy() for a in cache]
    ref = oracle.kv4_attn_decode(q.astype(np.float64), S, *host, scale)
    rest = np.arange(S) != loud
    K, V = (np.abs(oracle.kv4_dequant(host[i], host[i + 1], 0, S))[rest] for i in (0, 2))
    for h in range(H_q):
        score = scale * np.abs(q[h].astype(np.float64)) @ K[:, h * H_kv // H_q].max(axis=0)
        bound = 2.0 ** -20 * (1 + score) * V[:, h * H_kv // H_q].max()
        assert np.abs(out[h].double().cpu().numpy() - ref[h]).max() <= bound, h


@pytest.mark.parametrize("H_q,H_kv", [(8, 8), (8, 4), (16, 4), (16, 2)])
def test_sums_over_long_contexts_keep_their_precision(H_q, H_kv):
    """The average of 30000 values that nearly cancel.  A sum of centred codes walks about zero: its partial sums stay below
    sqrt(512) codes in a wavefront, so that roundings of 2^-24 of them and of the output (0.3 of a value's standard deviation)
    leave less than 2^-24 of the deviation: 0.2 to 0.4 of it here, 0.4 to 0.5 with sums over few tokens a lane on the vector
    unit.  Sums of the codes 0 .. 15 grow with every token: 0.9."""
    print(f"kv4 long context H_q={H_q} H_kv={H_kv}", flush=True)
    S, scale = 30000, 128 ** -0.5
    cache = []
    for name in ("k", "v"):
        c, p = rcp.kv4_new_cache(H_kv, S, DEV)
        rcp.kv4_append(torch.from_numpy(rcp_synth.kv_vectors(81, name, S, H_kv)).to(DEV), 0, c, p)
        cache += [c, p]
    q = torch.from_numpy(rcp_synth.query_vectors(81, f"q{H_q}", H_q)).to(DEV)
    rcp.set_option("kv_tokens", 2048)
    try:
        out = rcp.kv4_attn_decode(q, S, *cache, scale)
    finally:
        rcp.set_option("reset", 0)
    host = [a.cpu().numpy() for a in cache]
    ref = oracle.kv4_attn_decode(q.double().cpu().numpy(), S, *host, scale)
    V = oracle.kv4_dequant(host[2], host[3], 0, S).std(axis=0).repeat(H_q // H_kv, axis=0)
    err = (out.double().cpu().numpy() - ref) / V
    assert np.sqrt((err ** 2).mean()) <= 0.6 * 2.0 ** -24


def _attention_of_heads(q64, lengths, host, scale, heads, B, H_kv):
    """The oracle for some heads of every sequence, one query head per cache head."""
    for b in range(B):
        for h in heads:
            at = slice(b * H_kv + h, b * H_kv + h + 1)
            yield b, h, oracle.kv4_attn_decode(q64[b, h:h + 1], lengths[b], *[np.ascontiguousarray(a[at]) for a in host], scale)[0]


@pytest.mark.parametrize("H,lengths", [
    (32, [4095]), (32, [4096]), (32, [4097]),        # all loads at once up to here, the streaming form, the matrix-core form
    (32, [7500]), (32, [8192]), (16, [15361]),       # streaming: an odd number, all and one token of the last split
    (32, [430] * 8 + [257, 512, 300, 299, 64 * 6 + 1, 64 * 6 + 16, 64 * 6 + 17, 400]),   # its wavefronts with and without a last chunk
    (8, [1024] * 16), (32, [2048, 2047, 1985, 2033]), (64, [1797, 1900]),
    (48, [887, 1024, 513, 961, 1, 16, 17, 960, 1009, 1000]), (32, [1098] * 7),       # on 1024 tokens, in three splits
    (5, [52500]),                    # an odd number of heads
    (8, [81900]), (8, [81920]),      # splits of the most tokens, the last one not full and full
    (16, [600, 4000, 1, 2900, 1500]),
])
@pytest.mark.parametrize("q_dtype", [torch.float16, torch.float32, torch.bfloat16])
def test_attention_with_one_query_head_per_cache_head(H, lengths, q_dtype):
    print(f"kv4 one query head per cache head H={H} {lengths} {q_dtype}", flush=True)
    B, S, scale = len(lengths), max(lengths), 0.2
    cache = []
    for name in ("k", "v"):
        c, p = rcp.kv4_new_cache(B * H, S + 2, DEV)
        for b, n in enumerate(lengths):
            rcp.kv4_append(torch.from_numpy(rcp_synth.kv_vectors(91 + b, name, n, H)).to(DEV), 0, c[b * H:(b + 1) * H], p[b * H:(b + 1) * H])
        cache += [c, p]
    q = torch.from_numpy(np.stack([rcp_synth.query_vectors(91 + b, f"q{H}", H) for b in range(B)])).to(DEV).to(q_dtype)
    if B == 1:
        out = rcp.kv4_attn_decode(q[0], S, *cache, scale)[None]
        rotated = rcp.kv4_rotate_attn_decode(q[0], S, *cache, scale)
        apart = rcp.kv4_attn_decode(rcp.rotate_act(q[0], rcp.Rotation.wht(128)), S, *cache, scale)
        assert torch.equal(rotated, apart)
    else:
        out = rcp.kv4_attn_decode_batched(q, lengths, *cache, scale)
    host, q64 = [a.cpu().numpy() for a in cache], q.double().cpu().numpy()
    for b, h, ref in _attention_of_heads(q64, lengths, host, scale, (0, H // 2, H - 1), B, H):
        K, V = (np.abs(oracle.kv4_dequant(host[i][b * H + h:b * H + h + 1], host[i + 1][b * H + h:b * H + h + 1], 0, lengths[b])) for i in (0, 2))
        score = scale * np.abs(q64[b, h]) @ K[:, 0].max(axis=0)
        # as in test_attention_of_grouped_heads_on_the_matrix_cores
        assert np.abs(out[b, h].double().cpu().numpy() - ref).max() <= 2.0 ** -20 * (1 + score) * V.max(), (b, h)


@pytest.mark.parametrize("rep", [2, 4, 8, 16])
def test_query_heads_of_a_cache_head_do_not_touch_each_other(rep):
    """One head with an infinite element, one with a NaN and one 2^30 times as large as the rest leave the other heads of
    their cache head what they are without them."""
    print(f"kv4 mfma independent heads rep={rep}", flush=True)
    S, H_kv = 700, 4
    cache = []
    for name in ("k", "v"):
        c, p = rcp.kv4_new_cache(H_kv, S, DEV)
        rcp.kv4_append(torch.from_numpy(rcp_synth.kv_vectors(61, name, S, H_kv)).to(DEV), 0, c, p)
        cache += [c, p]
    q = torch.from_numpy(rcp_synth.query_vectors(61, f"q{rep}", rep * H_kv)).float().to(DEV)
    bad = q.clone()
    bad[0, 5], bad[rep, 7] = float("inf"), float("nan")
    bad[2 * rep] *= 2.0 ** 30
    rcp.set_option("kv_tokens", 512)
    try:
        want, got = (rcp.kv4_attn_decode(x, S, *cache, 0.1).cpu() for x in (q, bad))
    finally:
        rcp.set_option("reset", 0)
    changed = {0, rep, 2 * rep}
    for h in range(rep * H_kv):
        assert h in changed or torch.equal(got[h], want[h]), h
    assert not torch.isfinite(got[0]).any() and not torch.isfinite(got[rep]).any()


@pytest.mark.parametrize("N,K", [
    (8204, 512),     # groups one at a time; three blocks of rows per workgroup, the last workgroup ragged
    (4100, 2048),    # the most groups of that form, two blocks
    (4100, 2176),    # batches of four groups from here on: 17 groups, the last batch with one
    (8204, 4096),
    (1028, 8320),    # 65 groups: seventeen batches in two rounds, the third round of units one group wide
])
@pytest.mark.parametrize("M", [2, 4, 7, 9, 16])
def test_grouped_products_of_several_row_blocks(N, K, M):
    print(f"grouped gemm N={N} K={K} M={M}", flush=True)
    NG = K // 128
    idx = rcp_synth.random_indices(41, f"gb{N}x{K}", N, K)
    q = rcp_synth.random_int4(41 + M, f"gb{K}", M, K)
    rng = np.random.default_rng(41)
    cb = np.sort(rng.standard_normal((N // 4, NG, 4, 4)) * 0.03, axis=3).astype(np.float16)
    sc = (np.abs(rng.standard_normal(M)) * 0.2 + 0.05).astype(np.float16)
    xq = ((q[:, 0::2].astype(np.uint8) & 0xF) | ((q[:, 1::2].astype(np.uint8) & 0xF) << 4)).astype(np.uint8)
    packed = oracle.pack_indices_grouped(idx)
    ref, P = oracle.w2a4_gemv_grouped(packed, cb.view(np.uint16).ravel(), N, K, xq, sc.view(np.uint16), M=M)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (packed, cb, xq, sc)]
    out = rcp.w2a4_gemm_grouped(dev[0], dev[1], N, K, dev[2], dev[3], M, out_dtype=torch.float32).cpu().numpy()
    lut = np.abs(cb.astype(np.float64)).transpose(0, 2, 1, 3).reshape(N, NG, 4)
    terms = np.abs(P.reshape(M, N, NG, 4).astype(np.float64))
    # binary32 multiply-adds on exact sums: at most 4 NG + 20 roundings, each relative to the magnitudes met so far (the
    # sums of the bit planes times differences of levels: up to twice the levels' own, and `spread`)
    cond = sc.astype(np.float64)[:, None] * np.einsum("mngl,ngl->mn", terms, lut)
    spread = sc.astype(np.float64)[:, None] * (8 * 128 * lut.max(axis=2).sum(axis=1))[None]
    assert np.all(np.abs(out - ref.reshape(M, N)) <= (4 * NG + 20) * 2.0 ** -24 * (2 * cond + spread))
    assert np.linalg.norm(out - ref.reshape(M, N)) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("N,K,M", [
    (16388, 1024, 16), (16388, 2176, 5),                    # five row blocks per workgroup: single groups, batches of four
    (24580, 4096, 3), (24580, 4096, 7),                     # seven, B operands of four and of eight tokens
    (28676, 2176, 2), (28676, 4096, 8), (28676, 2176, 16),  # eight, the last workgroup with one row group
    (33028, 8192, 16),                                      # the cap of eight: more workgroups than compute units, sixteen
])                                                          # wavefronts, the largest LDS
def test_grouped_products_of_many_row_blocks(N, K, M):
    print(f"grouped gemm N={N} K={K} M={M}", flush=True)
    NG, rng = K // 128, np.random.default_rng(47)
    rows = np.unique(np.r_[0:64, rng.integers(0, N, 512), N - 160:N])
    idx = rcp_synth.random_indices(47, f"mb{N}x{K}", N, K)
    q = rcp_synth.random_int4(47 + M, f"mb{K}", M, K)
    cb = np.sort(rng.standard_normal((N // 4, NG, 4, 4), dtype=np.float32) * 0.03, axis=3).astype(np.float16)
    sc = (np.abs(rng.standard_normal(M)) * 0.2 + 0.05).astype(np.float16)
    xq = ((q[:, 0::2].astype(np.uint8) & 0xF) | ((q[:, 1::2].astype(np.uint8) & 0xF) << 4)).astype(np.uint8)
    dev = [torch.from_numpy(a).to(DEV) for a in (oracle.pack_indices_grouped(idx), cb, xq, sc)]
    out = rcp.w2a4_gemm_grouped(dev[0], dev[1], N, K, dev[2], dev[3], M, out_dtype=torch.float32)[:, rows].cpu().numpy()
    lut = cb.astype(np.float64)[rows // 4, :, rows % 4]
    w = np.take_along_axis(lut, idx[rows].reshape(-1, NG, 128).astype(np.int64), axis=2).reshape(-1, K)
    ref = (q.astype(np.float64) @ w.T) * sc.astype(np.float64)[:, None]
    # as in test_grouped_products_of_several_row_blocks, with the sums of |q| for those of each level
    cond = (np.abs(q).astype(np.float64) @ np.abs(w).T) * sc.astype(np.float64)[:, None]
    spread = sc.astype(np.float64)[:, None] * (8 * 128 * np.abs(lut).max(axis=2).sum(axis=1))[None]
    assert np.all(np.abs(out - ref) <= (4 * NG + 20) * 2.0 ** -24 * (2 * cond + spread))
    assert np.linalg.norm(out - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("rows", [16, 44])
@pytest.mark.parametrize("M", [3, 8, 9, 12])   # one operand for both halves of q (a column per half) and two, with unused columns
def test_largest_sums_of_several_tokens_are_exact(M, rows):
    """Every q at an end of its range over the longest input, all weights at one level per row of a nibble: the sums
    |F| = 8 K and T / 2 - F are the largest that the accumulators, and the integers made of them, have to hold."""
    N, K = 48, 32768
    rcp.set_option("gemv_variant", 2)
    rcp.set_option("gemm_rows", rows)
    idx = np.empty((N, K), np.uint8)
    idx[:] = ((np.arange(N) + np.arange(N) // 4) % 4)[:, None]
    q = np.where(np.arange(M) % 2 == 0, -8, 7).astype(np.int8)[:, None] * np.ones((1, K), np.int8)
    xq = ((q[:, 0::2].astype(np.uint8) & 0xF) | ((q[:, 1::2].astype(np.uint8) & 0xF) << 4)).astype(np.uint8)
    cb = np.tile(np.array([-2, -1, 1, 3], np.float16), (N, 1))
    packed = torch.from_numpy(oracle.pack_indices(idx)).to(DEV)
    try:
        out, P = rcp.w2a4_gemv(packed, torch.from_numpy(cb).to(DEV), N, K, torch.from_numpy(xq).to(DEV),
                               torch.ones(M, dtype=torch.float16, device=DEV), M, out_dtype=torch.float32, want_partial_sums=True)
    finally:
        rcp.set_option("reset", 0)
    want = np.zeros((M, N, 4), np.int64)
    for l in range(4):
        want[:, :, l] = np.where(idx[:, 0] == l, 1, 0)[None, :] * (q[:, :1].astype(np.int64) * K)
    assert np.array_equal(P.cpu().numpy().reshape(M, N, 4), want)
    assert np.array_equal(out.cpu().numpy(), (want * cb.astype(np.int64)[None]).sum(axis=2).astype(np.float32))


@pytest.mark.parametrize("K", [512, 2176, 4096])   # groups one at a time, batches of four with a rest, whole batches
@pytest.mark.parametrize("M", [3, 8, 16])
def test_the_four_rows_of_a_nibble_are_computed_alike(K, M):
    """Rows of equal weights and levels give equal bits, whichever bit of the nibble holds them, at levels far apart (sums of
    levels that need more than 24 bits)."""
    print(f"grouped gemm equal rows K={K} M={M}", flush=True)
    N, NG = 48, K // 128
    idx = np.repeat(rcp_synth.random_indices(43, f"er{K}", N // 4, K), 4, axis=0)
    q = rcp_synth.random_int4(43 + M, f"er{K}", M, K)
    rng = np.random.default_rng(43)
    levels = (rng.standard_normal((N // 4, NG, 1, 4)) * np.exp2(rng.integers(-12, 8, (N // 4, NG, 1, 4)))).astype(np.float16)
    cb = np.ascontiguousarray(np.repeat(levels, 4, axis=2))
    sc = np.ones(M, np.float16)
    xq = ((q[:, 0::2].astype(np.uint8) & 0xF) | ((q[:, 1::2].astype(np.uint8) & 0xF) << 4)).astype(np.uint8)
    dev = [torch.from_numpy(a).to(DEV) for a in (oracle.pack_indices_grouped(idx), cb, xq, sc)]
    out = rcp.w2a4_gemm_grouped(dev[0], dev[1], N, K, dev[2], dev[3], M, out_dtype=torch.float32).view(M, N // 4, 4)
    assert torch.equal(out, out[:, :, :1].expand_as(out))


@pytest.mark.parametrize("N,K", [(4100, 2176), (16420, 2304), (40, 8320)])   # two blocks of rows, five, one; ragged N and K
@pytest.mark.parametrize("M", [2, 8, 9, 16])
def test_per_group_sums_of_several_tokens_are_exact(N, K, M):
    print(f"grouped gemm sums N={N} K={K} M={M}", flush=True)
    NG, rows = K // 128, np.r_[0:8, N // 2:N // 2 + 8, N - 8:N]
    idx = rcp_synth.random_indices(45, f"ps{N}x{K}", N, K)
    q = rcp_synth.random_int4(45 + M, f"ps{K}", M, K)
    cb = np.sort(np.random.default_rng(45).standard_normal((N // 4, NG, 4, 4)) * 0.03, axis=3).astype(np.float16)
    xq = ((q[:, 0::2].astype(np.uint8) & 0xF) | ((q[:, 1::2].astype(np.uint8) & 0xF) << 4)).astype(np.uint8)
    dev = [torch.from_numpy(a).to(DEV) for a in (oracle.pack_indices_grouped(idx), cb, xq, np.ones(M, np.float16))]
    out, P = rcp.w2a4_gemm_grouped(dev[0], dev[1], N, K, dev[2], dev[3], M, out_dtype=torch.float32, want_partial_sums=True)
    onehot = (idx[rows].reshape(-1, NG, 128)[None, ..., None] == np.arange(4))
    want = (q.reshape(M, 1, NG, 128, 1).astype(np.int32) * onehot).sum(axis=3)
    assert np.array_equal(P.view(M, N, NG, 4)[:, rows].cpu().numpy(), want)
    lut = cb.astype(np.float64).transpose(0, 2, 1, 3).reshape(N, NG, 4)[rows]
    ref = (want * lut).sum(axis=(2, 3))
    assert np.linalg.norm(out[:, rows].cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
    # eight wavefronts stand for up to sixteen here: the same bits as without the sums
    assert torch.equal(out, rcp.w2a4_gemm_grouped(dev[0], dev[1], N, K, dev[2], dev[3], M, out_dtype=torch.float32))


@pytest.mark.parametrize("n", [15, 16, 17, 32, 47])   # a workgroup takes sixteen vectors of any heads, then sixteen tokens of one
@pytest.mark.parametrize("rotate", [False, True])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
def test_appended_prompts_are_exact(n, rotate, dtype):
    """Codes, steps and zero points byte for byte, at magnitudes from steps below the smallest binary16 number to quotients
    beyond binary32 (there the quantiser divides)."""
    print(f"kv4 append n={n} rotate={rotate} {dtype}", flush=True)
    H, pos = 5, 3
    x = rcp_synth.kv_vectors(51, f"prompt{n}", n, H).astype(np.float32)
    x *= np.exp2(np.linspace(-30, 8 if dtype == torch.float16 else 30, n)).astype(np.float32)[:, None, None]
    if not rotate:
        x[1, 1], x[2, 2] = (6e4, -6e4) if dtype == torch.float16 else (3e38, -3e38)   # constant vectors: step 1
        x[3, 3, ::2] = x[1, 1, 0]
    xd = torch.from_numpy(x).to(DEV).to(dtype)
    codes, params = rcp.kv4_new_cache(H, n + 5, DEV)
    rcp.kv4_append(xd, pos, codes, params, rotate=rotate)
    rc, rp = oracle.kv4_new_cache(H, n + 5)
    oracle.kv4_append(xd.float().cpu().numpy(), pos, 0.95, rc, rp, rotate=rotate)
    assert np.array_equal(params.cpu().numpy(), rp)
    assert np.array_equal(codes.cpu().numpy(), rc)
