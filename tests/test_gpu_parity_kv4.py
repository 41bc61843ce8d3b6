"""GPU-vs-oracle parity of the 4-bit KV cache through the C ABI: codes, step sizes and zero points
bit-exact, attention outputs within 1e-3 of the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_15779_amd as rcp
import rcp_synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 128
TOL = 1e-3


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _say(msg):
    print(msg, flush=True)


@pytest.fixture(autouse=True)
def _auto_options():
    yield
    rcp.set_option("kv_tokens", 0)


def _as_dtype(x16, dtype):
    """(device tensor, the same values as float32 numpy)."""
    if dtype == "f16":
        return _t(x16), x16.astype(np.float32)
    if dtype == "f32":
        x32 = x16.astype(np.float32) * np.float32(1.0009765)
        return _t(x32), x32
    xb = _t(x16.astype(np.float32)).to(torch.bfloat16)
    return xb, xb.float().cpu().numpy()


def _oracle_cache(x32, S_max, pos=0, clip=0.95):
    codes, params = oracle.kv4_new_cache(x32.shape[1], S_max)
    oracle.kv4_append(x32, pos, clip, codes, params)
    return codes, params


@pytest.mark.parametrize("n,H,dtype", [(1, 1, "f16"), (1, 32, "f16"), (3, 5, "f32"), (17, 8, "bf16"), (300, 32, "f16"),
                                       (64, 3, "f32")])
def test_append_bit_exact(n, H, dtype):
    _say(f"kv4 append n={n} H={H} {dtype}")
    xd, x32 = _as_dtype(rcp_synth.kv_vectors(2, f"app{n}x{H}", n, H), dtype)
    S_max, pos = n + 7, 4
    codes, params = rcp.kv4_new_cache(H, S_max, DEV)
    codes.fill_(0xEE)
    params.fill_(0x77)
    rcp.kv4_append(xd, pos, codes, params)
    torch.cuda.synchronize()
    rc, rp = oracle.kv4_new_cache(H, S_max)
    rc[:], rp[:] = 0xEE, 0x77
    oracle.kv4_append(x32, pos, 0.95, rc, rp)
    assert np.array_equal(params.cpu().numpy(), rp)
    assert np.array_equal(codes.cpu().numpy(), rc)


def test_append_values_on_rounding_boundaries_and_degenerate_groups():
    _say("kv4 append boundaries")
    rng = np.random.default_rng(3)
    n, H = 40, 4
    x = np.zeros((n, H, D), dtype=np.float32)
    for i in range(n):
        for h in range(H):
            step = np.float32(2.0 ** rng.integers(-6, 3))
            base = np.float32(rng.integers(-40, 10)) * step
            k = rng.integers(0, 16, size=D).astype(np.float32)
            k[:2] = (0, 15)
            half = rng.integers(0, 2, size=D).astype(np.float32) * np.float32(0.5)   # exact ties: round half to even
            half[:2] = 0
            x[i, h] = base + step * (k + half)
    x[0, 0] = 0.0                 # zero range
    x[1, 1] = -7.25               # constant group
    x[2, 2] = 6.0e4               # large constant
    x[3, 3, :] = 1e-9             # step underflows in fp16
    x[3, 3, 5] = -1e-9
    for clip in (1.0, 0.95, 0.5):
        codes, params = rcp.kv4_new_cache(H, n, DEV)
        rcp.kv4_append(_t(x), 0, codes, params, clip_ratio=clip)
        torch.cuda.synchronize()
        rc, rp = _oracle_cache(x, n, clip=clip)
        assert np.array_equal(params.cpu().numpy(), rp)
        assert np.array_equal(codes.cpu().numpy(), rc)


@pytest.mark.parametrize("n,H,dtype", [(1, 1, "f16"), (1, 32, "f16"), (5, 3, "f32"), (33, 8, "bf16"), (200, 32, "f16")])
def test_rotated_append_bit_exact(n, H, dtype):
    """rotate = 1: the order-128 Hadamard transform of every head vector (R3 on the keys), then the quantiser."""
    _say(f"kv4 rotated append n={n} H={H} {dtype}")
    xd, x32 = _as_dtype(rcp_synth.kv_vectors(13, f"rot{n}x{H}", n, H), dtype)
    codes, params = rcp.kv4_new_cache(H, n + 2, DEV)
    rcp.kv4_append(xd, 1, codes, params, rotate=True)
    torch.cuda.synchronize()
    rc, rp = oracle.kv4_new_cache(H, n + 2)
    oracle.kv4_append(x32, 1, 0.95, rc, rp, rotate=True)
    assert np.array_equal(params.cpu().numpy(), rp)
    assert np.array_equal(codes.cpu().numpy(), rc)


def test_rotated_queries_and_keys_through_the_whole_path():
    """q and k rotated online (rcp_rotate_act over the 32 query head vectors, rotate = 1 in the append), values
    as they are: against the oracle doing the same, and close to attention over the unquantised vectors."""
    _say("kv4 whole path with R3")
    H, S = 32, 600
    k = rcp_synth.kv_vectors(14, "k", S, H)
    v = rcp_synth.kv_vectors(14, "v", S, H)
    q = rcp_synth.query_vectors(14, "q", H)
    kc, kp = rcp.kv4_new_cache(H, S, DEV)
    vc, vp = rcp.kv4_new_cache(H, S, DEV)
    rcp.kv4_append(_t(k), 0, kc, kp, rotate=True)
    rcp.kv4_append(_t(v), 0, vc, vp)
    q_rot = rcp.rotate_act(_t(q), rcp.Rotation.wht(D))           # 32 rows of 128
    out = rcp.kv4_attn_decode(q_rot, S, kc, kp, vc, vp, 1.0 / np.sqrt(D))
    torch.cuda.synchronize()
    rkc, rkp = oracle.kv4_new_cache(H, S)
    rvc, rvp = oracle.kv4_new_cache(H, S)
    oracle.kv4_append(k.astype(np.float32), 0, 0.95, rkc, rkp, rotate=True)
    oracle.kv4_append(v.astype(np.float32), 0, 0.95, rvc, rvp)
    q64 = oracle.rotate(q.astype(np.float64), oracle.ROT_WHT, D, 1)
    ref = oracle.kv4_attn_decode(q64, S, rkc, rkp, rvc, rvp, 1.0 / np.sqrt(D))
    got = out.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= TOL * (1.0 + np.abs(ref)))
    # the rotation leaves q . k unchanged, so the result stays near full-precision attention (4-bit noise only)
    k64, v64, qf = k.astype(np.float64), v.astype(np.float64), q.astype(np.float64)
    sc = np.einsum("hd,thd->ht", qf, k64) / np.sqrt(D)
    p = np.exp(sc - sc.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    full = np.einsum("ht,thd->hd", p, v64)
    assert np.linalg.norm(got - full) <= 0.1 * np.linalg.norm(full)


def test_append_token_by_token_equals_one_call():
    _say("kv4 append incremental")
    H, n = 8, 21
    x = _t(rcp_synth.kv_vectors(4, "inc", n, H))
    c1, p1 = rcp.kv4_new_cache(H, 32, DEV)
    c2, p2 = rcp.kv4_new_cache(H, 32, DEV)
    rcp.kv4_append(x, 5, c1, p1)
    for i in range(n):
        rcp.kv4_append(x[i:i + 1], 5 + i, c2, p2)
    rcp.kv4_append(x[:0], 0, c2, p2)          # nothing to append
    torch.cuda.synchronize()
    assert torch.equal(c1, c2) and torch.equal(p1, p2)


def _build_cache(seed, S, H_kv, S_max):
    k = rcp_synth.kv_vectors(seed, "k", S, H_kv)
    v = rcp_synth.kv_vectors(seed, "v", S, H_kv)
    kc, kp = rcp.kv4_new_cache(H_kv, S_max, DEV)
    vc, vp = rcp.kv4_new_cache(H_kv, S_max, DEV)
    rcp.kv4_append(_t(k), 0, kc, kp)
    rcp.kv4_append(_t(v), 0, vc, vp)
    torch.cuda.synchronize()
    return kc, kp, vc, vp


def _check_attention(q_dev, q64, S, cache, scale, out_dtype=torch.float32, heads=None):
    kc, kp, vc, vp = cache
    out = rcp.kv4_attn_decode(q_dev, S, kc, kp, vc, vp, scale, out_dtype=out_dtype)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    host = [a.cpu().numpy() for a in cache]
    if heads is None:
        ref = oracle.kv4_attn_decode(q64, S, *host, scale)
    else:       # sampled query heads (full-size case)
        rep = q64.shape[0] // host[0].shape[0]
        ref = np.stack([oracle.kv4_attn_decode(q64[h:h + 1], S, *[np.ascontiguousarray(a[h // rep:h // rep + 1]) for a in host],
                                               scale)[0] for h in heads])
        got = got[heads]
    tol = TOL if out_dtype == torch.float32 else 2 * TOL
    bound = tol * (1.0 + np.abs(ref))
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - ref) <= bound), float(np.max(np.abs(got - ref) / (1.0 + np.abs(ref))))


@pytest.mark.parametrize("H_q,H_kv,S,S_max", [(1, 1, 1, 1), (2, 2, 3, 8), (4, 4, 63, 64), (4, 4, 64, 64), (4, 4, 65, 70),
                                              (8, 8, 257, 300), (32, 32, 700, 1024), (32, 8, 333, 400), (16, 2, 1500, 1500),
                                              (3, 1, 5000, 5003), (1, 1, 9000, 9000), (1, 1, 70001, 70001), (32, 32, 8200, 8200)])
@pytest.mark.parametrize("q_dtype", ["f16", "f32", "bf16"])
def test_attention_matches_oracle(H_q, H_kv, S, S_max, q_dtype):
    _say(f"kv4 attn H_q={H_q} H_kv={H_kv} S={S} S_max={S_max} {q_dtype}")
    cache = _build_cache(5, S, H_kv, S_max)
    qd, q32 = _as_dtype(rcp_synth.query_vectors(5, f"q{H_q}", H_q), q_dtype)
    _check_attention(qd, q32.astype(np.float64), S, cache, 1.0 / np.sqrt(D))


@pytest.mark.parametrize("tokens", [64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("H_q,H_kv,S", [(4, 4, 1), (4, 2, 130), (8, 8, 1000), (2, 1, 3333), (2, 2, 17), (1, 1, 2049), (2, 1, 5000)])
@pytest.mark.parametrize("q_dtype", ["f16", "f32", "bf16"])
def test_attention_every_split_length(tokens, H_q, H_kv, S, q_dtype):
    # every (query type, tokens per workgroup) instantiation of the per-split kernel, and the matrix-core form on longer splits
    _say(f"kv4 attn tokens/workgroup={tokens} H_q={H_q} H_kv={H_kv} S={S} {q_dtype}")
    cache = _build_cache(11, S, H_kv, S + 3)
    qd, q32 = _as_dtype(rcp_synth.query_vectors(11, f"q{H_q}", H_q), q_dtype)
    rcp.set_option("kv_tokens", tokens)
    _check_attention(qd, q32.astype(np.float64), S, cache, 1.0 / np.sqrt(D))


def test_attention_reads_only_the_first_S_tokens_and_fp16_output():
    _say("kv4 attn prefix / fp16 out")
    H, S_max = 4, 512
    cache = _build_cache(6, S_max, H, S_max)
    qd, q32 = _as_dtype(rcp_synth.query_vectors(6, "q", H), "f16")
    for S in (1, 100, 320, 512):
        _check_attention(qd, q32.astype(np.float64), S, cache, 0.09)
    _check_attention(qd, q32.astype(np.float64), 200, cache, 0.09, out_dtype=torch.float16)


@pytest.mark.parametrize("tokens", [0, 512])
def test_attention_peaked_and_flat_score_distributions(tokens):
    _say(f"kv4 attn peaked / flat, tokens/workgroup={tokens}")
    rcp.set_option("kv_tokens", tokens)
    H, S = 4, 900
    cache = _build_cache(7, S, H, S)
    K = oracle.kv4_dequant(cache[0].cpu().numpy(), cache[1].cpu().numpy(), 0, S)
    # a query along one key: scores of several hundred, one weight near 1
    q = (3.0 * K[123]).astype(np.float16)
    _check_attention(_t(q), q.astype(np.float64), S, cache, 1.0)
    # zero query: uniform weights
    z = np.zeros((H, D), dtype=np.float16)
    _check_attention(_t(z), z.astype(np.float64), S, cache, 1.0)
    # large negative and positive scores in different splits
    q = (-2.0 * K[800]).astype(np.float16)
    _check_attention(_t(q), q.astype(np.float64), S, cache, 1.0)


def test_attention_full_size_sampled_heads():
    # LLaMA-2-7B: 32 heads of 128, 4096 cached tokens; the oracle checks four of the 32 heads
    _say("kv4 attn full size")
    H, S = 32, 4096
    cache = _build_cache(8, S, H, S)
    qd, q32 = _as_dtype(rcp_synth.query_vectors(8, "q", H), "f16")
    _check_attention(qd, q32.astype(np.float64), S, cache, 1.0 / np.sqrt(D), heads=[0, 7, 18, 31])


@pytest.mark.parametrize("q_dtype", ["f32", "bf16"])
def test_attention_full_size_as_benchmarked(q_dtype):
    # the call of bench.py's chained decoder-layer step: binary32 (rotated) queries of 32 heads over 4096 cached
    # tokens, automatic split length (256 tokens per workgroup); the oracle checks four of the 32 heads
    _say(f"kv4 attn full size, {q_dtype} queries, automatic split")
    H, S = 32, 4096
    cache = _build_cache(12, S, H, S)
    qd, q32 = _as_dtype(rcp_synth.query_vectors(12, "q", H), q_dtype)
    _check_attention(qd, q32.astype(np.float64), S, cache, 1.0 / np.sqrt(D), heads=[1, 9, 22, 30])


def test_workspace_is_reusable_and_too_small_is_refused():
    _say("kv4 attn workspace")
    H, S = 4, 300
    cache = _build_cache(9, S, H, S)
    qd, q32 = _as_dtype(rcp_synth.query_vectors(9, "q", H), "f16")
    need = rcp.kv4_workspace_bytes(H, S)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)     # NaN bit patterns: nothing may be read before written
    a = rcp.kv4_attn_decode(qd, S, *cache, 0.1, workspace=ws)
    b = rcp.kv4_attn_decode(qd, 40, *cache, 0.1, workspace=ws)
    c = rcp.kv4_attn_decode(qd, S, *cache, 0.1, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(a, c) and torch.isfinite(b).all()
    with pytest.raises(rcp.RcpError):
        rcp.kv4_attn_decode(qd, S, *cache, 0.1, workspace=ws[:need - 16])
    with pytest.raises(rcp.RcpError):
        rcp.kv4_attn_decode(qd, S + 1, *cache, 0.1)


# ---- several sequences at once -------------------------------------------------------------------------
def _pooled(seed, lengths, H_kv, S_max):
    """Pooled device caches of len(lengths) sequences filled through single-sequence appends, and the host
    copies per sequence for the oracle."""
    B = len(lengths)
    kc, kp = rcp.kv4_new_cache(B * H_kv, S_max, DEV)
    vc, vp = rcp.kv4_new_cache(B * H_kv, S_max, DEV)
    for b, S in enumerate(lengths):
        k = rcp_synth.kv_vectors(seed, f"k{b}", S, H_kv)
        v = rcp_synth.kv_vectors(seed, f"v{b}", S, H_kv)
        sl = slice(b * H_kv, (b + 1) * H_kv)
        rcp.kv4_append(_t(k), 0, kc[sl], kp[sl], rotate=True)
        rcp.kv4_append(_t(v), 0, vc[sl], vp[sl])
    torch.cuda.synchronize()
    return kc, kp, vc, vp


@pytest.mark.parametrize("lengths,H_q,H_kv,S_max", [([5], 4, 4, 8), ([1, 64, 65, 700], 8, 8, 700), ([300, 2, 129, 128, 127], 8, 2, 512),
                                                    ([1500] * 3 + [1], 32, 32, 1500), (list(range(1, 17)), 4, 4, 16),
                                                    ([2100, 40], 16, 4, 2100)])
@pytest.mark.parametrize("tokens", [0, 64, 256, 512, 1024])
def test_batched_attention_matches_the_oracle_sequence_by_sequence(lengths, H_q, H_kv, S_max, tokens):
    _say(f"kv4 batched attn lengths={lengths[:5]}.. H_q={H_q} H_kv={H_kv} tokens/workgroup={tokens}")
    B = len(lengths)
    cache = _pooled(20, lengths, H_kv, S_max)
    q16 = np.stack([rcp_synth.query_vectors(20, f"q{b}", H_q) for b in range(B)])
    rcp.set_option("kv_tokens", tokens)
    out = rcp.kv4_attn_decode_batched(_t(q16), lengths, *cache, 1.0 / np.sqrt(D))
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    host = [a.cpu().numpy() for a in cache]
    for b, S in enumerate(lengths):
        sl = slice(b * H_kv, (b + 1) * H_kv)
        ref = oracle.kv4_attn_decode(q16[b].astype(np.float64), S, *[np.ascontiguousarray(a[sl]) for a in host], 1.0 / np.sqrt(D))
        assert np.all(np.abs(got[b] - ref) <= TOL * (1.0 + np.abs(ref))), (b, S)
        if tokens:      # with the split length fixed, the batched rows are the single-sequence results
            single = rcp.kv4_attn_decode(_t(q16[b]), S, *[a[sl] for a in cache], 1.0 / np.sqrt(D))
            torch.cuda.synchronize()
            assert torch.equal(single, out[b])


def _random_pool(seed, heads, S_max):
    """Caches of arbitrary codes, steps 2^-4 .. 2^-2 and zero points 4 .. 11: (k codes, k params, v codes, v params)."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    pool = []
    for _ in range(2):
        pool.append(torch.randint(0, 256, (heads, S_max, 64), generator=g, device=DEV, dtype=torch.uint8))
        step = torch.exp2(-4 + 2 * torch.rand((heads, S_max), generator=g, device=DEV)).half()
        z = torch.randint(4, 12, (heads, S_max), generator=g, device=DEV, dtype=torch.int16)
        pool.append(torch.stack((step.view(torch.int16), z), dim=-1).view(torch.uint8))
    return pool


# more workgroups than compute units in a grid for the longest sequence: only splits with tokens have one, found from the lengths
@pytest.mark.parametrize("H_q,H_kv,lengths", [
    (32, 32, [1300, 1, 512, 513]), (40, 10, [3000, 1, 2, 511, 1024, 700, 5, 1536, 2999]), (32, 32, [2049, 256]),
    (20, 20, [600] * 7 + [1]), (160, 8, [1, 1025, 2500, 40, 40, 40, 512, 512]), (64, 32, [1, 2600, 1]),
    (32, 8, [97 * i + 1 for i in range(16)][::-1]), (64, 16, [3000] + [1] * 14 + [2999])])
def test_a_row_of_a_ragged_batch_is_the_single_call(H_q, H_kv, lengths):
    """At a fixed split length, bit for bit: the single calls take the plain grid."""
    _say(f"kv4 ragged batch H_q={H_q} H_kv={H_kv} lengths={lengths}")
    B = len(lengths)
    pool = _random_pool(H_q + B, B * H_kv, max(lengths) // 4 * 4 + 8)  # (each sequence's share of it aligned)
    q = torch.randn((B, H_q, D), generator=torch.Generator(device=DEV).manual_seed(B), device=DEV)
    rcp.set_option("kv_tokens", 512)
    assert -(-max(lengths) // 512) * H_kv * B > 256
    out = rcp.kv4_attn_decode_batched(q, lengths, *pool, 0.0625)
    for b, S in enumerate(lengths):
        assert torch.equal(out[b], rcp.kv4_attn_decode(q[b], S, *[a[b * H_kv:(b + 1) * H_kv] for a in pool], 0.0625)), (b, S)


@pytest.mark.parametrize("H_q,H_kv,lengths", [
    (32, 8, [4100, 300, 1, 2048, 5000]), (64, 32, [1700, 900]), (32, 4, [5000]), (32, 8, [9000]), (64, 16, [1000] * 15 + [17]),
    (32, 8, [319] * 4), (32, 8, [340, 320, 310, 310]), (32, 32, [300] + [65] * 15), (32, 32, [117] * 16), (32, 32, [117] * 15 + [130]),
    (64, 4, [480, 200]), (64, 4, [703, 1]), (64, 4, [1407, 1300]), (32, 4, [511, 512, 500, 500]), (32, 4, [512, 512, 512, 513]),   # around the
    (8, 1, [1747, 1600, 1700, 1726]), (20, 10, [1200, 1100]), (32, 16, [2047]), (32, 16, [2049]), (16, 4, [4095]), (16, 4, [4097]),   # forms' meeting
    (64, 8, [2047]), (64, 8, [2049])])                                                                                              # points
def test_attention_on_automatic_splits(H_q, H_kv, lengths):
    """The split length that the lengths ask for, against the oracle on the first and the last sequence's first and last heads."""
    _say(f"kv4 automatic splits H_q={H_q} H_kv={H_kv} lengths={lengths[:5]}")
    B = len(lengths)
    pool = _random_pool(7 * H_q + B, B * H_kv, max(lengths) + 3)
    q = torch.randn((B, H_q, D), generator=torch.Generator(device=DEV).manual_seed(H_kv), device=DEV)
    if B == 1:
        out = rcp.kv4_attn_decode(q[0], lengths[0], *pool, 0.0625).unsqueeze(0)
        apart = rcp.kv4_attn_decode(rcp.rotate_act(q[0], rcp.Rotation.wht(D)), lengths[0], *pool, 0.0625)
        assert torch.equal(rcp.kv4_rotate_attn_decode(q[0], lengths[0], *pool, 0.0625), apart)
    else:
        out = rcp.kv4_attn_decode_batched(q, lengths, *pool, 0.0625)
    got, q64, rep = out.cpu().numpy().astype(np.float64), q.cpu().numpy().astype(np.float64), H_q // H_kv
    for b in sorted({0, B - 1}):
        for h in (0, H_q - 1):
            k = b * H_kv + h // rep
            ref = oracle.kv4_attn_decode(q64[b, h:h + 1], lengths[b], *[np.ascontiguousarray(a[k:k + 1].cpu().numpy()) for a in pool], 0.0625)
            assert np.all(np.abs(got[b, h] - ref[0]) <= TOL * (1.0 + np.abs(ref[0]))), (b, h)


def test_batched_append_equals_single_appends():
    _say("kv4 batched append")
    B, H, S_max = 5, 8, 40
    positions = [0, 39, 7, 7, 20]
    x = rcp_synth.kv_vectors(21, "newtok", B, H)
    for rotate in (False, True):
        c1, p1 = rcp.kv4_new_cache(B * H, S_max, DEV)
        c2, p2 = rcp.kv4_new_cache(B * H, S_max, DEV)
        c1.fill_(0x5A), p1.fill_(0x33), c2.fill_(0x5A), p2.fill_(0x33)
        rcp.kv4_append_batched(_t(x), positions, c1, p1, rotate=rotate)
        for b in range(B):
            sl = slice(b * H, (b + 1) * H)
            rcp.kv4_append(_t(x[b:b + 1]), positions[b], c2[sl], p2[sl], rotate=rotate)
        torch.cuda.synchronize()
        assert torch.equal(c1, c2) and torch.equal(p1, p2)
        # and against the oracle for one of the sequences
        rc, rp = oracle.kv4_new_cache(H, S_max)
        rc[:], rp[:] = 0x5A, 0x33
        oracle.kv4_append(x[2:3].astype(np.float32), positions[2], 0.95, rc, rp, rotate=rotate)
        assert np.array_equal(c1[2 * H:3 * H].cpu().numpy(), rc) and np.array_equal(p1[2 * H:3 * H].cpu().numpy(), rp)
    with pytest.raises(rcp.RcpError):
        rcp.kv4_append_batched(_t(x), [0, 40, 1, 2, 3], c1, p1)


# ------------------------------------------------------------------------------------------
# fewer launches: keys and values appended together, rotation of the query and the merge of the splits
# inside the attention launch
# ------------------------------------------------------------------------------------------
@pytest.mark.parametrize("rotate_k", [False, True])
@pytest.mark.parametrize("n,H,dtype", [(1, 32, "f16"), (1, 1, "f32"), (5, 3, "bf16"), (70, 8, "f16")])
def test_append_kv_equals_the_two_appends(n, H, dtype, rotate_k):
    """rcp_kv4_append_kv: bit for bit the two rcp_kv4_append calls, and the oracle's codes and parameters."""
    _say(f"kv4 append_kv n={n} H={H} {dtype} rotate_k={rotate_k}")
    kd, k32 = _as_dtype(rcp_synth.kv_vectors(21, f"akv_k{n}x{H}", n, H), dtype)
    vd, v32 = _as_dtype(rcp_synth.kv_vectors(21, f"akv_v{n}x{H}", n, H), dtype)
    S_max, pos = n + 5, 3
    kc, kp = rcp.kv4_new_cache(H, S_max, DEV)
    vc, vp = rcp.kv4_new_cache(H, S_max, DEV)
    for t in (kc, kp, vc, vp):
        t.fill_(0x5A)
    rcp.kv4_append_kv(kd, vd, pos, kc, kp, vc, vp, rotate_k=rotate_k)
    torch.cuda.synchronize()
    for x32, rot, c, p in ((k32, rotate_k, kc, kp), (v32, False, vc, vp)):
        rc, rp = oracle.kv4_new_cache(H, S_max)
        rc[:], rp[:] = 0x5A, 0x5A
        oracle.kv4_append(x32, pos, 0.95, rc, rp, rotate=rot)
        assert np.array_equal(p.cpu().numpy(), rp)
        assert np.array_equal(c.cpu().numpy(), rc)
    kc2, kp2 = rcp.kv4_new_cache(H, S_max, DEV)
    kc2.fill_(0x5A)
    kp2.fill_(0x5A)
    rcp.kv4_append(kd, pos, kc2, kp2, rotate=rotate_k)
    torch.cuda.synchronize()
    assert torch.equal(kc, kc2) and torch.equal(kp, kp2)


@pytest.mark.parametrize("tokens", [0, 128, 256, 1024])
@pytest.mark.parametrize("qdtype", ["f16", "f32", "bf16"])
@pytest.mark.parametrize("S,H_q,H_kv", [(1, 4, 4), (129, 8, 2), (600, 32, 32), (2100, 8, 8), (4096, 32, 8)])
def test_rotating_attention_equals_the_separate_launches(S, H_q, H_kv, qdtype, tokens):
    """rcp_kv4_rotate_attn_decode = rcp_rotate_act on the query followed by rcp_kv4_attn_decode, bit for bit, and within
    the tolerance of the oracle on queries it rotated itself."""
    _say(f"kv4 rotating attention S={S} H_q={H_q} H_kv={H_kv} {qdtype} kv_tokens={tokens}")
    rcp.set_option("kv_tokens", tokens)
    k = rcp_synth.kv_vectors(31, f"fk{S}", S, H_kv)
    v = rcp_synth.kv_vectors(31, f"fv{S}", S, H_kv)
    qd, q32 = _as_dtype(rcp_synth.query_vectors(31, f"fq{S}x{H_q}", H_q), qdtype)
    kc, kp = rcp.kv4_new_cache(H_kv, S, DEV)
    vc, vp = rcp.kv4_new_cache(H_kv, S, DEV)
    rcp.kv4_append_kv(_t(k), _t(v), 0, kc, kp, vc, vp, rotate_k=True)
    scale = 0.08838834764831845
    q_rot = rcp.rotate_act(qd, rcp.Rotation.wht(D))
    ref = rcp.kv4_attn_decode(q_rot, S, kc, kp, vc, vp, scale)
    ref16 = rcp.kv4_attn_decode(q_rot, S, kc, kp, vc, vp, scale, out_dtype=torch.float16)
    a = rcp.kv4_rotate_attn_decode(qd, S, kc, kp, vc, vp, scale)
    a16 = rcp.kv4_rotate_attn_decode(qd, S, kc, kp, vc, vp, scale, out_dtype=torch.float16)
    torch.cuda.synchronize()
    assert torch.equal(a, ref) and torch.equal(a16, ref16), "query rotation inside the kernel differs from rcp_rotate_act"
    # against the oracle (its own rotation of the query, in binary32 as the kernels do)
    ok, okp = oracle.kv4_new_cache(H_kv, S)
    ov, ovp = oracle.kv4_new_cache(H_kv, S)
    oracle.kv4_append(k.astype(np.float32), 0, 0.95, ok, okp, rotate=True)
    oracle.kv4_append(v.astype(np.float32), 0, 0.95, ov, ovp)
    qr = np.stack([oracle.fwht_f32(q32[h]) for h in range(H_q)])
    want = oracle.kv4_attn_decode(qr, S, ok, okp, ov, ovp, scale)
    got = a.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - want) <= TOL * (1.0 + np.abs(want)))


def test_rotating_attention_full_size_as_benchmarked():
    """32 heads x 4096 cached tokens, fp16 query rotated inside the kernel: the bits of the path with the rotation as a
    launch of its own, on a workspace filled with NaN patterns beforehand."""
    H, S = 32, 4096
    k = rcp_synth.kv_vectors(41, "full_k", S, H)
    v = rcp_synth.kv_vectors(41, "full_v", S, H)
    q = _t(rcp_synth.query_vectors(41, "full_q", H))
    kc, kp = rcp.kv4_new_cache(H, S, DEV)
    vc, vp = rcp.kv4_new_cache(H, S, DEV)
    rcp.kv4_append_kv(_t(k), _t(v), 0, kc, kp, vc, vp, rotate_k=True)
    scale = 0.08838834764831845
    ref = rcp.kv4_attn_decode(rcp.rotate_act(q, rcp.Rotation.wht(D)), S, kc, kp, vc, vp, scale)
    ws = torch.empty(rcp.kv4_workspace_bytes(H, S), dtype=torch.uint8, device=DEV)
    for _ in range(3):
        ws.fill_(0xFF)   # NaN patterns: nothing stale may be read
        out = rcp.kv4_rotate_attn_decode(q, S, kc, kp, vc, vp, scale, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
