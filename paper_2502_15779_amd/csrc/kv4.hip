// 4-bit KV cache (Appendix table of quantisation configurations: asymmetric, groups of 128 = one
// head vector, clipping ratio 0.95; the quantiser is Eqn. 1 with N = 4) and one-token attention
// over it (Section 2.1: R3 rotates queries and keys so that the cache can be held in 4 bits).
//
// Layout of one cached tensor (keys or values) of one layer, head size 128:
//   codes   [H][S_max][64 bytes]  element j of a head vector in byte j / 2, bits 4 * (j % 2) ...
//   params  [H][S_max] dwords     bits 0..15 the binary16 step s, bits 16..31 the int16 zero point z
// Head-major, so that the tokens one head attends to are contiguous: a wavefront reads 1 KiB
// (16 tokens) per load instruction.
#include <math.h>

#include <type_traits>

#include "kv4_plan.hpp"
#include "rcp_internal.hpp"

namespace rcp {

constexpr int KV_D = 128;

// Batched calls: per-sequence lengths (attention) or positions (append) travel by value.
struct KvBatch {
    int v[RCP_MAX_M];
    int H_q, H_kv;
    int n;                 // sequences,
    int first[RCP_MAX_M];  // and in a compact grid the first workgroup of each (beyond the last one: the number of all)
};

// ---------------------------------------------------------------------------------------
// append: quantise n_tokens x H head vectors into cache positions pos ...
// Sixteen lanes (one DPP row) own a head vector, eight consecutive elements each.
// ROT: the vector first goes through the normalised order-128 Hadamard transform: butterflies in
// ascending stride order (1, 2, 4 in registers, 8 .. 64 between the sixteen lanes), each output
// one IEEE add or subtract, then one multiplication by (float)(1/sqrt(128)).
//
// A prompt of thousands of tokens was bound by instruction issue, not by memory (2000 tokens of 8 heads, bf16 keys and
// values, are 10 MB: 2 us at the rate of a copy), so the quantiser runs without divisions and the exchanges between lanes
// are operands of the additions.  That launch: 6.7 -> 4.7 us; 2000 tokens of 32 heads 18.4 -> 13.1 us; one token of 32
// heads 2.8 -> 2.4 us.
// ---------------------------------------------------------------------------------------
// a / s, correctly rounded, for s with at most eleven significant bits and rs = 1 / s up to a unit in the last place: the
// residual a - q0 s of q0 = a rs is exact, so that q0 + (a - q0 s) rs misses the quotient by less than 2^-20 units in the
// last place before its rounding, while a quotient by an eleven-bit divisor is 2^-12 units away from every midpoint of
// two floats (it cannot be one: midpoint times divisor needs more than 24 bits).  Holds while q0 is finite; where the
// quotient underflows both round to the integer 0.
__device__ __forceinline__ float kv_quotient(float a, float s, float rs)
{
    const float q0 = __fmul_rn(a, rs);
    return __fmaf_rn(__fmaf_rn(-q0, s, a), rs, q0);
}

template <int CTRL>
__device__ __forceinline__ float kv_dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

struct KvCode {
    uint32_t word;   // eight codes of this lane
    uint32_t param;  // step and zero point of the vector
};

// Quantises the vector of a lane row from its eight elements per lane.  EXACT: divides; otherwise `far` is set where a
// quotient may overflow, and the caller starts again with the divisions.
template <int DT, bool ROT, bool EXACT>
__device__ __forceinline__ KvCode kv4_quantise_vector(const Raw8<DT>& raw, int l, float clip_ratio, bool& far)
{
    // every product and difference below is rounded on its own (hi_c - lo_c must not become a
    // fused multiply-add: for a constant vector it has to be exactly zero).  The pragma covers
    // the operators written in this body, hence plain * and - rather than the __f*_rn wrappers.
#pragma clang fp contract(off)
    float v[8];
    widen8<DT>(raw, v);
    if constexpr (ROT) {
        register_stages<3>(v, 0);
        // element stride 8 * m: the partner is lane l ^ m of the row.  partner - v in the upper lane of a pair is written
        // partner + (-v): one sign flip and one addition that reads the partner's lane
        auto stage = [&](int m, auto partner) {
            const uint32_t sign = (l & m) != 0 ? 0x80000000u : 0u;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = partner(v[e]) + __uint_as_float(__float_as_uint(v[e]) ^ sign);
        };
        stage(1, [](float z) { return kv_dpp<0xB1>(z); });                 // quad 1,0,3,2
        stage(2, [](float z) { return kv_dpp<0x4E>(z); });                 // quad 2,3,0,1
        stage(4, [](float z) { return kv_dpp<0x1B>(kv_dpp<0x141>(z)); });  // half row mirrored, quads mirrored back
        stage(8, [](float z) { return kv_dpp<0x128>(z); });                // row rotated by eight
        const float norm = 0.088388347648318440550f;  // (float)(1 / sqrt(128))
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = v[e] * norm;
    }
    float lo = v[0], hi = v[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) {
        lo = fminf(lo, v[j]);
        hi = fmaxf(hi, v[j]);
    }
#define RCP_ROW_MINMAX(ctrl)          \
    lo = fminf(lo, kv_dpp<ctrl>(lo)); \
    hi = fmaxf(hi, kv_dpp<ctrl>(hi))
    RCP_ROW_MINMAX(0x128);
    RCP_ROW_MINMAX(0x124);
    RCP_ROW_MINMAX(0x122);
    RCP_ROW_MINMAX(0x121);
#undef RCP_ROW_MINMAX
    const float lo_c = clip_ratio * lo, hi_c = clip_ratio * hi;
    const float range = hi_c - lo_c;
    // (an infinite range ends at the largest step either way)
    uint16_t sb = __half_as_ushort(round_to_half(EXACT ? __fdiv_rn(range, 15.0f) : kv_quotient(range, 15.0f, 0.066666670143604279f)));
    if ((sb & 0x7fffu) == 0) sb = 0x3c00u;
    if ((sb & 0x7fffu) >= 0x7c00u) sb = 0x7bffu;
    const float s = half_bits_to_float(sb);
    const float rs = __builtin_amdgcn_rcpf(s);
    far = !(fmaxf(fabsf(lo), fabsf(hi)) * rs < 1.0e38f);
    float zf = -rintf(EXACT ? __fdiv_rn(lo_c, s) : kv_quotient(lo_c, s, rs));
    zf = fminf(fmaxf(zf, -32768.0f), 32767.0f);
    const int z = static_cast<int>(zf);
    zf = static_cast<float>(z);
    float q[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        q[j] = __builtin_amdgcn_fmed3f(rintf(EXACT ? __fdiv_rn(v[j], s) : kv_quotient(v[j], s, rs)) + zf, 0.0f, 15.0f);
    // four codes as one exact integer below 2^16
    const float w0 = fmaf(q[3], 4096.0f, fmaf(q[2], 256.0f, fmaf(q[1], 16.0f, q[0])));
    const float w1 = fmaf(q[7], 4096.0f, fmaf(q[6], 256.0f, fmaf(q[5], 16.0f, q[4])));
    return {static_cast<uint32_t>(w0) | (static_cast<uint32_t>(w1) << 16),
            static_cast<uint32_t>(sb) | (static_cast<uint32_t>(z & 0xffff) << 16)};
}

template <int DT, bool ROT>
__device__ __forceinline__ KvCode kv4_quantise(const Raw8<DT>& raw, int l, float clip_ratio)
{
    bool far;
    KvCode c = kv4_quantise_vector<DT, ROT, false>(raw, l, clip_ratio, far);
    // uniform: the lanes of a row exchange values in there
    if (__builtin_expect(__any(far), 0)) c = kv4_quantise_vector<DT, ROT, true>(raw, l, clip_ratio, far);
    return c;
}

// Few tokens: sixteen consecutive (token, head) vectors per workgroup.
// BATCHED: row i of x belongs to sequence i (one new token each), whose cache starts at head
// i * H of the pooled cache and whose position is batch.v[i].
template <int DT, bool ROT, bool BATCHED>
__device__ __forceinline__ void kv4_append_rows(const void* __restrict__ x, int rows, int H, int S_max, int pos, float clip_ratio,
                                                uint32_t* __restrict__ codes, uint32_t* __restrict__ params, const KvBatch& batch,
                                                int block)
{
    const int row = block * 16 + (threadIdx.x >> 4);
    const int l = threadIdx.x & 15;
    const int rr = min(row, rows - 1);  // surplus lanes repeat the last vector and store nothing
    const Raw8<DT> raw = load8_raw<DT>(x, static_cast<size_t>(rr) * KV_D + 8 * l);
    const int i = rr / H, h = rr - i * H;
    const size_t slot = BATCHED ? static_cast<size_t>(rr) * S_max + batch.v[i]
                                : static_cast<size_t>(h) * S_max + (pos + i);
    const KvCode c = kv4_quantise<DT, ROT>(raw, l, clip_ratio);
    if (row < rows) {
        codes[slot * 16 + l] = c.word;
        if (l == 0) params[slot] = c.param;
    }
}

// Many tokens: sixteen consecutive tokens of one head per workgroup, so that its codes and parameters are contiguous in
// the cache (consecutive rows of x leave a parameter by itself in each 128-byte line).  Two or four vectors per lane with
// their loads side by side are slower throughout: there are enough wavefronts, and fewer of them hide less.
template <int DT, bool ROT>
__device__ __forceinline__ void kv4_append_tokens(const void* __restrict__ x, int n_tokens, int H, int S_max, int pos, float clip_ratio,
                                                  uint32_t* __restrict__ codes, uint32_t* __restrict__ params, int block, int h)
{
    const int i = block * 16 + (threadIdx.x >> 4);
    const int l = threadIdx.x & 15;
    const Raw8<DT> raw = load8_raw<DT>(x, (static_cast<size_t>(min(i, n_tokens - 1)) * H + h) * KV_D + 8 * l);
    const KvCode c = kv4_quantise<DT, ROT>(raw, l, clip_ratio);
    if (i < n_tokens) {
        const size_t slot = static_cast<size_t>(h) * S_max + (pos + i);
        codes[slot * 16 + l] = c.word;
        if (l == 0) params[slot] = c.param;
    }
}

// TOKENS: blockIdx = (block of tokens, head) instead of blocks of rows
template <int DT, bool ROT, bool BATCHED, bool TOKENS = false>
__global__ __launch_bounds__(256) void kv4_append_kernel(const void* __restrict__ x, int rows, int H, int S_max, int pos,
                                                         float clip_ratio, uint32_t* __restrict__ codes,
                                                         uint32_t* __restrict__ params, KvBatch batch)
{
    if constexpr (TOKENS) kv4_append_tokens<DT, ROT>(x, rows, H, S_max, pos, clip_ratio, codes, params, blockIdx.x, blockIdx.y);
    else kv4_append_rows<DT, ROT, BATCHED>(x, rows, H, S_max, pos, clip_ratio, codes, params, batch, blockIdx.x);
}

// The new keys and the new values of the same tokens in one launch: blockIdx.z = 0 quantises the keys (rotated when
// rotate_k is set), blockIdx.z = 1 the values (never rotated) -- the arithmetic of kv4_append_kernel on each.
template <int DT, bool TOKENS>
__global__ __launch_bounds__(256) void kv4_append_kv_kernel(const void* __restrict__ k, const void* __restrict__ v, int rows, int H,
                                                            int S_max, int pos, int rotate_k, float clip_ratio,
                                                            uint32_t* __restrict__ k_codes, uint32_t* __restrict__ k_params,
                                                            uint32_t* __restrict__ v_codes, uint32_t* __restrict__ v_params)
{
    auto append = [&](auto rot, const void* x, uint32_t* codes, uint32_t* params) {
        constexpr bool ROT = decltype(rot)::value;
        const KvBatch none = {};
        if constexpr (TOKENS) kv4_append_tokens<DT, ROT>(x, rows, H, S_max, pos, clip_ratio, codes, params, blockIdx.x, blockIdx.y);
        else kv4_append_rows<DT, ROT, false>(x, rows, H, S_max, pos, clip_ratio, codes, params, none, blockIdx.x);
    };
    if (blockIdx.z == 0 && rotate_k) append(std::true_type{}, k, k_codes, k_params);
    else if (blockIdx.z == 0) append(std::false_type{}, k, k_codes, k_params);
    else append(std::false_type{}, v, v_codes, v_params);
}

// ---------------------------------------------------------------------------------------
// one-token attention, split along the sequence.
// Workgroup (split, query head): L = 64, 128 or 256 cached tokens.  Four lanes own a token, 16 bytes (32
// elements) of its vector each; a wavefront covers 16 tokens per load, the workgroup 64.
//   pass 1  scores q . K_t (kept in registers), their maximum m
//   pass 2  p_t = exp(score_t - m), l = sum p_t, acc_j = sum_t p_t * V_tj
// and (m, l, acc) go to the workspace; kv4_combine_kernel merges the splits.
// With x_tj = s_t * (c_tj - z_t):  q . K_t = s_t * (sum_j q_j c_tj - z_t * sum_j q_j)  and
// sum_t p_t V_tj = sum_t (p_t s_t) c_tj - sum_t p_t s_t z_t, so the codes enter as plain integers.
//
// Register r = 8 d + 4 e + b of a lane stands for element 8 d + 2 b + e of its 32 (dword d of
// the 16 bytes, byte b, nibble e): the order in which the nibbles come out of two masks.
// ---------------------------------------------------------------------------------------
constexpr int KV_THREADS = 256;
constexpr int KV_PART = KV_D + 4;      // floats per partial result: acc[128], m, l, 2 unused

// The four low nibbles and the four high nibbles of a dword as bytes.  The empty asm keeps the
// compiler from folding the mask into each later byte extraction (a 4-bit field extract plus a
// conversion per element); with the bytes opaque, (x >> 8 b) & 0xff becomes one
// v_cvt_f32_ubyte<b> per element.
__device__ __forceinline__ void nibble_bytes(uint32_t w, uint32_t& lo, uint32_t& hi)
{
    lo = w & 0x0f0f0f0fu;
    hi = (w >> 4) & 0x0f0f0f0fu;
    asm("" : "+v"(lo), "+v"(hi));
}

// Four bytes b in 0..15 -> four floats b * unit in two instructions: read as FP8 (E4M3) numbers, the codes
// 0..7 are subnormals and 8..15 the first binade, both linear in b, so v_cvt_pk_f32_fp8 converts two at a
// time; `kv_fp8_unit()` is what it gives for the byte 1 (a power of two), divided out again by the callers.
typedef float v2f __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void bytes_to_floats(uint32_t x, float (&f)[4])
{
    const v2f a = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(x), false);
    const v2f b = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(x), true);
    f[0] = a[0];
    f[1] = a[1];
    f[2] = b[0];
    f[3] = b[1];
}

__device__ __forceinline__ float kv_fp8_unit() { return __builtin_amdgcn_cvt_pk_f32_fp8(1, false)[0]; }

__device__ __forceinline__ int kv_elem_of_reg(int r) { return 8 * (r >> 3) + 2 * (r & 3) + ((r >> 2) & 1); }

__device__ __forceinline__ float quad_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false));  // lanes 1,0,3,2
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, false));  // lanes 2,3,0,1
    return v;
}

// sum over the four tokens of a row of 16 lanes (lanes 4 apart hold the same piece)
__device__ __forceinline__ float row_tokens_sum(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, false));  // row_ror 4
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, false));  // row_ror 8
    return v;
}

// The query values of a lane (32 consecutive elements of a head vector, the four lanes of a quad hold all 128) through
// the normalised order-128 Hadamard transform: butterflies in ascending stride order (1 .. 16 in registers, 32 and 64
// between the lanes of the quad), each output one IEEE add or subtract, then one multiplication by (float)(1/sqrt(128)):
// bit for bit what rcp_rotate_act gives for a row of 128.
__device__ __forceinline__ void kv_rotate_query(float (&t)[32], int piece)
{
#pragma clang fp contract(off)
#pragma unroll
    for (int st = 1; st < 32; st <<= 1)
#pragma unroll
        for (int e = 0; e < 32; ++e)
            if ((e & st) == 0) {
                const float a = t[e], b = t[e + st];
                t[e] = a + b;
                t[e + st] = a - b;
            }
#pragma unroll
    for (int e = 0; e < 32; ++e) {  // stride 32: the partner is lane piece ^ 1 of the quad
        const float other = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t[e]), 0xB1, 0xf, 0xf, false));
        t[e] = (piece & 1) ? other - t[e] : t[e] + other;
    }
#pragma unroll
    for (int e = 0; e < 32; ++e) {  // stride 64: lane piece ^ 2
        const float other = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t[e]), 0x4E, 0xf, 0xf, false));
        t[e] = (piece & 2) ? other - t[e] : t[e] + other;
    }
    const float norm = 0.088388347648318440550f;  // (float)(1 / sqrt(128))
#pragma unroll
    for (int e = 0; e < 32; ++e) t[e] = t[e] * norm;
}

// The same with the four pieces of a head in lanes 16 apart (piece = lane / 16) instead of neighbouring ones.
__device__ __forceinline__ void kv_rotate_query_rows(float (&t)[32], int piece)
{
#pragma clang fp contract(off)
#pragma unroll
    for (int st = 1; st < 32; st <<= 1)
#pragma unroll
        for (int e = 0; e < 32; ++e)
            if ((e & st) == 0) {
                const float a = t[e], b = t[e + st];
                t[e] = a + b;
                t[e + st] = a - b;
            }
#pragma unroll
    for (int e = 0; e < 32; ++e) {  // stride 32; the swap leaves (value of the even row, value of the odd row) in every lane
        auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(t[e]), __float_as_uint(t[e]), false, false);
        const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
        t[e] = (piece & 1) ? a - b : a + b;
    }
#pragma unroll
    for (int e = 0; e < 32; ++e) {  // stride 64
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[e]), __float_as_uint(t[e]), false, false);
        const float a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
        t[e] = (piece & 2) ? a - b : a + b;
    }
    const float norm = 0.088388347648318440550f;  // (float)(1 / sqrt(128))
#pragma unroll
    for (int e = 0; e < 32; ++e) t[e] = t[e] * norm;
}

// This lane's 32 query values in register order (r = 8 d + 4 e + b <-> element 8 d + 2 b + e) and their sum.
template <int QDT>
__device__ __forceinline__ float kv_query_registers(const Raw8<QDT> (&qraw)[4], bool rotate, int piece, float (&qr)[32])
{
    float t[32];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        float t8[8];
        widen8<QDT>(qraw[d], t8);
#pragma unroll
        for (int e = 0; e < 8; ++e) t[8 * d + e] = t8[e];
    }
    if (rotate) kv_rotate_query(t, piece);  // uniform
    float qsum = 0.0f;
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                qr[8 * d + 4 * e + b] = t[8 * d + 2 * b + e];
                qsum += qr[8 * d + 4 * e + b];
            }
    return qsum;
}

// out_hj = sum_i e^(m_i - M) acc_ij / sum_i e^(m_i - M) l_i over the splits i of one head (src: its partial results).
// `groups` x 128 (virtual) threads: thread (g, j) merges the splits i = g, g + groups, ... of column j, four at a time so
// that their loads are in flight together, against its own running maximum; the groups meet in LDS and are merged the
// same way.
constexpr int KV_CT = 1024;
struct KvMergeLds {
    float red[KV_CT / KV_D][KV_D];
    float dred[KV_CT / KV_D], mred[KV_CT / KV_D];
};

// unit: log2(e) when the m_i are in units of e, 1 when they are powers of two.
__device__ __forceinline__ void kv_merge_head(const float* __restrict__ src, int splits, int groups, float unit, void* __restrict__ out,
                                              bool out_f16, int h, KvMergeLds& lds, int nthreads)
{
    auto power = [unit](float x) { return __builtin_amdgcn_exp2f(x * unit); };
    for (int vt = threadIdx.x; vt < groups * KV_D; vt += nthreads) {
        const int j = vt & (KV_D - 1), g = vt >> 7;
        float M = -INFINITY, num = 0.0f, den = 0.0f;
        for (int i0 = g; i0 < splits; i0 += 4 * groups) {
            float mi[4], li[4], ai[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = min(i0 + groups * u, splits - 1);
                mi[u] = *(src + i * KV_PART + KV_D);
                li[u] = *(src + i * KV_PART + KV_D + 1);
                ai[u] = *(src + i * KV_PART + j);
            }
            float mb = M;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + groups * u < splits) mb = fmaxf(mb, mi[u]);
            const float r = power(M - mb);  // 0 on the first round (M = -inf, mb finite)
            num *= r;
            den *= r;
            M = mb;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float e = (i0 + groups * u < splits) ? power(mi[u] - M) : 0.0f;
                num = fmaf(e, ai[u], num);
                den = fmaf(e, li[u], den);
            }
        }
        lds.red[g][j] = num;  // a group without a split leaves M = -inf, num = den = 0
        if (j == 0) {
            lds.dred[g] = den;
            lds.mred[g] = M;
        }
    }
    __syncthreads();
    if (threadIdx.x < KV_D) {
        const int tid = threadIdx.x;
        float Mt = lds.mred[0];
        for (int w = 1; w < groups; ++w) Mt = fmaxf(Mt, lds.mred[w]);
        float n = 0.0f, d = 0.0f;
        for (int w = 0; w < groups; ++w) {
            const float e = power(lds.mred[w] - Mt);
            n = fmaf(e, lds.red[w][tid], n);
            d = fmaf(e, lds.dred[w], d);
        }
        const float r = n / d;
        if (out_f16) static_cast<__half*>(out)[h * KV_D + tid] = __float2half_rn(r);
        else static_cast<float*>(out)[h * KV_D + tid] = r;
    }
}

// BATCHED: blockIdx.z is the sequence; its length is batch.v[z], its caches start at head z * H_kv of
// the pooled buffers, its query and partial results at row z * H_q; workgroups past its end leave.
// Which (split, query head, cache head) a workgroup works on.  Workgroups go to the eight dies (each with
// its own L2) in turn by their index, so the H_q / H_kv query heads that read the same cache head over the
// same split are given indices 8 apart: they run on one die at about the same time and the cache bytes come
// from HBM once instead of once per query head.  Unit u = (split, cache head); index = u % 8 + 8 * (rep * (u / 8) + r)
// for query head r of the group.  With rep = 1 this is the plain order.  False for the padding of the grid.
__device__ __forceinline__ bool kv_place(unsigned index, int splits, int rep, int H_kv, int& split, int& h, int& hk)
{
    const unsigned die = index & 7u, t = index >> 3;
    const unsigned r = t % static_cast<unsigned>(rep), k = t / static_cast<unsigned>(rep);
    const unsigned u = 8u * k + die;
    if (u >= static_cast<unsigned>(splits) * static_cast<unsigned>(H_kv)) return false;
    split = static_cast<int>(u % static_cast<unsigned>(splits));
    hk = static_cast<int>(u / static_cast<unsigned>(splits));
    h = hk * rep + static_cast<int>(r);
    return true;
}

// QROT: the query first goes through the order-128 Hadamard transform (R3), in the prologue, while the cache loads are
// in flight.
template <int QDT, int ITERS, bool BATCHED, bool QROT = false>
__global__ __launch_bounds__(KV_THREADS) void kv4_attn_kernel(const void* __restrict__ q, int S, int S_max, int rep, int splits,
                                                              float softmax_scale, const u32x4* __restrict__ k_codes,
                                                              const uint32_t* __restrict__ k_params,
                                                              const u32x4* __restrict__ v_codes,
                                                              const uint32_t* __restrict__ v_params,
                                                              float* __restrict__ part, KvBatch batch)
{
    __shared__ float red[4][KV_D];
    __shared__ float wmax[4], lrow[4][4], zrow[4][4];
    constexpr int L = 64 * ITERS;
    int split, h, hk;
    if (!kv_place(blockIdx.x, splits, rep, batch.H_kv, split, h, hk)) return;  // padding of the grid
    const int tid = threadIdx.x, slot = tid >> 2, piece = tid & 3, wave = tid >> 6;
    const int t0 = split * L;
    if constexpr (BATCHED) {
        const int seq = blockIdx.z;
        S = batch.v[seq];
        if (t0 >= S) return;  // the whole workgroup: this sequence has fewer splits
        h += seq * batch.H_q;
        hk += seq * batch.H_kv;
    }
    const int t_end = min(S, t0 + L);
    const size_t head_base = static_cast<size_t>(hk) * S_max;

    // every load of the workgroup is issued before the first use: the query, then the keys,
    // then the values (slots past the end repeat the last token and get weight 0)
    Raw8<QDT> qraw[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) qraw[d] = load8_raw<QDT>(q, static_cast<size_t>(h) * KV_D + 32 * piece + 8 * d);
    u32x4 kw[ITERS], vw[ITERS];
    uint32_t kp[ITERS], vp[ITERS];
    bool valid[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int t = t0 + it * 64 + slot;
        valid[it] = t < t_end;
        const size_t at = head_base + (valid[it] ? t : t_end - 1);
        // the cache is read once per call: loads with the non-temporal hint (6.6 -> 6.0 us at 1024 tokens, 13.2 -> 12.5 at
        // 8192, 57 -> 51 us for 16 sequences of 4096)
        kw[it] = __builtin_nontemporal_load(k_codes + (at * 4 + piece));
        kp[it] = __builtin_nontemporal_load(k_params + at);
    }
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int t = t0 + it * 64 + slot;
        const size_t at = head_base + (valid[it] ? t : t_end - 1);
        vw[it] = __builtin_nontemporal_load(v_codes + (at * 4 + piece));
        vp[it] = __builtin_nontemporal_load(v_params + at);
    }

    // this lane's 32 query values in register order (the softmax scale goes onto the score)
    float qr[32];
    const float qsum = kv_query_registers<QDT>(qraw, QROT, piece, qr);

    const float unit = kv_fp8_unit(), inv_unit = 1.0f / unit;
    const float scale_by_unit = softmax_scale * inv_unit, qsum_unit = qsum * unit;

    // ---- pass 1: scores (all four lanes of a token end up holding its score) ----
    float score[ITERS];
    float top = -INFINITY;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t lo, hi;
            nibble_bytes(kw[it][d], lo, hi);
            float fl[4], fh[4];
            bytes_to_floats(lo, fl);
            bytes_to_floats(hi, fh);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                dot[d] = fmaf(qr[8 * d + b], fl[b], dot[d]);
                dot[d] = fmaf(qr[8 * d + 4 + b], fh[b], dot[d]);
            }
        }
        // dot = unit * sum q c: the unit (a power of two) is taken out exactly
        const float s = half_bits_to_float(static_cast<uint16_t>(kp[it] & 0xffffu)) * scale_by_unit;
        const float z = static_cast<float>(static_cast<int>(kp[it]) >> 16);
        float sc = s * (((dot[0] + dot[1]) + (dot[2] + dot[3])) - z * qsum_unit);
        sc = quad_sum(sc);
        score[it] = valid[it] ? sc : -INFINITY;
        top = fmaxf(top, score[it]);
    }
    top = wave_max(top);
    if ((tid & 63) == 0) wmax[wave] = top;
    __syncthreads();
    const float m = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));

    // ---- pass 2: weights and the value sum ----
    float acc[32];
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[r] = 0.0f;
    float lsum = 0.0f, zacc = 0.0f;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const float p = __expf(score[it] - m);  // exp(-inf) = 0 for the surplus slots
        const float w0 = p * half_bits_to_float(static_cast<uint16_t>(vp[it] & 0xffffu));
        const float w = w0 * inv_unit;  // the converted codes carry the factor unit
        lsum += p;
        zacc = fmaf(w0, static_cast<float>(static_cast<int>(vp[it]) >> 16), zacc);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t lo, hi;
            nibble_bytes(vw[it][d], lo, hi);
            float fl[4], fh[4];
            bytes_to_floats(lo, fl);
            bytes_to_floats(hi, fh);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                acc[8 * d + b] = fmaf(w, fl[b], acc[8 * d + b]);
                acc[8 * d + 4 + b] = fmaf(w, fh[b], acc[8 * d + 4 + b]);
            }
        }
    }

    // ---- the 64 tokens of a workgroup pass are summed: rows of 16 lanes by DPP, the four rows
    // by two register folds (after which a lane of row w holds registers 4 k + w), the four
    // wavefronts through LDS ----
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[r] = row_tokens_sum(acc[r]);
    lsum = row_tokens_sum(lsum);
    zacc = row_tokens_sum(zacc);
    float f16v[16], f32v[8];
#pragma unroll
    for (int k = 0; k < 16; ++k) f16v[k] = fold16f(acc[2 * k], acc[2 * k + 1]);
#pragma unroll
    for (int k = 0; k < 8; ++k) f32v[k] = fold32f(f16v[2 * k], f16v[2 * k + 1]);
    const int rw = (tid >> 4) & 3;
    if ((tid & 12) == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) red[wave][32 * piece + kv_elem_of_reg(4 * k + rw)] = f32v[k];
        if (piece == 0) {
            lrow[wave][rw] = lsum;
            zrow[wave][rw] = zacc;
        }
    }
    __syncthreads();
    float* dst = part + (static_cast<size_t>(h) * splits + split) * KV_PART;
    if (tid < KV_D) {
        float zs = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int r = 0; r < 4; ++r) zs += zrow[w][r];
        dst[tid] = ((red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid])) - zs;
    } else if (tid == KV_D) {
        float ls = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int r = 0; r < 4; ++r) ls += lrow[w][r];
        dst[KV_D] = m;
        dst[KV_D + 1] = ls;
    }
}

// ---------------------------------------------------------------------------------------
// The streaming form for one query head per cache head where splits of 512 tokens, or of 1024, give every compute unit one workgroup or a few
// (kv_stream_tokens has its figures): a matrix product with one row of sixteen in use is a longer chain behind each load.  Workgroup = (split, head
// [, sequence]).  The split is cut into chunks of 16 tokens; wavefront w takes chunks w, w + 4, ... and walks them on its own: no
// workgroup barrier inside the loop, the loads of its next two chunks in flight while it computes one.  Each wavefront keeps a
// reference m (uniform over the wavefront; the running maximum, raised lazily) and rescales its sums when a chunk raises
// it:  acc <- acc * 2^(m_old - m_new);  p_t = 2^(score_t - m_new), scores in units of log 2.
// At the end the four wavefronts merge in LDS with the same rule and (m, l, acc) of the split goes to the workspace for
// kv4_combine_kernel.  The sums of a lane (eight or sixteen tokens) are centred before they are added up over lanes, wavefronts and splits, as
// the value codes of the matrix-core form are: left as they are, they grow with the tokens and cancel (24 drawn calls, error against 64
// bits: 2.2e-7 on average without, 1.4e-7 with, 1.5e-7 in the matrix-core form; the time is the same).
// ---------------------------------------------------------------------------------------
constexpr float KV_LAZY = 40.0f;  // how far a score may exceed the reference before it is raised
struct KvChunk {
    u32x4 kw, vw;
    uint32_t kp, vp;
    bool valid;
};

template <int QDT, bool BATCHED, bool QROT>
__global__ __launch_bounds__(KV_THREADS) void kv4_attn_stream_kernel(const void* __restrict__ q, int S, int S_max, int splits,
                                                                     float softmax_scale, const u32x4* __restrict__ k_codes,
                                                                     const uint32_t* __restrict__ k_params,
                                                                     const u32x4* __restrict__ v_codes,
                                                                     const uint32_t* __restrict__ v_params, int L,
                                                                     float* __restrict__ part, KvBatch batch)
{
    __shared__ float red[4][KV_D];
    __shared__ float wm[4], lrow[4][4], zrow[4][4];
    int h = static_cast<int>(blockIdx.x) / splits;
    const int split = static_cast<int>(blockIdx.x) - h * splits;
    const int tid = threadIdx.x, lane = tid & 63, slot = lane >> 2, piece = tid & 3;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = split * L;
    if constexpr (BATCHED) {
        const int seq = blockIdx.z;
        S = batch.v[seq];
        if (t0 >= S) return;  // the whole workgroup: this sequence has fewer splits
        h += seq * batch.H_q;
    }
    const int t_end = min(S, t0 + L);
    const size_t head_base = static_cast<size_t>(h) * S_max;
    // chunks of this wavefront that hold at least one cached token
    const int span = t_end - t0 - 16 * wave;
    const int nchunks = span > 0 ? (span + 63) >> 6 : 0;

    auto load = [&](int c, KvChunk& r) {  // chunk c of this wavefront: tokens t0 + 16 (4 c + wave) ...; past the end: the last token, weight 0
        const int t = t0 + 16 * (4 * c + wave) + slot;
        r.valid = t < t_end;
        const size_t at = head_base + (r.valid ? t : t_end - 1);
        // read once per call: non-temporal loads, as in kv4_attn_kernel
        r.kw = __builtin_nontemporal_load(k_codes + (at * 4 + piece));
        r.kp = __builtin_nontemporal_load(k_params + at);
        r.vw = __builtin_nontemporal_load(v_codes + (at * 4 + piece));
        r.vp = __builtin_nontemporal_load(v_params + at);
    };

    Raw8<QDT> qraw[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) qraw[d] = load8_raw<QDT>(q, static_cast<size_t>(h) * KV_D + 32 * piece + 8 * d);
    KvChunk cA, cB;
    load(0, cA);
    load(1, cB);

    float qr[32];
    const float qsum = kv_query_registers<QDT>(qraw, QROT, piece, qr);
    const float unit = kv_fp8_unit(), inv_unit = 1.0f / unit;
    const float scale_by_unit = softmax_scale * 1.44269504088896340736f * inv_unit, qsum_unit = qsum * unit;

    float acc[32];
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[r] = 0.0f;
    float lsum = 0.0f, zacc = 0.0f, wsum = 0.0f;
    float m = -INFINITY;  // uniform over the wavefront
    int chunk = 0;

    auto step = [&](KvChunk& cur) {
        float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t lo, hi;
            nibble_bytes(cur.kw[d], lo, hi);
            float fl[4], fh[4];
            bytes_to_floats(lo, fl);
            bytes_to_floats(hi, fh);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                dot[d] = fmaf(qr[8 * d + b], fl[b], dot[d]);
                dot[d] = fmaf(qr[8 * d + 4 + b], fh[b], dot[d]);
            }
        }
        const float s = half_bits_to_float(static_cast<uint16_t>(cur.kp & 0xffffu)) * scale_by_unit;
        const float z = static_cast<float>(static_cast<int>(cur.kp) >> 16);
        float sc = quad_sum(s * (((dot[0] + dot[1]) + (dot[2] + dot[3])) - z * qsum_unit));
        sc = cur.valid ? sc : -INFINITY;
        // The reference m only has to keep the powers in range, so it is raised lazily: when some score
        // of the chunk exceeds it by more than KV_LAZY (always on the first chunk, where m = -inf; every chunk
        // that is stepped holds a cached token, so the new maximum is finite).  Weights then stay below
        // 2^KV_LAZY and the sums of a split far inside the binary32 range.
        if (__builtin_amdgcn_ballot_w64(sc > m + KV_LAZY) != 0) {  // uniform
            const float m_new = fmaxf(m, wave_max(sc));
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);  // 0 on the first chunk
#pragma unroll
            for (int r = 0; r < 32; ++r) acc[r] *= alpha;
            lsum *= alpha;
            zacc *= alpha;
            wsum *= alpha;
            m = m_new;
        }
        const float p = __builtin_amdgcn_exp2f(sc - m);
        const float w0 = p * half_bits_to_float(static_cast<uint16_t>(cur.vp & 0xffffu));
        const float w = w0 * inv_unit;
        lsum += p;
        wsum += w0;
        zacc = fmaf(w0, static_cast<float>((static_cast<int>(cur.vp) >> 16) - 8), zacc);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t lo, hi;
            nibble_bytes(cur.vw[d], lo, hi);
            float fl[4], fh[4];
            bytes_to_floats(lo, fl);
            bytes_to_floats(hi, fh);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                acc[8 * d + b] = fmaf(w, fl[b], acc[8 * d + b]);
                acc[8 * d + 4 + b] = fmaf(w, fh[b], acc[8 * d + 4 + b]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        load(chunk + 2, cur);  // refill with the chunk two steps ahead (past the end: a harmless repeat of the last token)
        __builtin_amdgcn_sched_barrier(0);
        ++chunk;
    };
    // steps counted up front and run in pairs: one loop body, one exit (four chunks in flight instead of
    // two: 130 registers and no gain)
    for (int i = 0; i < nchunks / 2; ++i) {
        step(cA);
        step(cB);
    }
    if (nchunks & 1) step(cA);

    // ---- the 16 tokens of a wavefront's chunks are summed as in kv4_attn_kernel; the four wavefronts
    // merge through LDS, each weighted by 2^(its m - the largest m) ----
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[r] = row_tokens_sum(fmaf(-8.0f, wsum, acc[r]));
    lsum = row_tokens_sum(lsum);
    zacc = row_tokens_sum(zacc);
    float f16v[16], f32v[8];
#pragma unroll
    for (int k = 0; k < 16; ++k) f16v[k] = fold16f(acc[2 * k], acc[2 * k + 1]);
#pragma unroll
    for (int k = 0; k < 8; ++k) f32v[k] = fold32f(f16v[2 * k], f16v[2 * k + 1]);
    const int rw = (tid >> 4) & 3;
    if ((tid & 12) == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) red[wave][32 * piece + kv_elem_of_reg(4 * k + rw)] = f32v[k];
        if (piece == 0) {
            lrow[wave][rw] = lsum;
            zrow[wave][rw] = zacc;
        }
    }
    if (lane == 0) wm[wave] = m;
    __syncthreads();
    float* dst = part + (static_cast<size_t>(h) * splits + split) * KV_PART;
    if (tid <= KV_D) {
        const float M = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));  // wavefront 0 always has a token: finite
        float total = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float e = __builtin_amdgcn_exp2f(wm[w] - M);  // 0 for a wavefront without tokens
            float v;
            if (tid < KV_D) v = red[w][tid] - ((zrow[w][0] + zrow[w][1]) + (zrow[w][2] + zrow[w][3]));
            else v = (lrow[w][0] + lrow[w][1]) + (lrow[w][2] + lrow[w][3]);
            total = fmaf(e, v, total);
        }
        if (tid < KV_D) dst[tid] = total;
        else {
            dst[KV_D] = M;
            dst[KV_D + 1] = total;
        }
    }
}

// ---------------------------------------------------------------------------------------
// The matrix-core form for long contexts, batches and grouped query heads.  Workgroup = (split of L tokens, cache head
// [, sixteen of its query heads] [, sequence]); all query heads that read the cache head are rows of one matrix
// product, so the codes are fetched and unpacked once for all of them.  Wavefront w of the four walks the chunks
// w, w + 4, ... of 64 tokens on its own (no workgroup barrier inside the loop).
//
// Operands.  A code in a byte of its own is c * 2^-9 as an E4M3 number, and one instruction turns two of those into
// binary16 numbers (7 operations for the eight codes of a dword).  Left as binary16 subnormals c * 2^-24 they would take
// five, but the matrix unit aligns products by their nominal exponents: outputs were off by 4e-5 instead of 3e-7.
// The other operand (query, softmax weights) is a sum of two binary16 numbers, hi + lo, in two instructions; products are
// exact and the sums binary32.  A piece keeps 11 bits down to 2^-14 and an absolute 2^-25 below, so the operands are scaled:
// the query by a power of two per head (largest element 2^13 .. 2^14), the weights through their reference (below).  Both
// then hold 22 bits and more of every value down to 2^-12 of the largest, and 2^-34 of the largest below that.
// The (s, z) of a token stay outside the products:
//   score = s_t (q . c_t - z_t sum q),   out = sum_t (p_t s_t) (c_t - 8) - sum_t p_t s_t (z_t - 8).
// Value codes enter less 8: the two sums of `out` grow with the tokens and cancel, and their binary32 roundings with them
// (60000 tokens of 32 heads, error against 64 bits: 4.6e-7 with 0 .. 15, 1.2e-7 with -8 .. 7; the vector form 2.5e-7).  That
// costs nine operations for the eight codes of a dword instead of seven: 1 to 3 % of the call where several query heads share
// a cache head (16 sequences of up to 6000 tokens 23.5 -> 23.6 us, 40000 tokens of 32 over 16 heads 24.4 -> 25.0).  (The same for the keys costs as much again and gains only
// where the elements of a query share an offset.)
//   scores   rows = query heads, columns = 16 tokens, k = the 128 elements: the codes go from memory to registers in
//            operand order (lane = token l % 16, 16 bytes l / 16 of it)
//   values   rows = query heads, columns = 16 elements, k = 32 tokens: the codes go to LDS as they lie in memory and
//            come back transposed by ds_read_b64_tr_b4 (16 tokens of one element per lane); the 16-byte pieces of a
//            token are permuted by the token's position so that sixteen rows fall into different banks
// Between the two a lane holds the scores of its token(s) for up to four heads; the weights pass through LDS.
// What bounds it, by the counters of 16 sequences of 300 to 6000 tokens, 32 over 8 heads (18.4 us by the trace for 9.6 us of bytes,
// 22.5 with fixed splits and workgroups without tokens): no unit.  A SIMD holds 1.3 wavefronts on average, its vector unit issues
// in 41 % of the cycles and its matrix unit is busy in 15 %; a wavefront spends a third of its life waiting for memory or
// LDS and 27 % for its own previous instructions: the chain of one chunk, which too few wavefronts hide.
// RP: query heads per cache head, rounded up to a power of two.
// Registers: four wavefronts a SIMD for one and two heads (124 and 128 registers; left at 130, 120000 tokens of 16 over 8
// heads take 34.3 us instead of 31.6), three for the others.
// ---------------------------------------------------------------------------------------
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef int v2i __attribute__((ext_vector_type(2)));
constexpr float KV_W_TOP = 14.0f;      // the weights of a head stay below 2^14 (binary16 ends at 2^16) ...
constexpr float KV_W_REF = 9.0f;       // ... and a raised reference puts the largest so far at 2^9
constexpr int KV_WSTRIDE = 68;         // dwords per head of the weights in LDS: 64 tokens, padded off the bank period

union KvHalves {
    uint32_t w[4];
    v8h h;
};

// eight codes of a dword as binary16 numbers, elements 0,2 | 4,6 | 1,3 | 5,7
__device__ __forceinline__ v8h kv_code_halves(uint32_t w)
{
    const int lo = static_cast<int>(w & 0x0f0f0f0fu), hi = static_cast<int>((w >> 4) & 0x0f0f0f0fu);
    const v2h a = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 512.0f, false), b = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 512.0f, true);
    const v2h c = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 512.0f, false), d = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 512.0f, true);
    return v8h{a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}
// which element of the dword stands in half e of register r of that operand
__device__ __forceinline__ constexpr int kv_half_element(int r, int e) { return ((r & 2) >> 1) + 4 * (r & 1) + 2 * e; }

// The eight codes of a dword less 8, elements 0,4 | 1,5 | 2,6 | 3,7: a code under the exponent of 1024 reads as 1024 + c, in
// the next four bits up as 1024 + 16 c.
__device__ __forceinline__ v8h kv_centred_halves(uint32_t w)
{
    uint32_t base = 0x64006400u;
    asm("" : "+v"(base));
    auto pair = [&](uint32_t x, uint32_t mask) { return __builtin_bit_cast(v2h, (x & mask) | base); };
    const v2h by = {0.0625f, 0.0625f}, less = {-1032, -1032}, less16 = {-72, -72};
    const uint32_t u = w >> 8;
    const v2h a = pair(w, 0x000f000fu) + less, b = __builtin_elementwise_fma(pair(w, 0x00f000f0u), by, less16);
    const v2h c = pair(u, 0x000f000fu) + less, d = __builtin_elementwise_fma(pair(u, 0x00f000f0u), by, less16);
    return v8h{a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}
// which token stands in half e of register r of that operand
__device__ __forceinline__ constexpr int kv_centred_element(int r, int e) { return r + 4 * e; }

__device__ __forceinline__ uint32_t half_bits(float v) { return __half_as_ushort(__float2half_rn(v)); }

// v as hi + lo, two binary16 numbers: hi in the low 16 bits
__device__ __forceinline__ uint32_t kv_split_half(float v)
{
    const uint32_t hi = half_bits(v);
    return hi | (half_bits(v - half_bits_to_float(static_cast<uint16_t>(hi))) << 16);
}

// maximum / sum over the lanes that hold values of the same head in the score layout
template <int RP>
__device__ __forceinline__ float kv_head_max(float v)
{
#define RCP_ROW_MAX(ctrl) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, false)))
    RCP_ROW_MAX(0x128);
    RCP_ROW_MAX(0x124);
    RCP_ROW_MAX(0x122);
    RCP_ROW_MAX(0x121);
#undef RCP_ROW_MAX
    if constexpr (RP <= 4) {
        auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    if constexpr (RP <= 8) {
        auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    return v;
}

template <int RP>
__device__ __forceinline__ float kv_head_sum(float v)
{
    v = row_sum16f(v);
    if constexpr (RP <= 4) v = fold16f(v, v);
    if constexpr (RP <= 8) v = fold32f(v, v);
    return v;
}

template <int RP>
struct KvMfmaLds {
    union {
        struct {
            u32x4 v[4][256];                       // a chunk's value codes of each wavefront
            float2 qc[4][RP];                      // sum of q in the units of the products, products -> score in powers of two
            uint32_t w[4][RP * KV_WSTRIDE];        // its softmax weights, hi | lo << 16
        } run;
        struct {
            float red[4][RP][KV_D];
            float m[4][RP], l[4][RP];
        } end;
    };
};

template <int RP, bool COMPACT>
__global__ __launch_bounds__(KV_THREADS, RP <= 2 ? 4 : 3) void kv4_attn_mfma_kernel(const void* __restrict__ q, int q_dt, int rotate, int S_max, int rep,
                                                                   int splits, float softmax_scale, const u32x4* __restrict__ k_codes,
                                                                   const uint32_t* __restrict__ k_params,
                                                                   const u32x4* __restrict__ v_codes,
                                                                   const uint32_t* __restrict__ v_params, int L,
                                                                   float* __restrict__ part, KvBatch batch)
{
    constexpr int HV = RP < 4 ? RP : 4;                       // heads a lane holds scores of
    constexpr int SETS = RP <= 4 ? 1 : RP == 8 ? 2 : 4;       // tokens a lane holds scores of
    __shared__ KvMfmaLds<RP> lds;
    int seq = 0, S = batch.v[0];
    // plain grid (splits of the longest sequence, cache heads [, sequences]): from arguments that arrive with the wavefront
    int hk0 = static_cast<int>(blockIdx.x) / splits, split = static_cast<int>(blockIdx.x) - hk0 * splits;
    if constexpr (COMPACT) {
        // Only splits that hold tokens have a workgroup: among those of a plain grid the early leavers upset the order in which the
        // compute units are filled (16 sequences of up to 6000 tokens, 44000 in all, 360 of 768 workgroups at work on 256
        // units: 24.0 -> 19.4 us at the same split length).
        int start = 0;
        auto look = [&](int lo, int hi) {  // selects on arguments that are all fetched together
#pragma unroll
            for (int b = lo; b < hi; ++b) {
                const bool from = static_cast<int>(blockIdx.x) >= batch.first[b];
                seq = from ? b : seq;
                start = from ? batch.first[b] : start;
                S = from ? batch.v[b] : S;
            }
        };
        look(1, 4);
        if (batch.n > 4) look(4, 8);  // uniform
        if (batch.n > 8) look(8, RCP_MAX_M);
        const int within = static_cast<int>(blockIdx.x) - start;
        split = within / batch.H_kv;
        hk0 = within - split * batch.H_kv;
    } else {
        seq = blockIdx.z;
        S = batch.v[seq];
        if (split * L >= S) return;  // the whole workgroup: this sequence has fewer splits
    }
    const int t0 = split * L;
    const int t_end = min(S, t0 + L);
    const int hk = hk0 + seq * batch.H_kv;
    const int R = min(RP, rep - static_cast<int>(blockIdx.y) * RP);  // query heads of this workgroup
    const int h0 = seq * batch.H_q + hk0 * rep + static_cast<int>(blockIdx.y) * RP;
    const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int first = t0 + 64 * wave;
    const int nchunks = t_end > first ? (t_end - first + 255) >> 8 : 0;  // of this wavefront; uniform

    // One resource per tensor and cache head that ends with this workgroup's last token: what lies beyond reads as
    // zero (code 0 of weight 0), so no address is clamped.  The cache is read once per call: non-temporal loads.
    const size_t head_base = static_cast<size_t>(hk) * S_max;
    auto resource = [&](const void* p, int bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(static_cast<const char*>(p)) + head_base * bytes, 0, t_end * bytes, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t kc = resource(k_codes, 64), vc = resource(v_codes, 64), kr = resource(k_params, 4), vr = resource(v_params, 4);
    constexpr int NT = 2;
    u32x4 kw[4];
    uint32_t kp[SETS], vp[SETS];
    auto set_token = [&](int s) { return RP <= 4 ? lane : RP == 8 ? 32 * s + 16 * (g >> 1) + i : 16 * s + i; };
    const int k_lane = i * 64 + g * 16, v_lane = (lane >> 2) * 64 + ((lane & 3) ^ g) * 16, p_lane = set_token(0) * 4;
    constexpr int P_SET = RP == 8 ? 128 : 64;  // bytes of parameters from one set to the next
    auto load_keys = [&](int base) {
#pragma unroll
        for (int n = 0; n < 4; ++n) kw[n] = __builtin_amdgcn_raw_buffer_load_b128(kc, k_lane + base * 64 + 1024 * n, 0, NT);
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            kp[s] = __builtin_amdgcn_raw_buffer_load_b32(kr, p_lane + base * 4 + P_SET * s, 0, NT);
            vp[s] = __builtin_amdgcn_raw_buffer_load_b32(vr, p_lane + base * 4 + P_SET * s, 0, NT);
        }
    };
    auto load_values = [&](int base) {  // lane -> (token lane / 4, piece lane % 4 of it after the permutation)
#pragma unroll
        for (int n = 0; n < 4; ++n)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(vc, (__attribute__((address_space(3))) void*)(&lds.run.v[wave][64 * n]), 16,
                                                     v_lane + base * 64 + 1024 * n, 0, 0, NT);
    };
    // ---- the query: lane = (head i, elements 32 g ...) ----
    v8h qhi[4], qlo[4];
    if (nchunks > 0) {
        // the query is requested first: memory answers in order and it is needed first
        float t[32];
        const size_t qat = static_cast<size_t>(h0 + min(i, R - 1)) * KV_D + 32 * g;
        if (q_dt == RCP_F32) {  // uniform
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const float4 x = reinterpret_cast<const float4*>(static_cast<const float*>(q) + qat)[d];
                t[4 * d] = x.x;
                t[4 * d + 1] = x.y;
                t[4 * d + 2] = x.z;
                t[4 * d + 3] = x.w;
            }
            __builtin_amdgcn_sched_barrier(0);
            load_keys(first);
            load_values(first);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            Raw8<RCP_F16> raw[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) raw[d] = load8_raw<RCP_F16>(q, qat + 8 * d);
            __builtin_amdgcn_sched_barrier(0);
            load_keys(first);
            load_values(first);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t w[4] = {raw[d].a.x, raw[d].a.y, raw[d].a.z, raw[d].a.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint16_t x = static_cast<uint16_t>(w[e] & 0xffffu), y = static_cast<uint16_t>(w[e] >> 16);
                    t[8 * d + 2 * e] = q_dt == RCP_F16 ? half_bits_to_float(x) : bf16_bits_to_float(x);
                    t[8 * d + 2 * e + 1] = q_dt == RCP_F16 ? half_bits_to_float(y) : bf16_bits_to_float(y);
                }
            }
        }
        if (rotate) kv_rotate_query_rows(t, g);  // uniform
        float top = 0.0f, sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            if (i >= R) t[e] = 0.0f;
            top = fmaxf(top, fabsf(t[e]));
        }
        // The head's largest element becomes 2^13 .. 2^14.  One power of two per head and not one for the sixteen: an
        // infinite element must not push the other heads out of binary16, nor a large head the small ones below it.
        {
            auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(top), __float_as_uint(top), false, false);
            top = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
            r = __builtin_amdgcn_permlane32_swap(__float_as_uint(top), __float_as_uint(top), false, false);
            top = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        }
        const int E = __builtin_amdgcn_frexp_expf(top);
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            t[e] = ldexpf(t[e], 14 - E);
            sum += t[e];
        }
        sum = fold32f(fold16f(sum, sum), fold16f(sum, sum));
        if (g == 0 && i < RP) lds.run.qc[wave][i] = make_float2(sum, ldexpf(softmax_scale * 1.44269504088896340736f, E - 14));
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            KvHalves hi, lo;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t x = kv_split_half(t[8 * d + kv_half_element(r, 0)]), y = kv_split_half(t[8 * d + kv_half_element(r, 1)]);
                hi.w[r] = __builtin_amdgcn_perm(y, x, 0x05040100u);
                lo.w[r] = __builtin_amdgcn_perm(y, x, 0x07060302u);
            }
            qhi[d] = hi.h;
            qlo[d] = lo.h;
        }
    }

    v4f acc[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) acc[b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    float m[HV], lsum[HV], zacc[HV];
#pragma unroll
    for (int v = 0; v < HV; ++v) {
        m[v] = -INFINITY;
        lsum[v] = zacc[v] = 0.0f;
    }

    for (int c = 0; c < nchunks; ++c) {
        const int base = first + 256 * c;
        v4f D[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            D[n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const v8h b = kv_code_halves(kw[n][d]);
                D[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qlo[d], b, D[n], 0, 0, 0);
                D[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qhi[d], b, D[n], 0, 0, 0);
            }
        }
        float ks[SETS], kz[SETS], sv[SETS], zv[SETS];
        bool valid[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            ks[s] = half_bits_to_float(static_cast<uint16_t>(kp[s] & 0xffffu));
            kz[s] = static_cast<float>(static_cast<int>(kp[s]) >> 16);
            sv[s] = half_bits_to_float(static_cast<uint16_t>(vp[s] & 0xffffu));
            zv[s] = static_cast<float>((static_cast<int>(vp[s]) >> 16) - 8);
            valid[s] = base + set_token(s) < t_end;
            // computed before the next parameters arrive in the same registers
            asm volatile("" : "+v"(ks[s]), "+v"(kz[s]), "+v"(sv[s]), "+v"(zv[s]));
        }
        __builtin_amdgcn_sched_barrier(0);
        load_keys(base + 256);  // past the end: zeros
        __builtin_amdgcn_sched_barrier(0);

        // rows of sixteen lanes without a head are filled with the other tokens' scores
        float sc[SETS][HV];
#pragma unroll
        for (int v = 0; v < HV; ++v) {
            if constexpr (RP <= 4) {
                auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(D[0][v]), __float_as_uint(D[1][v]), false, false);
                auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(D[2][v]), __float_as_uint(D[3][v]), false, false);
                auto r = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
                sc[0][v] = __uint_as_float(r[0]);
            } else if constexpr (RP == 8) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(D[2 * s][v]), __float_as_uint(D[2 * s + 1][v]), false, false);
                    sc[s][v] = __uint_as_float(r[0]);
                }
            } else {
#pragma unroll
                for (int s = 0; s < SETS; ++s) sc[s][v] = D[s][v];
            }
        }
        float2 qc[HV];  // fetched anew for each chunk: held, they would cost the third wavefront of a SIMD
        {
            int at = RP <= 4 ? 0 : RP == 8 ? 4 * (g & 1) : 4 * g;
            asm("" : "+v"(at) : "s"(c));
#pragma unroll
            for (int v = 0; v < HV; ++v) qc[v] = lds.run.qc[wave][at + v];
        }
        // A weight of the product is p s = 2^(score - m) s, so the reference m of a head is held against score + log2 s: with
        // the largest score alone, or the largest step of the chunk, one token of a large step and no attention would push
        // the weights that matter below the binary16 pieces.  p itself stays below 2^(14 + 24) (the smallest step), as does
        // a step of zero (a slot that was never written) with the same bound in its place.
        float top[HV];  // the largest of score + log2 s of this lane's tokens
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const float ls = __builtin_amdgcn_logf(__builtin_amdgcn_fmed3f(fabsf(sv[s]), 0x1p-24f, 65504.0f));
#pragma unroll
            for (int v = 0; v < HV; ++v) {
                float x = fmaf(-kz[s], qc[v].x, sc[s][v]) * (ks[s] * qc[v].y);
                asm("" : "+v"(x));  // a select: the branch that the compiler makes of it costs 2 % of a call
                sc[s][v] = valid[s] ? x : -INFINITY;
                top[v] = s == 0 ? sc[s][v] + ls : fmaxf(top[v], sc[s][v] + ls);
            }
        }
        bool raise = false;
#pragma unroll
        for (int v = 0; v < HV; ++v) raise |= top[v] > m[v] + KV_W_TOP;
        // It only has to keep the weights in range and moves when one would leave it (always on the first chunk, whose
        // first token is valid), for that head alone: what a head returns does not depend on its neighbours.
        if (__builtin_amdgcn_ballot_w64(raise) != 0) {  // uniform
#pragma unroll
            for (int v = 0; v < HV; ++v) {
                const float t = kv_head_max<RP>(top[v]);
                const float m_new = t > m[v] + KV_W_TOP ? t - KV_W_REF : m[v];
                const float alpha = __builtin_amdgcn_exp2f(m[v] - m_new);  // 0 on the first chunk
                m[v] = m_new;
                lsum[v] *= alpha;
                zacc[v] *= alpha;
#pragma unroll
                for (int b = 0; b < 8; ++b) acc[b][v] *= alpha;
            }
        }
        uint32_t* const ww = lds.run.w[wave];
#pragma unroll
        for (int s = 0; s < SETS; ++s)
#pragma unroll
            for (int v = 0; v < HV; ++v) {
                const float p = __builtin_amdgcn_exp2f(sc[s][v] - m[v]);  // 0 for the surplus tokens
                const float w0 = p * sv[s];
                lsum[v] += p;
                zacc[v] = fmaf(w0, zv[s], zacc[v]);
                const int head = RP <= 4 ? v : RP == 8 ? 4 * (g & 1) + v : 4 * g + v;
                ww[head * KV_WSTRIDE + set_token(s)] = kv_split_half(w0);
            }
        // weights back as operands: lane = (head i, tokens 16 g + 8 h ...)
        v8h phi[2], plo[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x4* const src = reinterpret_cast<const u32x4*>(ww + min(i, RP - 1) * KV_WSTRIDE + 16 * g + 8 * h);
            const u32x4 w03 = src[0], w47 = src[1];
            const uint32_t ws[8] = {w03.x, w03.y, w03.z, w03.w, w47.x, w47.y, w47.z, w47.w};
            KvHalves hi, lo;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t x = ws[kv_centred_element(r, 0)], y = ws[kv_centred_element(r, 1)];
                hi.w[r] = __builtin_amdgcn_perm(y, x, 0x05040100u);
                lo.w[r] = __builtin_amdgcn_perm(y, x, 0x07060302u);
            }
            phi[h] = hi.h;
            plo[h] = lo.h;
        }
        // the values of this chunk are in LDS once no more loads than the keys requested above are outstanding
        constexpr int AFTER = 4 + 2 * SETS;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt((AFTER & 15) | (7 << 4) | (15 << 8));
        __builtin_amdgcn_sched_barrier(0);
        const int tok = 16 * g + i;
        const char* const row = reinterpret_cast<const char*>(&lds.run.v[wave][0]) + tok * 64;
        const int f = (tok >> 2) & 3;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const v2i r = __builtin_amdgcn_ds_read_tr4_b64_v2i32(
                (__attribute__((address_space(3))) v2i*)(row + (((b >> 1) ^ f) * 16 + (b & 1) * 8)));
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const v8h x = kv_centred_halves(static_cast<uint32_t>(r[h]));
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(plo[h], x, acc[b], 0, 0, 0);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(phi[h], x, acc[b], 0, 0, 0);
            }
        }
        // every read of the chunk has returned before the next one overwrites it
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
        load_values(base + 256);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int v = 0; v < HV; ++v) {
        lsum[v] = kv_head_sum<RP>(lsum[v]);
        zacc[v] = kv_head_sum<RP>(zacc[v]);
    }
    __builtin_amdgcn_s_waitcnt(0);  // the surplus values have landed: LDS changes hands
    __syncthreads();
    if (4 * g < RP) {
#pragma unroll
        for (int v = 0; v < HV; ++v) {
#pragma unroll
            for (int b = 0; b < 8; ++b) lds.end.red[wave][4 * g + v][16 * b + i] = acc[b][v] - zacc[v];
            if (i == 0) {
                lds.end.m[wave][4 * g + v] = m[v];
                lds.end.l[wave][4 * g + v] = lsum[v];
            }
        }
    }
    __syncthreads();
    for (int idx = tid; idx < R * KV_D; idx += KV_THREADS) {
        const int h = idx >> 7, j = idx & (KV_D - 1);
        float M = lds.end.m[0][h];  // wavefront 0 always has a token: finite
#pragma unroll
        for (int w = 1; w < 4; ++w) M = fmaxf(M, lds.end.m[w][h]);
        float total = 0.0f, ls = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float e = __builtin_amdgcn_exp2f(lds.end.m[w][h] - M);  // 0 for a wavefront without tokens
            total = fmaf(e, lds.end.red[w][h][j], total);
            ls = fmaf(e, lds.end.l[w][h], ls);
        }
        float* const dst = part + (static_cast<size_t>(h0 + h) * splits + split) * KV_PART;
        dst[j] = total;
        if (j == 0) {
            dst[KV_D] = M;
            dst[KV_D + 1] = ls;
        }
    }
}

// The merge of the splits as a kernel of its own: one workgroup of `groups` x 128 threads per head (kv_merge_head).
// BATCHED: blockIdx.x = sequence * H_q + head; a sequence of length batch.v[z] has written only its
// first ceil(length / L) of the `splits` slots of each head.
template <bool OUT_F16, bool BATCHED>
__global__ __launch_bounds__(KV_CT) void kv4_combine_kernel(const float* __restrict__ part, int splits, int groups,
                                                            void* __restrict__ out, int L, float unit, KvBatch batch)
{
    __shared__ KvMergeLds lds;
    const int h = blockIdx.x;
    const float* src = part + static_cast<size_t>(h) * splits * KV_PART;
    if constexpr (BATCHED) {
        // the sequence's own number of splits and thread groups, so that the merge runs in the same order
        // as in a call for this sequence alone
        splits = (batch.v[h / batch.H_q] + L - 1) / L;
        groups = min(groups, (splits + 3) / 4);
    }
    kv_merge_head(src, splits, groups, unit, out, OUT_F16, h, lds, groups * KV_D);
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
// Tokens per workgroup are chosen in launch_kv4_attn (measured: 64 never wins, the per-workgroup
// reduction then weighs too much); the "kv_tokens" option overrides.
size_t kv4_workspace_bytes(int H_q, int S)
{
    const int splits = (S + 63) / 64;  // the most any split length needs
    return static_cast<size_t>(H_q) * splits * KV_PART * sizeof(float);
}

// From sixteen tokens on (a lane row of a workgroup each) a workgroup takes tokens of one head; below, where lane rows
// would be left without work, vectors in the order of x.
static bool kv4_by_tokens(int n_tokens) { return n_tokens >= 16; }

static dim3 kv4_append_grid(int n_tokens, int H, bool by_tokens, unsigned tensors)
{
    if (by_tokens) return dim3(static_cast<unsigned>((n_tokens + 15) / 16), static_cast<unsigned>(H), tensors);
    return dim3(static_cast<unsigned>((n_tokens * H + 15) / 16), 1u, tensors);
}

// positions == nullptr: n_tokens tokens of one sequence from `pos` on; otherwise one token for each of
// n_tokens sequences of a pooled cache, at positions[i]
int launch_kv4_append(const void* x, rcp_dtype dt, int n_tokens, int H, int S_max, int pos, const int* positions, bool rotate,
                      float clip_ratio, void* codes, void* params, hipStream_t st)
{
    if (n_tokens * H == 0) return RCP_OK;
    auto* c = static_cast<uint32_t*>(codes);
    auto* p = static_cast<uint32_t*>(params);
    KvBatch batch = {};
    const bool batched = positions != nullptr;
    if (batched)
        for (int i = 0; i < n_tokens; ++i) batch.v[i] = positions[i];
    const bool by_tokens = !batched && kv4_by_tokens(n_tokens) && H <= 65535;
    const dim3 grid = kv4_append_grid(n_tokens, H, by_tokens, 1u);
    auto launch = [&](auto kernel) {
        enqueue(kernel, grid, 256, 0, st, x, by_tokens ? n_tokens : n_tokens * H, H, S_max, pos, clip_ratio, c, p, batch);
    };
#define RCP_KV_APPEND(DT)                                                          \
    do {                                                                           \
        if (batched) {                                                             \
            if (rotate) launch(&kv4_append_kernel<DT, true, true>);                \
            else launch(&kv4_append_kernel<DT, false, true>);                      \
        } else if (by_tokens) {                                                    \
            if (rotate) launch(&kv4_append_kernel<DT, true, false, true>);         \
            else launch(&kv4_append_kernel<DT, false, false, true>);               \
        } else {                                                                   \
            if (rotate) launch(&kv4_append_kernel<DT, true, false>);               \
            else launch(&kv4_append_kernel<DT, false, false>);                     \
        }                                                                          \
    } while (0)
    if (dt == RCP_F32) RCP_KV_APPEND(RCP_F32);
    else if (dt == RCP_F16) RCP_KV_APPEND(RCP_F16);
    else RCP_KV_APPEND(RCP_BF16);
#undef RCP_KV_APPEND
    return check_launch("rcp_kv4_append");
}

// keys and values of the same n_tokens tokens in one launch
int launch_kv4_append_kv(const void* k, const void* v, rcp_dtype dt, int n_tokens, int H, int S_max, int pos, bool rotate_k,
                         float clip_ratio, void* k_codes, void* k_params, void* v_codes, void* v_params, hipStream_t st)
{
    if (n_tokens * H == 0) return RCP_OK;
    const bool by_tokens = kv4_by_tokens(n_tokens) && H <= 65535;
    const dim3 grid = kv4_append_grid(n_tokens, H, by_tokens, 2u);
    auto launch = [&](auto kernel) {
        enqueue(kernel, grid, 256, 0, st, k, v, by_tokens ? n_tokens : n_tokens * H, H, S_max, pos, rotate_k ? 1 : 0, clip_ratio,
                                     static_cast<uint32_t*>(k_codes), static_cast<uint32_t*>(k_params),
                                     static_cast<uint32_t*>(v_codes), static_cast<uint32_t*>(v_params));
    };
#define RCP_KV_APPEND(DT)                                                              \
    by_tokens ? launch(&kv4_append_kv_kernel<DT, true>) : launch(&kv4_append_kv_kernel<DT, false>)
    if (dt == RCP_F32) RCP_KV_APPEND(RCP_F32);
    else if (dt == RCP_F16) RCP_KV_APPEND(RCP_F16);
    else RCP_KV_APPEND(RCP_BF16);
#undef RCP_KV_APPEND
    return check_launch("rcp_kv4_append_kv");
}

// lengths == nullptr: one sequence of S tokens; otherwise B sequences of a pooled cache, lengths[b] tokens each
// rotate_q (single sequence only): the order-128 Hadamard rotation of the query inside the attention kernel
int launch_kv4_attn(const void* q, rcp_dtype q_dt, int B, int H_q, int H_kv, int S_max, int S, const int* lengths,
                    const void* k_codes, const void* k_params, const void* v_codes, const void* v_params,
                    float softmax_scale, void* out, rcp_dtype out_dt, void* workspace, hipStream_t st, bool rotate_q)
{
    const bool batched = lengths != nullptr;
    const bool fused = !batched && rotate_q;
    KvBatch batch = {};
    if (batched) {
        S = 0;
        for (int b = 0; b < B; ++b) {
            batch.v[b] = lengths[b];
            S = lengths[b] > S ? lengths[b] : S;  // the longest sequence sizes the grid
        }
    }
    batch.H_q = H_q;
    batch.H_kv = H_kv;
    if (!batched) batch.v[0] = S;
    const unsigned nseq = static_cast<unsigned>(batched ? B : 1);
    batch.n = static_cast<int>(nseq);
    const int rep = H_q / H_kv, per = (rep + 15) / 16;  // sixteen query heads at most per workgroup of the matrix-core form
    const KvPlan plan = kv_plan(batch.v, static_cast<int>(nseq), batched, H_q, H_kv, num_compute_units(), options().kv_tokens);
    const bool matrix = plan.form == KvForm::matrix;
    const int L = plan.tokens;
    const int splits = (S + L - 1) / L;
    auto* kc = static_cast<const u32x4*>(k_codes);
    auto* vc = static_cast<const u32x4*>(v_codes);
    auto* kp = static_cast<const uint32_t*>(k_params);
    auto* vp = static_cast<const uint32_t*>(v_params);
    auto* part = static_cast<float*>(workspace);
    if (matrix) {
        // the plain grid for one sequence and while it has no more workgroups than there are units (finding the sequence costs 0.1 to
        // 0.3 us: 11 sequences of 2500 tokens in all, 64 over 8 heads, 9.7 against 10.0)
        const bool compact = nseq > 1 && static_cast<long long>(splits) * H_kv * per * nseq > num_compute_units();
        int groups = 0;
        for (int b = 0; b < RCP_MAX_M; ++b) {
            batch.first[b] = groups;
            if (b < static_cast<int>(nseq)) groups += (batch.v[b] + L - 1) / L * H_kv;
        }
        const dim3 grid(static_cast<unsigned>(compact ? groups : splits * H_kv), static_cast<unsigned>(per), compact ? 1u : nseq);
        auto launch = [&](auto kernel) {
            enqueue(kernel, grid, KV_THREADS, 0, st, q, static_cast<int>(q_dt), fused ? 1 : 0, S_max, rep, splits, softmax_scale, kc, kp, vc, vp, L,
                                                part, batch);
        };
        auto form = [&](auto gapless) {
            constexpr bool COMPACT = decltype(gapless)::value;
            if (rep == 1) launch(&kv4_attn_mfma_kernel<1, COMPACT>);
            else if (rep == 2) launch(&kv4_attn_mfma_kernel<2, COMPACT>);
            else if (rep <= 4) launch(&kv4_attn_mfma_kernel<4, COMPACT>);
            else if (rep <= 8) launch(&kv4_attn_mfma_kernel<8, COMPACT>);
            else launch(&kv4_attn_mfma_kernel<16, COMPACT>);
        };
        if (compact) form(std::true_type{});
        else form(std::false_type{});
    } else if (plan.form == KvForm::stream) {
        const dim3 grid(static_cast<unsigned>(splits) * static_cast<unsigned>(H_kv), 1u, nseq);
        auto launch = [&](auto kernel) {
            enqueue(kernel, grid, KV_THREADS, 0, st, q, S, S_max, splits, softmax_scale, kc, kp, vc, vp, L, part, batch);
        };
        auto form = [&](auto dt) {
            constexpr int QDT = decltype(dt)::value;
            if (batched) launch(&kv4_attn_stream_kernel<QDT, true, false>);
            else if (fused) launch(&kv4_attn_stream_kernel<QDT, false, true>);
            else launch(&kv4_attn_stream_kernel<QDT, false, false>);
        };
        if (q_dt == RCP_F32) form(std::integral_constant<int, RCP_F32>{});
        else if (q_dt == RCP_F16) form(std::integral_constant<int, RCP_F16>{});
        else form(std::integral_constant<int, RCP_BF16>{});
    } else {
        const dim3 grid(static_cast<unsigned>(kv_at_once_groups(splits, rep, H_kv)), 1u, nseq);
        auto launch = [&](auto kernel) {
            enqueue(kernel, grid, KV_THREADS, 0, st, q, S, S_max, rep, splits, softmax_scale, kc, kp, vc, vp, part, batch);
        };
#define RCP_KV_LAUNCH(QDT, ITERS)                                        \
    do {                                                                 \
        if (batched) launch(&kv4_attn_kernel<QDT, ITERS, true>);         \
        else if (fused) launch(&kv4_attn_kernel<QDT, ITERS, false, true>); \
        else launch(&kv4_attn_kernel<QDT, ITERS, false>);                \
    } while (0)
#define RCP_KV_DISPATCH(QDT)                                                          \
    do {                                                                              \
        if (L == 64) RCP_KV_LAUNCH(QDT, 1);                                           \
        else if (L == 128) RCP_KV_LAUNCH(QDT, 2);                                     \
        else RCP_KV_LAUNCH(QDT, 4);                                                   \
    } while (0)
        if (q_dt == RCP_F32) RCP_KV_DISPATCH(RCP_F32);
        else if (q_dt == RCP_F16) RCP_KV_DISPATCH(RCP_F16);
        else RCP_KV_DISPATCH(RCP_BF16);
#undef RCP_KV_DISPATCH
#undef RCP_KV_LAUNCH
    }
    int rc = check_launch("rcp_kv4_attn_decode");
    if (rc != RCP_OK) return rc;
    int groups = (splits + 3) / 4;
    if (groups > KV_CT / KV_D) groups = KV_CT / KV_D;
    const unsigned cgrid = static_cast<unsigned>(H_q) * (batched ? B : 1);
    auto combine = [&](auto kernel) { enqueue(kernel, cgrid, groups * KV_D, 0, st, part, splits, groups, out, L, plan.form == KvForm::at_once ? 1.44269504088896340736f : 1.0f, batch); };
    if (batched) {
        if (out_dt == RCP_F16) combine(&kv4_combine_kernel<true, true>);
        else combine(&kv4_combine_kernel<false, true>);
    } else {
        if (out_dt == RCP_F16) combine(&kv4_combine_kernel<true, false>);
        else combine(&kv4_combine_kernel<false, false>);
    }
    return check_launch("rcp_kv4_attn_decode(combine)");
}

}  // namespace rcp
