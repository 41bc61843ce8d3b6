// Skinny W2A4 GEMM (several tokens) with group-wise look-up tables on the matrix cores: the
// scheme of gemm_mfma.hip (masked bit-plane words as FP4 operands of the 16x16x128 matrix
// instruction) applied to the paper's deployed weight setting, one LUT per (row, 128 input
// channels) (Appendix table of quantisation configurations; Section 4.4 for the product).
//
//     P[m][h][g][l] = sum_{k in group g : idx[h][k] = l} q[m][k]              (exact)
//     O[m][h]       = S[m] * sum_g sum_l LUT[h][g][l] * P[m][h][g][l]        (fp32)
//
// One 128-column step of the matrix instruction is exactly one quantisation group, so the
// accumulators are not carried from step to step: after three instructions (one per bit plane; the
// 16 rows of the A operand are (row group, row in the nibble) pairs as in gemm_mfma.hip, the mask
// a per-lane value, the int4 activations FP8 bytes)
// a lane holds the exact plane sums F_p of four rows for one token, times the power of two that the
// operands' units leave in them (where several groups are taken at a time), and adds their products with
// the group's levels to four running fp32 outputs.  The power of two is taken out of the levels, once
// for all tokens and without a rounding: a scaled instruction would take the vector unit four
// cycles longer (eight layers of 4096 / 14336 at 6 tokens,
// quantisers and rotations included, 359.2 -> 356.6 us).  The per-group sum T of q that level 0 needs comes
// from one more instruction with an all-ones A operand.  The fourth row of a nibble is the FP4 sign
// bit; its lanes shift it down by one.
//
// Work decomposition.  A wavefront takes a batch of four neighbouring groups, converts the
// activations of the batch once, and walks the sixteen-row blocks of its workgroup with the next
// block's weights and levels in flight: small loads that arrive one after the other, so that the
// products overlap the stream.  (With 64 rows at a time in registers all wavefronts waited for the
// end of the stream and computed after it; and the conversion weighs as much as the products of
// sixteen rows.)  The four lanes of a quad share a row group: each fetches one group of the batch,
// 64 consecutive bytes together -- in memory the same unit of neighbouring groups lies side by side,
// while row groups are K/16 units apart -- and a step takes its group from one of the four lanes.
// (Fetched in operand order, every lane is a request of its own and every cache line is asked for by
// four wavefronts at different times: the loads alone took 13.6 of 16.1 us on 28672 x 4096.)
// Token l%16 feeds the B operand; up to 8 (4) tokens, lanes 8 (4) apart convert different groups of
// the batch and the operand of each is rotated into place.
// The levels of the 64 (row, group) pairs of a block and batch come one pair to a lane, which turns
// the four levels into the coefficients of (sum of q, F_b0, F_b1, F_b0&b1),
//     O += L0*T + (L1-L0)*F0 + (L2-L0)*F1 + (L3-L2-L1+L0)*F3      (= sum_l L_l * P_l),
// once for all token lanes; they are read back from a wavefront-private LDS buffer as broadcasts.
// Every wavefront parks its partial outputs in LDS and the workgroup adds them in a fixed order
// (deterministic), scales and stores.
#include <type_traits>

#include "rcp_internal.hpp"

namespace rcp {

constexpr int MG_WAVES = 16;   // wavefronts per workgroup at most
constexpr int MG_P_WAVES = 8;  // with batches of four and the per-group sums
constexpr int MG_MAX_BLOCKS = 8;   // sixteen-row blocks per workgroup at most (partial outputs in LDS)

// every lane of a quad gets what lane s of it holds
template <int S>
__device__ __forceinline__ uint32_t quad_broadcast(uint32_t v)
{
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), S * 0x55, 0xf, 0xf, true));
}

struct MgBlock {
    u32x4 wa, wb;  // two units of (row group quad % 4, group quad lane): 4 rows x 16 columns each, planes interleaved per cell
    uint2 lut;     // the levels of one (row, group)
};

// BATCH: groups a wavefront takes at a time: four (one 64-byte piece per row group and unit), or one (short K, where four
// would leave most wavefronts without work).
// TK: tokens a B operand holds (16, 8 or 4): the smallest of them that is not below M.
// WANTP: the per-group sums are written to Pout as well (a verification output), the four groups of a batch together, so that
// a cache line is not left half written while the other wavefronts' lines push it out.  With batches of four that takes 144
// registers and leaves eight wavefronts, each of which stands for one or two of the W that the partial outputs are counted
// in, so that the outputs have the same bits.  (Sixteen wavefronts with 101 registers spilled: 28672 x 4096 at 2 / 16 tokens
// 100 / 247 us; now 24 / 95.)
template <bool OUT_F16, bool WANTP, int BATCH, int TK>
__global__ __launch_bounds__(64 * (WANTP && BATCH == 4 ? MG_P_WAVES : MG_WAVES)) void gemm_mfma_grouped_kernel(const uint4* __restrict__ packed,
                                                                       const uint4* __restrict__ codebook, int N, int K,
                                                                       const uint4* __restrict__ xq,
                                                                       const uint16_t* __restrict__ scale, int M, int W, int NB,
                                                                       void* __restrict__ out, int32_t* __restrict__ Pout)
{
    extern __shared__ float4 mg_lds[];
    // (W wavefronts and NB blocks of the workgroup are arguments: the launch dimensions would have to be fetched from memory)
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float4* const coef = mg_lds + wave * (BATCH * 16);                    // [group][row]: of (T, F0, F1, F3)
    const int stride = 16 * NB + 1;                                          // floats per token: conflict-free
    float* const slab = reinterpret_cast<float*>(mg_lds + W * (BATCH * 16));  // [wavefront][token][row]
    const int i = lane & 15, kb = lane >> 4, t = lane & 3;
    const int U = K / 16, G = N / 4, NG = K / RCP_GROUP;
    const int rg0 = static_cast<int>(blockIdx.x) * 4 * NB;
    // this lane's row of the nibble as a mask, how far it is shifted down (the fourth row is the FP4 sign bit), and the
    // power of two that undoes the 0.5 / 1 / 2 / 2 it then stands for and the activations' unit
    const uint32_t row_mask = 0x11111111u << t, row_shift = t == 3 ? 1u : 0u;
    // (one group at a time the levels are as many as the instructions, and the scaled instruction does it: 130000 x 1536 at
    // 2 tokens 28.2 us, 28.5 with the levels multiplied)
    constexpr bool SCALED = BATCH == 1;
    constexpr float INT_UNIT = SCALED ? 1.0f : FP8_INT_UNIT;
    constexpr int SC_ONE = SCALED ? 0x7f : 0, SC_INT = SCALED ? FP8_INT_SCALE : 0;
    const float row_unit = SCALED ? 1.0f : FP8_INT_UNIT * (t == 0 ? 2.0f : t == 1 ? 1.0f : 0.5f);
    const int row_scale = SCALED ? (t == 0 ? 0x80 : t == 1 ? 0x7f : 0x7e) : 0;

    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint4*>(packed), 0, static_cast<int>(static_cast<unsigned>(G) * static_cast<unsigned>(U) * 16u), 0x00020000);
    const __amdgpu_buffer_rsrc_t cres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint4*>(codebook), 0, static_cast<int>(static_cast<unsigned>(G) * static_cast<unsigned>(NG) * 32u), 0x00020000);
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(xq), 0, M * (K / 2), 0x00020000);
    constexpr unsigned OUTSIDE = 0x80000000u;            // beyond every resource: reads as zero
    constexpr int PER = 16 / TK, NX = BATCH / PER;
    static_assert(BATCH == 4 || (BATCH == 1 && TK == 16), "");    // groups per converted operand, conversions per batch

    const int batches = (NG + BATCH - 1) / BATCH;
    const int lg = BATCH == 1 ? 0 : (lane >> 2) & 3;  // the group of this lane's levels; row group lane / 16, row lane % 4
    const int wg = BATCH == 1 ? 0 : t;                // the group of this lane's weights
    // Groups past the end of K and row groups past the end of N lie outside the resources: they read zeros and add zeros.
    auto load = [&](int b, int block, MgBlock& st) {
        const int g0 = BATCH * b, round = g0 >> 5;
        const int R = min(32, NG - 32 * round);
        const unsigned unit = 256u * round + static_cast<unsigned>(a4b8_unit(kb)) * R + (g0 & 31) + wg;  // the second unit is 2 R further
        const unsigned wo = g0 + wg < NG ? static_cast<unsigned>(rg0 + 4 * block + (i >> 2)) * U * 16u + unit * 16u : OUTSIDE;
        const unsigned lo = g0 + lg < NG ? (static_cast<unsigned>(rg0 + 4 * block + kb) * NG + g0 + lg) * 32u + t * 8u : OUTSIDE;
        st.wa = __builtin_amdgcn_raw_buffer_load_b128(wres, static_cast<int>(wo), 0, 0);
        st.wb = __builtin_amdgcn_raw_buffer_load_b128(wres, static_cast<int>(wo), g0 < NG ? R * 32 : 0, 0);
        const auto l = __builtin_amdgcn_raw_buffer_load_b64(cres, static_cast<int>(lo), 0, 0);
        st.lut = make_uint2(l[0], l[1]);
    };
    u32x4 xv[NX];
    auto load_tokens = [&](int b) {
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            const int g = BATCH * b + PER * n + i / TK;  // tokens beyond M lie outside the resource
            xv[n] = __builtin_amdgcn_raw_buffer_load_b128(
                xres, static_cast<int>(((g < NG) & (i % TK < M)) ? static_cast<unsigned>(i % TK) * (K / 2) + kb * 16u + 64u * g : OUTSIDE), 0, 0);
        }
    };
    // the B operands of a batch's groups and the sums of q for this lane's token
    v8i bop[BATCH];
    float tq[BATCH];
    const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
    auto convert = [&]() {
        const v8i ones = {0x22222222, 0x22222222, 0x22222222, 0x22222222, 0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < BATCH; ++s) {
            if (s % PER == 0) {
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    int first, second;
                    int4_to_fp8(xv[s / PER][d], first, second);
                    bop[s][2 * d] = first;
                    bop[s][2 * d + 1] = second;
                }
            } else {  // this group was converted by the lanes TK further up: rotate them down
#pragma unroll
                for (int d = 0; d < 8; ++d) bop[s][d] = __builtin_amdgcn_mov_dpp(bop[s - 1][d], 0x120 + 16 - TK, 0xf, 0xf, true);
            }
            tq[s] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ones, bop[s], zero, 4, 0, 0, SC_ONE, 0, SC_INT)[0];
        }
    };
    // rows 4 * kb + v of the block, this lane's token
    auto products = [&](const MgBlock& cur, int block, int g0, float (&o)[4]) {
        {
            const float c0 = half_bits_to_float(static_cast<uint16_t>(cur.lut.x & 0xffffu));
            const float c1 = half_bits_to_float(static_cast<uint16_t>(cur.lut.x >> 16));
            const float c2 = half_bits_to_float(static_cast<uint16_t>(cur.lut.y & 0xffffu));
            const float c3 = half_bits_to_float(static_cast<uint16_t>(cur.lut.y >> 16));
            // (row_unit times L0, L1-L0, .. with the same roundings: it is a power of two)
            const float u0 = row_unit * c0;
            const float4 c = make_float4(INT_UNIT * c0, fmaf(row_unit, c1, -u0), fmaf(row_unit, c2, -u0),
                                         fmaf(row_unit, (c3 - c2) - c1, u0));
            coef[16 * lg + 4 * kb + t] = c;
        }
        int4 sums[4][BATCH];
        auto step = [&](auto index) {
            constexpr int s = decltype(index)::value;
            const uint32_t p0[4] = {cur.wa.x, cur.wa.z, cur.wb.x, cur.wb.z};
            const uint32_t p1[4] = {cur.wa.y, cur.wa.w, cur.wb.y, cur.wb.w};
            v8i an[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) an[p] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                an[0][d] = static_cast<int>(((BATCH == 1 ? p0[d] : quad_broadcast<s>(p0[d])) & row_mask) >> row_shift);
                an[1][d] = static_cast<int>(((BATCH == 1 ? p1[d] : quad_broadcast<s>(p1[d])) & row_mask) >> row_shift);
                an[2][d] = an[0][d] & an[1][d];
            }
            v4f F[3];
#pragma unroll
            for (int p = 0; p < 3; ++p)
                if constexpr (SCALED)
                    F[p] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(an[p], bop[s], zero, 4, 0, 0, row_scale, 0, SC_INT);
                else F[p] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(an[p], bop[s], zero, 4, 0, 0, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float4 c = coef[16 * s + 4 * kb + v];
                float val = fmaf(c.x, tq[s], o[v]);
                val = fmaf(c.y, F[0][v], val);
                val = fmaf(c.z, F[1][v], val);
                o[v] = fmaf(c.w, F[2][v], val);
                if constexpr (WANTP) {
                    const float unit = SCALED ? 1.0f : FP8_INT_UNIT * (v == 0 ? 2.0f : v == 1 ? 1.0f : 0.5f);
                    const float T = INT_UNIT * tq[s], F0 = unit * F[0][v], F1 = unit * F[1][v], F3 = unit * F[2][v];
                    sums[v][s] = make_int4(static_cast<int>(T - F0 - F1 + F3), static_cast<int>(F0 - F3), static_cast<int>(F1 - F3),
                                           static_cast<int>(F3));
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // one step's operands and sums live at a time
        };
        step(std::integral_constant<int, 0>{});
        if constexpr (BATCH == 4) {
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
        }
        // (the products run in all lanes: the compiler would move them into the branch, which switches rows off)
        asm volatile("" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(o[3]));
        if constexpr (WANTP) {
            const int group = rg0 + 4 * block + kb;
            if (i < M && group < G)
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int s = 0; s < BATCH; ++s)
                        if (g0 + s < NG) reinterpret_cast<int4*>(Pout)[(static_cast<size_t>(i) * N + 4 * group + v) * NG + g0 + s] = sums[v][s];
        }
    };
    auto park = [&](int part, int block, bool first, const float (&o)[4]) {
        if (i < TK) {
            float* const dst = slab + (part * TK + i) * stride + 16 * block + 4 * kb;
#pragma unroll
            for (int v = 0; v < 4; ++v) dst[v] = first ? o[v] : dst[v] + o[v];
        }
    };
    auto stream = [&](int part) {
        MgBlock cur;
        load_tokens(part);
        load(part, 0, cur);
        for (int b = part; b < batches; b += W) {  // uniform
            __builtin_amdgcn_sched_barrier(0);
            convert();
            __builtin_amdgcn_sched_barrier(0);
            // the activations of the next batch (sixteen tokens leave no registers for that: 128 keep sixteen wavefronts on a
            // compute unit)
            if constexpr (TK < 16) load_tokens(b + W);
            for (int block = 0; block < NB; ++block) {
                MgBlock next;  // the next block, or the first one of the next batch, is in flight while this one is computed
                const bool last = block + 1 == NB;
                // (one group at a time there is no next batch, and its loads would delay the barrier behind the loop by their
                // latency: 4096 x 2048 3.89 -> 3.75 us.  The condition itself costs the overlap where blocks and batches follow.)
                if (BATCH != 1 || !last || b + W < batches) load(last ? b + W : b, last ? 0 : block + 1, next);
                __builtin_amdgcn_sched_barrier(0);
                float o[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                products(cur, block, BATCH * b, o);
                park(part, block, b == part, o);
                cur = next;
            }
            if (TK == 16 && (BATCH != 1 || b + W < batches)) load_tokens(b + W);
        }
    };
    constexpr bool SHARED = WANTP && BATCH == 4;
    if constexpr (SHARED)
        for (int part = wave; part < W; part += MG_P_WAVES) stream(part);
    else stream(wave);
    __syncthreads();

    for (int idx = tid; idx < M * 16 * NB; idx += 64 * (SHARED ? min(W, MG_P_WAVES) : W)) {
        const int n = idx / (16 * NB), hh = idx - n * (16 * NB);
        const int h = 4 * rg0 + hh;
        if (h >= N) continue;
        float val = 0.0f;
        for (int w = 0; w < W; ++w) val += slab[(w * TK + n) * stride + hh];  // fixed order
        val *= half_bits_to_float(scale[n]);
        const size_t oi = static_cast<size_t>(n) * N + h;
        if constexpr (OUT_F16) static_cast<__half*>(out)[oi] = __float2half_rn(val);
        else static_cast<float*>(out)[oi] = val;
    }
}

int launch_gemm_mfma_grouped(const void* packed, const void* codebook, int N, int K, const void* xq,
                             const void* scale, int M, void* out, rcp_dtype out_dt, int32_t* P, hipStream_t st)
{
    if (static_cast<long long>(N) * K / 4 >= (1LL << 31))
        return fail(RCP_ERR_SHAPE, "rcp_w2a4_gemm_grouped: packed matrix of %lld bytes exceeds 2 GiB",
                    static_cast<long long>(N) * K / 4);
    const int NG = K / RCP_GROUP;
    // One workgroup per compute unit, of as many sixteen-row blocks as that takes ("gemm_rows" sets the rows): the converted
    // activations serve all of them, and no unit carries more than its share.  At 6 tokens, blocks per workgroup 1 / 2 / 3 /
    // 4: 12288 x 4096 8.0 / 7.2 / 6.4 / 7.0 us, 28672 x 4096 15.7 / 12.6 / 12.8 / 11.2, and 10.6 with seven; the first form
    // of this kernel (64 or 16 rows, one group at a time): 7.7 and 15.3.
    const int total = (N + 15) / 16, cus = num_compute_units();
    int nb = (total + cus - 1) / cus;
    if (nb > MG_MAX_BLOCKS) nb = MG_MAX_BLOCKS;
    if (options().gemm_rows != 0) nb = (options().gemm_rows + 15) / 16;
    // One group at a time up to K = 2048, where batches of four would leave most of the wavefronts without work (256 x 512 at
    // 16 tokens 3.8 against 2.5 us, 8192 x 2048 4.8 against 4.3), else four (4096 x 4096 at 16 tokens 5.0 against 5.2).
    const int batch = NG <= 16 ? 1 : 4;
    // As few wavefronts as take the batches in the same number of rounds as the most would: sixteen (4096 x 14336, 6 tokens:
    // 9.9 us with at most eight, 9.0 with fourteen).
    const int batches = (NG + batch - 1) / batch;
    int waves = options().gemm_waves != 0 ? options().gemm_waves : MG_WAVES;
    const int rounds = (batches + waves - 1) / waves;
    waves = (batches + rounds - 1) / rounds;
    const int blocks = (total + nb - 1) / nb;
    auto* pk = static_cast<const uint4*>(packed);
    auto* cb = static_cast<const uint4*>(codebook);
    auto* x4 = static_cast<const uint4*>(xq);
    auto* sc = static_cast<const uint16_t*>(scale);
    const int tk = P != nullptr || batch == 1 || M > 8 ? 16 : M > 4 ? 8 : 4;
    const int resident = P != nullptr && batch == 4 && waves > MG_P_WAVES ? MG_P_WAVES : waves;
    const size_t lds = static_cast<size_t>(waves) * (batch * 16 * sizeof(float4) + tk * (16 * nb + 1) * sizeof(float));
#define RCP_MG(F16, P_, B_, TK)                                                                                                 \
    do {                                                                                                                        \
        if (lds > 64 * 1024) {                                                                                                  \
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_mfma_grouped_kernel<F16, P_, B_, TK>), \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));        \
            if (e != hipSuccess) return fail(RCP_ERR_HIP, "rcp_w2a4_gemm_grouped: LDS opt-in failed: %s", hipGetErrorString(e)); \
        }                                                                                                                       \
        enqueue(&gemm_mfma_grouped_kernel<F16, P_, B_, TK>, blocks, resident * 64, lds, st, pk, cb, N, K, x4, sc, M, waves, nb, out, P); \
    } while (0)
#define RCP_MG_TK(F16)                               \
    do {                                             \
        if (batch == 1) {                            \
            if (P != nullptr) RCP_MG(F16, true, 1, 16);  \
            else RCP_MG(F16, false, 1, 16);          \
        } else if (P != nullptr) RCP_MG(F16, true, 4, 16);  \
        else if (tk == 4) RCP_MG(F16, false, 4, 4);  \
        else if (tk == 8) RCP_MG(F16, false, 4, 8);  \
        else RCP_MG(F16, false, 4, 16);              \
    } while (0)
    if (out_dt == RCP_F16) RCP_MG_TK(true);
    else RCP_MG_TK(false);
#undef RCP_MG_TK
#undef RCP_MG
    return check_launch("rcp_w2a4_gemm_grouped");
}

}  // namespace rcp
