// Decoder glue between the W4A4 linears of a Llama-shaped layer: rotary position embedding,
// causal softmax attention over a short prefix, residual add.  (RMSNorm and the SwiGLU gate are
// fused into the activation quantizer, quantize.hip.)  The paper does not restate the decoder;
// these follow the published architecture (Su et al. 2021 in the half-split pairing used by
// Llama; Vaswani et al. 2017).  Attention of head sizes 64 and 128 runs on the matrix cores (attention.hip); the small
// head sizes take binary32 FMAs over LDS tiles with an online softmax, here.
#include <algorithm>

#include "common.h"
#include "quant_math.h"
#include "decode_attn.h"

namespace sqap {

// v'_i = v_i cos a - v_{i+d/2} sin a,  v'_{i+d/2} = v_{i+d/2} cos a + v_i sin a,
// a = pos * base^(-2i/d); angle, sine and cosine in binary64, products in binary64, one rounding
// to half.  One thread per (token, head, i); consecutive threads take consecutive i.
__global__ __launch_bounds__(256) void rope_kernel(__half *__restrict__ X, int64_t ld, const int32_t *__restrict__ pos,
                                                   int S, int H, int d, double base, const RopeFreq freq)
{
    const int half_d = d >> 1;
    const int64_t total = (int64_t)S * H * half_d;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int i = (int)(idx % half_d);
    const int64_t sh = idx / half_d;
    const int h = (int)(sh % H);
    const int s = (int)(sh / H);
    __half *v = X + (int64_t)s * ld + (int64_t)h * d;
    const double a = rope_angle(freq, pos[s], i, d, base);
    double sn, cs;
    sincos(a, &sn, &cs);
    const double lo = (double)__half2float(v[i]), hi = (double)__half2float(v[i + half_d]);
    v[i] = __float2half_rn((float)(lo * cs - hi * sn));
    v[i + half_d] = __float2half_rn((float)(hi * cs + lo * sn));
}

// Rotary embedding of a fused q|k|v row block with the key/value cache append folded in: queries are rotated
// in place, keys are rotated on their way into the cache row (the copy in the q|k|v buffer stays as it was),
// values are copied.  Same arithmetic as rope_kernel; one launch instead of a rotation and a row copy.
// One thread per (token, head-or-value slot, i): slots 0 .. H-1 queries, H .. 2H-1 keys, 2H .. 3H-1 values.
__global__ __launch_bounds__(256) void rope_append_kernel(__half *__restrict__ QKV, int64_t ld,
                                                          const int32_t *__restrict__ pos, int S, int H, int d,
                                                          double base, __half *__restrict__ KV, int64_t ldkv, const RopeFreq freq)
{
    const int half_d = d >> 1;
    const int64_t total = (int64_t)S * 3 * H * half_d;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int i = (int)(idx % half_d);
    const int64_t sh = idx / half_d;
    const int slot = (int)(sh % (3 * H));
    const int s = (int)(sh / (3 * H));
    const __half *src = QKV + (int64_t)s * ld + (int64_t)slot * d;
    if (slot >= 2 * H) {                                      // value: plain copy of the pair
        __half *dst = KV + (int64_t)s * ldkv + (int64_t)(slot - H) * d;
        dst[i] = src[i];
        dst[i + half_d] = src[i + half_d];
        return;
    }
    const double a = rope_angle(freq, pos[s], i, d, base);
    double sn, cs;
    sincos(a, &sn, &cs);
    const double lo = (double)__half2float(src[i]), hi = (double)__half2float(src[i + half_d]);
    const __half r0 = __float2half_rn((float)(lo * cs - hi * sn));
    const __half r1 = __float2half_rn((float)(hi * cs + lo * sn));
    __half *dst = slot < H ? QKV + (int64_t)s * ld + (int64_t)slot * d : KV + (int64_t)s * ldkv + (int64_t)(slot - H) * d;
    dst[i] = r0;
    dst[i + half_d] = r1;
}

// The same in 16-byte pieces, for head sizes that are a power of two from 16 to 256 and rows that lie 16 bytes aligned: a
// workgroup takes one token (or a share of its heads, where tokens are few), evaluates the d/2 angles of its position
// once and shares sines and cosines through LDS; a thread keeps the eight pairs of its piece in registers and rotates that
// piece of head after head, two 16-byte loads and stores each, the first head's asked for before the angles.
// APPEND: slots 0 .. H-1 queries, H .. 2H-1 keys (into the cache), 2H .. 3H-1 values (copied).
// What bounds it: memory with many tokens (77 MB at 2368 tokens x 64 heads of 128, 15 us at the rate of a copy), the sine
// and cosine with few.  Measured (us): 2368 tokens 15.1 (one pair per thread and step: 26.2), 148 with append 3.4 (5.9).
// Where a thread per pair, or from kRopeTokenKernelFrom tokens on rope_token_kernel, is quicker: few pairs (append, 8 tokens of 64
// heads of 256 2.42 against 2.66, 64 of 32 heads of 64 2.42 against 2.55, 512 of 8 heads of 32 2.48 against 2.58; the other way
// round 130 of 8 heads of 128 2.52 against 2.68), and tokens that fill less than half a wavefront, of which the workgroup has
// four (2400 tokens, 4 heads of 64: 3.90 against 4.60, 8 heads 4.45 against 4.41; append, 1 head of 64: 2.93 against 4.65).
template <bool APPEND>
__global__ __launch_bounds__(256) void rope_pieces_kernel(__half *__restrict__ X, int64_t ld, const int32_t *__restrict__ pos, int H,
                                                          int d, double base, __half *__restrict__ KV, int64_t ldkv,
                                                          const RopeFreq freq)
{
    __shared__ double cs[kRopeTableMax], sn[kRopeTableMax];
    const int half_d = d >> 1, s = blockIdx.x, t = threadIdx.x;
    const int pieces = half_d >> 3, piece = t & (pieces - 1);         // (a power of two)
    const int slots = APPEND ? 3 * H : H, step = 256 / pieces * gridDim.y;
    int slot = t / pieces + 256 / pieces * blockIdx.y;
    __half *row = X + (int64_t)s * ld + piece * 8;
    union Piece { sqap_v4u v; __half2 h[4]; };
    Piece lo, hi;
    lo.v = hi.v = sqap_v4u{0u, 0u, 0u, 0u};
    auto fetch = [&] {
        lo.v = *reinterpret_cast<const sqap_v4u *>(row + (int64_t)slot * d);
        hi.v = *reinterpret_cast<const sqap_v4u *>(row + (int64_t)slot * d + half_d);
    };
    if (slot < slots) fetch();
    if (t < half_d) {
        double sv, cv;
        sincos(rope_angle(freq, pos[s], t, d, base), &sv, &cv);
        sn[t] = sv;
        cs[t] = cv;
    }
    __syncthreads();
    double c8[8], s8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        c8[e] = cs[piece * 8 + e];
        s8[e] = sn[piece * 8 + e];
    }
    while (slot < slots) {
        __half *to = !APPEND || slot < H ? row + (int64_t)slot * d : KV + (int64_t)s * ldkv + (int64_t)(slot - H) * d + piece * 8;
        if (!APPEND || slot < 2 * H) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const float2 a = __half22float2(lo.h[p]), b = __half22float2(hi.h[p]);
                const double a0 = (double)a.x, a1 = (double)a.y, b0 = (double)b.x, b1 = (double)b.y;
                lo.h[p] = __halves2half2(__float2half_rn((float)(a0 * c8[2 * p] - b0 * s8[2 * p])),
                                         __float2half_rn((float)(a1 * c8[2 * p + 1] - b1 * s8[2 * p + 1])));
                hi.h[p] = __halves2half2(__float2half_rn((float)(b0 * c8[2 * p] + a0 * s8[2 * p])),
                                         __float2half_rn((float)(b1 * c8[2 * p + 1] + a1 * s8[2 * p + 1])));
            }
        }
        *reinterpret_cast<sqap_v4u *>(to) = lo.v;
        *reinterpret_cast<sqap_v4u *>(to + half_d) = hi.v;
        slot += step;
        if (slot < slots) fetch();
    }
}

constexpr int kRopeTokenKernelFrom = 512;        // tokens
constexpr int kRopePiecesMinThreads = 32;        // with work, of a workgroup

template <bool APPEND>
static bool launch_rope_pieces(__half *X, int64_t ld, const int32_t *pos, int S, int H, int d, double base, __half *KV,
                               int64_t ldkv, hipStream_t st)
{
    if (d < 16 || d > 2 * kRopeTableMax || (d & (d - 1)) != 0 || (ld & 7) != 0 || (reinterpret_cast<uintptr_t>(X) & 15u) != 0) return false;
    if (APPEND && ((ldkv & 7) != 0 || (reinterpret_cast<uintptr_t>(KV) & 15u) != 0)) return false;
    const int64_t threads = (int64_t)(APPEND ? 3 * H : H) * (d / 16);         // that a token has work for
    const int from = !APPEND && S >= kRopeTokenKernelFrom ? 1 << 17 : S < 128 ? 1 << 18 : (3 << 16) + 1;        // pairs
    if (threads < kRopePiecesMinThreads || S * threads * 8 < from) return false;
    // few tokens: a token's heads are dealt to as many workgroups as they fill, up to four per compute unit in all
    const int rounds = ((APPEND ? 3 * H : H) * (d / 16) + 255) / 256;
    const int shares = S >= 1024 ? 1 : std::min(rounds, std::min(64, 1024 / S + 1));
    hipLaunchKernelGGL(rope_pieces_kernel<APPEND>, dim3(S, shares), dim3(256), 0, st, X, ld, pos, H, d, base, KV, ldkv,
                       rope_frequencies(d, base));
    return true;
}

sqap_status launch_rope_append(__half *QKV, int64_t ld, const int32_t *pos, int S, int H, int d, double base,
                               __half *KV, int64_t ldkv, hipStream_t st)
{
    const int64_t total = (int64_t)S * 3 * H * (d / 2);
    if (total == 0) return SQAP_OK;
    if (launch_rope_pieces<true>(QKV, ld, pos, S, H, d, base, KV, ldkv, st)) {
        SQAP_HIP_CHECK(hipGetLastError());
        return SQAP_OK;
    }
    hipLaunchKernelGGL(rope_append_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, QKV, ld, pos, S, H, d,
                       base, KV, ldkv, rope_frequencies(d, base));
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// What the pieces leave, many tokens: one workgroup per token evaluates the d/2 angles of its position once (the
// binary64 power, sine and cosine are a few hundred instructions per pair) and shares them between the
// heads through LDS.  With few tokens the per-pair kernel is faster (more threads in flight: 6.7 against
// 8.8 us at 84 tokens); at 2368 tokens this one takes a tenth of its time.
constexpr int kRopeMaxHalfD = 256;

__global__ __launch_bounds__(256) void rope_token_kernel(__half *__restrict__ X, int64_t ld,
                                                         const int32_t *__restrict__ pos, int H, int d, double base,
                                                         const RopeFreq freq)
{
    __shared__ double cs[kRopeMaxHalfD], sn[kRopeMaxHalfD];
    const int half_d = d >> 1, s = blockIdx.x;
    for (int i = threadIdx.x; i < half_d; i += 256) {
        const double a = rope_angle(freq, pos[s], i, d, base);
        double sv, cv;
        sincos(a, &sv, &cv);
        sn[i] = sv;
        cs[i] = cv;
    }
    __syncthreads();
    __half *row = X + (int64_t)s * ld;
    for (int idx = threadIdx.x; idx < H * half_d; idx += 256) {
        const int h = idx / half_d, i = idx - h * half_d;
        __half *v = row + (int64_t)h * d;
        const double lo = (double)__half2float(v[i]), hi = (double)__half2float(v[i + half_d]);
        v[i] = __float2half_rn((float)(lo * cs[i] - hi * sn[i]));
        v[i + half_d] = __float2half_rn((float)(hi * cs[i] + lo * sn[i]));
    }
}

sqap_status launch_rope(__half *X, int64_t ld, const int32_t *pos, int S, int H, int d, double base, hipStream_t st)
{
    const int64_t total = (int64_t)S * H * (d / 2);
    if (total == 0) return SQAP_OK;
    if (launch_rope_pieces<false>(X, ld, pos, S, H, d, base, nullptr, 0, st)) {
        SQAP_HIP_CHECK(hipGetLastError());
        return SQAP_OK;
    }
    if (S >= kRopeTokenKernelFrom && d / 2 <= kRopeMaxHalfD) {
        hipLaunchKernelGGL(rope_token_kernel, dim3(S), dim3(256), 0, st, X, ld, pos, H, d, base, rope_frequencies(d, base));
        SQAP_HIP_CHECK(hipGetLastError());
        return SQAP_OK;
    }
    hipLaunchKernelGGL(rope_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, X, ld, pos, S, H, d, base,
                       rope_frequencies(d, base));
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// Causal attention.  Query i (of Sq) sits at sequence position Sk - Sq + i and sees keys 0 ..
// Sk - Sq + i.  A batch of sequences is a stack of row blocks (Sq rows of Q and O, Sk rows of K
// and V per sequence).  This scalar form serves the small head sizes (16 and 32): one workgroup per
// (head, block of 32 queries, sequence); keys and values pass through LDS in tiles of 64.  Thread t
// works for query t/8: in the score phase on keys 8(t%8) .. +7 of the tile, in the output phase on
// the D/8 consecutive head-dimension columns from (t%8) D/8 on.  Running maximum m, running sum l
// and the output row are rescaled when a tile raises the maximum (the usual online softmax); all in
// binary32.
constexpr int kAttQ = 32, kAttK = 64;

template <int D>
__global__ __launch_bounds__(256) void attention_kernel(const __half *__restrict__ Q, int64_t ldq,
                                                        const __half *__restrict__ Kc, int64_t ldk,
                                                        const __half *__restrict__ V, int64_t ldv, int Sq, int Sk,
                                                        int H, __half *__restrict__ O, int64_t ldo)
{
    constexpr int PITCH = D + 8;                 // halves per LDS row: keeps 16-byte alignment, staggers the banks
    constexpr int CPT = D / 8;                   // output columns per thread
    __shared__ __attribute__((aligned(16))) __half qs[kAttQ * PITCH];
    __shared__ __attribute__((aligned(16))) __half ks[kAttK * PITCH];
    __shared__ __attribute__((aligned(16))) __half vs[kAttK * PITCH];
    __shared__ float ps[kAttQ * (kAttK + 1)];
    const int t = threadIdx.x, h = blockIdx.x, q0 = blockIdx.y * kAttQ;
    const int qi = t >> 3, sub = t & 7;
    Q += (int64_t)blockIdx.z * Sq * ldq;
    O += (int64_t)blockIdx.z * Sq * ldo;
    Kc += (int64_t)blockIdx.z * Sk * ldk;
    V += (int64_t)blockIdx.z * Sk * ldv;
    const int shift = Sk - Sq;                   // query i sees keys <= i + shift
    const float inv_sqrt_d = 1.0f / sqrtf((float)D);

    for (int u = t; u < kAttQ * (D / 8); u += 256) {
        const int r = u / (D / 8), c = u % (D / 8);
        uint4 raw = make_uint4(0u, 0u, 0u, 0u);
        if (q0 + r < Sq) raw = *reinterpret_cast<const uint4 *>(Q + (int64_t)(q0 + r) * ldq + (int64_t)h * D + c * 8);
        *reinterpret_cast<uint4 *>(qs + r * PITCH + c * 8) = raw;
    }
    float o[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) o[c] = 0.f;
    float m = -INFINITY, l = 0.f;
    const int my_q = q0 + qi;
    const int last_key = min(Sk - 1, min(q0 + kAttQ - 1, Sq - 1) + shift);      // of the whole block
    for (int k0 = 0; k0 <= last_key; k0 += kAttK) {
        __syncthreads();                                                        // previous tile consumed (and qs written)
        for (int u = t; u < kAttK * (D / 8); u += 256) {
            const int r = u / (D / 8), c = u % (D / 8);
            uint4 kr = make_uint4(0u, 0u, 0u, 0u), vr = kr;
            if (k0 + r < Sk) {
                kr = *reinterpret_cast<const uint4 *>(Kc + (int64_t)(k0 + r) * ldk + (int64_t)h * D + c * 8);
                vr = *reinterpret_cast<const uint4 *>(V + (int64_t)(k0 + r) * ldv + (int64_t)h * D + c * 8);
            }
            *reinterpret_cast<uint4 *>(ks + r * PITCH + c * 8) = kr;
            *reinterpret_cast<uint4 *>(vs + r * PITCH + c * 8) = vr;
        }
        __syncthreads();
        // scores of this thread's 8 keys
        float sc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sc[j] = 0.f;
        for (int c = 0; c < D; c += 8) {
            const uint4 qraw = *reinterpret_cast<const uint4 *>(qs + qi * PITCH + c);
            const __half2 *q2 = reinterpret_cast<const __half2 *>(&qraw);
            float qf[8];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const float2 f = __half22float2(q2[p]);
                qf[2 * p] = f.x;
                qf[2 * p + 1] = f.y;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint4 kraw = *reinterpret_cast<const uint4 *>(ks + (sub * 8 + j) * PITCH + c);
                const __half2 *k2 = reinterpret_cast<const __half2 *>(&kraw);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const float2 f = __half22float2(k2[p]);
                    sc[j] = fmaf(qf[2 * p], f.x, sc[j]);
                    sc[j] = fmaf(qf[2 * p + 1], f.y, sc[j]);
                }
            }
        }
        float tile_max = -INFINITY;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int key = k0 + sub * 8 + j;
            const bool seen = key < Sk && key <= my_q + shift && my_q < Sq;
            sc[j] = seen ? sc[j] * inv_sqrt_d : -INFINITY;
            tile_max = fmaxf(tile_max, sc[j]);
        }
        for (int x = 1; x < 8; x <<= 1) tile_max = fmaxf(tile_max, __shfl_xor(tile_max, x));
        const float m_new = fmaxf(m, tile_max);
        // a query that has seen no key yet keeps m = -inf; exp(-inf - -inf) is avoided
        const float rescale = m_new == -INFINITY ? 1.f : expf(m - m_new);
        float tile_sum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float pj = sc[j] == -INFINITY ? 0.f : expf(sc[j] - m_new);
            ps[qi * (kAttK + 1) + sub * 8 + j] = pj;
            tile_sum += pj;
        }
        for (int x = 1; x < 8; x <<= 1) tile_sum += __shfl_xor(tile_sum, x);
        l = l * rescale + tile_sum;
        m = m_new;
        __syncthreads();                                                        // ps complete
#pragma unroll
        for (int c = 0; c < CPT; ++c) o[c] *= rescale;
        const int kmax = min(min(kAttK, Sk - k0), my_q + shift - k0 + 1);      // (no infinite value times the zero of a query that does not see it)
        for (int j = 0; j < kmax; ++j) {
            const float pj = ps[qi * (kAttK + 1) + j];
            const __half *vrow = vs + j * PITCH + sub * CPT;
#pragma unroll
            for (int c = 0; c < CPT; c += 2) {
                const float2 f = __half22float2(*reinterpret_cast<const __half2 *>(vrow + c));
                o[c] = fmaf(pj, f.x, o[c]);
                o[c + 1] = fmaf(pj, f.y, o[c + 1]);
            }
        }
    }
    if (my_q < Sq) {
        __half *dst = O + (int64_t)my_q * ldo + (int64_t)h * D + sub * CPT;
        const float inv_l = 1.0f / l;
#pragma unroll
        for (int c = 0; c < CPT; c += 2)
            *reinterpret_cast<__half2 *>(dst + c) = __floats2half2_rn(o[c] * inv_l, o[c + 1] * inv_l);
    }
}

sqap_status launch_attention(const __half *Q, int64_t ldq, const __half *Kc, int64_t ldk, const __half *V,
                             int64_t ldv, int batch, int Sq, int Sk, int H, int d, __half *O, int64_t ldo, hipStream_t st)
{
    if (Sq == 0 || batch == 0) return SQAP_OK;
    if (d == 64 || d == 128) return launch_attention_tiles(Q, ldq, Kc, ldk, V, ldv, batch, Sq, Sk, H, d, O, ldo, st);
    const dim3 grid(H, (Sq + kAttQ - 1) / kAttQ, batch);
#define SQAP_ATT_CASE(DD)                                                                                          \
    case DD:                                                                                                       \
        hipLaunchKernelGGL(attention_kernel<DD>, grid, dim3(256), 0, st, Q, ldq, Kc, ldk, V, ldv, Sq, Sk, H, O, ldo); \
        break;
    switch (d) {
        SQAP_ATT_CASE(16)
        SQAP_ATT_CASE(32)
    default:
        return fail(SQAP_EUNSUPPORTED, "attention: head size %d (16, 32, 64 or 128)", d);
    }
#undef SQAP_ATT_CASE
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// The workgroup (of T threads) that arrives last, of n_groups, quantizes the whole output row, as quantize_rows_kernel does.  The outputs
// were stored past the caches (agent scope), are complete once the vector-memory counter has drained, and are read past the caches
// here: no fence, which would write back and invalidate a whole L2 per workgroup.
// row_lds: width halves of LDS, wave_max: T / 64 floats.
template <int T>
__device__ __forceinline__ void quantize_by_the_last(float *row_lds, float *wave_max, int *last_flag, const __half *O, int width,
                                                     int n_groups, uint8_t *Xq, __half *sx, unsigned int *counter)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's outputs have arrived before the workgroup does
    lds_barrier();
    if (t == 0) *last_flag = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned int)(n_groups - 1);
    lds_barrier();
    if (!*last_flag) return;
    __half *row = reinterpret_cast<__half *>(row_lds);
    const int groups = width >> 3;
    float amax = 0.f;
    for (int g = t; g < groups; g += T) {
        union { unsigned long long u[2]; uint4 v; } raw;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            raw.u[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(O) + 2 * g + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        reinterpret_cast<uint4 *>(row)[g] = raw.v;
        float f[8];
        unpack_halves(raw.v, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(f[e]));
    }
    amax = wavefront_max(amax);
    if (lane == 0) wave_max[wave] = amax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < T / 64; ++w) amax = fmaxf(amax, wave_max[w]);
    const __half sh = row_scale(amax);
    const float sf = __half2float(sh);
    const Reciprocal rcp = scale_reciprocal(sf);
    if (t == 0) {
        sx[0] = sh;
        __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);       // the next call starts from zero again
    }
    for (int g = t; g < groups; g += T) {
        float f[8];
        unpack_halves(reinterpret_cast<const uint4 *>(row)[g], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = quotient(f[e], rcp);
        reinterpret_cast<uint32_t *>(Xq)[g] = pack_codes8(f);
    }
}

// One decode step's attention in a single launch: the new token's query and key are rotated (same
// arithmetic as rope_kernel), the rotated key and the value go into row `past` of the cache, and the
// query attends to cache rows 0 .. past.  One workgroup per head.  At one token each of the three
// launches this replaces (rotation + append, attention, activation quantizer) is a few microseconds
// of latency and no work, so the quantizer of the following linear is folded in as well: the
// workgroup that finishes last (a device-wide arrival counter) quantizes the whole output row.
//
// Scores: 16 lanes per key, lane c holding columns 8c .. 8c+7 (one 16-byte load per key row); softmax over
// chunks of 192 keys with the usual running maximum and sum; output: the same lane layout over the value
// rows, the 16 key groups added through LDS.  All binary32.  A chunk's key AND value rows (12 of each per
// lane) are asked for at once, the first chunk's before the rotation, whose binary64 sine and cosine are a
// longer dependent chain than the rest of the kernel: a prefix of up to 191 positions costs one round of loads.
__global__ __launch_bounds__(256) void decode_attention_kernel(const __half *__restrict__ QKV,
                                                               const int32_t *__restrict__ pos, int H, int d,
                                                               double base, __half *KV, int64_t ldkv, int past,
                                                               __half *O, uint8_t *__restrict__ Xq,
                                                               __half *__restrict__ sx, unsigned int *counter,
                                                               const RopeFreq freq)
{
    __shared__ DecodeAttnLds lds;
    __shared__ int last_flag;
    decode_attention_head<false>(lds, blockIdx.x, QKV, pos[0], H, d, base, KV, ldkv, past, O, nullptr, freq, nullptr, nullptr, 0, Xq != nullptr);
    if (!Xq) return;

    quantize_by_the_last<256>(lds.ored, lds.wred, &last_flag, O, H * d, H, Xq, sx, counter);
}

// The same for a long cache.  decode_attention_head walks the chunks one after the other with four wavefronts, one per
// SIMD, and waits for its own instructions (2.6 us per chunk of 192 keys; with the rows of three chunks in flight no less).
// Its arithmetic leaves more freedom than that: every score is a sum of its own, every column of every key group a chain
// of its own, and the chunks' running maxima follow from the scores.  Eight wavefronts work out all scores (32 keys at
// a time, the sums over lanes for eight of them together), then maxima, probabilities and group sums of all chunks side by side, then
// the output, two key groups per wavefront and four columns per lane.  The same operations in the same order per value: the same bits.
// SHARES: workgroups of a head.  Each works out all scores and takes a share of the value columns, so they need not meet; the first
// one appends to the cache.
// What bounds it: a compute unit takes in a cache line of 128 bytes every four cycles or so (65 GB/s, however many rows are on their way:
// 16 or 24 per lane instead of 8 in the scores gave nothing), and a head's rows go through one unit: 512 bytes per position, with two units
// keys and half of the values, 384 each (replayed from a graph, from 1500 to 3000 positions: 5.8 ns per position with two, 66 GB/s
// per unit; 7.5 in the form before, 68 GB/s; heads of 96, one unit and 384 bytes, 6.6, 58 GB/s).  Many heads are bound by memory: 130 heads
// of 128 16.5 ns, 4 TB/s.
// Measured with the quantizer folded in (32 heads of 128, us; one workgroup per head; the form before, which also summed key by key and
// fenced a whole L2 before it arrived): 400 positions 9.5 (10.6; 13.9), 800 11.4 (13.1; 16.5), 1500 13.5 (16.5; 20.7), 3000 24.6 (28.8; 32.3);
// 64, in the kernel above, 7.5 (8.7).  As a launch of its own the quantizer takes as long or a little longer (64 positions 7.8 in all, folded in
// 8.0; 400 9.9 and 10.0; 800 13.1 and 12.8; 3000 25.0 and 24.7; from a graph).  Without the quantizer the kernel above took 7.5 at 192 positions, 15.9 at 800: this one from two chunks on.
// Two shares where a share of a value row still is whole lines and the heads leave the units for it.
// What a unit has on its way is limited too (64 KB or so), so that from memory its rate is that over a microsecond's latency.  The units that
// have no head are near the same memory: two more workgroups per head touch the lines ahead of the two that attend, which then find them
// in their L2.  Replayed over twelve caches in turn (from memory; without helpers in brackets), us: 32 heads of 128, 800 positions 12.1
// (12.4), 1500 14.6 (20.4), 3000 24.2 (33.2); 16 heads 1500 13.4 (15.5), 3000 21.8 (33.8); 4 heads 3000 19.1 (23.8); 32 heads of 64 1500 16.6
// (16.8), 3000 26.1 (35.2).  400 positions 10.2 (9.9): the keys asked for at once are most of them.  One, three, four and six helpers: 0 to 20 % slower
// at 32 heads (four 2 to 14 %), up to 7 % faster at 16 heads and 3000 positions.
// Scores wait in LDS, 4 bytes per position: up to kDecLongMax of them (with the rest 52 KiB).
constexpr int kDecLongMin = 2 * kDecChunk;
constexpr int kDecLongT = 512, kDecLongMax = 42 * kDecChunk, kDecLongChunks = kDecLongMax / kDecChunk;
constexpr int kDecLongKeys = 8;            // keys per lane that are summed together, and rows on their way
constexpr int kDecLongFirst = kDecLongT / 16 * kDecLongKeys;       // keys that a workgroup asks for at once, before anything else
typedef unsigned int sqap_v2u __attribute__((ext_vector_type(2)));
constexpr int kDecLongAhead = 2;           // chunks whose value rows are on their way during the output
constexpr int kDecHelpMin = 3 * kDecChunk;  // cached positions from which on a head gets helpers

// Touches the cache lines of head h that the workgroups attending behind the same L2 are about to read, in the order in which they read them:
// one word of each, dropped.  `columns` of the values from `first_column` on.  This is helper `index` of `count` >= 1.
__device__ __forceinline__ void warm_cache(const __half *KV, int64_t ldkv, int past, int h, int H, int d, int first_column, int columns, int index, int count)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const char *key = reinterpret_cast<const char *>(KV + (int64_t)h * d), *value = reinterpret_cast<const char *>(KV + (int64_t)(H + h) * d + first_column);
    auto touch = [&](const char *base, int bytes, int first_row) {
        const int lines = (bytes + 127) >> 7, n = past * lines;
        for (int i = first_row * lines + (wave * count + index) * 64 + lane; i < n; i += count * kDecLongT) {
            const int row = i / lines, line = i - row * lines;
            const unsigned word = *reinterpret_cast<const unsigned *>(base + (int64_t)row * ldkv * 2 + min(line * 128, bytes - 4));
            asm volatile("" ::"v"(word));
        }
    };
    touch(key, d * 2, kDecLongFirst);
    touch(value, columns * 2, 0);
}

template <int SHARES>
__global__ __launch_bounds__(kDecLongT) void decode_attention_long_kernel(const __half *__restrict__ QKV,
                                                                          const int32_t *__restrict__ pos, int H, int d,
                                                                          double base, __half *KV, int64_t ldkv, int past,
                                                                          __half *O, uint8_t *__restrict__ Xq,
                                                                          __half *__restrict__ sx, unsigned int *counter,
                                                                          const RopeFreq freq)
{
    extern __shared__ __attribute__((aligned(16))) float sc[];        // scores, then probabilities; whole chunks
    __shared__ __attribute__((aligned(16))) float qf[kDecMaxD];
    __shared__ __attribute__((aligned(16))) __half knew[kDecMaxD], vnew[kDecMaxD];
    __shared__ __attribute__((aligned(16))) float ored[kDecRedFloats];
    __shared__ float cmax[kDecLongChunks], mrun[kDecLongChunks], resc[kDecLongChunks], psg[kDecLongChunks * 16], lw[4], wave_max[kDecLongT / 64];
    __shared__ int last_flag;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, h = blockIdx.x, share = SHARES == 1 ? 0 : blockIdx.y;
    if ((int)blockIdx.y >= SHARES) {                     // (helpers: launch_decode_attention)
        const int helpers = gridDim.y - SHARES, index = blockIdx.y - SHARES;
        if (H % 8 == 0) warm_cache(KV, ldkv, past, h, H, d, 0, d, index, helpers);
        else warm_cache(KV, ldkv, past, h, H, d, (index % SHARES) * (d / SHARES), d / SHARES, index / SHARES, (helpers - index % SHARES + SHARES - 1) / SHARES);
        return;
    }
    const int half_d = d >> 1, width = H * d, Sk = past + 1, n_chunks = (Sk + kDecChunk - 1) / kDecChunk;
    const __half *q = QKV + (int64_t)h * d, *k = q + width, *v = k + width;
    __half fresh[6] = {};
    if (t < half_d) {
        fresh[0] = q[t];
        fresh[1] = q[t + half_d];
        fresh[2] = k[t];
        fresh[3] = k[t + half_d];
        fresh[4] = v[t];
        fresh[5] = v[t + half_d];
    }
    const int kg = t >> 4, c = t & 15;
    const bool col_ok = c * 8 < d;
    // a uniform base and a 32-bit lane offset per load; past the last cached row that row again (its score is not used)
    constexpr int KSTEP = kDecLongT / 16;
    const uint32_t pitch = (uint32_t)ldkv * 2u, k_limit = (uint32_t)(past - 1) * pitch + (col_ok ? c * 16 : 0);
    const char *kbase = reinterpret_cast<const char *>(KV + (int64_t)h * d);
    uint32_t k_at = (uint32_t)kg * pitch + (col_ok ? c * 16 : 0);
    auto next_key_row = [&] {
        const sqap_v4u raw = *reinterpret_cast<const sqap_v4u *>(kbase + min(k_at, k_limit));
        k_at += KSTEP * pitch;
        return raw;
    };
    sqap_v4u kraw[kDecLongKeys];
#pragma unroll
    for (int u = 0; u < kDecLongKeys; ++u) kraw[u] = next_key_row();

    // rotation of this head's query and key; the value is copied (as in decode_attention_head)
    if (t < half_d) {
        double sn, cs;
        sincos(rope_angle(freq, pos[0], t, d, base), &sn, &cs);
        __half *krow = KV + (int64_t)past * ldkv + (int64_t)h * d, *vrow = krow + width;
        double lo = (double)__half2float(fresh[0]), hi = (double)__half2float(fresh[1]);
        qf[t] = __half2float(__float2half_rn((float)(lo * cs - hi * sn)));
        qf[t + half_d] = __half2float(__float2half_rn((float)(hi * cs + lo * sn)));
        lo = (double)__half2float(fresh[2]);
        hi = (double)__half2float(fresh[3]);
        const __half k0 = __float2half_rn((float)(lo * cs - hi * sn)), k1 = __float2half_rn((float)(hi * cs + lo * sn));
        knew[t] = k0;
        knew[t + half_d] = k1;
        vnew[t] = fresh[4];
        vnew[t + half_d] = fresh[5];
        if (share == 0) {
            global_store_half(krow + t, k0);
            global_store_half(krow + t + half_d, k1);
            global_store_half(vrow + t, fresh[4]);
            global_store_half(vrow + t + half_d, fresh[5]);
        }
    }
    lds_barrier();

    // scores
    float q8[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) q8[e] = col_ok ? qf[c * 8 + e] : 0.f;
    const float inv_sqrt_d = 1.0f / sqrtf((float)d);
    // where a key's score goes: the twelve keys of a chunk that a key group has lie side by side
    auto place_of = [](int key) {
        const int chunk = key / kDecChunk, r = key - chunk * kDecChunk;
        return chunk * kDecChunk + (r & 15) * kDecKeys + (r >> 4);
    };
    auto dot = [&](const uint4 raw) {
        float kf[8];
        unpack_halves(raw, kf);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s = fmaf(q8[e], kf[e], s);
        return col_ok ? s : 0.f;                          // (a lane past the head's columns read some other ones)
    };
    auto score = [&](const uint4 raw) {
        float s = dot(raw);
        s += dpp_move_f<kDppXor1>(s);
        s += dpp_move_f<kDppXor2>(s);
        s += dpp_move_f<kDppHalfMirror>(s);
        s += dpp_move_f<kDppMirror>(s);
        return s * inv_sqrt_d;
    };
    // Eight keys at a time: at each of the first three steps of the sums over 16 lanes a lane goes on with half of the keys, so that
    // lane c ends with the sum of key c % 8: 26 instructions for eight sums instead of 40, one product and one store instead of
    // eight.  The pairs added are those of score(), so are the bits.
    const bool odd1 = c & 1, odd2 = c & 2, odd4 = c & 4;
    auto xor4 = [](float v) {                             // lane c ^ 4's
        const int w = (int)__float_as_uint(v);
        const int up = __builtin_amdgcn_update_dpp(0, w, 0x104, 0xf, 0x5, false);         // row_shl:4 into lanes 0-3 and 8-11
        return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(up, w, 0x114, 0xf, 0xa, false));      // row_shr:4 into the others
    };
    for (int k0 = 0; k0 < past; k0 += KSTEP * kDecLongKeys) {
        float s[kDecLongKeys];
#pragma unroll
        for (int u = 0; u < kDecLongKeys; ++u) {
            s[u] = dot(make_uint4(kraw[u].x, kraw[u].y, kraw[u].z, kraw[u].w));
            kraw[u] = next_key_row();
        }
#pragma unroll
        for (int u = 0; u < 8; u += 2) s[u] = (odd1 ? s[u + 1] : s[u]) + dpp_move_f<kDppXor1>(odd1 ? s[u] : s[u + 1]);
#pragma unroll
        for (int u = 0; u < 8; u += 4) s[u] = (odd2 ? s[u + 2] : s[u]) + dpp_move_f<kDppXor2>(odd2 ? s[u] : s[u + 2]);
        s[0] = (odd4 ? s[4] : s[0]) + xor4(odd4 ? s[0] : s[4]);
        s[0] += dpp_move_f<0x128>(s[0]);                  // row_ror:8
        const int key = k0 + (c & 7) * KSTEP + kg;
        if (c < 8 && key < past) sc[place_of(key)] = s[0] * inv_sqrt_d;
    }
    const float s_new = score(lds_load16(knew + (col_ok ? c * 8 : 0)));
    // the first value rows, on their way during the softmax (a wavefront: two key groups, C columns per lane)
    constexpr int C = 4 / SHARES;
    typedef typename std::conditional<SHARES == 1, sqap_v2u, unsigned>::type piece_t;
    const int vg = 2 * wave + (lane >> 5), vc = share * (kDecMaxD / SHARES) + (lane & 31) * C;
    const bool v_ok = vc < d;
    const char *vbase = reinterpret_cast<const char *>(KV + width + (int64_t)h * d);
    const uint32_t v_col = v_ok ? vc * 2 : 0, v_first = (uint32_t)vg * pitch + v_col;
    // a chunk's value rows: a uniform base, lane offsets that stop at the last cached row
    auto load_values = [&](piece_t (&rows)[kDecKeys], int i) {
        const int first = min(min(i, n_chunks - 1) * kDecChunk, past - 1);
        const char *from = vbase + (int64_t)first * pitch;
        const uint32_t limit = (uint32_t)(past - 1 - first) * pitch + v_col;
#pragma unroll
        for (int j = 0; j < kDecKeys; ++j) rows[j] = *reinterpret_cast<const piece_t *>(from + min(v_first + (uint32_t)j * 16u * pitch, limit));
    };
    piece_t vraw[kDecLongAhead][kDecKeys];
#pragma unroll
    for (int a = 0; a < kDecLongAhead; ++a) load_values(vraw[a], a);
    lds_barrier();
    for (int key = past + t; key < n_chunks * kDecChunk; key += kDecLongT) sc[place_of(key)] = key == past ? s_new : -INFINITY;     // (t = 0: the new token)
    lds_barrier();

    // chunk maxima, running maxima, rescaling factors
    for (int i = wave; i < n_chunks; i += kDecLongT / 64) {
        float m = fmaxf(fmaxf(sc[i * kDecChunk + lane], sc[i * kDecChunk + 64 + lane]), sc[i * kDecChunk + 128 + lane]);
        for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
        if (lane == 0) cmax[i] = m;
    }
    lds_barrier();
    if (t < n_chunks) {
        float before = -INFINITY, m = -INFINITY;
        for (int i = 0; i <= t; ++i) {
            before = m;
            m = fmaxf(m, cmax[i]);
        }
        mrun[t] = m;
        resc[t] = expf(before - m);
    }
    lds_barrier();
    for (int key = t; key < n_chunks * kDecChunk; key += kDecLongT) {
        const float s = sc[key];
        sc[key] = s == -INFINITY ? 0.f : expf(s - mrun[key / kDecChunk]);
    }
    lds_barrier();
    for (int i = t; i < n_chunks * 16; i += kDecLongT) {
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < kDecKeys; ++j) sum += sc[i * kDecKeys + j];
        psg[i] = sum;
    }
    lds_barrier();

    if (wave == kDecLongT / 64 - 1 && lane < 4) {         // the running sums of the four sets of key groups
        float l = 0.f;
        for (int i = 0; i < n_chunks; ++i) {
            const float *p = psg + i * 16 + lane * 4;
            l = l * resc[i] + ((p[0] + p[1]) + (p[2] + p[3]));
        }
        lw[lane] = l;
    }
    float o[C] = {};
    auto value_chunk = [&](piece_t (&rows)[kDecKeys], int i, auto last_c) {
        constexpr bool LAST = decltype(last_c)::value;
        const float f = resc[i];
        float p[kDecKeys];
#pragma unroll
        for (int j = 0; j < kDecKeys; j += 4) {
            const float4 four = *reinterpret_cast<const float4 *>(sc + (i * 16 + vg) * kDecKeys + j);
            p[j] = four.x;
            p[j + 1] = four.y;
            p[j + 2] = four.z;
            p[j + 3] = four.w;
        }
#pragma unroll
        for (int e = 0; e < C; ++e) o[e] *= f;
#pragma unroll
        for (int j = 0; j < kDecKeys; ++j) {
            const int key = i * kDecChunk + 16 * j + vg;
            union { piece_t v; __half2 h2[C / 2]; } raw;
            raw.v = rows[j];
            if (LAST && key >= past)                      // the new token's row, and zeros past it
                raw.v = key == past && v_ok ? *reinterpret_cast<const piece_t *>(vnew + vc) : piece_t{};
#pragma unroll
            for (int e = 0; e < C; e += 2) {
                const float2 v = __half22float2(raw.h2[e / 2]);
                o[e] = fmaf(p[j], v.x, o[e]);
                o[e + 1] = fmaf(p[j], v.y, o[e + 1]);
            }
        }
        if (!LAST) load_values(rows, i + kDecLongAhead);
    };
    for (int i0 = 0; i0 < n_chunks; i0 += kDecLongAhead) {
#pragma unroll
        for (int a = 0; a < kDecLongAhead; ++a) {
            if (i0 + a < n_chunks - 1) value_chunk(vraw[a], i0 + a, std::false_type{});
            else if (i0 + a == n_chunks - 1) value_chunk(vraw[a], i0 + a, std::true_type{});
        }
    }
    if (v_ok) {
#pragma unroll
        for (int e = 0; e < C; ++e) ored[vg * kDecMaxD + vc + e] = o[e];
    }
    lds_barrier();
    float acc = 0.f;
    const int first = share * (kDecMaxD / SHARES), columns = min(d, kDecMaxD / SHARES);
    if (t < columns) {
#pragma unroll
        for (int g = 0; g < 16; ++g) acc += ored[g * kDecMaxD + first + t];
    }
    store_head_output(O + (int64_t)h * d + first, columns, acc * (1.0f / ((lw[0] + lw[1]) + (lw[2] + lw[3]))), Xq != nullptr);
    if (Xq) quantize_by_the_last<kDecLongT>(ored, wave_max, &last_flag, O, width, H * SHARES, Xq, sx, counter);
}

sqap_status launch_decode_attention(const __half *QKV, const int32_t *pos, int H, int d, double base, __half *KV,
                                    int64_t ldkv, int past, __half *O, uint8_t *Xq, __half *sx,
                                    unsigned int *counter, hipStream_t st)
{
    if (past >= kDecLongMin && past < kDecLongMax && (int64_t)(past + 1024) * ldkv * 2 < (int64_t)1 << 31) {
        const size_t lds = (size_t)(past / kDecChunk + 1) * kDecChunk * sizeof(float);
        const auto launch = [&](auto kernel, int shares) {
            hipLaunchKernelGGL(kernel, dim3(H, shares), dim3(kDecLongT), lds, st, QKV, pos, H, d, base, KV, ldkv, past, O, Xq, sx, counter,
                               rope_frequencies(d, base));
        };
        // (Where the output or the cache row lies over the token's own q|k|v: one workgroup reads all of a head's columns before it
        // writes any, of two one may still have to.)
        const auto begin = [](const __half *p) { return reinterpret_cast<uintptr_t>(p); };
        const int64_t width = (int64_t)H * d;
        const __half *row = KV + (int64_t)past * ldkv;
        const bool in_place = (begin(O) < begin(QKV + 3 * width) && begin(QKV) < begin(O + width)) ||
                              (begin(row) < begin(QKV + 3 * width) && begin(QKV) < begin(row + 2 * width));
        const int cus = device_cu_count(), shares = d == kDecMaxD && 2 * H <= cus && !in_place ? 2 : 1;
        // Helpers behind the same L2 as the workgroups that attend (workgroup i of a launch runs on XCD i % 8; were it otherwise, they would
        // only be of no use): two where all of a head's workgroups are behind one, two for each share otherwise.  Fewer positions are
        // there as fast without.
        const int wanted = H % 8 == 0 ? 2 : 2 * shares;
        const int helpers = H * shares % 8 == 0 && past >= kDecHelpMin ? std::max(0, std::min(wanted, cus / H - shares)) : 0;
        if (shares == 2) launch(decode_attention_long_kernel<2>, 2 + helpers);
        else launch(decode_attention_long_kernel<1>, 1 + helpers);
    } else {
        hipLaunchKernelGGL(decode_attention_kernel, dim3(H), dim3(256), 0, st, QKV, pos, H, d, base, KV, ldkv, past, O, Xq,
                           sx, counter, rope_frequencies(d, base));
    }
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// x <- half(float(x) + float(delta)), rows of K halves with pitches; 8 elements per thread
__global__ __launch_bounds__(256) void residual_add_kernel(__half *__restrict__ X, int64_t ldx,
                                                           const __half *__restrict__ Dl, int64_t ldd, int M, int K)
{
    const int groups = K >> 3;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)M * groups) return;
    const int g = (int)(idx % groups);
    const int64_t r = idx / groups;
    uint4 *xp = reinterpret_cast<uint4 *>(X + r * ldx) + g;
    uint4 a = *xp;
    const uint4 b = reinterpret_cast<const uint4 *>(Dl + r * ldd)[g];
    __half2 *a2 = reinterpret_cast<__half2 *>(&a);
    const __half2 *b2 = reinterpret_cast<const __half2 *>(&b);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const float2 x = __half22float2(a2[p]), y = __half22float2(b2[p]);
        float s0 = x.x + y.x, s1 = x.y + y.y;
        asm volatile("" : "+v"(s0), "+v"(s1));       // binary32 sums first, then one conversion each
        a2[p] = __floats2half2_rn(s0, s1);
    }
    *xp = a;
}

sqap_status launch_residual_add(__half *X, int64_t ldx, const __half *Dl, int64_t ldd, int M, int K, hipStream_t st)
{
    const int64_t total = (int64_t)M * (K >> 3);
    if (total == 0) return SQAP_OK;
    hipLaunchKernelGGL(residual_add_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, X, ldx, Dl, ldd, M, K);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

}  // namespace sqap
