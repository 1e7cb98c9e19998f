// W4A4 linear for up to 16 token rows: every workgroup owns complete outputs and its wavefronts are one stream of weights.
//
// With so few rows the weights are all there is to move, each byte of them once, and what a launch costs beyond that is its
// start-up: the first loads, and every point at which loads stop being in flight.  So a wavefront has a share of K (an eighth,
// where K is long enough) and walks the 16-channel groups of its workgroup one after the other as ONE sequence of 1 KiB
// pieces (16 channels x 128 codes: the operand order of v_mfma_i32_16x16x64_i8 as packed), a ring of R of them on its way all the
// time; nothing stops at the end of a group: the wavefront adds its 16 x 16 partial sums into LDS (integers, any order, the
// same result) and goes on.  The token rows sit in LDS in operand order, staged once by all wavefronts while the
// first weights are on their way.  Two barriers in all.
// What bounds it: short launches their start-up (arguments, token rows, first weights: 2.5 us at 512 x 512), long ones the weights'
// arrival (32000 x 4096 at 13.5 us: 4.9 TB/s).  Every instruction in front of the first loads counts: with divisions at run time
// and conditional address arithmetic per load 512 x 512 took 3.5 us and 32000 x 4096 14.6; with the arguments of several weights
// read by index three weights of 4096 x 4096 took 8.6 us, 7.6 with selects.  Weights read past the caches: 4 to 15 % slower.
// Measured against the kernel of gemm_rows.hip, which these shapes had before (M = 4, us, that kernel in brackets): 512 x 512 2.5 (3.0),
// 1024 x 2816 3.0 (3.7), 4096 x 4096 3.9 (5.2), 12288 x 4096 7.2 (8.5), 22016 x 4096 10.4 (14.5), K = 11008 6.9 (7.6), 32000 x 4096 13.7
// (18.3), three of 4096 x 4096 7.6 (9.1), two of 11008 x 4096 10.9 (15.7); 16 rows 0 to 9 % above these but for K = 11008
// (7.8; 7.7).  Against the streaming kernel, which keeps launches of many problems: 100000 x 4096 at M = 1 / 8 33.9 / 34.6 (47 / 48).
#include <algorithm>

#include "common.h"

namespace sqap {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kFewWaves = 8, kFewThreads = 64 * kFewWaves;
constexpr int kFewMaxRows = 16, kFewMaxGroups = 32;      // token rows; 16-channel groups of a workgroup
constexpr int kFewMaxLds = 160 * 1024;

struct FewParams {
    const uint8_t *Xq;     // [M, K/2] canonical
    const __half *sx;      // [M]
    unsigned long long *error_word;        // of the caller's workspace, nullable: cleared (no wait can fail here)
    int M, chunks, c16;    // c16: 16-channel groups in all
    uint32_t wg_inv;       // ceil(2^32 / workgroups)
    uint32_t n4_inv[2];    // 2^20 / (4 n) + 1 for the smaller and the larger number n of groups of a workgroup
    uint32_t seg_inv;      // 2^16 / segs + 1
    uint32_t per_xcd_pitch;        // workgroups of an XCD; << 16: bytes from one chunk of 32 codes to the next in LDS, 16 per row and 16 more (banks)
    // 64-chunk segments per row; << 8: log2 of the shares K is cut into (the other wavefronts take other groups); << 16: rows staged
    // - 1; << 24: weights the input is multiplied with.  (Fields of less than a word would be vector loads.)
    uint32_t segs_klog_mask_count;
    RowsWeight w[kRowsMaxWeights];
};

__device__ __forceinline__ void few_widen(const v4i p, v4i &lo, v4i &hi)
{
    const v4i mask = {(int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0};
    lo = (p << 4) & mask;
    hi = p & mask;
}

template <int R, bool MULTI>
__global__ __launch_bounds__(kFewThreads, 1) void gemm_few_kernel(const FewParams p)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    // the arguments are asked for together: behind the first branch they would be a second trip to memory
    asm volatile("" ::"s"(p.Xq), "s"(p.sx), "s"(p.error_word), "s"(p.M), "s"(p.w[0].Wd), "s"(p.w[0].sw), "s"(p.w[0].N));
    if (MULTI)
        asm volatile("" ::"s"(p.w[1].Wd), "s"(p.w[1].sw), "s"(p.w[1].g_begin), "s"(p.w[2].Wd), "s"(p.w[2].sw), "s"(p.w[2].g_begin),
                     "s"(p.w[3].Wd), "s"(p.w[3].sw), "s"(p.w[3].g_begin));
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    if (blockIdx.x == 0 && t == 0 && p.error_word) *p.error_word = 0ull;
    const int per_xcd = p.per_xcd_pitch & 0xffff, pitch = p.per_xcd_pitch >> 16;
    const int segs = p.segs_klog_mask_count & 255, k_log = (p.segs_klog_mask_count >> 8) & 255;
    const int row_mask = (p.segs_klog_mask_count >> 16) & 255, count = p.segs_klog_mask_count >> 24;
    const uint32_t i_wg = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const int g_begin = (int)__umulhi((uint32_t)p.c16 * i_wg, p.wg_inv), g_end = (int)__umulhi((uint32_t)p.c16 * (i_wg + 1), p.wg_inv);
    const int n = g_end - g_begin;
    if (n == 0) return;
    const int chunks = p.chunks, blocks = (chunks + 3) >> 2, ks = 1 << k_log, gs = kFewWaves >> k_log;
    const int kq = wave & (ks - 1), gsh = wave >> k_log;
    const int b0 = (blocks * kq) >> k_log, nbw = ((blocks * (kq + 1)) >> k_log) - b0;
    const int T = gsh < n ? ((n - gsh + gs - 1) >> (3 - k_log)) * nbw : 0;       // pieces of this wavefront

    // the weight that channel group g belongs to: selects, not an indexed read of the arguments (a trip to memory each)
    auto weight_of = [&](int g) {
        RowsWeight w = p.w[0];
        if (MULTI) {
#pragma unroll
            for (int i = 1; i < kRowsMaxWeights; ++i)
                if (i < count && g >= p.w[i].g_begin) w = p.w[i];
        }
        return w;
    };
    auto group_ptr = [&](int g) {
        const uint8_t *wd = p.w[0].Wd;
        if (MULTI) {
            int first = 0;
#pragma unroll
            for (int i = 1; i < kRowsMaxWeights; ++i)
                if (i < count && g >= p.w[i].g_begin) {
                    wd = p.w[i].Wd;
                    first = p.w[i].g_begin;
                }
            g -= first;
        }
        return wd + (size_t)(g >> 1) * (uint32_t)(chunks * 512) + ((g & 1) * 256 + b0 * 2048);
    };

    // ---- token rows: a wavefront load is 64 chunks of one row
    constexpr int XL = 12;
    const int pairs = p.M * segs;
    v4i xr[XL];
    auto load_x = [&](int j) {
        const int pr = min(wave + j * kFewWaves, pairs - 1), row = (pr * p.seg_inv) >> 16, c = (pr - row * segs) * 64 + lane;
        return *reinterpret_cast<const v4i *>(p.Xq + ((size_t)row * chunks + min(c, chunks - 1)) * 16);
    };
    auto store_x = [&](int j, const v4i v) {
        const int pr = wave + j * kFewWaves, row = (pr * p.seg_inv) >> 16, c = (pr - row * segs) * 64 + lane;
        if (pr < pairs && c < blocks * 4)
            *reinterpret_cast<v4i *>(smem + c * pitch + row * 16) = c < chunks ? v : v4i{0, 0, 0, 0};
    };
    const int per_wave = (pairs + kFewWaves - 1) / kFewWaves;
    xr[0] = load_x(0);
    if (per_wave > 1) xr[1] = load_x(1);
    if (per_wave > 2) {
#pragma unroll
        for (int j = 2; j < 4; ++j) xr[j] = load_x(j);
    }
    if (per_wave > 4) {
#pragma unroll
        for (int j = 4; j < 8; ++j) xr[j] = load_x(j);
    }
    if (per_wave > 8) {
#pragma unroll
        for (int j = 8; j < XL; ++j) xr[j] = load_x(j);
    }

    // ---- the weight stream
    const uint32_t woff = (uint32_t)(lane >> 4) * 512 + (lane & 15) * 16;
    int lblk = nbw, lg = min(g_begin + gsh, g_end - 1);
    const uint8_t *lptr = group_ptr(lg);
    v4i ring[R];
    auto next_piece = [&] {                                      // (past the last piece: the last group's again)
        const v4i v = *reinterpret_cast<const v4i *>(lptr + woff);
        lptr += 2048;
        if (__builtin_expect(--lblk == 0, 0)) {
            lblk = nbw;
            if (lg + gs < g_end) lg += gs;
            lptr = group_ptr(lg);
        }
        return v;
    };
#pragma unroll
    for (int r = 0; r < R; ++r) ring[r] = next_piece();

    // scales of the outputs this thread will store
    const int M = p.M, n4 = 4 * n, total = n4 * M;
    const uint32_t inv_n4 = p.n4_inv[n * 8 * per_xcd > p.c16];      // u / n4 = (u * inv) >> 20 for u * n4 < 2^20
    struct Out { int token, g, col; };
    auto out_of = [&](int u) {
        Out o;
        o.token = (int)(((uint32_t)u * inv_n4) >> 20);
        const int c = u - o.token * n4;
        o.g = c >> 2;
        const RowsWeight w = weight_of(g_begin + o.g);
        o.col = (g_begin + o.g - w.g_begin) * 16 + (c & 3) * 4;
        return o;
    };
    auto scales_of = [&](int u, __half &sxv, uint2 &swv) {
        const Out o = out_of(min(u, total - 1));
        sxv = p.sx[o.token];
        swv = *reinterpret_cast<const uint2 *>(weight_of(g_begin + o.g).sw + o.col);      // zero padded past N
    };
    __half sx_own;
    uint2 sw_own;
    scales_of(t, sx_own, sw_own);

    // ---- LDS: sums to zero, tokens in
    int *sums = reinterpret_cast<int *>(smem + blocks * 4 * pitch);
    for (int i = t; i < n * 64; i += kFewThreads) reinterpret_cast<v4i *>(sums)[i] = v4i{0, 0, 0, 0};
    store_x(0, xr[0]);
    if (per_wave > 1) store_x(1, xr[1]);
    if (per_wave > 2) {
#pragma unroll
        for (int j = 2; j < 4; ++j) store_x(j, xr[j]);
    }
    if (per_wave > 4) {
#pragma unroll
        for (int j = 4; j < 8; ++j) store_x(j, xr[j]);
    }
    if (per_wave > 8) {
#pragma unroll
        for (int j = 8; j < XL; ++j) store_x(j, xr[j]);
        for (int j = XL; j < per_wave; ++j) store_x(j, load_x(j));
    }
    lds_barrier();

    // ---- products
    if (T > 0) {
        const uint8_t *const x_first = smem + (b0 * 4 + (lane >> 4)) * pitch + (lane & 15 & row_mask) * 16, *x_at = x_first;
        int left = nbw, ug = gsh;
        v4i acc = {0, 0, 0, 0};
        auto use = [&](const v4i w) {
            v4i wl, wh, xl, xh;
            const v4i xf = *reinterpret_cast<const v4i *>(x_at);
            x_at += 4 * pitch;
            few_widen(w, wl, wh);
            few_widen(xf, xl, xh);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(wl, xl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh, xh, acc, 0, 0, 0);
            if (__builtin_expect(--left == 0, 0)) {              // the group's share is complete
                left = nbw;
                x_at = x_first;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    __hip_atomic_fetch_add(sums + (ug * 4 + e) * 64 + lane, acc[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                acc = v4i{0, 0, 0, 0};
                ug += gs;
            }
        };
        int i = 0;
        for (; i + R < T; i += R) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const v4i w = ring[r];
                ring[r] = next_piece();
                use(w);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (i + r < T) use(ring[r]);
    }
    lds_barrier();

    // ---- outputs: four channels of one token per thread
    for (int u = t; u < total; u += kFewThreads) {
        if (u != t) scales_of(u, sx_own, sw_own);
        const Out o = out_of(u);
        const RowsWeight w = weight_of(g_begin + o.g);
        const int *s = sums + o.g * 256 + ((o.col >> 2) & 3) * 16 + o.token;
        const int v[4] = {s[0], s[64], s[128], s[192]};
        if (o.col >= w.N) continue;
        // two binary32 products, then one rounding to half; the sums are 256 times the integer
        const float sxf = __half2float(sx_own) * 0.00390625f;
        const __half2 *sw2 = reinterpret_cast<const __half2 *>(&sw_own);
        const float2 s01 = __half22float2(sw2[0]), s23 = __half22float2(sw2[1]);
        float y0 = ((float)v[0] * sxf) * s01.x, y1 = ((float)v[1] * sxf) * s01.y;
        float y2 = ((float)v[2] * sxf) * s23.x, y3 = ((float)v[3] * sxf) * s23.y;
        asm volatile("" : "+v"(y0), "+v"(y1), "+v"(y2), "+v"(y3));
        union { __half2 h[2]; uint2 u; __half e[4]; } pk;
        pk.h[0] = __floats2half2_rn(y0, y1);
        pk.h[1] = __floats2half2_rn(y2, y3);
        __half *dst = w.Y + (size_t)o.token * w.ldy + o.col;
        if (o.col + 4 <= w.N) {
            *reinterpret_cast<halves4_any *>(dst) = halves4_any{pk.u.x, pk.u.y};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (o.col + e < w.N) dst[e] = pk.e[e];
        }
        if (w.acc_out) {
            int32_t *ad = w.acc_out + (size_t)o.token * w.N + o.col;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (o.col + e < w.N) ad[e] = v[e] >> 8;
        }
    }
}

static int few_k_log(int blocks) { return blocks >= 8 ? 3 : blocks >= 4 ? 2 : blocks >= 2 ? 1 : 0; }

int few_k_shares(int K) { return 1 << few_k_log((K / 32 + 3) / 4); }

// R: pieces in flight per wavefront, no more than it has, so that none is asked for twice: four.  A compute unit takes in 1 KiB per 15 ns, so the
// 32 KiB of eight wavefronts with four pieces each are half a microsecond of arrivals, and every load in front of the first product is start-up.
// Measured with up to sixteen in flight in brackets (4 rows, 8 of the last; us, replayed): weights in the caches 12288 x 4096 4.9 (5.1), 22016 x
// 4096 9.3 (10.0), 4096 x 11008 4.9 (5.1), 32000 x 4096 12.1 (13.5); copies of them in turn, from memory 12288 x 4096 6.9 (7.8), 22016 x 4096 10.6
// (10.9), 4096 x 11008 7.2 (7.9), 32000 x 4096 13.7 (14.4).  Two, three, five, six and eight: no shape more than 2 % faster than with four but
// 4096 x 4096 and 4096 x 11008 from memory (two 4.1 against 4.3; six 6.9 against 7.2), others up to 15 % slower.
// Rows staged: 8 or 16, the lanes of a token that is not there read another's.
static bool few_plan(int M, int c16, int K, int cus, FewParams *p, int *pieces, int *lds)
{
    if (K % 32 != 0 || c16 < 1 || M < 1 || M > kFewMaxRows) return false;
    const int per_xcd = std::max(1, cus / 8), W = 8 * per_xcd, n = (c16 + W - 1) / W;
    const int blocks = (K / 32 + 3) / 4, rows = M <= 8 ? 8 : 16;
    p->chunks = K / 32;
    p->c16 = c16;
    const int k_log = few_k_log(blocks), segs = (blocks * 4 + 63) / 64, pitch = 16 * rows + 16;
    const int ks = 1 << k_log, gs = kFewWaves / ks;
    p->per_xcd_pitch = (uint32_t)per_xcd | (uint32_t)pitch << 16;
    p->segs_klog_mask_count = (uint32_t)segs | (uint32_t)k_log << 8 | (uint32_t)(rows - 1) << 16;
    p->seg_inv = 65536u / segs + 1;
    p->wg_inv = (uint32_t)((0xffffffffull + W) / W);
    p->n4_inv[0] = (1u << 20) / (4 * std::max(1, c16 / W)) + 1;
    p->n4_inv[1] = (1u << 20) / (4 * (c16 / W + 1)) + 1;
    *pieces = ((n + gs - 1) / gs) * ((blocks + ks - 1) / ks);
    *lds = blocks * 4 * pitch + n * 1024;
    return n <= kFewMaxGroups && *lds <= kFewMaxLds;
}

// (a device's compute units, of which a launch uses multiples of eight)
static int few_cus(int cus) { return cus > 256 ? 256 : cus < 8 ? 8 : cus; }

bool few_kernel_applies(int M, int channel_groups, int K, int compute_units)
{
    FewParams p = {};
    int pieces, lds;
    return few_plan(M, channel_groups, K, few_cus(compute_units), &p, &pieces, &lds);
}

template <int R, bool MULTI>
static sqap_status launch_few_k(const FewParams &p, int lds, hipStream_t st)
{
    static std::atomic<bool> configured[kMaxDeviceSlots];
    const int dslot = device_slot();
    if (!configured[dslot].load(std::memory_order_acquire)) {
        SQAP_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_few_kernel<R, MULTI>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kFewMaxLds));
        configured[dslot].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((gemm_few_kernel<R, MULTI>), dim3(8 * (p.per_xcd_pitch & 0xffff)), dim3(kFewThreads), lds, st, p);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

template <bool MULTI>
static sqap_status launch_few_r(const FewParams &p, int pieces, int lds, hipStream_t st)
{
    if (pieces <= 2) return launch_few_k<2, MULTI>(p, lds, st);
    return launch_few_k<4, MULTI>(p, lds, st);
}

sqap_status launch_few_linear(const uint8_t *Xq, const __half *sx, int M, int K, const RowsWeight *weights, int count,
                              unsigned long long *error_word, hipStream_t st)
{
    FewParams p = {};
    p.Xq = Xq;
    p.sx = sx;
    p.M = M;
    p.error_word = error_word;
    int groups = 0;
    for (int i = 0; i < count; ++i) {
        p.w[i] = weights[i];
        p.w[i].g_begin = groups;
        groups += (weights[i].N + 15) / 16;
    }
    int pieces, lds;
    if (!few_plan(M, groups, K, few_cus(device_cu_count()), &p, &pieces, &lds))
        return fail(SQAP_EUNSUPPORTED, "sqap_w4a4_linear: M = %d, %d channels, K = %d outside the few-rows kernel's range", M, groups * 16, K);
    p.segs_klog_mask_count |= (uint32_t)count << 24;
    return count > 1 ? launch_few_r<true>(p, pieces, lds, st) : launch_few_r<false>(p, pieces, lds, st);
}

}  // namespace sqap
