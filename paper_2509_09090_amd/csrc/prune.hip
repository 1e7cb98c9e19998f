// Token selection kernels: retention score, top-k (Eq. 1 of the paper), the
// surviving row list and the row gather.
#include "common.h"

namespace sqap {

// Monotone map from a score to an unsigned key: larger score <=> larger key,
// -0 and +0 share a key, every NaN maps to 0 (below -inf, whose key is 0x007fffff).
__device__ __forceinline__ uint32_t score_key(float s)
{
    uint32_t b = __float_as_uint(s);
    if ((b & 0x7fffffffu) > 0x7f800000u) return 0u;
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Exclusive prefix sum of one 0/1 flag per thread over a 256-thread block.
// Returns the thread's offset; *total receives the block sum.  `wave_sums`
// is 4 ints of LDS.  Contains two barriers.
__device__ __forceinline__ int block_scan_flags(bool flag, int *wave_sums, int *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long m = __ballot(flag);
    int before = __popcll(m & ((1ull << lane) - 1ull));
    __syncthreads();                       // previous users of wave_sums are done
    if (lane == 0) wave_sums[wave] = __popcll(m);
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        int c = wave_sums[w];
        if (w < wave) off += c;
        tot += c;
    }
    *total = tot;
    return off + before;
}

constexpr int kTopkWaveMax = 2048;         // tokens that one wavefront holds

// A wavefront's scores as keys, lane l holding tokens l, l + 64, ...; no key past the end.  All loads are on their way before the first is
// looked at (under a condition each they were four round trips in a row: 256 tokens, whole kernel 5.4 us against 3.6).
template <int PL>
__device__ __forceinline__ void load_keys(const float *__restrict__ s, int n, int lane, uint32_t (&key)[PL])
{
    float raw[PL];
#pragma unroll
    for (int r = 0; r < PL; ++r) raw[r] = s[min(lane + 64 * r, n - 1)];
#pragma unroll
    for (int r = 0; r < PL; ++r) key[r] = lane + 64 * r < n ? score_key(raw[r]) : 0u;
}

// A value that at least k of the wavefront's keys reach, such that k tokens remain if those above it are taken and then the first
// ones equal to it: bit by bit from the top, up to the first value that exactly k reach (usually after half of the 32 bits), else
// the k-th largest key.  Keys are compared with values above zero, which keys past the end do not reach.
template <int PL>
__device__ __forceinline__ uint32_t kth_key(const uint32_t (&key)[PL], int k)
{
    uint32_t T = 0;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t cand = T | (1u << bit);
        int reach = 0;
#pragma unroll
        for (int r = 0; r < PL; ++r) reach += __popcll(__ballot(key[r] >= cand));
        if (reach >= k) T = cand;
        if (reach == k) break;
    }
    return T;
}

// n <= 2048: one wavefront per observation, no
// barriers and no LDS traffic in the ranking.  Lane l owns tokens l, l + 64, ...: tokens
// 64 r .. 64 r + 63 sit in lane order, so "lower index first" is "lower row, then lower lane".
// Keys above kth_key's T are kept, and of the keys equal to T the first ones by index.  Outputs are compacted with ballot prefixes.
// PL = tokens per lane.  What bounds it: one trip to memory, the ballot rounds, the stores; us with the row list: 64 tokens 1.9, 3 x 256
// 3.8, 576 8.6, 4 x 1024 10.2, 2 x 1500 17.3 (loads one after the other, all 32 rounds: 4.4, 5.4, 17.4, 19.4; the last by counting ranks
// in LDS, 233).
template <int PL>
__global__ __launch_bounds__(64) void topk_wave_kernel(const float *__restrict__ scores, int n, int keep_k,
                                                       int32_t *__restrict__ idx_out, int seq_len, int vis_begin,
                                                       int32_t *__restrict__ rows_out)
{
    __shared__ uint8_t keptf[64 * PL];
    const int lane = threadIdx.x, b = blockIdx.x;
    const float *s = scores + (size_t)b * n;
    const unsigned long long below = (1ull << lane) - 1ull;
    bool valid[PL], kept[PL];
    uint32_t key[PL];
    if (keep_k > 0) {
        load_keys<PL>(s, n, lane, key);
    } else {                                                     // (there may be no scores)
#pragma unroll
        for (int r = 0; r < PL; ++r) key[r] = 0u;
    }
#pragma unroll
    for (int r = 0; r < PL; ++r) valid[r] = lane + 64 * r < n;
    const uint32_t T = kth_key<PL>(key, keep_k);
    int above = 0;
#pragma unroll
    for (int r = 0; r < PL; ++r) above += __popcll(__ballot(valid[r] && key[r] > T));
    const int need_eq = keep_k - above;
    int32_t *out = idx_out + (size_t)b * keep_k;
    int eq_seen = 0, base = 0;
#pragma unroll
    for (int r = 0; r < PL; ++r) {
        const bool eq = valid[r] && key[r] == T;
        const unsigned long long me = __ballot(eq);
        kept[r] = valid[r] && (key[r] > T || (eq && eq_seen + __popcll(me & below) < need_eq));
        eq_seen += __popcll(me);
        const unsigned long long mk = __ballot(kept[r]);
        if (kept[r]) out[base + __popcll(mk & below)] = lane + 64 * r;
        base += __popcll(mk);
        if (rows_out && valid[r]) keptf[lane + 64 * r] = kept[r];
    }
    if (rows_out) {
        // LDS operations of one wavefront complete in order: the flags written above are visible
        __builtin_amdgcn_wave_barrier();
        int32_t *rows = rows_out + (size_t)b * (seq_len - n + keep_k);
        int rbase = 0;
        for (int c0 = 0; c0 < seq_len; c0 += 64 * 4) {           // (four flags on their way at a time)
            bool keep[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int sq = c0 + 64 * u + lane, v = sq - vis_begin;
                const uint8_t flag = keptf[min(max(v, 0), max(n - 1, 0))];
                keep[u] = sq < seq_len && (v < 0 || v >= n || flag);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long mk = __ballot(keep[u]);
                if (keep[u]) rows[rbase + __popcll(mk & below)] = b * seq_len + c0 + 64 * u + lane;
                rbase += __popcll(mk);
            }
        }
    }
}

static bool launch_topk_wave(const float *scores, int batch, int n, int keep_k, int32_t *idx, int seq_len,
                             int vis_begin, int32_t *rows, hipStream_t st)
{
    if (n > kTopkWaveMax) return false;
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(batch), dim3(64), 0, st, scores, n, keep_k, idx, seq_len, vis_begin, rows);
    };
    if (n <= 64) launch(topk_wave_kernel<1>);
    else if (n <= 256) launch(topk_wave_kernel<4>);
    else if (n <= 512) launch(topk_wave_kernel<8>);
    else if (n <= 1024) launch(topk_wave_kernel<16>);
    else launch(topk_wave_kernel<32>);
    return true;
}

// Any n: radix select, 8 bits per pass from the top, finds the key T of the
// keep_k-th ranked element and how many elements equal to T are kept; a last
// pass in index order keeps key > T and the first `need_eq` with key == T.
__global__ __launch_bounds__(256) void topk_radix_kernel(const float *__restrict__ scores, int n,
                                                         int keep_k, int32_t *__restrict__ idx_out)
{
    __shared__ int hist[256];
    __shared__ int wave_sums[4];
    __shared__ int sel_digit, sel_remaining;
    const int t = threadIdx.x;
    const float *s = scores + (size_t)blockIdx.x * n;
    int32_t *out = idx_out + (size_t)blockIdx.x * keep_k;
    uint32_t prefix = 0, mask = 0;
    int remaining = keep_k;
    for (int shift = 24; shift >= 0; shift -= 8) {
        hist[t] = 0;
        __syncthreads();
        for (int i = t; i < n; i += 256) {
            uint32_t k = score_key(s[i]);
            if ((k & mask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1);
        }
        __syncthreads();
        int above = 0;
        for (int d = t + 1; d < 256; ++d) above += hist[d];
        if (above < remaining && above + hist[t] >= remaining) {
            sel_digit = t;
            sel_remaining = remaining - above;
        }
        __syncthreads();
        prefix |= (uint32_t)sel_digit << shift;
        mask |= 0xffu << shift;
        remaining = sel_remaining;
        __syncthreads();
    }
    const uint32_t T = prefix;
    const int need_eq = remaining;
    int base = 0, eq_seen = 0;
    for (int c = 0; c < n; c += 256) {
        const int i = c + t;
        uint32_t k = i < n ? score_key(s[i]) : 0u;
        bool gt = i < n && k > T, eq = i < n && k == T;
        int eq_total;
        int eq_rank = eq_seen + block_scan_flags(eq, wave_sums, &eq_total);
        bool keep = gt || (eq && eq_rank < need_eq);
        int total;
        int pos = block_scan_flags(keep, wave_sums, &total);
        if (keep) out[base + pos] = i;
        base += total;
        eq_seen += eq_total;
    }
}

sqap_status launch_prune_topk(const float *scores, int batch, int n, int keep_k, int32_t *idx,
                              hipStream_t st)
{
    if (!launch_topk_wave(scores, batch, n, keep_k, idx, 0, 0, nullptr, st))
        hipLaunchKernelGGL(topk_radix_kernel, dim3(batch), dim3(256), 0, st, scores, n, keep_k, idx);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

sqap_status launch_kept_rows(const int32_t *idx, int batch, int keep_k, int seq_len,
                             int vis_begin, int n_vis, int32_t *rows, hipStream_t st);

// top-k and the surviving rows; one launch when the scores fit a wavefront
sqap_status launch_prune_rows(const float *scores, int batch, int n, int keep_k, int seq_len, int vis_begin,
                              int32_t *idx, int32_t *rows, hipStream_t st)
{
    if (launch_topk_wave(scores, batch, n, keep_k, idx, seq_len, vis_begin, rows, st)) {
        SQAP_HIP_CHECK(hipGetLastError());
        return SQAP_OK;
    }
    sqap_status stt = launch_prune_topk(scores, batch, n, keep_k, idx, st);
    if (stt != SQAP_OK) return stt;
    return launch_kept_rows(idx, batch, keep_k, seq_len, vis_begin, n, rows, st);
}

// ---------------------------------------------------------------------------
// Full selection rule of Section 3.2: K_attn (Eq. 1) + K_ring (Eq. 2-4) + K_fps
// (Eq. 5).  Lane l owns tokens l, l + 64, ... (at most 1024 tokens, 16 per lane).  Four wavefronts per
// observation hold the same tokens: the distances to the set the sampling starts from, one member at a time,
// are shared out by lane number mod 4; then the first wavefront samples alone (a pick depends on the one before, and a
// barrier per pick would cost more than the arithmetic it shares out).  Everything after the projection is
// integer work, so the result is exact.
// A serial chain bounds it: up to 32 ballot rounds of the top-k search, then the picks, of which those at squared distances 1 and 2 (four in
// five where half of the tokens are kept) are made at once, see Words; a pick before them is three instructions per 64 tokens, a
// wavefront maximum and the decoding of the winner.  A token's state is one word, squared distance * 1024 + inverted index: the
// largest word is the next pick, a member's distance is zero, which keeps it out without further tests.  Coordinates are packed
// halves, 32 times as large (1023 * 32 fits), so that one subtraction and one dot product, which adds the inverted index, give the
// state for a new member, and a minimum does the rest.  Measured per call, 16 observations, us (every pick by itself in brackets): 16 x 16
// tokens, 128 kept 8.5 (11.7); 24 x 24, 300 kept 25.2 (46.0); 32 x 32, 512 kept 34.5 (69.5); 12 x 12, 72 kept 7.8 (9.5).
constexpr int kSelectCamera = 26;          // doubles per observation: K (9), [R|t] (12), point (3), patch w, h
constexpr uint32_t kFarAway = 1u << 30;    // above any state on a grid of <= 1024 tokens: a squared distance is below 2^20

// Eq. 2-3 in binary64, dot products summed left to right, no contraction.
__device__ __forceinline__ bool project_token(const double *c, int &tu, int &tv)
{
    const double *Km = c, *Rt = c + 9, *p = c + 21;
    double cam[3], h[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
        cam[i] = ((Rt[4 * i] * p[0] + Rt[4 * i + 1] * p[1]) + Rt[4 * i + 2] * p[2]) + Rt[4 * i + 3];
#pragma unroll
    for (int i = 0; i < 3; ++i) h[i] = (Km[3 * i] * cam[0] + Km[3 * i + 1] * cam[1]) + Km[3 * i + 2] * cam[2];
    if (!(h[2] > 0.0)) return false;
    const double fu = floor((h[0] / h[2]) / c[24]), fv = floor((h[1] / h[2]) / c[25]);
    if (!(fabs(fu) <= 1073741824.0) || !(fabs(fv) <= 1073741824.0)) return false;
    tu = (int)fu;
    tv = (int)fv;
    return true;
}

// Maximum over the 64 lanes, returned in every lane.  Row-shift steps fold each row of 16
// lanes into its lane 15, two row broadcasts fold the four rows into lane 63; lanes whose
// source does not exist take 0, the identity here.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#define SQAP_DPP_MAX(ctrl, row_mask, bank_mask)                                                      \
    {                                                                                                \
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, row_mask, bank_mask, false); \
        v = o > v ? o : v;                                                                           \
    }
    SQAP_DPP_MAX(0x111, 0xf, 0xf)    // row_shr:1
    SQAP_DPP_MAX(0x112, 0xf, 0xf)    // row_shr:2
    SQAP_DPP_MAX(0x114, 0xf, 0xe)    // row_shr:4, lanes 4-15 of a row
    SQAP_DPP_MAX(0x118, 0xf, 0xc)    // row_shr:8, lanes 8-15 of a row
    SQAP_DPP_MAX(0x142, 0xa, 0xf)    // lane 15 of rows 0 and 2 into rows 1 and 3
    SQAP_DPP_MAX(0x143, 0xc, 0xf)    // lane 31 into rows 2 and 3
#undef SQAP_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

typedef short v2s __attribute__((ext_vector_type(2)));
constexpr int kSelectWaves = 4;

// squared distance of packed (32 u, 32 v) * 1024 + the inverted index
__device__ __forceinline__ uint32_t state_of(uint32_t a, uint32_t b, int inverted)
{
    const v2s d = __builtin_bit_cast(v2s, a) - __builtin_bit_cast(v2s, b);
    return (uint32_t)__builtin_amdgcn_sdot2(d, d, inverted, false);
}

// The states after a new member at `at`.  Four dot products at a time, each in a register of its own: a result can be read three
// wait states later, and in one register they would wait for each other.
template <int PL>
__device__ __forceinline__ void add_member(uint32_t (&state)[PL], const uint32_t (&uv)[PL], const int (&inverted)[PL], uint32_t at)
{
#pragma unroll
    for (int r = 0; r < PL; r += 4) {
        uint32_t t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = state_of(uv[r + e], at, inverted[r + e]);
        asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
#pragma unroll
        for (int e = 0; e < 4; ++e) state[r + e] = min(state[r + e], t[e]);
    }
}

// The last picks at once.  At squared distance 2 a pick only touches candidates beside, above or below it (theirs becomes 1; the
// others' stays 2), and nothing new becomes a candidate: taken in order of index, the picks are the candidates that no pick of a lower
// index lies beside.  All undecided candidates without an undecided one beside them at a lower index are picks, whatever comes later; their
// neighbours are out; and again until all are decided.  Grids of up to 64 columns, as one word of 64 tokens per lane: word r in lane r.
struct Words {
    unsigned long long not_last;               // tokens that are not in the last column
    int gw;
    // tokens right of and below those of x
    __device__ __forceinline__ unsigned long long after(unsigned long long x) const
    {
        const unsigned long long r = x & not_last, up = (r >> 63) | (x >> (64 - gw));
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)up, 0x111, 0xf, 0xf, false);         // from the lane before
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(up >> 32), 0x111, 0xf, 0xf, false);
        return (r << 1) | (gw < 64 ? x << gw : 0ull) | (unsigned long long)hi << 32 | lo;
    }
    __device__ __forceinline__ unsigned long long picks(unsigned long long candidates) const
    {
        unsigned long long picked = 0;
        while (__any(candidates != 0ull)) {                                          // (each time round the lowest is decided, at least)
            const unsigned long long now = candidates & ~after(candidates);
            picked |= now;
            candidates &= ~(now | after(now));
        }
        return picked;
    }
};

// word r of 64 tokens, for lane r
template <int PL>
__device__ __forceinline__ unsigned long long to_words(const bool (&is)[PL], int lane)
{
    unsigned long long word = 0;
#pragma unroll
    for (int r = 0; r < PL; ++r) {
        const unsigned long long mk = __ballot(is[r]);
        word = lane == r ? mk : word;
    }
    return word;
}

// Keeps the first `left` of the tokens that `is` says; how many that leaves.
template <int PL>
__device__ __forceinline__ int keep_first(const bool (&is)[PL], bool (&kept)[PL], unsigned long long below, int left)
{
#pragma unroll
    for (int r = 0; r < PL; ++r) {
        const unsigned long long mk = __ballot(is[r]);
        kept[r] = kept[r] || (is[r] && (int)__popcll(mk & below) < left);
        left -= (int)__popcll(mk);
    }
    return left;
}

template <int PL>     // tokens per lane: at most 64 * PL tokens
__global__ __launch_bounds__(64 * kSelectWaves) void prune_select_kernel(const float *__restrict__ scores, int gw, int gh,
                                                          int k_attn, int keep_total,
                                                          const double *__restrict__ camera, int radius,
                                                          int32_t *__restrict__ idx_out, int cap,
                                                          int32_t *__restrict__ count_out)
{
    __shared__ uint32_t part[kSelectWaves][64 * PL];
    const int lane = threadIdx.x & 63, b = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = gw * gh;
    const float *s = scores + (size_t)b * n;
    const unsigned long long below = (1ull << lane) - 1ull;      // lanes with a lower number

    // own tokens: lane + 64 r.  Tokens 64 r .. 64 r + 63 sit in lane order, so "lower index
    // first" is "lower row first, then lower lane".
    bool valid[PL], kept[PL];
    uint32_t key[PL], uv[PL];
    load_keys<PL>(s, n, lane, key);
#pragma unroll
    for (int r = 0; r < PL; ++r) {
        const int i = lane + 64 * r;
        valid[r] = i < n;
        uv[r] = valid[r] ? ((uint32_t)(i % gw) | ((uint32_t)(i / gw) << 16)) << 5 : 0u;
    }
    int cu = 0, cv = 0;
    bool have_ring = false;
    if (camera) have_ring = project_token(camera + (size_t)b * kSelectCamera, cu, cv);

    // Eq. 1: keys above T and the first tokens equal to T
    const uint32_t T = kth_key<PL>(key, k_attn);
    int above = 0;
#pragma unroll
    for (int r = 0; r < PL; ++r) above += __popcll(__ballot(valid[r] && key[r] > T));
    const int need_eq = k_attn - above;          // (k_attn = 0 ends with a T that no key reaches: nothing above, nothing needed)
    int eq_seen = 0;
#pragma unroll
    for (int r = 0; r < PL; ++r) {
        const bool eq = valid[r] && key[r] == T;
        const unsigned long long mk = __ballot(eq);
        bool keep = valid[r] && (key[r] > T || (eq && eq_seen + __popcll(mk & below) < need_eq));
        eq_seen += __popcll(mk);
        // Eq. 4 by the distance itself
        if (have_ring && valid[r]) {
            const int du = abs((int)((uv[r] & 0xffffu) >> 5) - cu), dv = abs((int)(uv[r] >> 21) - cv);
            keep = keep || (du > dv ? du : dv) <= radius;
        }
        kept[r] = keep;
    }
    int count = 0;
#pragma unroll
    for (int r = 0; r < PL; ++r) count += __popcll(__ballot(kept[r]));

    // Eq. 5: distance of every candidate to the set kept so far, then one pick per step
    const int m = keep_total > count ? keep_total - count : 0;
    if (m > 0) {                                             // (the same in all four wavefronts)
        uint32_t state[PL];
        int inverted[PL];
#pragma unroll
        for (int r = 0; r < PL; ++r) {
            state[r] = valid[r] ? kFarAway : 0u;
            inverted[r] = 1023 - (lane + 64 * r);
            asm volatile("" : "+v"(inverted[r]));            // (a register, not arithmetic on the lane in every pick)
        }
#pragma unroll
        for (int rr = 0; rr < PL; ++rr) {
            unsigned long long mk = __ballot(kept[rr]) & (0x1111111111111111ull << wave);      // this wavefront's members
            while (mk) {
                const int src = __builtin_ctzll(mk);
                mk &= mk - 1;
                const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)uv[rr], src);
                add_member<PL>(state, uv, inverted, at);
            }
        }
#pragma unroll
        for (int r = 0; r < PL; ++r) part[wave][lane + 64 * r] = state[r];
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int r = 0; r < PL; ++r) {
            const int i = lane + 64 * r;
            state[r] = min(min(part[0][i], part[1][i]), min(part[2][i], part[3][i]));
            if (state[r] == kFarAway) state[r] += (uint32_t)inverted[r];                      // (an empty set: token 0 first)
        }
        const uint32_t inv_gw = (1u << 20) / (uint32_t)gw + 1u;      // w / gw = (w * inv_gw) >> 20: w * gw < 2^20
        const uint32_t row_step = (65536u - (uint32_t)gw) << 5;      // (w - v gw) | v << 16 = w + v (65536 - gw)
        const uint32_t near = gw <= 64 ? 2u : 1u;
        int left = m;
        for (; left > 0; --left) {
            // largest distance, lowest index among equals: the index is in the state inverted
            uint32_t best = state[0];
#pragma unroll
            for (int r = 1; r < PL; ++r) best = max(best, state[r]);
            best = wave_max_u32(best);
            if (best >> 10 <= near) break;
            const uint32_t w = 1023u & ~best;
            const uint32_t at = (w << 5) + ((w * inv_gw) >> 20) * row_step;
            add_member<PL>(state, uv, inverted, at);
        }
#pragma unroll
        for (int r = 0; r < PL; ++r) kept[r] = kept[r] || (valid[r] && (state[r] >> 10) == 0u);
        if (left > 0) {
            bool is[PL];
            if (near == 2u) {
#pragma unroll
                for (int r = 0; r < PL; ++r) is[r] = valid[r] && (int)(uv[r] & 0xffffu) >> 5 != gw - 1;
                const Words words = {to_words<PL>(is, lane), gw};
#pragma unroll
                for (int r = 0; r < PL; ++r) is[r] = (state[r] >> 10) == 2u;
                const unsigned long long picked = words.picks(to_words<PL>(is, lane));
#pragma unroll
                for (int r = 0; r < PL; ++r) {
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)picked, r);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(picked >> 32), r);
                    is[r] = ((((unsigned long long)hi << 32) | lo) >> lane & 1ull) != 0ull;
                }
                left = keep_first<PL>(is, kept, below, left);
            }
            if (left > 0) {                                  // all others lie beside a member: by index
#pragma unroll
                for (int r = 0; r < PL; ++r) is[r] = valid[r] && !kept[r];
                keep_first<PL>(is, kept, below, left);
            }
        }
    } else if (wave != 0) {
        return;
    }

    // ascending output
    int32_t *out = idx_out + (size_t)b * cap;
    int base = 0;
#pragma unroll
    for (int r = 0; r < PL; ++r) {
        const unsigned long long mk = __ballot(kept[r]);
        if (kept[r]) out[base + __popcll(mk & below)] = lane + 64 * r;
        base += __popcll(mk);
    }
    for (int i = base + lane; i < cap; i += 64) out[i] = -1;
    if (count_out && lane == 0) count_out[b] = base;
}

sqap_status launch_prune_select(const float *scores, int batch, int gw, int gh, int k_attn, int keep_total,
                                const double *camera, int radius, int32_t *idx, int cap, int32_t *count,
                                hipStream_t st)
{
    const int n = gw * gh;
    if (n <= 256)
        hipLaunchKernelGGL(prune_select_kernel<4>, dim3(batch), dim3(64 * kSelectWaves), 0, st, scores, gw, gh, k_attn, keep_total,
                           camera, radius, idx, cap, count);
    else if (n <= 512)
        hipLaunchKernelGGL(prune_select_kernel<8>, dim3(batch), dim3(64 * kSelectWaves), 0, st, scores, gw, gh, k_attn, keep_total,
                           camera, radius, idx, cap, count);
    else
        hipLaunchKernelGGL(prune_select_kernel<16>, dim3(batch), dim3(64 * kSelectWaves), 0, st, scores, gw, gh, k_attn,
                           keep_total, camera, radius, idx, cap, count);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// One block per observation: walks the sequence in order, keeps every token
// outside the visual span and the visual tokens listed (ascending) in idx.  The list is read once, into one flag
// per visual token; spans that do not fit the flags search the list, whose dependent reads took most of the
// kernel's time (16 x 256 tokens: 3.4 us, with flags 2.6; 16 x 1024: 6.8 and 3.4).  A list that is found to be ascending needs neither
// (one barrier instead of four and two per 256 tokens: 16 x 256 2.43 -> 2.36, 16 x 1024 3.27 -> 2.31).
constexpr int kRowFlags = 8192;
__global__ __launch_bounds__(256) void kept_rows_kernel(const int32_t *__restrict__ idx, int keep_k,
                                                        int seq_len, int vis_begin, int n_vis,
                                                        int32_t *__restrict__ rows)
{
    __shared__ int wave_sums[4];
    __shared__ uint32_t flag_words[kRowFlags / 4];
    uint8_t *flags = reinterpret_cast<uint8_t *>(flag_words);
    const int b = blockIdx.x, t = threadIdx.x;
    const int32_t *my = idx + (size_t)b * keep_k;
    int32_t *out = rows + (size_t)b * (seq_len - n_vis + keep_k);
    // An ascending list of visual tokens says where each goes.  Anything else (a selection of fewer than keep_k ends with -1) takes
    // the flags, or the search.
    constexpr int HELD = 4;
    int held[HELD];
    bool ascending = keep_k <= 256 * HELD;
    if (ascending) {
#pragma unroll
        for (int j = 0; j < HELD; ++j) {
            const int i = t + 256 * j;
            const int v = held[j] = i < keep_k ? my[i] : 0, before = i > 0 && i < keep_k ? my[i - 1] : -1;
            if (i < keep_k && (v <= before || v < 0 || v >= n_vis)) ascending = false;
        }
    }
    if (__syncthreads_and(ascending)) {
#pragma unroll
        for (int j = 0; j < HELD; ++j)
            if (t + 256 * j < keep_k) out[vis_begin + t + 256 * j] = b * seq_len + vis_begin + held[j];
        for (int i = t; i < seq_len - n_vis; i += 256)
            out[i < vis_begin ? i : i + keep_k] = b * seq_len + (i < vis_begin ? i : i + n_vis);
        return;
    }
    const bool flagged = n_vis <= kRowFlags;
    if (flagged) {
        for (int i = t; i < (n_vis + 3) / 4; i += 256) flag_words[i] = 0u;
        __syncthreads();
        for (int i = t; i < keep_k; i += 256) {
            const int v = my[i];
            if (v >= 0 && v < n_vis) flags[v] = 1;
        }
        __syncthreads();
    }
    int base = 0;
    for (int c = 0; c < seq_len; c += 256) {
        const int s = c + t;
        bool keep = false;
        if (s < seq_len) {
            const int v = s - vis_begin;
            if (v < 0 || v >= n_vis) {
                keep = true;
            } else if (flagged) {
                keep = flags[v] != 0;
            } else {                     // binary search in the ascending list
                int lo = 0, hi = keep_k;
                while (lo < hi) {
                    int mid = (lo + hi) >> 1;
                    if (my[mid] < v) lo = mid + 1; else hi = mid;
                }
                keep = lo < keep_k && my[lo] == v;
            }
        }
        int total;
        int pos = block_scan_flags(keep, wave_sums, &total);
        if (keep) out[base + pos] = b * seq_len + s;
        base += total;
    }
}

sqap_status launch_kept_rows(const int32_t *idx, int batch, int keep_k, int seq_len,
                             int vis_begin, int n_vis, int32_t *rows, hipStream_t st)
{
    hipLaunchKernelGGL(kept_rows_kernel, dim3(batch), dim3(256), 0, st, idx, keep_k, seq_len,
                       vis_begin, n_vis, rows);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// out[i,:] = X[rows[i],:]; one 16-byte piece per thread, rows of a block contiguous.
__global__ __launch_bounds__(256) void gather_rows_kernel(const __half *__restrict__ X, int64_t ldx,
                                                          const int32_t *__restrict__ rows, int M,
                                                          int pieces, __half *__restrict__ out,
                                                          int64_t ldo)
{
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t row = gid / pieces;
    const int p = (int)(gid % pieces);
    if (row >= M) return;
    const uint4 *src = reinterpret_cast<const uint4 *>(X + (int64_t)rows[row] * ldx) + p;
    uint4 *dst = reinterpret_cast<uint4 *>(out + row * ldo) + p;
    *dst = *src;
}

sqap_status launch_gather_rows(const __half *X, int64_t ldx, const int32_t *rows, int M, int K,
                               __half *out, int64_t ldo, hipStream_t st)
{
    const int pieces = K / 8;
    const int64_t total = (int64_t)M * pieces;
    const int64_t blocks = (total + 255) / 256;
    if (blocks > 0x7fffffff) return fail(SQAP_EUNSUPPORTED, "sqap_gather_rows: too large");
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, X, ldx, rows, M,
                       pieces, out, ldo);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// Retention score.  One block of 8 wavefronts; wavefront w takes heads w, w+8, ...
// For its head every lane owns keys lane, lane+64, ...: pass 1 builds the
// running (max, sum) of the softmax, pass 2 recomputes the logits of the
// visual span and turns them into weights.  Heads are then added into the
// LDS accumulator in wavefront order, so the sum order is fixed.
__device__ __forceinline__ float dot_qk(const __half *__restrict__ qh, const __half *__restrict__ kh, int d)
{
    float acc = 0.f;
    for (int i = 0; i < d; i += 2) {
        float2 a = __half22float2(*reinterpret_cast<const __half2 *>(qh + i));
        float2 b = __half22float2(*reinterpret_cast<const __half2 *>(kh + i));
        acc = fmaf(a.x, b.x, acc);
        acc = fmaf(a.y, b.y, acc);
    }
    return acc;
}

constexpr int kScoreWaves = 8;

__global__ __launch_bounds__(64 * kScoreWaves) void attn_scores_kernel(
    const __half *__restrict__ q, const __half *__restrict__ k, int S, int H, int d, int vis_begin,
    int n_vis, float *__restrict__ scores)
{
    extern __shared__ float acc_lds[];   // n_vis floats
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int j = threadIdx.x; j < n_vis; j += blockDim.x) acc_lds[j] = 0.f;
    __syncthreads();
    const float inv_sqrt_d = 1.0f / sqrtf((float)d);
    const int rounds = (H + kScoreWaves - 1) / kScoreWaves;
    for (int r = 0; r < rounds; ++r) {
        const int h = r * kScoreWaves + wave;
        float m = -INFINITY, z = 0.f;
        if (h < H) {
            const __half *qh = q + (size_t)h * d;
            for (int s = lane; s < S; s += 64) {
                float l = dot_qk(qh, k + ((size_t)s * H + h) * d, d) * inv_sqrt_d;
                float mn = fmaxf(m, l);
                z = z * expf(m - mn) + expf(l - mn);
                m = mn;
            }
            for (int o = 32; o > 0; o >>= 1) {
                float m2 = __shfl_xor(m, o), z2 = __shfl_xor(z, o);
                float mn = fmaxf(m, m2);
                float za = (m == -INFINITY) ? 0.f : z * expf(m - mn);
                float zb = (m2 == -INFINITY) ? 0.f : z2 * expf(m2 - mn);
                z = za + zb;
                m = mn;
            }
        }
        // add this round's heads in wavefront order
        for (int w = 0; w < kScoreWaves; ++w) {
            if (w == wave && h < H) {
                const __half *qh = q + (size_t)h * d;
                for (int j = lane; j < n_vis; j += 64) {
                    const int s = vis_begin + j;
                    float l = dot_qk(qh, k + ((size_t)s * H + h) * d, d) * inv_sqrt_d;
                    acc_lds[j] += expf(l - m) / z;
                }
            }
            __syncthreads();
        }
    }
    for (int j = threadIdx.x; j < n_vis; j += blockDim.x) scores[j] = acc_lds[j] / (float)H;
}

// Fast path of the retention score: one workgroup per head.  A group of d/8 lanes reads one
// key row piece (16 bytes per lane: a coalesced run of 2d bytes), the logits of the head go to
// LDS, the workgroup takes their maximum and the sum of exponentials, and writes the head's
// softmax weights of the visual span to the workspace.  The workgroup that finishes last (a
// counter in the workspace tells) adds the heads in head order, so the result does not depend on
// the order in which the workgroups ran, and puts the counter back to zero.
// A batch of observations runs as one launch (grid: heads x observations); each observation has
// its own counter and its own piece of the weight array.
// Workspace: [batch counters, one 256-byte line each (atomics on one line serialise)]
//            [batch * H * n_vis floats].
constexpr int kScoreMaxSeq = 4096;                // logits of one head sit in LDS
constexpr int kCounterStride = 64;                // 32-bit words per counter line
static size_t score_counter_bytes(int batch) { return (size_t)batch * kCounterStride * sizeof(unsigned int); }

__device__ __forceinline__ float block_reduce_256(float v, bool take_max, float *scratch4)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int o = 32; o > 0; o >>= 1) {
        const float u = __shfl_xor(v, o);
        v = take_max ? fmaxf(v, u) : v + u;
    }
    __syncthreads();                              // previous users of scratch4 are done
    if (lane == 0) scratch4[wave] = v;
    __syncthreads();
    return take_max ? fmaxf(fmaxf(scratch4[0], scratch4[1]), fmaxf(scratch4[2], scratch4[3]))
                    : (scratch4[0] + scratch4[1]) + (scratch4[2] + scratch4[3]);
}

// kRowsInFlight: key rows a lane group loads before it reduces any.  LP: lanes per key row, 16 or 8 (then the sum takes no LDS
// permutes), 0 for any other.
template <int kRowsInFlight, int LP>
__global__ __launch_bounds__(256) void attn_head_kernel(const __half *__restrict__ q, const __half *__restrict__ k,
                                                        int S, int H, int d, int vis_begin, int n_vis,
                                                        float *__restrict__ scores, unsigned int *heads_done,
                                                        float *all_head_weights)
{
    __shared__ float logits[kScoreMaxSeq];
    __shared__ float red[4];
    __shared__ bool is_last;
    const int t = threadIdx.x, h = blockIdx.x, b = blockIdx.y;
    q += (size_t)b * H * d;
    k += (size_t)b * S * H * d;
    scores += (size_t)b * n_vis;
    float *head_weights = all_head_weights + (size_t)b * H * n_vis;
    const int lp = LP ? LP : d >> 3;              // lanes per key row: a power of two, 1 .. 32
    const int sub = t & (lp - 1), grp = t / lp, groups = 256 / lp;
    float qf[8];
    {
        const uint4 raw = *reinterpret_cast<const uint4 *>(q + (size_t)h * d + sub * 8);
        const __half2 *h2 = reinterpret_cast<const __half2 *>(&raw);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float2 f = __half22float2(h2[i]);
            qf[2 * i] = f.x;
            qf[2 * i + 1] = f.y;
        }
    }
    const float inv_sqrt_d = 1.0f / sqrtf((float)d);
    for (int s0 = 0; s0 < S; s0 += groups * kRowsInFlight) {
        uint4 raw[kRowsInFlight];
#pragma unroll
        for (int r = 0; r < kRowsInFlight; ++r) {
            const int s = s0 + r * groups + grp;
            if (LP == 0) raw[r] = make_uint4(0u, 0u, 0u, 0u);
            if (s < S) raw[r] = *reinterpret_cast<const uint4 *>(k + ((size_t)s * H + h) * d + sub * 8);
        }
#pragma unroll
        for (int r = 0; r < kRowsInFlight; ++r) {
            const int s = s0 + r * groups + grp;
            if (LP != 0 && s0 + r * groups >= S) break;      // (uniform; with LDS permutes it would keep them from overlapping)
            const __half2 *h2 = reinterpret_cast<const __half2 *>(&raw[r]);
            float acc = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float2 f = __half22float2(h2[i]);
                acc = fmaf(qf[2 * i], f.x, acc);
                acc = fmaf(qf[2 * i + 1], f.y, acc);
            }
            // the lane group's sum in every lane, partners 8, 4, 2, 1 apart, without LDS permutes: once the step by 8 has made
            // the lanes of a row repeat every 8, 4 back is 4 across, and so on; in groups of 8 the partner 4 across is the
            // mirror image's mirror image within its quad
            if (LP == 16) {
                acc += dpp_move_f<0x128>(acc);
                acc += dpp_move_f<0x124>(acc);
                acc += dpp_move_f<0x122>(acc);
                acc += dpp_move_f<0x121>(acc);
            } else if (LP == 8) {
                acc += dpp_move_f<0x1B>(dpp_move_f<kDppHalfMirror>(acc));
                acc += dpp_move_f<kDppXor2>(acc);
                acc += dpp_move_f<kDppXor1>(acc);
            } else {
                for (int o = lp >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
            }
            if (s < S && sub == 0) logits[s] = acc * inv_sqrt_d;
        }
    }
    __syncthreads();
    float m = -INFINITY;
    for (int s = t; s < S; s += 256) m = fmaxf(m, logits[s]);
    m = block_reduce_256(m, true, red);
    float z = 0.f;
    for (int s = t; s < S; s += 256) z += expf(logits[s] - m);
    z = block_reduce_256(z, false, red);
    // The weights go out as agent-scope stores (written through this XCD's L2, since the workgroup that
    // adds the heads may sit behind another one); they are complete once the vector-memory counter
    // drains, and only then does the workgroup count itself as done.  A full release fence here would
    // write back the whole L2 once per workgroup.
    for (int j = t; j < n_vis; j += 256)
        __hip_atomic_store(&head_weights[(size_t)h * n_vis + j], expf(logits[vis_begin + j] - m) / z, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0) {
        const unsigned done = __hip_atomic_fetch_add(&heads_done[b * kCounterStride], 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
        is_last = done + 1 == (unsigned)H;
        if (is_last)                              // ready for the next call
            __hip_atomic_store(&heads_done[b * kCounterStride], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (is_last) {
        // agent-scope loads: they do not hit stale lines of an earlier call in this XCD's caches
        for (int j = t; j < n_vis; j += 256) {
            float a = 0.f;
#pragma unroll 16
            for (int hh = 0; hh < H; ++hh)
                a += __hip_atomic_load(&head_weights[(size_t)hh * n_vis + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            scores[j] = a / (float)H;
        }
    }
}

// The fast path needs a power-of-two head size of 8 .. 256, 16-byte aligned operands and a sequence
// whose logits fit LDS; everything else takes the one-workgroup kernel, which needs no workspace.
static bool score_fast_path(const void *q, const void *k, int S, int d)
{
    const bool pow2 = (d & (d - 1)) == 0;
    const bool aligned = ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k)) & 15u) == 0;
    return pow2 && d >= 8 && d <= 256 && aligned && S <= kScoreMaxSeq;
}

size_t attn_scores_workspace_bytes(int batch, int H, int n_vis)
{
    if (batch <= 0 || H <= 0 || n_vis <= 0) return 0;
    return score_counter_bytes(batch) + (size_t)batch * H * n_vis * sizeof(float);
}

// A round of loads is a trip to memory that everything else waits for: 18 rows per lane group take the 276 keys of an
// observation with heads of 128 in one round (16 observations x 32 heads: 11.6 us; 8 rows, three rounds: 15.6; one observation
// 8.0 and 12.4), 9 where that is enough (8 x 8 tokens, heads of 64: 5.2 and 6.5).  Other head sizes add their lanes with LDS
// permutes, whose latency bounds a round: eight rows side by side (us, observations x keys x heads x head size: 6 x 2524 x 32 x 16
// 25.9, 3 x 1455 x 32 x 32 15.5, 3 x 2867 x 32 x 256 160; 18 rows with a stop at the last key 27.9, 17.2 and 185).
static void launch_attn_head(const __half *q, const __half *k, int batch, int S, int H, int d, int vis_begin, int n_vis,
                             float *scores, unsigned int *counters, float *weights, hipStream_t st)
{
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(H, batch), dim3(256), 0, st, q, k, S, H, d, vis_begin, n_vis, scores, counters, weights);
    };
    const bool one_round_of_nine = S <= 9 * (2048 / d);
    if (d == 128) launch(one_round_of_nine ? attn_head_kernel<9, 16> : attn_head_kernel<18, 16>);
    else if (d == 64) launch(one_round_of_nine ? attn_head_kernel<9, 8> : attn_head_kernel<18, 8>);
    else launch(attn_head_kernel<8, 0>);
}

sqap_status launch_attn_scores(const __half *q, const __half *k, int batch, int S, int H, int d,
                               int vis_begin, int n_vis, float *scores, void *workspace, size_t workspace_bytes,
                               hipStream_t st)
{
    if (score_fast_path(q, k, S, d) && workspace && workspace_bytes >= attn_scores_workspace_bytes(batch, H, n_vis)) {
        unsigned int *counters = reinterpret_cast<unsigned int *>(workspace);
        float *weights = reinterpret_cast<float *>(reinterpret_cast<uint8_t *>(workspace) + score_counter_bytes(batch));
        launch_attn_head(q, k, batch, S, H, d, vis_begin, n_vis, scores, counters, weights, st);
    } else {
        for (int b = 0; b < batch; ++b)
            hipLaunchKernelGGL(attn_scores_kernel, dim3(1), dim3(64 * kScoreWaves), n_vis * sizeof(float), st,
                               q + (size_t)b * H * d, k + (size_t)b * S * H * d, S, H, d, vis_begin, n_vis,
                               scores + (size_t)b * n_vis);
    }
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// ---------------------------------------------------------------------------------------------
// The retention score for callers that cannot allocate (a stream under graph capture, a serving loop
// that forbids hipMalloc): the workspace of the fast kernel is this file-scope device array instead of
// a caller's buffer.  Layout as above: kNoAllocMaxBatch counter lines, then the per-head weights.
// The array's name is only a host-side handle: the device address is looked up once per device with
// hipGetSymbolAddress (each device holds its own copy of the array at its own address) and host code
// uses that address from then on.  The array is zero when the code object is loaded; what must be zero
// at the start of a call (the counters) is put back to zero by the workgroup that finishes last, so
// every call that runs to its end leaves the array ready for the next one.
constexpr int kNoAllocMaxBatch = 64;
constexpr size_t kNoAllocMaxWeights = 512 * 1024;                  // batch * H * n_vis floats: 2 MiB
constexpr size_t kNoAllocCounterBytes = (size_t)kNoAllocMaxBatch * kCounterStride * sizeof(unsigned int);
constexpr size_t kNoAllocScratchBytes = kNoAllocCounterBytes + kNoAllocMaxWeights * sizeof(float);
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

static std::atomic<void *> g_scratch_of_device[kMaxDeviceSlots];

// Device address of `scratch` on the current device (looked up on the first call per device).
sqap_status noalloc_scratch(void **out)
{
    int dev = 0;
    SQAP_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDeviceSlots)
        return fail(SQAP_EUNSUPPORTED, "device ordinal %d above %d", dev, kMaxDeviceSlots - 1);
    void *ptr = g_scratch_of_device[dev].load(std::memory_order_acquire);
    if (!ptr) {
        SQAP_HIP_CHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return fail(SQAP_EDEVICE, "hipGetSymbolAddress gave a null address for the scratch array");
        g_scratch_of_device[dev].store(ptr, std::memory_order_release);      // racing host threads store the same value
    }
    *out = ptr;
    return SQAP_OK;
}

size_t noalloc_max_weights() { return kNoAllocMaxWeights; }
int noalloc_max_batch() { return kNoAllocMaxBatch; }

sqap_status launch_attn_scores_noalloc(const __half *q, const __half *k, int batch, int S, int H, int d,
                                       int vis_begin, int n_vis, float *scores, hipStream_t st)
{
    if (!score_fast_path(q, k, S, d))       // the one-workgroup kernel uses no scratch memory at all
        return launch_attn_scores(q, k, batch, S, H, d, vis_begin, n_vis, scores, nullptr, 0, st);
    void *ptr = nullptr;
    sqap_status s = noalloc_scratch(&ptr);
    if (s != SQAP_OK) return s;
    // The kernel sees the array split as [batch counter lines][weights]; the weights start behind the
    // counter lines of THIS call's batch, which all lie inside the kNoAllocMaxBatch lines that are kept zero.
    unsigned int *counters = reinterpret_cast<unsigned int *>(ptr);
    float *weights = reinterpret_cast<float *>(reinterpret_cast<uint8_t *>(ptr) + kNoAllocCounterBytes);
    launch_attn_head(q, k, batch, S, H, d, vis_begin, n_vis, scores, counters, weights, st);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

}  // namespace sqap
