// W4A4 linear for 17 to a few hundred token rows (and for more where the channels are few): every workgroup owns complete outputs.
//
// At these sizes the output is too small to fill the machine with whole 256 x 256 tiles, and splitting K between workgroups costs a
// chain of global round trips (partial store, flag, reduction) that is longer than the arithmetic.  Here nothing crosses a
// workgroup: a workgroup (one per compute unit, eight wavefronts) owns a block of up to 96 token rows times up to six 16-channel
// groups, or two or three times as many one after the other, over the WHOLE reduction axis, and its wavefronts share out K:
//   up to three channel groups: K in eighths, every wavefront all rows and channels of the tile, so that a byte of tokens and a byte of
//   weights is widened to int8 by one wavefront only;
//   four to six (and three where K fits steps of 512 better than of 1024): K in quarters, two wavefronts per quarter with half of the channels each (all of them would not fit the registers).
// A step is 128 codes of K per share.  Token rows travel global -> LDS without passing registers, two steps ahead in three buffers, whole
// runs of 256 or 512 bytes of a row; 16-byte pieces are permuted (piece p of row r at p ^ (r % 16)), so that the operand reads (16
// rows, one piece) touch every bank once (counters: no conflicts).  Weights go straight to registers: the packed layout is the operand
// order of v_mfma_i32_16x16x64_i8 (lane l: channel l % 16, 16-byte piece l / 16).  One barrier per step, which waits by count for
// the loads of the step before the last.  At the end the shares are added through LDS.
// int4 -> int8 as in the large-M kernel: (x << 4) & 0xF0F0F0F0 and x & 0xF0F0F0F0 give 16 * code for the even and the odd codes; both
// operands are split the same way, so the accumulator is 256 * sum(x * w).
//
// What bounds it (cycle stamps, 148 x 12288 x 4096, 25 000 cycles per wavefront): issue of the vector ALU and the matrix cores together, which
// overlap in part only (two wavefronts of a SIMD with 12 widenings per 6 products each take 205 cycles if the widenings come in one piece
// before products that do not need them, 230 to 310 otherwise, products alone 205): 15 500 cycles in the steps, 7 700 of them
// products; 1 300 until the first load, 2 700 until the first step's operands are there, 5 500 for the reduction and the stores.
// Loads of a compute unit come in at 64 bytes per cycle, and all wavefronts' first step must not queue behind anybody's second.
// Without any loads after the first two steps the launch is 4 % shorter.  K-steps twice as long for four to six groups: 84 x 22016 x
// 4096 18.4 us against 15.9, because half of the weights had to arrive before the first product.
// Measured, us, the kernel before (160 rows, quarters of K x halves of the tokens, tokens through registers, three groups) in brackets:
// 32 x 512 x 512 3.0 (3.4); 84 x 4096 x 4096 6.0 (7.1), 84 x 12288 x 4096 9.6 (11.0), 84 x K = 11008 10.4 (12.0); 148 x 4096 x 4096 7.3
// (9.0), 148 x 12288 x 4096 12.4 (14.2), 148 x K = 11008 13.7 (15.4); 276 x 4096 x 4096 9.9 (11.2); 300 x 1000 x 1984 4.8 (6.0);
// 2000 x 700 x 5504 15.2 (19.1); but tall products of few channels whose K ends inside a step: 263 x 88 x 9728 7.5 (6.4), 433 x 104 x 5888
// 6.0 (5.4).  Against the tiles: 84 x 22016 x 4096 15.6 (20.3), 134 x 13896 x 4096 16.6 (21.7), 148 x 22016 x 4096 23.1
// (27.6), 276 x 12288 x 4096 22.5 (24.2), 451 x 8123 x 4160 29.6 (52.7), 679 x 4020 x 2816 17.9 (28.8); where they are faster, at
// whole_output_plan.
#include <algorithm>

#include "common.h"

namespace sqap {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kRowsThreads = 64 * kRowsWaves;
constexpr int kRowsMaxTG = 6;          // 16-token groups of a workgroup
constexpr int kRowsMaxCB = 3;          // 16-channel groups of a wavefront
constexpr int kRowsMaxTiles = 3;       // tiles of a workgroup, one after the other
constexpr int kRowsBufs = 3;
// a step: 128 codes of K for each of the ks shares
constexpr int rows_step_chunks(int ks) { return 4 * ks; }
constexpr int rows_scales_at(int tg, int cb, int ks)
{
    const int tokens = kRowsBufs * tg * 16 * rows_step_chunks(ks) * 16, reduce = kRowsWaves * tg * cb * 1024;
    return tokens > reduce ? tokens : reduce;
}
constexpr int rows_lds(int tg, int cb, int ks) { return rows_scales_at(tg, cb, ks) + 256 + 2 * kRowsMaxCB * 32; }

struct RowsParams {
    // (what a launch needs lies in two lines of 64 bytes: a cold line is a trip to memory in front of the first load)
    const uint8_t *Xq;     // [M, K/2] canonical
    const __half *sx;      // [M]
    unsigned long long *error_word;
    int M, chunks, c16;
    int rows_per_block;    // multiple of 16
    int tblocks, per_xcd;
    uint32_t wg_inv;       // ceil(2^32 / workgroups of a token block)
    uint32_t tb_inv;       // 2^16 / tblocks + 1
    int steps;
    int reserved;
    RowsWeight w;
};

__device__ __forceinline__ void rows_widen(const v4i p, v4i &lo, v4i &hi)
{
    const v4i mask = {(int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0};
    lo = (p << 4) & mask;
    hi = p & mask;
}

typedef float v2f_m __attribute__((ext_vector_type(2)));
typedef _Float16 v2h_m __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t rows_dequant_pair(int acc0, int acc1, float sx_over_256, float sw0, float sw1)
{
    float y0 = ((float)acc0 * sx_over_256) * sw0;
    float y1 = ((float)acc1 * sx_over_256) * sw1;
    asm volatile("" : "+v"(y0), "+v"(y1));
    const v2f_m y = {y0, y1};
    union { v2h_m h; uint32_t u; } r;
    r.h = __builtin_convertvector(y, v2h_m);
    return r.u;
}

template <int N>
__device__ __forceinline__ void wait_loads()
{
    // (the builtin, not assembly: the compiler then knows what has arrived)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | 7 << 4 | 15 << 8 | (N >> 4) << 14);
    asm volatile("" ::: "memory");
}

template <int TG, int CB, int KS, bool MASKED>
__device__ __forceinline__ void rows_tile(const RowsParams &p, uint8_t *smem, int row0, int row_end, int c0, int n)
{
    constexpr int STEP = rows_step_chunks(KS);          // chunks
    constexpr int GROUP = 16 * STEP * 16;              // bytes of a token group in a step
    constexpr int RPL = 64 / STEP;                     // rows per wavefront load
    constexpr int LOADS = TG * 16 / RPL, XL = (LOADS + kRowsWaves - 1) / kRowsWaves;      // token loads of a step, of a wavefront
    constexpr int PER_STEP = XL + CB;                  // loads of a wavefront and step
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int kq = wave & (KS - 1), half = KS == 8 ? 0 : wave >> 2;
    const int chunks = p.chunks, S = p.steps;
    const int rot = (int)(blockIdx.x >> 3) * S >> 5;
    auto step_of = [&](int i) { return i + rot >= S ? i + rot - S : i + rot; };
    // ---- token rows, global -> LDS, 16 STEP bytes of each per step: load e of a wavefront covers RPL rows, lane l takes slot l % STEP of
    // one of them, which holds piece slot ^ (row % 16).  (Where the loads do not come out even the last one is repeated.)
    const int lr = lane / STEP, first = LOADS < kRowsWaves ? wave % LOADS : wave;
    const int piece = (lane % STEP) ^ ((first * RPL + lr) & 15);       // (rows of one wavefront's loads are multiples of 16 apart)
    static_assert(kRowsWaves * RPL % 16 == 0, "one piece per lane");
    auto load_index = [&](int e) { return LOADS % kRowsWaves == 0 || e * kRowsWaves + first < LOADS ? e * kRowsWaves + first : max(e - 1, 0) * kRowsWaves + first; };
    uint32_t rowoff[XL];
#pragma unroll
    for (int e = 0; e < XL; ++e)
        rowoff[e] = (uint32_t)min(row0 + load_index(e) * RPL + lr, p.M - 1) * (uint32_t)(chunks * 16) + (MASKED ? 0 : piece * 16);
    auto issue_tokens = [&](int i) {
        const int step = step_of(i);
        uint8_t *const to = smem + (i % kRowsBufs) * TG * GROUP;
        const uint8_t *from = MASKED ? p.Xq : p.Xq + (size_t)step * (STEP * 16);
        const uint32_t po = MASKED ? (uint32_t)min(step * STEP + piece, chunks - 1) * 16 : 0;
#pragma unroll
        for (int e = 0; e < XL; ++e)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) v4i *)(from + (rowoff[e] + po)),
                                             (__attribute__((address_space(3))) void *)(to + load_index(e) * 1024), 16, 0, 0);
    };
    // ---- weights, straight to registers
    const uint8_t *wbase[CB];
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        const int g = min(c0 + half * CB + j, c0 + n - 1);
        wbase[j] = p.w.Wd + (size_t)(g >> 1) * chunks * 512 + (g & 1) * 256;
    }
    const uint32_t woff = (uint32_t)(kq * 4 + (lane >> 4)) * 512 + (lane & 15) * 16;
    v4i wr[2][CB];
    auto load_w = [&](int i, auto set_c) {
        constexpr int set = decltype(set_c)::value;
        const int step = step_of(i);
        const uint32_t clamped = (uint32_t)min(step * STEP + kq * 4 + (lane >> 4), chunks - 1) * 512 + (lane & 15) * 16;
#pragma unroll
        for (int j = 0; j < CB; ++j)
            wr[set][j] = MASKED ? *reinterpret_cast<const v4i *>(wbase[j] + clamped)
                                : *reinterpret_cast<const v4i *>(wbase[j] + (size_t)step * (STEP * 512) + woff);
    };
    constexpr std::integral_constant<int, 0> c0_{};
    constexpr std::integral_constant<int, 1> c1_{};

    __half sx_early = {};
    uint2 sw_early = {};
    const int sc = t - 2 * 64;
    if (t < TG * 16) sx_early = p.sx[min(row0 + t, p.M - 1)];
    if (sc >= 0 && sc < n * 4) sw_early = *reinterpret_cast<const uint2 *>(p.w.sw + (c0 + (sc >> 2)) * 16 + (sc & 3) * 4);       // zero padded past N

    // The waits below count loads: what is asked for in which order is fixed.  Every wavefront's first step comes before anybody's
    // second: a compute unit takes 64 bytes per cycle, and the queue is common.  An odd number of steps begins with register set 1,
    // so that the last step always has that one.
    const bool odd = S & 1;
    asm volatile("" ::: "memory");
    issue_tokens(0);
    asm volatile("" ::: "memory");
    if (odd) load_w(0, c1_);
    else load_w(0, c0_);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (S > 1) {
        issue_tokens(1);
        asm volatile("" ::: "memory");
        if (odd) load_w(1, c0_);
        else load_w(1, c1_);
    }
    __half *const sx_lds = reinterpret_cast<__half *>(smem + rows_scales_at(TG, CB, KS));
    uint2 *const sw_lds = reinterpret_cast<uint2 *>(smem + rows_scales_at(TG, CB, KS) + 256);
    if (t < TG * 16) sx_lds[t] = sx_early;
    if (sc >= 0 && sc < n * 4) sw_lds[sc] = sw_early;

    v4i acc[TG][CB];
#pragma unroll
    for (int i = 0; i < TG; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // operand order: token l % 16, piece l / 16 of a block
    const int tok = lane & 15;
    const int frag = tok * (STEP * 16) + (((kq * 4 + (lane >> 4)) ^ tok) * 16);

    auto step_body = [&](int i, auto par_c, auto more_c) {
        constexpr int PAR = decltype(par_c)::value;
        constexpr bool MORE = decltype(more_c)::value;
        constexpr std::integral_constant<int, PAR> cur{};
        // all operands of the step are on their way from LDS before anything waits for the first
        const uint8_t *from = smem + (i % kRowsBufs) * TG * GROUP + frag;
        v4i xf[TG];
#pragma unroll
        for (int g = 0; g < TG; ++g) xf[g] = *reinterpret_cast<const v4i *>(from + g * GROUP);
        __builtin_amdgcn_sched_barrier(0);
        if (MORE) issue_tokens(i + 2);
        asm volatile("" ::: "memory");
        if (MASKED) {
            const bool ok = step_of(i) * STEP + kq * 4 + (lane >> 4) < chunks;
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) wr[PAR][j][e] = ok ? wr[PAR][j][e] : 0;
        }
        v4i wl[CB], wh[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j) rows_widen(wr[PAR][j], wl[j], wh[j]);
        if (MORE) load_w(i + 2, cur);
        // a group is widened before the products of the group in front of it: the two wavefronts of a SIMD drift into taking turns
        // at the vector ALU and the matrix core (left to itself the compiler widens everything first, both wavefronts at once)
        v4i xl, xh;
        rows_widen(xf[0], xl, xh);
#pragma unroll
        for (int g = 0; g < TG; ++g) {
            __builtin_amdgcn_sched_barrier(0);
            v4i nl = xl, nh = xh;
            if (g + 1 < TG) rows_widen(xf[g + 1], nl, nh);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < CB; ++j) acc[g][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wl[j], xl, acc[g][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < CB; ++j) acc[g][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh[j], xh, acc[g][j], 0, 0, 0);
            xl = nl;
            xh = nh;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // step i needs everything asked for up to the end of step i - 2; what was asked for behind that may stay on its way
    constexpr std::true_type more{};
    constexpr std::false_type last{};
    auto next = [&] {
        wait_loads<PER_STEP>();
        lds_barrier();
    };
    auto final_step = [&] {
        wait_loads<0>();
        lds_barrier();
    };
    int i = 0;
    if (odd) {
        if (S > 1) {
            next();
            step_body(0, c1_, more);
        } else {
            final_step();
            step_body(0, c1_, last);
        }
        i = 1;
    }
    for (; i + 2 < S; i += 2) {
        next();
        step_body(i, c0_, more);
        next();
        step_body(i + 1, c1_, more);
    }
    if (i < S) {
        next();
        step_body(i, c0_, last);
        final_step();
        step_body(i + 1, c1_, last);
    }
    lds_barrier();                                     // everybody is done with the tokens

    // add the accumulators of the K shares through LDS
    int *red = reinterpret_cast<int *>(smem);
#pragma unroll
    for (int g = 0; g < TG; ++g)
#pragma unroll
        for (int j = 0; j < CB; ++j) *reinterpret_cast<v4i *>(red + ((wave * TG * CB + g * CB + j) * 64 + lane) * 4) = acc[g][j];
    lds_barrier();
    const int tok_in = lane & 15, ch4 = (lane >> 4) * 4;
    const RowsWeight &w = p.w;
    const bool a_vec = (w.N & 3) == 0 && w.acc_out && (reinterpret_cast<uintptr_t>(w.acc_out) & 15u) == 0;
    constexpr int OWN = (TG * CB + KS - 1) / KS;
    v4i sums[OWN];
#pragma unroll
    for (int m = 0; m < OWN; ++m) {
        const int *from = red + ((half * KS * TG * CB + min(m * KS + kq, TG * CB - 1)) * 64 + lane) * 4;
        sums[m] = *reinterpret_cast<const v4i *>(from);
#pragma unroll
        for (int s = 1; s < KS; ++s) sums[m] += *reinterpret_cast<const v4i *>(from + s * TG * CB * 256);
    }
#pragma unroll
    for (int m = 0; m < OWN; ++m) {
        const int tt = m * KS + kq;
        if (tt >= TG * CB) break;
        const int g = tt / CB, j = tt - g * CB, cg = half * CB + j;
        const v4i sum = sums[m];
        const int row = row0 + g * 16 + tok_in, col = (c0 + cg) * 16 + ch4;
        if (cg < n && row < row_end && col < w.N) {
            const float sxf = __half2float(sx_lds[g * 16 + tok_in]) * 0.00390625f;
            const uint2 swr = sw_lds[cg * 4 + (lane >> 4)];
            const __half2 *sw2 = reinterpret_cast<const __half2 *>(&swr);
            const float2 s01 = __half22float2(sw2[0]), s23 = __half22float2(sw2[1]);
            uint2 pk;
            pk.x = rows_dequant_pair(sum.x, sum.y, sxf, s01.x, s01.y);
            pk.y = rows_dequant_pair(sum.z, sum.w, sxf, s23.x, s23.y);
            __half *dst = w.Y + (size_t)row * w.ldy + col;
            if (col + 4 <= w.N) {
                *reinterpret_cast<halves4_any *>(dst) = halves4_any{pk.x, pk.y};
            } else {
                const __half *h = reinterpret_cast<const __half *>(&pk);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < w.N) dst[e] = h[e];
            }
            if (w.acc_out) {
                int32_t *ad = w.acc_out + (size_t)row * w.N + col;
                const v4i v = {sum.x >> 8, sum.y >> 8, sum.z >> 8, sum.w >> 8};
                if (a_vec && col + 4 <= w.N) {
                    *reinterpret_cast<v4i *>(ad) = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < w.N) ad[e] = v[e];
                }
            }
        }
    }
}

template <int TG, int CB, int KS, bool MASKED>
__global__ __launch_bounds__(kRowsThreads, 1) void gemm_rows_kernel(const RowsParams p)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    asm volatile("" ::"s"(p.Xq), "s"(p.sx), "s"(p.error_word), "s"(p.M), "s"(p.w.Wd), "s"(p.w.sw), "s"(p.w.N));
    if (blockIdx.x == 0 && threadIdx.x == 0 && p.error_word) *p.error_word = 0ull;
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int slot = (j * p.tb_inv) >> 16, tb = j - slot * p.tblocks;
    if (slot >= p.per_xcd) return;
    const uint32_t i = xcd * p.per_xcd + slot;
    const int g_begin = (int)__umulhi((uint32_t)p.c16 * i, p.wg_inv), g_end = (int)__umulhi((uint32_t)p.c16 * (i + 1), p.wg_inv);
    const int row0 = tb * p.rows_per_block;
    if (row0 >= p.M) return;
    const int row_end = min(p.M, row0 + p.rows_per_block);
    constexpr int MAXN = CB * (kRowsWaves / KS);
    int c0 = g_begin;
    for (int left = g_end - c0, tiles = (left + MAXN - 1) / MAXN; tiles > 0; --tiles) {
        const int n = tiles == 1 ? left : tiles == 2 ? (left + 1) / 2 : (left + 2) / 3;
        if (c0 != g_begin) lds_barrier();              // LDS is free for the next tile
        rows_tile<TG, CB, KS, MASKED>(p, smem, row0, row_end, c0, n);
        c0 += n;
        left -= n;
    }
}

// Token blocks, channel groups per workgroup and the shares of K: the plan with the lowest cost.  A step's products and widenings
// against the bytes a compute unit loads, or against what its XCD does (every XCD reads all token rows and an eighth of the weights;
// workgroups that share token rows are at different places of K, so rows that its L2 of 4 MB does not hold come once for each); the start
// and the reduction, once per tile.  All numbers are clock cycles but for the microseconds at the end, and fitted to every plan of 2028
// drawn shapes (17 to 3072 rows, 64 to 45000 channels, K of 384 to 14000, 7432 timings: half of them within 4 %).  The plan named is
// the fastest or within 3 % of it in 97 of 100 shapes, at worst 10 % off; without the masked steps of a K that ends inside one and without
// the L2, 22 shapes were 10 to 35 % off (148 x 4096 x 4800 9.0 us against 8.5, 1500 x 768 x 8192 19.8 and 14.9).
static bool rows_plan(int M, int c16, int K, int cus, WholePlan *plan, int *tiles_out, double *us_out)
{
    if (K % 32 != 0 || c16 < 1) return false;
    const int max_tiles = K < 1024 && K % 512 != 0 ? 1 : K > 8192 ? kRowsMaxTiles - 1 : kRowsMaxTiles;
    const int tb_min = (M + 16 * kRowsMaxTG - 1) / (16 * kRowsMaxTG), tb_max = std::min(cus / 8, 2 * tb_min + 2);
    double best = 0.0;
    for (int tb = tb_min; tb <= tb_max; ++tb) {
        const int rows = ((M + tb - 1) / tb + 15) / 16 * 16, tg = rows / 16;
        const int per_xcd = cus / 8 / tb, W = 8 * per_xcd, n_all = (c16 + W - 1) / W;
        const int tiles = (n_all + 2 * kRowsMaxCB - 1) / (2 * kRowsMaxCB);
        if (tiles > max_tiles) continue;
        const int n = (n_all + tiles - 1) / tiles;
        for (int ks = n <= kRowsMaxCB ? 8 : 4; ks >= (n < kRowsMaxCB ? 8 : 4); ks -= 4) {
            const bool eighths = ks == 8;
            const int cb = eighths ? n : (n + 1) / 2, halves = kRowsWaves / ks, step = rows_step_chunks(ks);
            const int steps = (K / 32 + step - 1) / step, blocks = steps * ks;         // of 128 codes
            const bool masked = K / 32 % step != 0;
            double issue = blocks * halves * (2.0 * tg * cb + 22.0 * (tg + cb));
            if (masked) issue += blocks * halves * cb * (eighths ? 17.0 : 6.5);
            const double bytes = (rows + 16.0 * n) * 64 * blocks / (eighths ? 38.0 : 31.0);
            const double x = 0.5 * M * K, w = (double)c16 * K / tiles, xcd = (x * (x + w > 4e6 ? per_xcd : 1) + w) / 650;
            const double us = 2.05 + tiles * (std::max(std::max(bytes, xcd), issue) + 1450 + 258.0 * tg * cb) * 0.00055;
            if (best == 0.0 || us < best) {
                best = us;
                *plan = {false, tb, rows, per_xcd, tg, cb, ks};
                *tiles_out = tiles;
            }
        }
    }
    *us_out = best;
    return best > 0.0;
}

static int rows_cus(int cus) { return cus > 256 ? 256 : cus < 8 ? 8 : cus; }

// Which of the two kernels with whole outputs per workgroup a shape takes, if any.  (Several weights with one input: few rows only.)
// At 9 to 16 rows both would do: gemm_few.hip's where a workgroup has few channels (4096 x 4096 4.0 us, 4.2 here, 1024 x 2816 3.3 and
// 3.5), this one's shorter start from three groups on (12288 x 4096 6.8 here, 7.4 there) and with a long K (11008: 6.9 to 7.1, 7.3 to 8.0).
// One tile per workgroup beats the other kernels' tiles wherever it fits (of 4773 drawn shapes 6 are slower by more than 3 %, none by
// more than 6 %).  A second and third tile pay start and reduction again, so there the two kernels' times are compared.  Taken always, they were
// up to 44 % slower than the other kernels (us, those in brackets: 313 x 14832 x 1024 16.1 (12.1), 1500 x 4608 x 512 15.4 (11.8), 148 x
// 30920 x 1792 23.1 (17.0), 154 x 28768 x 4992 39.9 (33.3), 3072 x 2304 x 8192 64.1 (62.0)) and never, up to 40 % (1024 x 2304 x 1024 9.8
// (15.5), 700 x 4608 x 2048 15.6 (25.3), 148 x 24576 x 8192 38.7 (45.5), 2048 x 1536 x 512 8.4 (10.7)).  Of 2000 drawn shapes with two or three
// tiles the comparison takes the faster kernel or one within 5 % of it in 97 of 100, at worst 17 % off.
bool whole_output_plan(int M, int channel_groups, int K, int compute_units, int weights, bool y_vectors, WholePlan *plan)
{
    if (M <= kSkinnyMaxM && K % 64 == 0 && K > 32768) return false;         // the streaming kernel's, which says what it refuses
    const int cus = rows_cus(compute_units);
    const bool few = few_kernel_applies(M, channel_groups, K, cus);
    const bool rather_rows = M > kSkinnyMaxM && (K > 8192 || channel_groups > 2 * cus);
    int tiles;
    double us;
    if ((!few || rather_rows) && weights == 1 && rows_plan(M, channel_groups, K, cus, plan, &tiles, &us) &&
        (tiles == 1 || M <= 16 || us <= tile_kernels_us(M, channel_groups, K, y_vectors)))
        return true;
    plan->few = few;
    return few;
}

template <int TG, int CB, int KS, bool MASKED>
static sqap_status launch_rows_k(const RowsParams &p, hipStream_t st)
{
    static std::atomic<bool> configured[kMaxDeviceSlots];
    const int dslot = device_slot();
    constexpr int lds = rows_lds(TG, CB, KS);
    static_assert(lds <= 160 * 1024, "");
    if (!configured[dslot].load(std::memory_order_acquire)) {
        SQAP_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_rows_kernel<TG, CB, KS, MASKED>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        configured[dslot].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((gemm_rows_kernel<TG, CB, KS, MASKED>), dim3(8 * p.per_xcd * p.tblocks), dim3(kRowsThreads), lds, st, p);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

template <int TG, int CB, int KS>
static sqap_status launch_rows_m(const RowsParams &p, hipStream_t st)
{
    if (p.chunks % rows_step_chunks(KS) != 0) return launch_rows_k<TG, CB, KS, true>(p, st);
    return launch_rows_k<TG, CB, KS, false>(p, st);
}

template <int TG>
static sqap_status launch_rows_c(const RowsParams &p, int cb, int ks, hipStream_t st)
{
    if (ks == 8) {
        if (cb == 1) return launch_rows_m<TG, 1, 8>(p, st);
        if (cb == 2) return launch_rows_m<TG, 2, 8>(p, st);
        return launch_rows_m<TG, 3, 8>(p, st);
    }
    if (cb == 2) return launch_rows_m<TG, 2, 4>(p, st);
    return launch_rows_m<TG, 3, 4>(p, st);
}

sqap_status launch_whole_outputs(const WholePlan &plan, const uint8_t *Xq, const __half *sx, int M, int K, const RowsWeight *weights, int count,
                                 unsigned long long *error_word, hipStream_t st)
{
    if (plan.few) return launch_few_linear(Xq, sx, M, K, weights, count, error_word, st);
    const int W = 8 * plan.per_xcd, step = rows_step_chunks(plan.k_shares);
    RowsParams p = {};
    p.Xq = Xq;
    p.sx = sx;
    p.error_word = error_word;
    p.M = M;
    p.chunks = K / 32;
    p.c16 = (weights[0].N + 15) / 16;
    p.rows_per_block = plan.rows_per_block;
    p.tblocks = plan.tblocks;
    p.per_xcd = plan.per_xcd;
    p.wg_inv = (uint32_t)((0xffffffffull + W) / W);
    p.tb_inv = 65536 / plan.tblocks + 1;
    p.steps = (p.chunks + step - 1) / step;
    p.w = weights[0];
    switch (plan.token_groups) {
    case 1: return launch_rows_c<1>(p, plan.channel_groups, plan.k_shares, st);
    case 2: return launch_rows_c<2>(p, plan.channel_groups, plan.k_shares, st);
    case 3: return launch_rows_c<3>(p, plan.channel_groups, plan.k_shares, st);
    case 4: return launch_rows_c<4>(p, plan.channel_groups, plan.k_shares, st);
    case 5: return launch_rows_c<5>(p, plan.channel_groups, plan.k_shares, st);
    default: return launch_rows_c<6>(p, plan.channel_groups, plan.k_shares, st);
    }
}

}  // namespace sqap
