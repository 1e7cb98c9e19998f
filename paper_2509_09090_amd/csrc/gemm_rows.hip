// W4A4 linear for a few hundred token rows (and for more where the channels are few): every workgroup owns complete outputs.
//
// At these sizes the output is too small to fill the machine with whole 256 x 256 tiles, and splitting K
// between workgroups costs a chain of global round trips (partial store, flag, reduction) that is longer
// than the arithmetic.  Here nothing crosses a workgroup: a workgroup (one per compute unit, eight
// wavefronts, two per SIMD) owns a block of up to 160 token rows times a short run of 16-channel groups
// over the WHOLE reduction axis.  Wavefront w takes quarter w % 4 of K and half w / 4 of the block's token
// groups; the four wavefronts of a half add their accumulators through LDS at the end.  Two wavefronts per
// SIMD matter: one wavefront issues at most one instruction every four cycles, and the int4 -> int8 widening
// costs about 2.5 vector-ALU instructions per matrix instruction, so a lone wavefront leaves the matrix
// core idle half of the time; with two, one's widening issues beside the other's products.
// Inside a workgroup every token byte is used by exactly one wavefront and every weight byte by two, so
// the main loop has no workgroup barrier:
//   weights   come straight from global memory into registers: the packed layout already is the operand
//             order of v_mfma_i32_16x16x64_i8 (lane l: channel l % 16, 16-byte piece l / 16);
//   tokens    are read with coalesced loads (8 rows x 128 bytes per wavefront load), parked in a slab of
//             LDS that belongs to the wavefront, and read back in operand order (lane l: token l % 16,
//             piece l / 16).  A slab row has a pitch of 144 bytes, which keeps both the row-wise stores
//             and the column-wise reads free of bank conflicts.  The rows of a pair of 16-token groups are
//             overwritten with the next step's rows as soon as the pair's products are issued, and
//             the registers they came from are reloaded for the step after that.
// int4 -> int8 as in the large-M kernel: (x << 4) & 0xF0F0F0F0 and x & 0xF0F0F0F0 give 16 * code for the even
// and the odd codes; both operands are split the same way, so the accumulator is 256 * sum(x * w).
// The price is that every workgroup reads all its token rows for the whole K (they come from the L2,
// which the 32 workgroups of an XCD share).  Up to 16 rows are gemm_few.hip's.
#include "common.h"

namespace sqap {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kRowsMaxAH = 5;          // 16-token groups per wavefront (a block of token rows has twice as many)
constexpr int kRowsMaxA = 2 * kRowsMaxAH;
constexpr int kRowsMaxB = 3;           // 16-channel groups per tile
constexpr int kRowsMaxBFew = 6;        // the same where a wavefront has one token group (AH = 1)
constexpr int rows_max_b(int ah) { return ah == 1 ? kRowsMaxBFew : kRowsMaxB; }
constexpr int kRowsStepCodes = 256;    // codes of K per main-loop step of a wavefront (two MFMA K-blocks of 128)
constexpr int kRowsPitch = 144;        // bytes per slab row: 128 of codes + 16 of padding
constexpr int kRowsSlabBytes = kRowsMaxAH * 16 * kRowsPitch;                           // 11520 per wavefront
constexpr int kRowsReduceBytes = kRowsWaves * kRowsMaxAH * kRowsMaxB * 1024;            // 8 wavefronts x 15 tiles x 1 KiB
constexpr int kRowsLdsBytes = kRowsReduceBytes > kRowsWaves * kRowsSlabBytes ? kRowsReduceBytes : kRowsWaves * kRowsSlabBytes;

struct RowsParams {
    // An argument whose line of 64 bytes is cold is a trip to memory in front of the first load of codes: what a launch
    // with one weight needs lies in the first two lines (spread over three, a launch of 4 to 10 us took 0.1 to 0.3 us longer)
    const uint8_t *Xq;     // [M, K/2] canonical
    const __half *sx;      // [M]
    unsigned long long *error_word;        // of the caller's workspace, nullable: cleared (no wait can fail here)
    int M, K, chunks;
    int c16;               // 16-channel groups in all
    int tblocks;           // blocks of token rows (1, 2, 4, 8 or 16)
    int rows_per_block;    // multiple of 16, at most 16 * kRowsMaxA
    int per_xcd;           // workgroups of an XCD that share its channel groups, per token block
    RowsWeight w;
};

__device__ __forceinline__ void widen16(const v4i p, v4i &lo, v4i &hi)
{
    const v4i mask = {(int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0, (int)0xF0F0F0F0};
    lo = (p << 4) & mask;
    hi = p & mask;
}

// same two-step rounding as the large-M epilogue: two binary32 products, then one rounding to half
typedef float v2f_r __attribute__((ext_vector_type(2)));
typedef _Float16 v2h_r __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t dequant_pair(int acc0, int acc1, float sx_over_256, float sw0, float sw1)
{
    float y0 = ((float)acc0 * sx_over_256) * sw0;
    float y1 = ((float)acc1 * sx_over_256) * sw1;
    asm volatile("" : "+v"(y0), "+v"(y1));
    const v2f_r y = {y0, y1};
    union { v2h_r h; uint32_t u; } r;
    r.h = __builtin_convertvector(y, v2h_r);
    return r.u;
}

// One tile: token rows [row0, row0 + 32 AH), channel groups [c0, c0 + B), all of K.  AH and B are
// compile-time constants: every main-loop iteration then issues the same loads and stores in the same
// order, which lets the compiler give each wait the exact count of younger loads that may stay in flight
// (with loads under run-time conditions it waits for all of them, i.e. for a full memory round trip per
// token group).  Token groups are taken two at a time so that consecutive products go to different
// accumulators, and the next pair's operands are read from LDS before the current pair is multiplied.
// RAGGED: K is any multiple of 32.  The last step then ends inside its 256 codes: token pieces past K are put into the slab as
// zeros (and weight pieces past K are any others), and a wavefront may have no step at all.
template <int AH, int B, bool RAGGED>
__device__ __forceinline__ void rows_tile(const RowsParams &p, uint8_t *smem, int row0, int row_end, int c0)
{
    static_assert(AH >= 1 && AH <= kRowsMaxAH && B >= 1 && B <= rows_max_b(AH), "tile shape");
    constexpr int PAIRS = (AH + 1) / 2;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int kq = wave & 3, th = wave >> 2;
    const int Kh = p.K >> 1;
    const int steps = RAGGED ? (p.K + kRowsStepCodes - 1) / kRowsStepCodes : p.K / kRowsStepCodes;
    const int s_begin = steps * kq / 4, s_end = steps * (kq + 1) / 4;
    // The wavefront takes its steps in rotated order, starting at a step that depends on the workgroup: all
    // workgroups of an XCD read the same token rows, and walking K in step they would all ask the same one
    // or two L2 channels for the same lines at the same time.
    const int own = s_end - s_begin, nst = RAGGED ? max(own, 1) : own, rot = (int)(blockIdx.x >> 3) % nst;
    auto step_of = [&](int i) {                                     // i-th step of this wavefront (i past the end: the last)
        int v = min(i, nst - 1) + rot;
        if (v >= nst) v -= nst;
        return s_begin + v;
    };
    uint8_t *slab = smem + wave * kRowsSlabBytes;
    const int wrow0 = row0 + th * AH * 16;                          // this wavefront's first token row

    // token rows: wavefront load i covers rows 8 i .. 8 i + 7 of the wavefront's rows, 128 bytes of each.  Byte
    // offset of this lane's piece in load i: (wrow0 + 8 i + lane / 8) * Kh + 16 * (lane % 8); rows past M - 1
    // re-read row M - 1 (never stored): one addition and one minimum per load instead of a pointer per load.
    const int lr = lane >> 3, piece = lane & 7;
    const uint32_t xoff0 = (uint32_t)(wrow0 + lr) * (uint32_t)Kh + (RAGGED ? 0 : piece * 16);
    const uint32_t xlimit = (uint32_t)(p.M - 1) * (uint32_t)Kh + (RAGGED ? 0 : piece * 16);
    const uint8_t *xbase = p.Xq;
    auto x_ptr = [&](int i, int step) {           // uniform base + 32-bit lane offset: no 64-bit lane arithmetic
        const uint32_t off = min(xoff0 + (uint32_t)(i * 8) * (uint32_t)Kh, xlimit);
        if (RAGGED) return reinterpret_cast<const v4i *>(xbase + (off + (uint32_t)min(step * 8 + piece, p.chunks - 1) * 16));
        return reinterpret_cast<const v4i *>(xbase + (size_t)step * 128 + off);
    };
    // what goes into the slab of a row piece loaded for `step`
    auto slab_piece = [&](const v4i v, int step) { return !RAGGED || step * 8 + piece < p.chunks ? v : v4i{0, 0, 0, 0}; };
    const int xdst = lr * kRowsPitch + piece * 16;                 // + i * 8 * pitch
    // operand order: lane l reads token l % 16, piece l / 16 (+ 4 for the second K-block of a step)
    const int xfrag = (lane & 15) * kRowsPitch + (lane >> 4) * 16;
    // weights: 16-channel group g = 2 * row group + half; chunk c of a row group sits at (rg * chunks + c) * 512
    // (uniform base per group + one 32-bit lane offset)
    const uint8_t *wbase[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const RowsWeight &w = p.w;
        const int g = c0 + j;
        wbase[j] = w.Wd + (size_t)(g >> 1) * p.chunks * 512 + (g & 1) * 256;
    }
    const uint32_t woff = (uint32_t)(lane >> 4) * 512 + (lane & 15) * 16;

    v4i acc[AH][B];
#pragma unroll
    for (int i = 0; i < AH; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    v4i xr[2 * AH];                   // token rows of step s + 1 in flight
    v4i wr[2][2][B];                  // weights: step s in set s & 1 (used now), step s + 1 in the other; [K-block][group]
    v4i xf[2];                        // operands of the token-group pair about to be multiplied

    auto load_x = [&](int step) {
#pragma unroll
        for (int i = 0; i < 2 * AH; ++i) xr[i] = *x_ptr(i, step);
    };
    auto load_w = [&](int step, auto set_c, auto q_c) {
        constexpr int set = decltype(set_c)::value, q = decltype(q_c)::value;
#pragma unroll
        for (int j = 0; j < B; ++j)
            wr[set][q][j] = RAGGED ? *reinterpret_cast<const v4i *>(wbase[j] + (uint32_t)min(step * 8 + q * 4 + (lane >> 4), p.chunks - 1) * 512 + (lane & 15) * 16)
                                   : *reinterpret_cast<const v4i *>(wbase[j] + (size_t)(step * 8 + q * 4) * 512 + woff);
    };
    auto read_pair = [&](int ip, int q, v4i (&dst)[2]) {
#pragma unroll
        for (int g = 0; g < 2; ++g)
            if (2 * ip + g < AH)
                dst[g] = *reinterpret_cast<const v4i *>(slab + (2 * ip + g) * 16 * kRowsPitch + xfrag + q * 64);
    };

    constexpr std::integral_constant<int, 0> c0_{};
    constexpr std::integral_constant<int, 1> c1_{};
    // prologue: step s_begin goes to the slab, step s_begin + 1 stays in the registers
    load_x(step_of(0));
    load_w(step_of(0), c0_, c0_);
    load_w(step_of(0), c0_, c1_);
    load_w(step_of(1), c1_, c0_);
    load_w(step_of(1), c1_, c1_);
#pragma unroll
    for (int i = 0; i < 2 * AH; ++i) *reinterpret_cast<v4i *>(slab + i * 8 * kRowsPitch + xdst) = slab_piece(xr[i], step_of(0));
    load_x(step_of(1));
    read_pair(0, 0, xf);

    // The i-th step of the wavefront; PAR = i & 1 names the register set that holds the step's weights.
    auto step_body = [&](int i, auto par_c) {
        constexpr int PAR = decltype(par_c)::value;
        constexpr std::integral_constant<int, PAR> cur{};
        const int s1 = step_of(i + 1), s2 = step_of(i + 2);
        (void)s1;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            v4i wl[B], wh[B];
#pragma unroll
            for (int j = 0; j < B; ++j) widen16(wr[PAR][q][j], wl[j], wh[j]);
            // the registers just consumed take the step after next
            if (q == 0) load_w(s2, cur, c0_);
            else load_w(s2, cur, c1_);
#pragma unroll
            for (int ip = 0; ip < PAIRS; ++ip) {
                v4i nx[2];
                if (ip + 1 < PAIRS) read_pair(ip + 1, q, nx);
                else if (q == 0) read_pair(0, 1, nx);
                v4i xl[2], xh[2];
#pragma unroll
                for (int g = 0; g < 2; ++g)
                    if (2 * ip + g < AH) widen16(xf[g], xl[g], xh[g]);
#pragma unroll
                for (int j = 0; j < B; ++j)
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        if (2 * ip + g < AH)
                            acc[2 * ip + g][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wl[j], xl[g], acc[2 * ip + g][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < B; ++j)
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        if (2 * ip + g < AH)
                            acc[2 * ip + g][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wh[j], xh[g], acc[2 * ip + g][j], 0, 0, 0);
                if (q == 1) {
                    // both K-blocks of this pair's rows are consumed: the next step's rows take their place in
                    // the slab and the registers they came from are asked for the step after that
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (4 * ip + r < 2 * AH) {
                            *reinterpret_cast<v4i *>(slab + (4 * ip + r) * 8 * kRowsPitch + xdst) = slab_piece(xr[4 * ip + r], s1);
                            xr[4 * ip + r] = *x_ptr(4 * ip + r, s2);
                        }
                }
                if (ip + 1 < PAIRS || q == 0) {
                    xf[0] = nx[0];
                    xf[1] = nx[1];
                }
            }
        }
        read_pair(0, 0, xf);                         // the next step's first pair (its rows were stored above)
    };
    int i = 0;
    for (; i + 1 < own; i += 2) {
        step_body(i, c0_);
        step_body(i + 1, c1_);
    }
    if (i < own) step_body(i, c0_);

    // add the accumulators of the four wavefronts that share a token half through LDS; wavefront (kq, th)
    // finishes tiles kq, kq + 4, ... of its half
    __syncthreads();                                   // every wavefront is done with its slab
    int *red = reinterpret_cast<int *>(smem);
#pragma unroll
    for (int i = 0; i < AH; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j)
            *reinterpret_cast<v4i *>(red + ((wave * AH * B + i * B + j) * 64 + lane) * 4) = acc[i][j];
    __syncthreads();
    const int tok_in = lane & 15, ch4 = (lane >> 4) * 4;
    for (int tt = kq; tt < AH * B; tt += 4) {
        const int i = tt / B, j = tt - i * B;
        v4i sum = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < 4; ++w)
            sum += *reinterpret_cast<const v4i *>(red + (((th * 4 + w) * AH * B + tt) * 64 + lane) * 4);
        const RowsWeight &w = p.w;
        const bool y_vec = (w.ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(w.Y) & 7u) == 0;
        const bool a_vec = (w.N & 3) == 0 && w.acc_out && (reinterpret_cast<uintptr_t>(w.acc_out) & 15u) == 0;
        const int row = wrow0 + i * 16 + tok_in, col = (c0 + j) * 16 + ch4;
        if (row < row_end && col < w.N) {
            const float sxf = __half2float(p.sx[row]) * 0.00390625f;
            const uint2 swr = *reinterpret_cast<const uint2 *>(w.sw + col);            // zero padded past N
            const __half2 *sw2 = reinterpret_cast<const __half2 *>(&swr);
            const float2 s01 = __half22float2(sw2[0]), s23 = __half22float2(sw2[1]);
            uint2 pk;
            pk.x = dequant_pair(sum.x, sum.y, sxf, s01.x, s01.y);
            pk.y = dequant_pair(sum.z, sum.w, sxf, s23.x, s23.y);
            __half *dst = w.Y + (size_t)row * w.ldy + col;
            if (y_vec && col + 4 <= w.N) {
                *reinterpret_cast<uint2 *>(dst) = pk;
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
    __syncthreads();                                   // LDS is free for the next tile
}

// Workgroup b runs on XCD b % 8 (the hardware deals consecutive workgroups to the XCDs in turn; nothing
// here depends on it for correctness, only for locality).  The 16-channel groups are dealt to the XCDs in
// contiguous runs, and inside an XCD to `per_xcd` workgroups per token block, so that the workgroups that
// read the same weights (one per token block) sit behind one L2.  AH = 16-token groups per wavefront: a
// block has 2 AH of them (rows past the block re-read other rows and are never stored).
template <int AH, bool RAGGED>
__global__ __launch_bounds__(64 * kRowsWaves, 1) void gemm_rows_kernel(const RowsParams p)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    if (blockIdx.x == 0 && threadIdx.x == 0 && p.error_word) *p.error_word = 0ull;
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int tb = j % p.tblocks, slot = j / p.tblocks;
    if (slot >= p.per_xcd) return;
    const int W = 8 * p.per_xcd, i = xcd * p.per_xcd + slot;
    const int g_begin = (int)((long long)p.c16 * i / W), g_end = (int)((long long)p.c16 * (i + 1) / W);
    const int row0 = tb * p.rows_per_block;
    if (row0 >= p.M) return;
    const int row_end = min(p.M, row0 + p.rows_per_block);      // rows past it belong to the next block (or to nobody)
    // tiles of at most MAXB groups, as even as possible (5 -> 3 + 2, 4 -> 2 + 2)
    constexpr int MAXB = rows_max_b(AH);
    const int n = g_end - g_begin, tiles = (n + MAXB - 1) / MAXB;
    for (int k = 0; k < tiles; ++k) {
        const int c0 = g_begin + n * k / tiles, b = g_begin + n * (k + 1) / tiles - c0;
        if constexpr (MAXB > kRowsMaxB) {
            if (b == 6) rows_tile<AH, 6, RAGGED>(p, smem, row0, row_end, c0);
            else if (b == 5) rows_tile<AH, 5, RAGGED>(p, smem, row0, row_end, c0);
            else if (b == 4) rows_tile<AH, 4, RAGGED>(p, smem, row0, row_end, c0);
        }
        if (b > 3) continue;
        if (b == 3) rows_tile<AH, 3, RAGGED>(p, smem, row0, row_end, c0);
        else if (b == 2) rows_tile<AH, 2, RAGGED>(p, smem, row0, row_end, c0);
        else rows_tile<AH, 1, RAGGED>(p, smem, row0, row_end, c0);
    }
}

// Token blocks: as few as hold M, more when the channel groups are too few to give every workgroup a run
// of its own (each workgroup then reads fewer token rows, and the weights are read once per block, the
// second time from the L2).  Cost of a workgroup in clock cycles: what its compute unit loads at 64 bytes
// per cycle against what its matrix cores multiply (a 16 x 16 x 64 product takes 16 cycles on one of four SIMDs).
// The plan with the lowest cost is taken, if a workgroup then has no more channel groups than rows_max_groups allows.
//
// How many groups of 16 channels a workgroup may have for this kernel to be the faster one (us, M x N x K, the other kernel behind
// "against").
// One tile (three groups; six up to 32 rows): always.  148 rows: N = 4096 9.1 against 15.0, N = 12288 15.7 against 20.8, K = 11008
// 15.2 against 22.1; where the 256 x 256 tiles are few or K is no multiple of 128, more: 522 x 1024 x 2816 8.2 against 25.4;
// 2000 x 700 x 5504 19.2 against 46.4; 148 x 2048 x 5504 10.2 against 16.5; 32 x 512 x 512 3.5 against 7.8; 450 x 300 x 4160 9.1
// against 57.
// A second tile reads the token rows again and pays the start-up of the load pipeline again.  Worth it
//   up to 64 rows: 64 x 22016 x 4096 17.5 against 19.7, 16 rows 12.9 against 18.3 (84 rows 21.6 against 20.9: not);
//   against the tiles with a guarded K: 300 x 12288 x 4160 33.9 against 50.7, 1200 x 3000 x 4160 33.1 against 50.6 (not with eight
//   groups at K = 1088: 600 x 8000 25.4 against 17.8);
//   four groups from 512 rows on: 600 x 4096 x 4096 23.4 against 31.2, 2368 x 1024 x 4096 25.1 against 31.3;
// not between otherwise (276 x 8192 x 4096 23.0 against 19.7), nor with a K too short to make up for a start-up (600 x 4096 x 512
// 12.4 against 11.0).
// Both sides compared on 800 drawn shapes (1 to 2600 rows, 16 to 60000 channels, K of 32 to 16384) and 120 groups: fifteen shapes more
// than 2 % slower with this rule than with the kernels they had before it, by up to 0.3 us at 3 to 8 us (5 % at one), 447 more than
// 2 % faster.
static int rows_max_groups(int M, int K)
{
    if (M <= 32) return M <= kSkinnyMaxM || K >= 1024 ? 2 * kRowsMaxBFew : kRowsMaxB;
    if (K < 1024) return kRowsMaxB;
    if (M <= 64) return 2 * kRowsMaxB;
    if (M > 160 && K % 128 != 0 && K >= 2048) return 2 * kRowsMaxB;
    return M >= 512 ? 4 : kRowsMaxB;
}

static bool rows_plan(int M, int c16, int K, int cus, RowsParams *p)
{
    if (K % 32 != 0 || c16 < 1) return false;
    const int max_groups = rows_max_groups(M, K);
    double best = 0.0;
    for (int tb = 1; tb <= 16; tb *= 2) {
        const int rows = ((M + tb - 1) / tb + 15) / 16 * 16;
        if (rows > 16 * kRowsMaxA) continue;
        const int a = (rows / 16 + 1) & ~1;                     // two wavefront halves of equal size
        int per_xcd = (cus / 8) / tb;
        if (per_xcd < 1) per_xcd = 1;
        const int W = 8 * per_xcd;
        const int n = (c16 + W - 1) / W;
        if (n > max_groups) continue;
        const double bytes = (a * 16.0 + 2 * 16.0 * n) * (K / 2);
        const double mfma = (double)a * n * (K / 128) * 2 * 16 / 4;
        const double cost = std::max(bytes / 64.0, mfma / 0.7);
        if (best == 0.0 || cost < best) {
            best = cost;
            p->tblocks = tb;
            p->rows_per_block = rows;
            p->per_xcd = per_xcd;
        }
    }
    p->c16 = c16;
    return best > 0.0;
}

static int rows_cus(int cus) { return cus > 256 ? 256 : cus < 8 ? 8 : cus; }

// Shapes that this kernel or the one for few rows takes: up to sixteen blocks of 160 token rows, and few enough channels per
// workgroup.  (Several weights with one input: few rows only.)
bool rows_kernel_applies(int M, int channel_groups, int K, int compute_units, int weights)
{
    if (M <= kSkinnyMaxM && K % 64 == 0 && K > 32768) return false;         // the streaming kernel's, which says what it refuses
    if (few_kernel_applies(M, channel_groups, K, compute_units)) return true;
    RowsParams p = {};
    return weights == 1 && rows_plan(M, channel_groups, K, rows_cus(compute_units), &p);
}

template <int AH, bool RAGGED>
static sqap_status launch_rows_k(const RowsParams &p, int blocks, hipStream_t st)
{
    static std::atomic<bool> configured[kMaxDeviceSlots];
    const int dslot = device_slot();
    if (!configured[dslot].load(std::memory_order_acquire)) {
        SQAP_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_rows_kernel<AH, RAGGED>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kRowsLdsBytes));
        configured[dslot].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((gemm_rows_kernel<AH, RAGGED>), dim3(blocks), dim3(64 * kRowsWaves), kRowsLdsBytes, st, p);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

template <int AH>
static sqap_status launch_rows_a(const RowsParams &p, int blocks, hipStream_t st)
{
    const bool ragged = p.K % kRowsStepCodes != 0 || p.K / kRowsStepCodes < 4;
    return ragged ? launch_rows_k<AH, true>(p, blocks, st) : launch_rows_k<AH, false>(p, blocks, st);
}

sqap_status launch_rows_linear(const uint8_t *Xq, const __half *sx, int M, int K, const RowsWeight *weights, int count,
                               unsigned long long *error_word, hipStream_t st)
{
    int groups = 0;
    for (int i = 0; i < count; ++i) groups += (weights[i].N + 15) / 16;
    if (few_kernel_applies(M, groups, K, device_cu_count())) return launch_few_linear(Xq, sx, M, K, weights, count, error_word, st);
    RowsParams p = {};
    p.Xq = Xq;
    p.sx = sx;
    p.M = M;
    p.K = K;
    p.chunks = K / 32;
    p.error_word = error_word;
    p.w = weights[0];
    if (!rows_plan(M, groups, K, rows_cus(device_cu_count()), &p))
        return fail(SQAP_EUNSUPPORTED, "sqap_w4a4_linear: M = %d, %d channels, K = %d outside the row kernel's range", M, groups * 16, K);
    const int blocks = 8 * p.per_xcd * p.tblocks;
    const int ah = (p.rows_per_block / 16 + 1) / 2;             // token groups per wavefront
    switch (ah) {
    case 1: return launch_rows_a<1>(p, blocks, st);
    case 2: return launch_rows_a<2>(p, blocks, st);
    case 3: return launch_rows_a<3>(p, blocks, st);
    case 4: return launch_rows_a<4>(p, blocks, st);
    default: return launch_rows_a<5>(p, blocks, st);
    }
}

}  // namespace sqap
