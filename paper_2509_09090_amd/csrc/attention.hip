// Causal softmax attention on the matrix cores, for head sizes 64 and 128.
#include "common.h"

namespace sqap {

// One workgroup: NQ query groups of 32 x NK key groups, one wavefront each; key and value tiles of 32 NK keys pass
// through LDS (two buffers, filled by global -> LDS loads that stay in flight while the other buffer is worked on)
// and are read by all the query groups; key group g takes keys 32 g .. of every tile, and the key groups'
// partial results are merged once at the end.  Everything is kept transposed so that no accumulator changes lanes:
//   S^T = K Q^T      v_mfma_f32_32x32x16_f16, A = 32 key rows, B = 32 query rows: lane l holds query l % 32,
//                    register i key 8 (i / 4) + 4 (l / 32) + i % 4;
//   softmax          over registers and the two lane halves;
//   O^T += V^T P^T   registers 8n .. 8n + 7 of P, converted to half, ARE the B operand of 16 keys (8 of them per lane
//                    half, in the order 16n + 4 (l / 32) + 0..3, 16n + 8 + 4 (l / 32) + 0..3); A = V^T comes from the
//                    row-major value tile by two transposing reads (ds_read_b64_tr_b16: a lane gets 4 keys of its column).
// A tile row is 2 D bytes without padding (the loads write 1 KiB per wavefront, contiguous); its 16-byte pieces are
// permuted (piece p of row r at p ^ swizzle(r)) so that both the 16-byte key reads (16 rows, one piece) and the
// transposing reads (4 rows, 4 pieces) touch every bank once (counters: no bank conflicts).
// Probabilities enter the second product as two halves (p = hi + lo, 22 bits): with one half each the result was 2.4e-4
// off (2-norm, 1024 queries x 2048 keys), with two 2.07e-4, which is the rounding of the output; the second set of
// products costs 10 % at that size.  That also makes the running maximum free to lag: it is only raised when
// a score exceeds it by more than 2^6 (scores are in units of ln 2), so O^T (64 registers) is seldom rescaled.
// What bounds it: not the loads (three or four buffers instead of two: no faster) nor any one unit (at 1024 x 2048 the
// matrix cores are busy in 45 % of the cycles in which a compute unit has work, the vector ALU in 45 %, LDS in 16 %; no bank conflicts), but
// the chain key reads -> products -> softmax -> products of a wavefront with two
// wavefronts per SIMD to fill it; having all LDS reads of a step in flight at once gave 12 %, addresses as a uniform base
// and a lane offset 15 %.  Slower: 64 keys per wavefront and step (the same at two waves per SIMD, worse with fewer),
// four or eight query groups on one tile, half of the key groups running half a step behind the others.
// Finding out whether outputs are finite and agreeing on it takes 0.1 to 0.2 us of a workgroup (16 x 148 x 148 22.7 without, 23.6 with,
// 1024 x 2048 50.7 and 51.0; a second time through the keys doubles a workgroup's time).  Heads of 64 are held to the 128 registers that
// four wavefronts per SIMD leave, which the second time through would pass (16 x 274 x 274, 32 heads 26.6, with 137 registers 28.0).
// Measured (us; the kernel before, one key tile per wavefront and 2-byte transposing reads, in brackets; heads of 128):
// 16 x 148 x 148, 32 heads 23.2 (62.8); 1024 x 2048, 32 heads 46.6 (126); 148 x 148, 32 heads 6.5 (8.2); 84 x 84 5.5 (6.2).
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));

constexpr float kRaiseBy = 6.0f;

// p - (half I of h), exact: one mixed-precision multiply-add instead of a conversion and a subtraction
template <int I>
__device__ __forceinline__ float remainder_of(const v2h h, float p)
{
    float r;
    if (I == 0) asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(p));
    else asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(p));
    return r;
}

template <int D>
__device__ __forceinline__ int swizzle(int r)
{
    if (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);             // 16 pieces per row, a row is all 64 banks
    return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);                    // 8 pieces per row, two rows are all banks
}

// two buffers of NK * 32 key rows and value rows; the merge reuses them for a (maximum, sum) pair per lane and the
// column tiles that a wavefront does not own, and a word behind these
template <int D, int NQ, int NK>
constexpr int merge_bytes() { return NQ * NK * 512 + NQ * NK * (NK - 1) * (D / 32 / NK) * 4096; }

template <int D, int NQ, int NK>
constexpr int attention_lds_bytes()
{
    const int tiles = 2 * NK * 32 * 2 * (2 * D), merge = merge_bytes<D, NQ, NK>() + 16;
    return tiles > merge ? tiles : merge;
}

// two halves: those of b where a's are not finite
__device__ __forceinline__ unsigned where_not_finite(unsigned a, unsigned b)
{
    const unsigned lo = (a & 0x7c00u) == 0x7c00u ? b : a, hi = (a & 0x7c000000u) == 0x7c000000u ? b : a;
    return (lo & 0xffffu) | (hi & 0xffff0000u);
}

// The A operands of 32 keys: per 16 keys and column tile two transposing reads (keys +0..3 and +8..11 of this lane half).
// lane_v: this lane's offsets in a tile's first 16 rows.  Written out because the compiler waits for every load in flight
// that lands in LDS (the next tile's) in front of the builtin; the wait for the reads is part of the block.
template <int D>
__device__ __forceinline__ void read_values(unsigned at, const unsigned (&lane_v)[2 * (D / 32)], v8h (&va)[2][D / 32])
{
    constexpr int NEXT = 16 * 2 * D;                                  // 16 rows on
    union Frag { struct { v2i lo, hi; } p; v8h v; } r[2][D / 32];
    if constexpr (D == 128)
        asm volatile("ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %17\n\tds_read_b64_tr_b16 %2, %18\n\tds_read_b64_tr_b16 %3, %19\n\t"
                     "ds_read_b64_tr_b16 %4, %20\n\tds_read_b64_tr_b16 %5, %21\n\tds_read_b64_tr_b16 %6, %22\n\tds_read_b64_tr_b16 %7, %23\n\t"
                     "ds_read_b64_tr_b16 %8, %16 offset:%24\n\tds_read_b64_tr_b16 %9, %17 offset:%24\n\tds_read_b64_tr_b16 %10, %18 offset:%24\n\t"
                     "ds_read_b64_tr_b16 %11, %19 offset:%24\n\tds_read_b64_tr_b16 %12, %20 offset:%24\n\tds_read_b64_tr_b16 %13, %21 offset:%24\n\t"
                     "ds_read_b64_tr_b16 %14, %22 offset:%24\n\tds_read_b64_tr_b16 %15, %23 offset:%24\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(r[0][0].p.lo), "=&v"(r[0][0].p.hi), "=&v"(r[0][1].p.lo), "=&v"(r[0][1].p.hi),
                       "=&v"(r[0][2].p.lo), "=&v"(r[0][2].p.hi), "=&v"(r[0][3].p.lo), "=&v"(r[0][3].p.hi),
                       "=&v"(r[1][0].p.lo), "=&v"(r[1][0].p.hi), "=&v"(r[1][1].p.lo), "=&v"(r[1][1].p.hi),
                       "=&v"(r[1][2].p.lo), "=&v"(r[1][2].p.hi), "=&v"(r[1][3].p.lo), "=&v"(r[1][3].p.hi)
                     : "v"(at + lane_v[0]), "v"(at + lane_v[1]), "v"(at + lane_v[2]), "v"(at + lane_v[3]), "v"(at + lane_v[4]),
                       "v"(at + lane_v[5]), "v"(at + lane_v[6]), "v"(at + lane_v[7]), "n"(NEXT)
                     : "memory");
    else
        asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %9\n\tds_read_b64_tr_b16 %2, %10\n\tds_read_b64_tr_b16 %3, %11\n\t"
                     "ds_read_b64_tr_b16 %4, %8 offset:%12\n\tds_read_b64_tr_b16 %5, %9 offset:%12\n\tds_read_b64_tr_b16 %6, %10 offset:%12\n\t"
                     "ds_read_b64_tr_b16 %7, %11 offset:%12\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(r[0][0].p.lo), "=&v"(r[0][0].p.hi), "=&v"(r[0][1].p.lo), "=&v"(r[0][1].p.hi),
                       "=&v"(r[1][0].p.lo), "=&v"(r[1][0].p.hi), "=&v"(r[1][1].p.lo), "=&v"(r[1][1].p.hi)
                     : "v"(at + lane_v[0]), "v"(at + lane_v[1]), "v"(at + lane_v[2]), "v"(at + lane_v[3]), "n"(NEXT)
                     : "memory");
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int ct = 0; ct < D / 32; ++ct) va[n][ct] = r[n][ct].v;
}

// The queries of a workgroup over all their keys: this wavefront's column tiles (OWN of them), as pairs of halves.
// FIRST: the fast way, with two assumptions.  Values are finite: an infinite one times the low half of a probability, which is
// zero or negative as often as not, is NaN where the probability times the value is infinite.  And scores are below 2^24 in
// units of ln 2: the maximum is a rounded product, the scores it is taken from are not, and beyond that the difference, which
// should be zero at the largest, is off by more than 1: the sum of the probabilities, at least 1 otherwise, is then below 1/2, or
// a probability overflows.  Where an assumption fails outputs are not finite, and the result is true (for a lane of them).  Not FIRST:
// one half per probability, rounded products, and zeros for the values past the last key, for which neither matters; no
// probability of a key that is seen, and no factor, is zero there, so that an infinite value stays one however small its weight
// (probabilities are 2^9 times as large: the smallest half adds 2^-33 of the largest).  In a tile of which some query does not see every
// key, values that are not finite take no part in the products, where they would be NaN times that query's zero (add_not_finite).
template <int D, int NQ, int NK, bool FIRST>
__device__ __forceinline__ bool attend(uint8_t *lds, int l, int wave, int qblock, const __half *__restrict__ Q, int64_t ldq,
                                        const __half *__restrict__ Kc, int64_t ldk, const __half *__restrict__ V, int64_t ldv,
                                        int Sq, int Sk, unsigned (&w)[D / 32 / NK][8])
{
    constexpr int NP = D / 16, CT = D / 32, TK = 32, TILE = NK * TK, ROW = 2 * D, PIECES = D / 8;
    constexpr int BUF = TILE * 2 * ROW;                               // keys, then values
    constexpr int RPI = 1024 / ROW;                                   // rows per wavefront load
    constexpr int WAVES = NQ * NK, LOADS_PER_WAVE = 2 * TILE / RPI / WAVES;
    static_assert(WAVES % 4 == 0 && (TILE / RPI) % WAVES == 0, "every wavefront asks for the same number of pieces");
    static_assert(NK > 1 && CT % NK == 0, "the key groups share the output's column tiles");
    const int c = l & 31, h = l >> 5;
    const int kg = wave / NQ, qg = wave % NQ;
    const int q0 = (qblock * NQ + qg) * 32;
    const int shift = Sk - Sq, my_q = q0 + c;
    const int block_last = min(Sk - 1, min((qblock + 1) * NQ * 32 - 1, Sq - 1) + shift);
    const int last_key = q0 < Sq ? min(q0 + 31, Sq - 1) + shift : -1; // of this wavefront
    const int n_iter = block_last / TILE + 1;

    // the next tile, global -> LDS: lane l fetches the piece that belongs at its place.  The wavefronts are a multiple of
    // four, so a lane's piece and its row within a load are the same for all its loads: a uniform base and a lane offset
    const int lr = l / PIECES, lp = ((l % PIECES) ^ swizzle<D>(wave * RPI + lr)) * 8;
    const int64_t koff = lr * ldk + lp, voff = lr * ldv + lp;
    auto issue_rows = [&](const __half *__restrict__ base, int64_t ld, int64_t off, int it, int at) {
        if ((it + 1) * TILE <= Sk) {
            const __half *from = base + (int64_t)(it * TILE + wave * RPI) * ld;
#pragma unroll
            for (int i = 0; i < LOADS_PER_WAVE / 2; ++i) {
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) v4i *)(from + off),
                                                 (__attribute__((address_space(3))) void *)(lds + at + (wave + i * WAVES) * 1024), 16, 0, 0);
                from += WAVES * RPI * ld;
            }
        } else {                                                      // rows past the end repeat the last one
#pragma unroll
            for (int i = 0; i < LOADS_PER_WAVE / 2; ++i) {
                const int64_t key = min(it * TILE + (wave + i * WAVES) * RPI + lr, Sk - 1);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) v4i *)(base + key * ld + lp),
                                                 (__attribute__((address_space(3))) void *)(lds + at + (wave + i * WAVES) * 1024), 16, 0, 0);
            }
        }
    };
    auto issue = [&](int it) {
        if (it < n_iter) {
            issue_rows(Kc, ldk, koff, it, (it & 1) * BUF);
            issue_rows(V, ldv, voff, it, (it & 1) * BUF + TILE * ROW);
        }
    };
    issue(0);

    v8h qf[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) {
        qf[m] = v8h{};
        if (my_q < Sq) qf[m] = *reinterpret_cast<const v8h *>(Q + (int64_t)my_q * ldq + 16 * m + 8 * h);
    }
    v16f ot[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) ot[ct][i] = 0.f;
    float mrun = -INFINITY, lrun = 0.f;                               // lrun: this lane half's keys only
    const float scale = 1.4426950408889634f / sqrtf((float)D);

    // V^T: lanes 16j .. 16j + 15 read 4 key rows x 16 columns
    const unsigned lds_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)lds;
    unsigned lane_v[2 * CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int r = 8 * b + 4 * h + ((l & 15) >> 2), piece = 4 * ct + 2 * ((l >> 4) & 1) + ((l & 3) >> 1);
            lane_v[2 * ct + b] = r * ROW + ((piece ^ swizzle<D>(r)) << 4) + ((l & 1) << 3);
        }

    int lane_k[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) lane_k[m] = c * ROW + (((2 * m + h) ^ swizzle<D>(c)) << 4);

    auto factor = [](float x) __attribute__((always_inline)) {
        const float f = __builtin_amdgcn_exp2f(x);
        return !FIRST && f < 0x1p-100f ? 0x1p-100f : f;               // (NaN stays)
    };
    auto probability = [&](float s, float m) __attribute__((always_inline)) {
        if (FIRST) return __builtin_amdgcn_exp2f(fmaf(s, scale, -m));
        const float p = __builtin_amdgcn_exp2f((s * scale - m) + 9.f);
        return p < 0x1p-24f && s > -INFINITY ? 0x1p-24f : p;
    };
    v16f st;
    auto scores = [&](int it) {
        const int key_tile = (it & 1) * BUF + kg * TK * ROW;
        v8h kf[NP];
#pragma unroll
        for (int m = 0; m < NP; ++m) kf[m] = *reinterpret_cast<const v8h *>(lds + key_tile + lane_k[m]);
        __builtin_amdgcn_sched_barrier(0);                            // (all of them in flight before the first product)
#pragma unroll
        for (int i = 0; i < 16; ++i) st[i] = 0.f;
#pragma unroll
        for (int m = 0; m < NP; ++m) st = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[m], qf[m], st, 0, 0, 0);
    };
    auto softmax_and_values = [&](int it) {
        const int k0 = it * TILE + kg * TK;
        // the values arrive while the products above are worked on
        v8h va[2][CT];
        read_values<D>(lds_base + (it & 1) * BUF + (TILE + kg * TK) * ROW, lane_v, va);
        if (k0 + TK - 1 > q0 + shift) {                               // the diagonal passes through this tile
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (k0 + 8 * (i >> 2) + 4 * h + (i & 3) > my_q + shift) st[i] = -INFINITY;
            if (!FIRST) {
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        union { v8h v; unsigned u[4]; } x;
                        x.v = va[n][ct];
#pragma unroll
                        for (int p = 0; p < 4; ++p) x.u[p] = where_not_finite(x.u[p], 0u);
                        va[n][ct] = x.v;
                    }
            }
        }
        float tmax = st[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, st[i]);
        const auto other = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
        tmax = fmaxf(__uint_as_float(other[0]), __uint_as_float(other[1])) * scale;
        if (__any(tmax > mrun + kRaiseBy)) {
            const float m_new = fmaxf(mrun, tmax);
            const float f = m_new == -INFINITY ? 1.f : factor(mrun - m_new);
            mrun = m_new;
            lrun *= f;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int i = 0; i < 16; ++i) ot[ct][i] *= f;
        }
        const float m_sub = mrun == -INFINITY ? 0.f : mrun;           // (a query that sees none of this group's keys so far)
        v8h ph[2], pl[2];
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float p0 = probability(st[i], m_sub), p1 = probability(st[i + 1], m_sub);
            lrun += p0 + p1;
            const v2h pk = {(_Float16)p0, (_Float16)p1};
            const v2h pr = {(_Float16)remainder_of<0>(pk, p0), (_Float16)remainder_of<1>(pk, p1)};
            ph[i >> 3][i & 7] = pk[0];
            ph[i >> 3][(i & 7) + 1] = pk[1];
            pl[i >> 3][i & 7] = pr[0];
            pl[i >> 3][(i & 7) + 1] = pr[1];
        }
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                ot[ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[n][ct], ph[n], ot[ct], 0, 0, 0);
                if (FIRST) ot[ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[n][ct], pl[n], ot[ct], 0, 0, 0);
            }
    };

    for (int it = 0; it < n_iter; ++it) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // this wavefront's part of tile `it` has landed
        lds_barrier();                                                // everybody's has; the other buffer is free
        if (!FIRST && (it + 1) * TILE > Sk) {                         // zeros instead of the last value row's repetitions
            for (int r = Sk - it * TILE + threadIdx.x / PIECES; r < TILE; r += 64 * WAVES / PIECES)
                *reinterpret_cast<uint4 *>(lds + (it & 1) * BUF + (TILE + r) * ROW + 16 * (threadIdx.x % PIECES)) = make_uint4(0u, 0u, 0u, 0u);
            lds_barrier();
        }
        issue(it + 1);
        if (it * TILE + kg * TK <= last_key) {
            scores(it);
            softmax_and_values(it);
        }
    }
    const auto lo = __builtin_amdgcn_permlane32_swap(__float_as_uint(lrun), __float_as_uint(lrun), false, false);
    lrun = __uint_as_float(lo[0]) + __uint_as_float(lo[1]);

    // merge of the key groups: group g collects column tiles g * CT / NK .. from the others
    constexpr int OWN = CT / NK;
    float *ml = reinterpret_cast<float *>(lds);                       // [wave][64] pairs (maximum, sum)
    float *pieces = ml + WAVES * 128;
    __syncthreads();                                                  // the tiles are no longer needed
    ml[(wave * 64 + l) * 2] = mrun;
    ml[(wave * 64 + l) * 2 + 1] = lrun;
    if (threadIdx.x == 0) *reinterpret_cast<int *>(lds + merge_bytes<D, NQ, NK>()) = 0;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int owner = ct / OWN;
        if (owner != kg) {
            float *dst = pieces + (((qg * NK + owner) * (NK - 1) + (kg < owner ? kg : kg - 1)) * OWN + ct % OWN) * 1024;
#pragma unroll
            for (int i = 0; i < 16; ++i) dst[i * 64 + l] = ot[ct][i];
        }
    }
    __syncthreads();
    float mall = -INFINITY, f[NK];
#pragma unroll
    for (int g = 0; g < NK; ++g) mall = fmaxf(mall, ml[((g * NQ + qg) * 64 + l) * 2]);
    float lall = 0.f;
#pragma unroll
    for (int g = 0; g < NK; ++g) {
        const float mg = ml[((g * NQ + qg) * 64 + l) * 2];
        f[g] = mg == -INFINITY ? 0.f : factor(mg - mall);
        lall += ml[((g * NQ + qg) * 64 + l) * 2 + 1] * f[g];
    }
    const float f_own = mrun == -INFINITY ? 0.f : factor(mrun - mall);
    const float inv_l = !FIRST || lall >= 0.5f ? 1.0f / lall : NAN;
    float zero[4] = {};                                               // NaN with the first output that is not finite
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        if (ct / OWN != kg) continue;
#pragma unroll
        for (int i = 0; i < 16; ++i) ot[ct][i] *= f_own;
#pragma unroll
        for (int g = 0; g < NK; ++g)
            if (g != kg) {
                const float *src = pieces + (((qg * NK + kg) * (NK - 1) + (g < kg ? g : g - 1)) * OWN + ct % OWN) * 1024;
#pragma unroll
                for (int i = 0; i < 16; ++i) ot[ct][i] = fmaf(src[i * 64 + l], f[g], ot[ct][i]);
            }
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            union { __half2 v; unsigned u; } pk;
            pk.v = __floats2half2_rn(ot[ct][i] * inv_l, ot[ct][i + 1] * inv_l);
            w[ct % OWN][i >> 1] = pk.u;
            zero[(i >> 1) & 3] = __builtin_amdgcn_fdot2(__builtin_bit_cast(v2h, pk.u), v2h{0, 0}, zero[(i >> 1) & 3], false);
        }
    }
    return my_q < Sq && (zero[0] + zero[1]) + (zero[2] + zero[3]) != 0.f;
}

// The infinities and NaN that attend<.., false> leaves out, to the outputs of the queries that see them: values at keys `from` .. `to`, of which
// this lane's query (its row Q) sees those up to `sees`.  V: this wavefront's columns.  A key whose score is -infinity has no weight: NaN.
template <int D, int OWN>
__device__ __forceinline__ void add_not_finite(unsigned (&w)[OWN][8], const __half *Q, const __half *Kc, int64_t ldk, const __half *V, int64_t ldv,
                                            int from, int to, int sees, int h)
{
    for (int key = from; key <= to; ++key) {
        unsigned x[OWN * 8];
        bool any = false;
#pragma unroll
        for (int i = 0; i < OWN * 4; ++i) {                           // columns 8 i + 4 h ..: register quad i % 4 of column tile i / 4
            const uint2 four = *reinterpret_cast<const uint2 *>(V + key * ldv + 8 * i + 4 * h);
            x[2 * i] = four.x;
            x[2 * i + 1] = four.y;
            any = any || where_not_finite(four.x, 0u) != four.x || where_not_finite(four.y, 0u) != four.y;
        }
        if (!any || key > sees) continue;
        float score = 0.f;
        for (int i = 0; i < D; ++i) score = fmaf(__half2float(Q[i]), __half2float(Kc[key * ldk + i]), score);
        const float weight = score == -INFINITY ? 0.f : 1.f;
#pragma unroll
        for (int i = 0; i < OWN * 8; ++i) {
            union { unsigned u; _Float16 f[2]; } value, out;
            value.u = x[i];
            out.u = w[i >> 3][i & 7];
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (!(fabsf((float)value.f[e]) < INFINITY)) out.f[e] = (_Float16)((float)out.f[e] + (float)value.f[e] * weight);
            w[i >> 3][i & 7] = out.u;
        }
    }
}

template <int D, int NQ, int NK, bool ROUNDS>
__global__ __launch_bounds__(64 * NQ * NK, D == 64 ? 4 : 2) void attention_tiles_kernel(const __half *__restrict__ Q, int64_t ldq,
                                                              const __half *__restrict__ Kc, int64_t ldk,
                                                              const __half *__restrict__ V, int64_t ldv, int Sq, int Sk,
                                                              __half *__restrict__ O, int64_t ldo, int round)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    constexpr int OWN = D / 32 / NK;
    const int l = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int rank = blockIdx.y;                                            // 0: the longest rows
    if (ROUNDS) {                                                     // every other round of the launch the other way about (launch_tiles)
        const int n = (gridDim.y + round - 1) / round, r = rank / round;
        if ((n - 1 - r) & 1) rank = (2 * r + 1) * round - 1 - rank;
    }
    const int qblock = gridDim.y - 1 - rank;
    Q += (int64_t)blockIdx.z * Sq * ldq + (int64_t)blockIdx.x * D;
    Kc += (int64_t)blockIdx.z * Sk * ldk + (int64_t)blockIdx.x * D;
    V += (int64_t)blockIdx.z * Sk * ldv + (int64_t)blockIdx.x * D;
    unsigned w[OWN][8];
    const bool bad = attend<D, NQ, NK, true>(lds, l, wave, qblock, Q, ldq, Kc, ldk, V, ldv, Sq, Sk, w);
    // If any wavefront has outputs that are not finite, the workgroup goes through its keys again and takes those from there.  (Nothing
    // has been stored yet: the queries may lie where the output goes.)
    int *again = reinterpret_cast<int *>(lds + merge_bytes<D, NQ, NK>());
    if (__any(bad) && l == 0) *again = 1;
    lds_barrier();
    if (*again != 0) {
        int l1 = l;
        asm volatile("" : "+v"(l1));                                  // (nothing of the first time is kept in registers for this)
        lds_barrier();                                                // everybody has read it: the tiles come back
        unsigned w1[OWN][8];
        attend<D, NQ, NK, false>(lds, l1, wave, qblock, Q, ldq, Kc, ldk, V, ldv, Sq, Sk, w1);
        const int q0 = (qblock * NQ + wave % NQ) * 32, q = q0 + (l1 & 31), shift = Sk - Sq;
        add_not_finite<D, OWN>(w1, Q + (int64_t)min(q, Sq - 1) * ldq, Kc, ldk, V + 32 * (wave / NQ) * OWN, ldv, (q0 + shift + 1) / 32 * 32,
                               min(q0 + 31, Sq - 1) + shift, q < Sq ? q + shift : -1, l1 >> 5);
        lds_barrier();                                                // (before anybody stores over queries that others read there)
#pragma unroll
        for (int t = 0; t < OWN; ++t)
#pragma unroll
            for (int i = 0; i < 8; ++i) w[t][i] = where_not_finite(w[t][i], w1[t][i]);
    }
    const int h = l >> 5, my_q = (qblock * NQ + wave % NQ) * 32 + (l & 31);
    O += (int64_t)blockIdx.z * Sq * ldo + (int64_t)blockIdx.x * D + (int64_t)my_q * ldo + 32 * (wave / NQ) * OWN;
#pragma unroll
    for (int t = 0; t < OWN; ++t) {
        // four consecutive columns per register quad; two quads make 16 bytes once the lane halves have exchanged
#pragma unroll
        for (int g = 0; g < 4; g += 2) {
            const auto a = __builtin_amdgcn_permlane32_swap(w[t][2 * g], w[t][2 * g + 2], false, false);
            const auto b = __builtin_amdgcn_permlane32_swap(w[t][2 * g + 1], w[t][2 * g + 3], false, false);
            if (my_q < Sq) *reinterpret_cast<uint4 *>(O + 32 * t + 8 * g + 8 * h) = make_uint4(a[0], b[0], a[1], b[1]);
        }
    }
}

template <int D, int NQ, int NK, bool ROUNDS = false>
static sqap_status launch_tiles(const __half *Q, int64_t ldq, const __half *Kc, int64_t ldk, const __half *V, int64_t ldv,
                                int batch, int Sq, int Sk, int H, __half *O, int64_t ldo, hipStream_t st, int round = 0)
{
    constexpr int bytes = attention_lds_bytes<D, NQ, NK>();
    static_assert(bytes <= 160 * 1024, "LDS of a compute unit");
    if constexpr (bytes > 48 * 1024) {
        static std::atomic<bool> allowed[kMaxDeviceSlots];
        const int slot = device_slot();
        if (!allowed[slot].load(std::memory_order_acquire)) {
            SQAP_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&attention_tiles_kernel<D, NQ, NK, ROUNDS>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
            allowed[slot].store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL((attention_tiles_kernel<D, NQ, NK, ROUNDS>), dim3(H, (Sq + 32 * NQ - 1) / (32 * NQ), batch), dim3(64 * NQ * NK), bytes, st,
                       Q, ldq, Kc, ldk, V, ldv, Sq, Sk, O, ldo, round);
    SQAP_HIP_CHECK(hipGetLastError());
    return SQAP_OK;
}

// Which form: two query groups x two key groups share a tile of 64 keys (two workgroups of four wavefronts per compute unit,
// their barriers independent of each other).  Where that leaves compute units without a workgroup, i.e. at most one query
// group per compute unit, and there are keys enough for more than one round (from 192 on: at 149 keys the two take the
// same time), one query group x four key groups.  Measured, us (batch x queries x keys, heads of 128; first form / second):
//   1x84x1000, 32 heads 19.7 / 14.7;  1x1024x1024, 8 heads 19.2 / 14.3;  1x64x384, 32 heads 9.6 / 7.7;
//   1x1x149, 32 heads 6.0 / 5.8;  1x148x148, 32 heads 6.3 / 6.5;  1x400x400, 32 heads 10.5 / 12.4;
//   16x148x148, 32 heads 22.2 / 49.3;  1x1024x2048, 32 heads 48.5 / 71.3.
// The second form needs four column tiles to share out: heads of 64 stay with the first, few queries over many keys among them
// (us, with four wavefronts along the keys and no sharing in brackets: 1x10x1341, 1 head 16.1 (17.6); 2x2x2917, 8 heads 32.9 (34.4);
// 1x7x2506, 32 heads 29.0 (30.6); 1x25x554, 8 heads 8.6 (10.0)).
sqap_status launch_attention_tiles(const __half *Q, int64_t ldq, const __half *Kc, int64_t ldk, const __half *V, int64_t ldv,
                                   int batch, int Sq, int Sk, int H, int d, __half *O, int64_t ldo, hipStream_t st)
{
    if (d == 64) return launch_tiles<64, 2, 2>(Q, ldq, Kc, ldk, V, ldv, batch, Sq, Sk, H, O, ldo, st);
    const int64_t groups = (int64_t)batch * H * ((Sq + 31) / 32);
    if (groups <= device_cu_count() && Sk >= 192)
        return launch_tiles<128, 1, 4>(Q, ldq, Kc, ldk, V, ldv, batch, Sq, Sk, H, O, ldo, st);
    // Later query blocks see more keys.  Where more blocks come than compute units have room for, the longest go first.  Where all
    // find room at once, one or two per compute unit, their order says which share a unit: the first round of them goes from short to
    // long, the second from long to short, so that long meets short, and where the second is not full the longest have a unit to
    // themselves.  32 heads unless said, us, both rounds from long to short in brackets: 1024 x 2048 46.6 (48.1), 1024 x 1024 21.8 (23.2),
    // 700 x 1500 28.8 (31.2), 600 x 600 13.5 (14.3), 900 x 900, 24 heads 17.7 (19.3).  Heads of 64, four blocks per unit: no gain (520 x
    // 1024 14.0 (13.5), 700 x 1200 16.0 (16.3)).
    const int cus = device_cu_count();
    const int64_t all = (int64_t)H * ((Sq + 63) / 64);
    if (batch == 1 && H <= cus && all > cus && all <= 2 * (int64_t)cus)
        return launch_tiles<128, 2, 2, true>(Q, ldq, Kc, ldk, V, ldv, batch, Sq, Sk, H, O, ldo, st, cus / H);
    return launch_tiles<128, 2, 2>(Q, ldq, Kc, ldk, V, ldv, batch, Sq, Sk, H, O, ldo, st);
}

}  // namespace sqap
