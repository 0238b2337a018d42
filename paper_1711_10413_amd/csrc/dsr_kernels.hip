/*
 * dsr_kernels.hip -- generic-mode region kernel of the data-sharing runtime.
 *
 * One workgroup per team.  The last wave is the master wave (section 4,
 * Figure 2: the master is isolated from the workers); it interprets the
 * region's program of PUSH / PUBLISH / POP operations, i.e. the sequential
 * code block that declares the shared locals.  Worker waves sit in the
 * await loop of Figure 3 and run whichever outlined body the master
 * publishes, reading the shared locals through the published frame
 * (section 5.1: sharing by reference), then reduce into the frame's shared
 * variable and join.  After its program the master publishes TERMINATE;
 * the last team to finish combines the teams' partial reductions.
 *
 * Exact fp64 reduction: every loop value y must be a multiple of 2^-75 with
 * |y| < 2^32.  Each lane splits y exactly into three parts on the grids
 * 2^-5, 2^-40 and 2^-75 (y + C - C rounding with a constant C whose last
 * bit has the grid's weight) and adds each part into its own fp64 bin.  A
 * bin's values have at most 37 significant bits above its grid, so up to
 * 2^16 of them sum exactly in fp64.  At the end of the loop each lane turns
 * its bins into one signed 192-bit integer of 2^-75 units; waves, teams and
 * the region add those integers, and the region total is rounded to double
 * once.  The result is the correctly rounded sum whatever the team, wave or
 * launch layout.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dsr.h"
#include "dsr_device.h"
#include "dsr_internal.h"

#if !defined(DSR_INST_MAXWG) || !defined(DSR_INST_VARIANT) || !defined(DSR_INST_TAG)
#error "compile with -DDSR_INST_MAXWG=<threads> -DDSR_INST_VARIANT=<v> -DDSR_INST_TAG=<tag>"
#endif

using namespace dsr;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));

/* Elements of a caller's buffer, moved together: the buffer's address is a
 * multiple of one element's size alone. */
typedef float x_pair __attribute__((ext_vector_type(2), aligned(4)));
typedef double y_pair __attribute__((ext_vector_type(2), aligned(8)));
typedef int32_t out_quad __attribute__((ext_vector_type(4), aligned(4)));

extern __shared__ __align__(16) uint8_t dsr_lds[];

/* Address-space qualifiers: loop buffers are global memory; without the
 * qualifier the compiler emits flat instructions for them, which also wait
 * on the LDS counter and cannot use scalar-base addressing. */
#define GLB __attribute__((address_space(1)))
#define LDSQ __attribute__((address_space(3)))

/* ---- exact accumulation ------------------------------------------------ */
struct i192 { uint64_t w0, w1, w2; };

__device__ __forceinline__ i192 add192(i192 a, i192 b)
{
    i192 r;
    r.w0 = a.w0 + b.w0;
    const uint64_t c0 = r.w0 < a.w0;
    const uint64_t t = a.w1 + b.w1;
    const uint64_t c1a = t < a.w1;
    r.w1 = t + c0;
    const uint64_t c1b = r.w1 < t;
    r.w2 = a.w2 + b.w2 + c1a + c1b;
    return r;
}

__device__ __forceinline__ i192 from_i64(int64_t v)
{
    return i192{(uint64_t)v, (uint64_t)(v >> 63), (uint64_t)(v >> 63)};
}

/* v * 2^sh for a signed 64-bit v and 0 <= sh < 128. */
__device__ __forceinline__ i192 shl192(int64_t v, int sh)
{
    const uint64_t ext = (uint64_t)(v >> 63);
    uint64_t w0 = (uint64_t)v, w1 = ext, w2 = ext;
    if (sh >= 64) { w2 = w1; w1 = w0; w0 = 0; sh -= 64; }
    if (sh) {
        w2 = (w2 << sh) | (w1 >> (64 - sh));
        w1 = (w1 << sh) | (w0 >> (64 - sh));
        w0 <<= sh;
    }
    return i192{w0, w1, w2};
}

struct lane_acc {
    double b1, b2, b3;   /* bins on the 2^-5, 2^-40 and 2^-75 grids        */
    int64_t i;           /* integer bodies: wrap-around int64 sum          */
    uint32_t bad;        /* a value fell outside the exact-sum window      */
    i192 big;            /* bins flushed so far, in 2^-75 units            */
};

__device__ __forceinline__ lane_acc acc_zero()
{
    lane_acc a;
    a.b1 = a.b2 = a.b3 = 0.0;
    a.i = 0;
    a.bad = 0;
    a.big = i192{0, 0, 0};
    return a;
}

__device__ __forceinline__ void acc_add_i64(lane_acc &a, int64_t v)
{
    a.i = (int64_t)((uint64_t)a.i + (uint64_t)v);
}

/* Split y exactly into y = t1 + t2 + r2 with t1 on the 2^-5 grid, t2 on
 * the 2^-40 grid and |r2| <= 2^-41, and add the parts to the bins.  r2 must
 * itself be on the 2^-75 grid (checked by rounding it there); the caller has
 * checked |y| < 2^32. */
__device__ __forceinline__ void acc_add_f64(lane_acc &a, double y)
{
    const double C1 = 0x1.8p47, C2 = 0x1.8p12, C3 = 0x1.8p-23;
    const double t1 = (y + C1) - C1;
    const double r1 = y - t1;
    const double t2 = (r1 + C2) - C2;
    const double r2 = r1 - t2;
    const double t3 = (r2 + C3) - C3;
    a.bad |= (uint32_t)(t3 != r2);
    a.b1 += t1;
    a.b2 += t2;
    a.b3 += r2;
}

/* The bins of a stream's values.  b1 and b2 start at the constants that
 * round to their grids, so one add both rounds a value to the grid and adds
 * it, and what was added is the bin's difference: seven adds per value
 * instead of acc_add_f64's eleven, and no compare.  Exact while a bin stays in
 * its constant's binade: fewer than 2^14 values below 2^32 each.  b3 takes
 * what is left below 2^-41, which is on the 2^-75 grid if the value is. */
struct bins_t {
    double b1, b2, b3;
};
#define DSR_BIN1 0x1.8p47
#define DSR_BIN2 0x1.8p12

__device__ __forceinline__ bins_t bins_zero()
{
    return bins_t{DSR_BIN1, DSR_BIN2, 0.0};
}

/* Value e goes to bins e & 1.  One wave alone on its SIMD waits for each
 * fp64 result it uses next, so the steps of G values go side by side: 2^21
 * elements, one scalar, 16 teams of 3 workers 53.4 -> 45.1 us per launch,
 * 2^20 with 48 scalars and an array 52.2 -> 46.9 us; 2^24 elements, 512
 * teams, 0.3-0.9 us less for 1 to 64 scalars. */
template <int G>
__device__ __forceinline__ void bins_add(bins_t (&B)[2], const double *y)
{
    double n[G], r[G];
#pragma unroll
    for (int e = 0; e < G; ++e) n[e] = (e < 2 ? B[e & 1].b1 : n[e < 2 ? 0 : e - 2]) + y[e];
#pragma unroll
    for (int e = 0; e < G; ++e) r[e] = n[e] - (e < 2 ? B[e & 1].b1 : n[e < 2 ? 0 : e - 2]);
#pragma unroll
    for (int e = 0; e < G; ++e) r[e] = y[e] - r[e];
    B[0].b1 = n[G - 2];
    B[1].b1 = n[G - 1];
#pragma unroll
    for (int e = 0; e < G; ++e) n[e] = (e < 2 ? B[e & 1].b2 : n[e < 2 ? 0 : e - 2]) + r[e];
    double t[G];
#pragma unroll
    for (int e = 0; e < G; ++e) t[e] = n[e] - (e < 2 ? B[e & 1].b2 : n[e < 2 ? 0 : e - 2]);
#pragma unroll
    for (int e = 0; e < G; ++e) r[e] -= t[e];
    B[0].b2 = n[G - 2];
    B[1].b2 = n[G - 1];
#pragma unroll
    for (int e = 0; e < G; ++e) B[e & 1].b3 += r[e];
}

/* Bins of the same grid add exactly while each holds fewer than 2^16
 * values. */
__device__ __forceinline__ void acc_merge(lane_acc &a, const bins_t &b)
{
    a.b1 += b.b1 - DSR_BIN1;
    a.b2 += b.b2 - DSR_BIN2;
    a.b3 += b.b3;
}

/* A lane's bins as one integer of 2^-75 units (bin values are integers of
 * their grid below 2^53 in magnitude, so the conversions are exact). */
__device__ __forceinline__ i192 bins_fixed(const lane_acc &a)
{
    const int64_t k1 = (int64_t)(a.b1 * 0x1p5);
    const int64_t k2 = (int64_t)(a.b2 * 0x1p40);
    const int64_t k3 = (int64_t)(a.b3 * 0x1p75);
    i192 s = add192(shl192(k1, 70), shl192(k2, 35));
    return add192(s, from_i64(k3));
}

/* Move the bins into the 192-bit accumulator (keeps them exact however
 * many values a lane adds). */
__device__ __forceinline__ void acc_flush(lane_acc &a)
{
    a.big = add192(a.big, bins_fixed(a));
    a.b1 = a.b2 = a.b3 = 0.0;
}

__device__ __forceinline__ i192 widen(const lane_acc &a)
{
    return add192(add192(a.big, bins_fixed(a)), from_i64(a.i));
}

/* One DPP step of the wave sum: every 32-bit part of v moved from the lane
 * the control selects (zero where that lane is outside the row, and in the
 * rows the mask leaves out), then added with carries. */
template <int CTRL, int ROWS>
__device__ __forceinline__ i192 dpp_add192(i192 v)
{
    const uint32_t p[6] = {(uint32_t)v.w0, (uint32_t)(v.w0 >> 32), (uint32_t)v.w1,
                           (uint32_t)(v.w1 >> 32), (uint32_t)v.w2, (uint32_t)(v.w2 >> 32)};
    uint32_t q[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) q[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)p[k], CTRL, ROWS, 0xf, true);
    return add192(v, i192{q[0] | ((uint64_t)q[1] << 32), q[2] | ((uint64_t)q[3] << 32), q[4] | ((uint64_t)q[5] << 32)});
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int lane)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

/* Sum over the first row (lanes 0 to 15), returned to every lane. */
__device__ __forceinline__ i192 row_sum192(i192 v)
{
    v = dpp_add192<0x111, 0x1>(v);   /* row_shr:1 */
    v = dpp_add192<0x112, 0x1>(v);   /* row_shr:2 */
    v = dpp_add192<0x114, 0x1>(v);   /* row_shr:4 */
    v = dpp_add192<0x118, 0x1>(v);   /* row_shr:8 */
    return i192{readlane64(v.w0, 15), readlane64(v.w1, 15), readlane64(v.w2, 15)};
}

/* Sum over the 64 lanes of a wave, returned to every lane: a running sum
 * inside each row of 16 lanes (row shifts by 1, 2, 4 and 8), then the row
 * totals carried across rows (lane 15 into row 1 and 3, lane 31 into rows 2
 * and 3), so lane 63 holds the total; all in VALU moves, no LDS round
 * trips.  Every lane of the wave takes part. */
__device__ __forceinline__ i192 wave_sum192(i192 v)
{
    v = dpp_add192<0x111, 0xf>(v);   /* row_shr:1 */
    v = dpp_add192<0x112, 0xf>(v);   /* row_shr:2 */
    v = dpp_add192<0x114, 0xf>(v);   /* row_shr:4 */
    v = dpp_add192<0x118, 0xf>(v);   /* row_shr:8 */
    v = dpp_add192<0x142, 0xa>(v);   /* row_bcast:15 into rows 1 and 3 */
    v = dpp_add192<0x143, 0xc>(v);   /* row_bcast:31 into rows 2 and 3 */
    return i192{readlane64(v.w0, 63), readlane64(v.w1, 63), readlane64(v.w2, 63)};
}

__device__ __forceinline__ uint64_t bits64(uint64_t w0, uint64_t w1, uint64_t w2, int p)
{
    const int q = p >> 6, r = p & 63;
    const uint64_t a = q == 0 ? w0 : (q == 1 ? w1 : w2);
    const uint64_t b = q == 0 ? w1 : (q == 1 ? w2 : 0ull);
    return r ? ((a >> r) | (b << (64 - r))) : a;
}

__device__ __forceinline__ bool any_below(uint64_t w0, uint64_t w1, uint64_t w2, int p)
{
    if (p <= 0) return false;
    const int q = p >> 6, r = p & 63;
    if (q > 0 && w0) return true;
    if (q > 1 && w1) return true;
    if (r == 0) return false;
    const uint64_t w = q == 0 ? w0 : (q == 1 ? w1 : w2);
    return (w & ((1ull << r) - 1ull)) != 0;
}

/* Nearest-even double of the signed 192-bit value times 2^-75. */
__device__ double fixed_to_double(i192 v)
{
    const bool neg = (int64_t)v.w2 < 0;
    uint64_t w0 = v.w0, w1 = v.w1, w2 = v.w2;
    if (neg) {
        w0 = ~w0; w1 = ~w1; w2 = ~w2;
        w0 += 1;
        uint64_t c = (w0 == 0);
        w1 += c;
        c = c && (w1 == 0);
        w2 += c;
    }
    int top;
    if (w2) top = 128 + 63 - __clzll((long long)w2);
    else if (w1) top = 64 + 63 - __clzll((long long)w1);
    else if (w0) top = 63 - __clzll((long long)w0);
    else return 0.0;
    uint64_t mant;
    bool round = false, sticky = false;
    if (top <= 52) {
        mant = w0 << (52 - top);
    } else {
        const int p = top - 52;
        mant = bits64(w0, w1, w2, p) & ((1ull << 53) - 1ull);
        round = bits64(w0, w1, w2, p - 1) & 1ull;
        sticky = any_below(w0, w1, w2, p - 1);
    }
    if (round && (sticky || (mant & 1ull))) {
        mant += 1;
        if (mant >> 53) { mant >>= 1; top += 1; }
    }
    const uint64_t E = (uint64_t)(top - 75 + 1023);
    const uint64_t bits = ((uint64_t)neg << 63) | (E << 52) | (mant & ((1ull << 52) - 1ull));
    return __longlong_as_double((long long)bits);
}

/* ---- loop bodies --------------------------------------------------------- */
/* A span is a range [lo, hi) of loop iterations shared cyclically by P
 * lanes, of which this lane is number p. */
struct span_t {
    uint64_t lo, hi;
    uint32_t p, P;
};

/* Drive a body over this lane's static share `sp` and then, under the
 * dynamic-tail schedule, over the blocks its wave claims from the loop's
 * device counter (the next claim is issued before the current block runs,
 * so its latency overlaps the work).  Claimed blocks are shared by the 64
 * lanes of the claiming wave. */
/* teams up to this many arrive at one counter (no group level) */
#ifndef DSR_FLAT_TEAMS
#define DSR_FLAT_TEAMS 512
#endif
#ifndef DSR_ARRIVE_FENCE
#define DSR_ARRIVE_FENCE 1
#endif
template <class F>
__device__ __forceinline__ void for_spans(const dsr_dloop &L, span_t sp, uint32_t lane,
                                          uint32_t *claim, lane_acc &A, F &&f)
{
    f(sp);
    if (L.schedule != DSR_SCHED_DYNAMIC_TAIL) return;
    uint32_t c = 0;
    if (lane == 0) c = atomicAdd(claim, 1u);
    c = (uint32_t)__shfl((int)c, 0, 64);
    uint32_t since = 0;
    for (;;) {
        const uint64_t lo = L.dyn_start + (uint64_t)c * L.block;
        if (lo >= L.n) break;
        uint32_t cn = 0;
        if (lane == 0) cn = atomicAdd(claim, 1u);
        f(span_t{lo, min(L.n, lo + (uint64_t)L.block), lane, 64u});
        /* a block adds at most 1024 values per lane: flush well before 2^16 */
        if (++since == 16) { acc_flush(A); since = 0; }
        c = (uint32_t)__shfl((int)cn, 0, 64);
    }
}

/* One lane's share of the affine loop: groups of four outputs (one 16-byte
 * store) from the first multiple of four on, the ends one by one.  A loop has
 * fewer than 2^31 iterations, so indices are 32 bits wide. */
__device__ __forceinline__ void affine_span(uint32_t a, uint32_t b, uint32_t c, uint32_t d,
                                            GLB int32_t *out, span_t sp, lane_acc &A)
{
    const uint32_t lo = (uint32_t)sp.lo, hi = (uint32_t)sp.hi;
    const uint32_t v0 = min(hi, (lo + 3u) & ~3u), v1 = max(v0, hi & ~3u);
    int64_t s = 0;
    auto value = [&](uint32_t i) { return (int32_t)(a * i + b - (c ^ i) + d); };
    for (uint32_t i = v0 + 4 * sp.p; i < v1; i += 4 * sp.P) {
        const i32x4 o = {value(i), value(i + 1), value(i + 2), value(i + 3)};
        __builtin_nontemporal_store(o, (GLB out_quad *)(out + i));
        s += ((int64_t)o.x + o.y) + ((int64_t)o.z + o.w);
    }
    /* at most three elements before the groups and three after */
    const uint32_t edge = sp.p < v0 - lo ? lo + sp.p : v1 + (sp.p - (v0 - lo));
    if (sp.p < (v0 - lo) + (hi - v1)) {
        const int32_t o = value(edge);
        out[edge] = o;
        s += o;
    }
    acc_add_i64(A, s);
}

/* ---- fma chains ----------------------------------------------------------
 * The chain y = a + s_0 x + s_1 x + ... rounds once per step, so its steps
 * run in order; what can be saved is steps that do not round.  The int32
 * scalars come first.  Let S_k be the sum of the first k of them.  While
 * a + S_k x is exact in fp64 for every k, each step's result is that value,
 * and one step with S = S_ni gives the same bits as ni steps:
 *   without an array (a = +0): x has 24 significant bits, so |S_k| <= 2^29
 *     suffices for every finite x, whatever its exponent;
 *   with an array element a: if x is a multiple of 2^-24, so is a + S_k x,
 *     and |a| + max|S_k| |x| < 2^29 bounds it to 53 bits.
 * Signed zeros agree as well: the chain starts at +0 or an integer, and an
 * exact sum that cancels is +0.  The first condition is checked once per body
 * (a scan over the scalars, one per lane), the second once per batch over the
 * batch's largest |x| and |a|; a non-finite x shows as a y outside the
 * exact-sum window.  A batch that fails runs every step.  Half of a 64-scalar
 * chain's steps and two thirds of a mixed region's fall away: 2^24 elements,
 * 512 teams x 256, 64 scalars 62.3 -> 49.7 us per launch (fp64-bound before,
 * HBM-bound like the short chains now), 38 scalars in a frame 57.8 -> 48.9 us;
 * launch and wait of 2^20 elements, 48 scalars and an 8128-element array on
 * 16 teams 108.7 -> 79.6 us; 10,000 mixed regions 3.79 -> 3.42 ms. */
__device__ __forceinline__ double readlane_f64(double v, uint32_t k)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, k);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), k);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <int E>
__device__ __forceinline__ void fma_all(double s, double (&acc)[E], const double (&xd)[E])
{
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = __builtin_fma(s, xd[e], acc[e]);
}

/* A double's exponent and leading bits: ordered as its magnitude, NaN above
 * all. */
__device__ __forceinline__ uint32_t magnitude(double y)
{
    return (uint32_t)((uint64_t)__double_as_longlong(y) >> 32) & 0x7FFFFFFFu;
}

/* Whether any of a lane's values lies outside the exact-sum window
 * (|y| >= 2^32 or not finite). */
template <int E>
__device__ __forceinline__ bool outside(const double (&y)[E])
{
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) m = max(m, magnitude(y[e]));
    return m >= 0x41F00000u;
}

/* Whether any of a lane's values inside the window is not on the 2^-75 grid.
 * All doubles of 2^-23 and more are on it; only a batch that holds a smaller
 * one is looked at value by value. */
template <int E>
__device__ __forceinline__ bool off_grid(const double (&y)[E])
{
    uint32_t m = 0x3FF00000u;
#pragma unroll
    for (int e = 0; e < E; ++e) m = min(m, magnitude(y[e]));
    bool w = false;
    if (__any(m < 0x3E800000u)) {
        asm volatile("");      /* keep the branch */
#pragma unroll
        for (int e = 0; e < E; ++e) w |= __builtin_rint(y[e] * 0x1p75) != y[e] * 0x1p75;
    }
    return w;
}

/* A chain with run-time counts: lane k holds scalar k as a double (at most
 * 64), and each step takes it with two readlanes shared by every element of
 * the batch.  Four steps at a time, so a batch of 16 elements issues 64
 * independent-enough fmas between reads. */
struct rt_chain {
    double sv;                /* lane k: scalar k                             */
    uint32_t ni, n;
    double S;                 /* sum of the int32 scalars                     */
    float M;                  /* largest partial sum in magnitude             */
    bool sum;                 /* the int32 steps may be taken as one          */

    template <int E>
    __device__ __forceinline__ void steps(double (&acc)[E], const double (&xd)[E], uint32_t k) const
    {
#pragma nounroll
        for (; k + 4 <= n; k += 4) {
            const double s0 = readlane_f64(sv, k), s1 = readlane_f64(sv, k + 1);
            const double s2 = readlane_f64(sv, k + 2), s3 = readlane_f64(sv, k + 3);
            fma_all<E>(s0, acc, xd);
            fma_all<E>(s1, acc, xd);
            fma_all<E>(s2, acc, xd);
            fma_all<E>(s3, acc, xd);
        }
#pragma nounroll
        for (; k < n; ++k) fma_all<E>(readlane_f64(sv, k), acc, xd);
    }

    /* Whether a batch's int32 steps may be taken as one.  Every lane of the
     * wave takes part, here and in eval. */
    template <bool ARR, int E>
    __device__ __forceinline__ bool choose(const float (&xf)[E], const int32_t (&a)[E]) const
    {
        if (!ARR || !sum) return sum;
        uint32_t mx = 0, frac = 0;
        int32_t hi = 0, lo = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            mx = max(mx, __float_as_uint(xf[e]) & 0x7FFFFFFFu);
            frac |= __float_as_uint(__builtin_amdgcn_fractf(xf[e] * 0x1p24f));
            hi = max(hi, a[e]);
            lo = min(lo, a[e]);
        }
        const float ma = (float)hi - (float)lo;
        /* (2^28 for 2^29: the bound itself is rounded) */
        return __all(frac == 0 && __builtin_fmaf(__uint_as_float(mx), M, ma) < 0x1p28f);
    }

    /* acc comes in as the chain's start; returns whether a value of this lane
     * is outside the window. */
    template <bool ARR, int E>
    __device__ __forceinline__ bool eval(double (&acc)[E], const double (&xd)[E], bool one) const
    {
        if (one) fma_all<E>(S, acc, xd);
        steps<E>(acc, xd, one ? ni : 0u);
        bool w = outside<E>(acc);
        if (!ARR && one && __any(w)) {
            /* all the steps of a batch with a value outside the window */
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = 0.0;
            steps<E>(acc, xd, 0);
            w = outside<E>(acc);
        }
        return w;
    }
};

/* A chain with its counts known at compile time, its fp64 scalars in
 * registers; `all` holds the int32 ones too, for what cannot be summed. */
template <int NI, int NF>
struct fixed_chain {
    double s[NF > 0 ? NF : 1];
    rt_chain all;

    template <bool ARR, int E>
    __device__ __forceinline__ bool choose(const float (&)[E], const int32_t (&)[E]) const
    {
        return NI == 1 || all.sum;
    }

    template <bool ARR, int E>
    __device__ __forceinline__ bool eval(double (&acc)[E], const double (&xd)[E], bool one) const
    {
        static_assert(!ARR, "fixed chains have no array");
        if (NI == 1 || one) {
            fma_all<E>(all.S, acc, xd);
#pragma unroll
            for (int k = 0; k < NF; ++k) fma_all<E>(s[k], acc, xd);
            const bool w = outside<E>(acc);
            if (NI == 1 || !__any(w)) return w;
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = 0.0;
        }
        all.template steps<E>(acc, xd, 0);
        return outside<E>(acc);
    }
};

/* One DPP step of a wave scan over doubles (zero where the source lane lies
 * outside the row). */
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_f64(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, true);
    return v + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ rt_chain make_chain(double sv, uint32_t ni, uint32_t nf, uint32_t lane)
{
    rt_chain c{sv, ni, ni + nf, ni ? readlane_f64(sv, 0) : 0.0, 0.0f, false};
    if (ni > 1) {
        /* partial sums of the int32 scalars: exact (at most 64 of 32 bits) */
        double p = lane < ni ? sv : 0.0;
        p = dpp_add_f64<0x111, 0xf>(p);
        p = dpp_add_f64<0x112, 0xf>(p);
        p = dpp_add_f64<0x114, 0xf>(p);
        p = dpp_add_f64<0x118, 0xf>(p);
        p = dpp_add_f64<0x142, 0xa>(p);
        p = dpp_add_f64<0x143, 0xc>(p);
        c.S = readlane_f64(p, 63);
        c.sum = __all(__builtin_fabs(p) <= 0x1p29);
        /* the largest magnitude, rounded up to a power of two: the highest
         * bit set in any lane */
        uint32_t m = c.sum ? (uint32_t)__builtin_fabs(p) : 0u;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) m |= (uint32_t)__shfl_xor((int)m, d, 64);
        m = uniform(m);
        c.M = m ? (float)(1ull << (32 - __builtin_clz(m))) : 0.0f;
    }
    return c;
}

/* The scalars read through the published reference list on every batch:
 * each chain step reads reference 1 + k (a space and an offset), then the
 * variable it names, as outlined code must when stores in its loop may
 * alias the shared variables (section 5.1's sharing by reference).  The
 * list is on chip or in a list frame on the HBM stack, the variables on
 * either stack; all of it is read through generic pointers, as the outlined
 * function receives them. */
struct list_chain {
    const uint32_t *lst;
    const uint8_t *stack_lds, *stack_hbm;
    uint32_t ni, nf;

    template <bool ARR, int E>
    __device__ __forceinline__ bool choose(const float (&)[E], const int32_t (&)[E]) const
    {
        return false;
    }

    template <bool ARR, int E>
    __device__ __forceinline__ bool eval(double (&acc)[E], const double (&xd)[E], bool) const
    {
        for (uint32_t k = 0; k < ni + nf; ++k) {
            const uint32_t sp = uniform(lst[2 * (1 + k)]), off = uniform(lst[2 * (1 + k) + 1]);
            const uint8_t *p = (sp == SPACE_LDS ? stack_lds : stack_hbm) + off;
            const double v = k < ni ? (double)*(const int32_t *)p : *(const double *)p;
            fma_all<E>(v, acc, xd);
        }
        return outside<E>(acc);
    }
};

__device__ __forceinline__ uint32_t mod_step(uint32_t j, uint32_t d, uint32_t m)
{
    j += d;
    return j >= m ? j - m : j;
}

/* How a body's array is read.  In an array of even length a pair of loop
 * iterations that starts on an even one never wraps inside the pair. */
enum { ARR_NONE = 0, ARR_EVEN = 1, ARR_ODD = 2 };

/* U element pairs of one lane: x, and the array elements they start from. */
template <int U, int ARR>
struct batch_t {
    f32x2 x[U];
    int32_t a[2 * U];
};

/* Streams the pairs of a range through a chain.  Pair b + lane + u * st of a
 * wave's batch at b (u < U) is the lane's u-th; a lane takes element pairs
 * (8 B of x, 16 B of y), so every load instruction of a wave covers 512
 * contiguous bytes of x and every store 1 KB of y.  The batch's place is
 * wave-uniform and the lane's offset inside it is fixed, so the addresses
 * cost the lanes nothing; the next batch's loads are in flight while the
 * current one computes.  What is left at the end, less than a batch for the
 * wave, is loaded in one round as well. */
template <int U, int ARR, class AP, class CH>
struct stream_t {
    const CH &ch;
    AP arr;
    uint32_t alen;
    const GLB char *xb;       /* pair 0 of the range                          */
    GLB char *yb;
    uint32_t nv;              /* pairs in the range                           */
    uint32_t first;           /* array index of pair 0's first element        */
    uint32_t inv;             /* floor((2^32 - 1) / alen)                     */
    uint32_t st, dj;          /* pair stride of a lane, as an array step      */
    uint32_t lane;
    lane_acc &A;
    bins_t B[2];

    template <int N, bool MASK>
    __device__ __forceinline__ void load(batch_t<U, ARR> &t, uint32_t b) const
    {
        uint32_t j = 0;
        /* (first + 2 v) mod alen; the quotient from the reciprocal is at most
         * one short */
        auto index = [&](uint32_t v) {
            const uint32_t k = first + 2u * v, m = k - __umulhi(k, inv) * alen;
            return m >= alen ? m - alen : m;
        };
        if constexpr (ARR != ARR_NONE && !MASK) j = index(b + lane);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const GLB char *base = xb + 8ull * (b + (uint32_t)u * st);
            uint32_t off = 8u * lane;
            if constexpr (MASK) {
                /* pairs past the end do the last one again, its array
                 * elements too (their results are dropped, but not whether
                 * they lie in the exact-sum window).  The byte offset fits 32
                 * bits: no range holds more than DSR_DEAL_MAX elements */
                const uint32_t v = min(b + (uint32_t)u * st + lane, nv - 1);
                base = xb;
                off = 8u * v;
                if constexpr (ARR != ARR_NONE) j = index(v);
            }
            t.x[u] = __builtin_nontemporal_load((const GLB x_pair *)(base + off));
            if constexpr (ARR == ARR_EVEN) {
                const i32x2 q = *(const typename AP::pair)(arr.p + j);
                t.a[2 * u] = q.x;
                t.a[2 * u + 1] = q.y;
                if constexpr (!MASK) j = mod_step(j, dj, alen);
            } else if constexpr (ARR == ARR_ODD) {
                t.a[2 * u] = arr.p[j];
                t.a[2 * u + 1] = arr.p[j + 1 == alen ? 0 : j + 1];
                if constexpr (!MASK) j = mod_step(j, dj, alen);
            }
        }
    }

    /* A loaded batch as the chain takes it: x as doubles, and the values the
     * chain starts from. */
    template <int N>
    struct terms_t {
        double xd[2 * N], y[2 * N];
        bool one;
    };

    template <int N>
    __device__ __forceinline__ void take(const batch_t<U, ARR> &t, terms_t<N> &q) const
    {
        float xf[2 * N];
        int32_t a[2 * N];
#pragma unroll
        for (int e = 0; e < 2 * N; ++e) {
            xf[e] = (e & 1) ? t.x[e / 2].y : t.x[e / 2].x;
            q.xd[e] = (double)xf[e];
            a[e] = ARR != ARR_NONE ? t.a[e] : 0;
        }
        q.one = ch.template choose<ARR != ARR_NONE, 2 * N>(xf, a);
    }

    template <int N>
    __device__ __forceinline__ void start(const batch_t<U, ARR> &t, terms_t<N> &q) const
    {
#pragma unroll
        for (int e = 0; e < 2 * N; ++e) q.y[e] = ARR != ARR_NONE ? (double)t.a[e] : 0.0;
    }

    template <int N>
    __device__ __forceinline__ void chain(terms_t<N> &q)
    {
        const bool w = ch.template eval<ARR != ARR_NONE, 2 * N>(q.y, q.xd, q.one);
        A.bad |= (uint32_t)(w || off_grid<2 * N>(q.y));
    }

    template <int N>
    __device__ __forceinline__ void add(const double (&y)[2 * N])
    {
        constexpr int G = N < 4 ? 2 * N : 8;
#pragma unroll
        for (int e = 0; e < 2 * N; e += G) bins_add<G>(B, y + e);
    }

    template <int N>
    __device__ __forceinline__ void store(const double (&y)[2 * N], uint32_t b) const
    {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const f64x2 r = {y[2 * u], y[2 * u + 1]};
            __builtin_nontemporal_store(r, (GLB y_pair *)(yb + 16ull * (b + (uint32_t)u * st) + 16u * lane));
        }
    }

    template <int N>
    __device__ __forceinline__ void rest(uint32_t b)
    {
        batch_t<U, ARR> t;
        terms_t<N> q;
        load<N, true>(t, b);
        take<N>(t, q);
        start<N>(t, q);
        chain<N>(q);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const f64x2 r = {q.y[2 * u], q.y[2 * u + 1]};
            const uint32_t v = b + (uint32_t)u * st;
            const bool in = v + lane < nv;
            if (in) __builtin_nontemporal_store(r, (GLB y_pair *)(yb + 16ull * (v + lane)));
            q.y[2 * u] = in ? r.x : 0.0;
            q.y[2 * u + 1] = in ? r.y : 0.0;
        }
        add<N>(q.y);
    }

    /* next(b): the wave's batch after the one at b.  Returns the first batch
     * that was not a full one.
     *
     * The counter that loads are waited for by is in order and counts stores
     * too.  So a batch's x is taken over first, then the previous batch's
     * results are stored, and the next batch's loads come last: the wait for
     * them, a batch later, then leaves nothing newer to wait for, and the
     * loads and the stores before them have had a batch's arithmetic to
     * complete.  With the loads of the next batch first, every batch waited
     * for the memory once: one scalar over 2^21 elements on 16 teams of 3
     * workers 45.1 -> 34.3 us per launch; 2^24 elements, 512 teams x 256, 1 /
     * 8 / 64 scalars 41.0 / 41.3 / 46.0 -> 40.3 / 40.3 / 43.2 us (the plain
     * streaming loop of the same traffic takes 40.2). */
    template <class NEXT>
    __device__ __forceinline__ uint32_t run(uint32_t b, NEXT &&next)
    {
        /* (32 bits wide: a scalar branch) */
        const uint32_t span = 63u + (uint32_t)(U - 1) * st, end = uniform(nv > span ? nv - span : 0u);
        auto full = [&](uint32_t q) { return uniform(q) < end; };
        B[0] = B[1] = bins_zero();
        if (full(b)) {
            batch_t<U, ARR> t;
            terms_t<U> q;
            load<U, false>(t, b);
            uint32_t since = 0, done = b;
            bool first = true, more = true;
            do {
                take<U>(t, q);
                /* here, not behind the stores */
#pragma unroll
                for (int e = 0; e < 2 * U; ++e) asm volatile("" : "+v"(q.xd[e]));
                if (!first) store<U>(q.y, done);
                start<U>(t, q);
                done = b;
                b = next(b);
                more = full(b);
                if (more) load<U, false>(t, b);
                chain<U>(q);
                add<U>(q.y);
                /* a batch adds U values to each bin: flush before 2^14 */
                if (++since == 1024) {
                    acc_merge(A, B[0]);
                    acc_merge(A, B[1]);
                    acc_flush(A);
                    B[0] = B[1] = bins_zero();
                    since = 0;
                }
                first = false;
            } while (more);
            store<U>(q.y, done);
        }
        if (b < nv) {
            const uint32_t left = min((uint32_t)U, (nv - b + st - 1) / st);
            if (U >= 8 && left > 4) rest<U>(b);
            else if (U >= 4 && left > 2) rest<U < 4 ? U : 4>(b);
            else rest<U < 2 ? U : 2>(b);
        }
        acc_merge(A, B[0]);
        acc_merge(A, B[1]);
        return b;
    }
};

/* A pointer to a body's array, and the type of a pair of its elements. */
struct lds_array {
    typedef const LDSQ i32x2 *pair;
    const LDSQ int32_t *p;
};
struct glb_array {
    typedef const GLB i32x2 *pair;
    const GLB int32_t *p;
};

/* The next block of the team's range, claimed by this wave from the counter
 * in the team's control block. */
__device__ __forceinline__ uint32_t claim_block(uint32_t lane)
{
    LDSQ uint32_t *ctr = (LDSQ uint32_t *)(dsr_lds + offsetof(cb_header, blocks));
    uint32_t c = 0;
    if (lane == 0) c = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return c;
}

/* A loop dealt to the waves of all teams, a batch at a time in turn: this wave
 * is number `wave` of `waves` (0: not dealt). */
struct deal_t {
    uint32_t wave, waves;
};

/* One range [sp.lo, sp.hi) of the loop through a chain, in one of three forms.
 * BLOCKS: the team's waves claim batches of 64 * U pairs from the team's counter,
 * so a wave on a SIMD it shares with fewer others takes more of them (three worker
 * waves per team and two teams per CU leave some SIMDs two worker waves and some
 * one); a claim is taken one batch ahead.  Dealt: the range is the whole loop,
 * up to DSR_DEAL_MAX elements, and the wave takes every `waves`-th batch of
 * 64 * U pairs.  Else lane sp.p of sp.P takes every sp.P-th pair; such a range, a team's or
 * a claimed block, holds at most 2^25 elements.  An odd first element and an odd
 * last one go to lanes 0 and 1 of the range; a dealt loop's odd last one goes to
 * the wave whose batch it would be in. */
template <int U, int ARR, bool BLOCKS, class AP, class CH>
__device__ __forceinline__ void chain_range(const CH &ch, AP arr, uint32_t alen, const dsr_dloop &L, span_t sp,
                                            deal_t deal, uint32_t lane, lane_acc &A)
{
    const uint32_t lo = uniform((uint32_t)sp.lo), hi = uniform((uint32_t)sp.hi);
    if (lo >= hi) return;
    const GLB float *x = (const GLB float *)L.in;
    GLB double *y = (GLB double *)L.out;
    const uint32_t p0 = (lo + 1) >> 1, p1 = max(p0, hi >> 1);
    bool edge = (sp.p == 0 && (lo & 1u)) || (sp.p == 1 && (hi & 1u));
    const uint32_t ie = sp.p == 0 ? lo : hi - 1;
    const float xe = edge ? x[ie] : 0.0f;
    const uint32_t st = BLOCKS ? 64u : uniform(sp.P);
    stream_t<U, ARR, AP, CH> S{ch, arr, alen, (const GLB char *)x + 8ull * p0, (GLB char *)y + 16ull * p0, p1 - p0,
                               ARR != ARR_NONE ? (2u * p0) % alen : 0u,
                               ARR != ARR_NONE ? 0xFFFFFFFFu / alen : 0u, st, ARR != ARR_NONE ? (2u * st) % alen : 0u,
                               lane, A, {}};
    constexpr uint32_t BATCH = 64u * U;
    uint32_t b = deal.waves ? deal.wave * BATCH : uniform(sp.p - lane), ahead = 0;
    const uint32_t step = deal.waves ? deal.waves * BATCH : U * st;
    if (BLOCKS) {
        b = uniform(claim_block(lane)) * BATCH;
        ahead = claim_block(lane);
    }
    b = S.run(b, [&](uint32_t q) {
        if (!BLOCKS) return q + step;
        const uint32_t n = uniform(ahead) * BATCH;
        ahead = claim_block(lane);
        return n;
    });
    /* a dealt loop's odd last element goes with the batch it would be in */
    if (deal.waves) edge = edge && b == S.nv / BATCH * BATCH;
    if (__any(edge)) {
        const float xf[1] = {xe};
        const double xd[1] = {(double)xe};
        int32_t a[1] = {0};
        if constexpr (ARR != ARR_NONE) a[0] = edge ? arr.p[ie % alen] : 0;
        double acc[1] = {ARR != ARR_NONE ? (double)a[0] : 0.0};
        const bool one = ch.template choose<ARR != ARR_NONE, 1>(xf, a);
        const bool w = ch.template eval<ARR != ARR_NONE, 1>(acc, xd, one);
        if (edge) {
            y[ie] = acc[0];
            A.bad |= (uint32_t)w;
            acc_add_f64(A, acc[0]);
        }
    }
}

/* A chain over the team's part of the loop: its static range by blocks, or
 * under the dynamic tail its static part and then the blocks its wave claims
 * from the loop's device counter.  The lean instances run static ranges only,
 * dealt or every wave its fixed per-lane share: the share was 0.3-1.0 us faster
 * there per 2^24-element region than blocks for 8 to 32 scalars, and the same
 * below (loops of that length are dealt now unless the caller sets a chunk). */
template <int U, int ARR, bool LEAN, class AP, class CH>
__device__ __forceinline__ void chain_loop(const CH &ch, AP arr, uint32_t alen, const dsr_dloop &L, span_t sp,
                                           deal_t deal, uint32_t lane, uint32_t *claim, lane_acc &A)
{
    if constexpr (LEAN) {
        chain_range<U, ARR, false>(ch, arr, alen, L, sp, deal, lane, A);
        return;
    }
    if (L.schedule == DSR_SCHED_STATIC) {
        chain_range<U, ARR, true>(ch, arr, alen, L, sp, deal, lane, A);
        return;
    }
    uint32_t c = 0, since = 0;
    for (bool tail = false;; tail = true) {
        /* the next claim is issued before the current block runs, so its
         * latency overlaps the work */
        if (tail && lane == 0) c = atomicAdd(claim, 1u);
        chain_range<U, ARR, false>(ch, arr, alen, L, sp, deal, lane, A);
        if (!tail && lane == 0) c = atomicAdd(claim, 1u);
        /* a block adds at most 1024 values per lane: flush well before 2^16 */
        if (++since == 16) { acc_flush(A); since = 0; }
        const uint64_t lo = L.dyn_start + (uint64_t)uniform(c) * L.block;
        if (lo >= L.n) return;
        sp = span_t{lo, min(L.n, lo + (uint64_t)L.block), lane, 64u};
    }
}

/* The chain's shared variables, published as a frame ([24 B exact sum][nf
 * fp64][ni int32][pad to 16][array]) or, REFS, as the list of references of
 * section 5.1: lane j reads reference 1 + j, then scalar j through it. */
template <int U, bool LEAN>
__device__ __forceinline__ void body_chain(const team_t &T, bool refs, frame_t f, const dsr_dloop &L, span_t sp,
                                           deal_t deal, lane_acc &A, uint32_t *claim, uint32_t lane)
{
    const uint32_t ni = uniform(L.ni), nf = uniform(L.nf), alen = uniform(L.alen);
    double sv = 0.0;
    uint32_t aspace = f.space, aoff = f.off + ((24 + 8 * nf + 4 * ni + 15) & ~15u);
    if (refs) {
        const uint32_t *lst = f.space == SPACE_LIST ? ref_list(T) : (const uint32_t *)frame_hbm(T, f);
        if (uniform(L.deref) && alen == 0) {
            const list_chain ch{lst, T.stack_lds, T.stack_hbm, ni, nf};
            chain_loop<U, ARR_NONE, LEAN>(ch, glb_array{nullptr}, 0, L, sp, deal, lane, claim, A);
            return;
        }
        if (lane < ni + nf) {
            const uint32_t sp_ = lst[2 * (1 + lane)], off = lst[2 * (1 + lane) + 1];
            const uint8_t *p = sp_ == SPACE_LDS ? T.stack_lds + off : T.stack_hbm + off;
            sv = lane < ni ? (double)*(const int32_t *)p : *(const double *)p;
        }
        if (alen) {
            aspace = uniform(lst[2 * (1 + ni + nf)]);
            aoff = uniform(lst[2 * (1 + ni + nf) + 1]);
        }
    } else if (f.space == SPACE_LDS) {
        const LDSQ uint8_t *fb = (const LDSQ uint8_t *)(dsr_lds + cb_bytes(T.nw) + f.off);
        if (lane < ni) sv = (double)*(const LDSQ int32_t *)(fb + 24 + 8 * nf + 4 * lane);
        else if (lane < ni + nf) sv = *(const LDSQ double *)(fb + 24 + 8 * (lane - ni));
    } else {
        const GLB uint8_t *fb = (const GLB uint8_t *)frame_hbm(T, f);
        if (lane < ni) sv = (double)*(const GLB int32_t *)(fb + 24 + 8 * nf + 4 * lane);
        else if (lane < ni + nf) sv = *(const GLB double *)(fb + 24 + 8 * (lane - ni));
    }
    const rt_chain ch = make_chain(sv, ni, nf, lane);
    /* batches of U pairs with an array too: half as many computed for less time
     * than memory takes to return the next batch's x (2^20 elements, 48 scalars,
     * 16 teams, per launch 63.0 -> 51.5 us; two such batches ahead 63.0); a second
     * full one ahead costs the general instances their registers */
    /* an array a list refers to may lie on a 4-byte boundary alone; in global
     * memory arrays are read element by element as well (one body less) */
    if (!alen)
        chain_loop<U, ARR_NONE, LEAN>(ch, glb_array{nullptr}, 0, L, sp, deal, lane, claim, A);
    else if (aspace != SPACE_LDS)
        chain_loop<U, ARR_ODD, LEAN>(ch, glb_array{(const GLB int32_t *)(T.stack_hbm + aoff)}, alen, L, sp, deal, lane, claim, A);
    else if ((alen & 1u) || (aoff & 7u))
        chain_loop<U, ARR_ODD, LEAN>(ch, lds_array{(const LDSQ int32_t *)(dsr_lds + cb_bytes(T.nw) + aoff)}, alen, L, sp, deal, lane,
                               claim, A);
    else
        chain_loop<U, ARR_EVEN, LEAN>(ch, lds_array{(const LDSQ int32_t *)(dsr_lds + cb_bytes(T.nw) + aoff)}, alen, L, sp, deal, lane,
                                claim, A);
}

/* Shared scalars are wave-uniform: read once as uniform values, they live in
 * scalar registers. */
__device__ __forceinline__ uint32_t uniform_u32(const uint8_t *p)
{
    return uniform(*(const uint32_t *)p);
}

/* Shared-array gather; arrays at `arr` (LDS or global pointer), `len`
 * elements each. */
__device__ __forceinline__ i32x4 load4(const LDSQ int32_t *p) { return *(const LDSQ i32x4 *)p; }
__device__ __forceinline__ i32x4 load4(const GLB int32_t *p) { return *(const GLB i32x4 *)p; }

/* V consecutive outputs of one lane. */
template <int V>
struct gather_vec {
    uint32_t e[V];
};

template <int NA, int V, class AP>
__device__ __forceinline__ gather_vec<V> gather_sum(AP arr, uint32_t len, uint32_t na, uint32_t idx)
{
    gather_vec<V> s;
#pragma unroll
    for (int k = 0; k < V; ++k) s.e[k] = 0;
    AP a = arr + idx;
    auto add = [&]() {
        if constexpr (V == 4) {
            const i32x4 v = load4(a);
            s.e[0] += (uint32_t)v.x;
            s.e[1] += (uint32_t)v.y;
            s.e[2] += (uint32_t)v.z;
            s.e[3] += (uint32_t)v.w;
        } else {
            s.e[0] += (uint32_t)*a;
        }
        a += len;
    };
    if constexpr (NA > 0) {
#pragma unroll
        for (int j = 0; j < NA; ++j) add();
    } else {
#pragma nounroll
        for (uint32_t j = 0; j < na; ++j) add();
    }
    return s;
}

template <int V>
__device__ __forceinline__ void gather_store(GLB int32_t *out, uint32_t i, const gather_vec<V> &s)
{
    if constexpr (V == 4) {
        const i32x4 r = {(int32_t)(s.e[0] + i), (int32_t)(s.e[1] + i + 1), (int32_t)(s.e[2] + i + 2),
                         (int32_t)(s.e[3] + i + 3)};
        __builtin_nontemporal_store(r, (GLB out_quad *)(out + i));
    } else {
        __builtin_nontemporal_store((int32_t)(s.e[0] + i), out + i);
    }
}

/* One lane's share of a gather: V outputs at i0, i0 + stride, ... below i1
 * (the last group may be cut short by i1).  V = 4 needs len and i0 to be
 * multiples of 4, so a group never wraps inside an array.  A loop has fewer
 * than 2^31 iterations, so every index is 32 bits wide, and the array index
 * is carried from group to group (one conditional subtraction) after one
 * division at the start (a 64-bit remainder per element had bound loops over
 * arrays of a ragged length).  Bound by the output stores; four groups go at
 * a time, their array reads (LDS or global) all in flight.  Launch and wait
 * of 10^7 outputs, 3 x 257, three levels: 68.0 -> 32.3 us; of 2^26 outputs,
 * 2 x 4096, two levels: 81.3 -> 66.7 us (with the lean instance, four
 * workgroups per CU instead of two). */
template <int NA, int V, class AP>
__device__ __forceinline__ void gather_run(AP arr, uint32_t len, uint32_t na, GLB int32_t *__restrict__ out,
                                           uint32_t i0, uint32_t i1, uint32_t stride)
{
    if (i0 >= i1) return;
    uint32_t i = i0, idx = i0 % len;
    const uint32_t step = stride % len;
#pragma nounroll
    for (; i + 3 * stride + V <= i1; i += 4 * stride) {
        const uint32_t x1 = mod_step(idx, step, len), x2 = mod_step(x1, step, len), x3 = mod_step(x2, step, len);
        const gather_vec<V> s0 = gather_sum<NA, V>(arr, len, na, idx), s1 = gather_sum<NA, V>(arr, len, na, x1),
                            s2 = gather_sum<NA, V>(arr, len, na, x2), s3 = gather_sum<NA, V>(arr, len, na, x3);
        gather_store<V>(out, i, s0);
        gather_store<V>(out, i + stride, s1);
        gather_store<V>(out, i + 2 * stride, s2);
        gather_store<V>(out, i + 3 * stride, s3);
        idx = mod_step(x3, step, len);
    }
#pragma nounroll
    for (; i + V <= i1; i += stride) {
        gather_store<V>(out, i, gather_sum<NA, V>(arr, len, na, idx));
        idx = mod_step(idx, step, len);
    }
    if constexpr (V > 1) {
#pragma nounroll
        for (; i < i1; ++i, ++idx) gather_store<1>(out, i, gather_sum<NA, 1>(arr, len, na, idx));
    }
}

/* Lane q of G lanes that share [lo, hi): groups of four outputs where the
 * arrays and the range allow it, single outputs otherwise; each store
 * instruction of the G lanes covers consecutive elements either way. */
template <int NA, class AP>
__device__ __forceinline__ void gather_lanes(AP arr, const dsr_dloop &L, uint32_t lo, uint32_t hi, uint32_t q,
                                             uint32_t G, bool vec)
{
    GLB int32_t *out = (GLB int32_t *)L.out;
    if (vec) gather_run<NA, 4>(arr, L.len, L.arrays, out, lo + 4 * q, hi, 4 * G);
    else gather_run<NA, 1>(arr, L.len, L.arrays, out, lo + q, hi, G);
}

/* ---- nested levels ----------------------------------------------------------
 * Part k of [lo, hi) cut into `parts` contiguous pieces whose lengths are
 * multiples of `gran` elements (4 keeps every piece on 16-byte vectors). */
__device__ __forceinline__ void split_range(uint64_t lo, uint64_t hi, uint32_t parts, uint32_t k, uint32_t gran,
                                            uint64_t &a, uint64_t &b)
{
    const uint64_t n = hi > lo ? hi - lo : 0;
    uint64_t per = (n + parts - 1) / parts;
    per = (per + gran - 1) / gran * gran;
    a = min(hi, lo + (uint64_t)k * per);
    b = min(hi, a + per);
}

/* The lanes of one gather loop: lane q of G shares [lo, hi) of the team frame
 * at (space, off). */
struct gather_t {
    uint32_t space, off, lo, hi, q, G;
};

/* The gather loop itself, at one place for the flat and the nested bodies:
 * the array count as a constant (0: more than four), the arrays in LDS or in
 * global memory, groups of four outputs or single ones. */
__device__ __forceinline__ void gather_loop(const team_t &T, const dsr_dloop &L, const gather_t &g, bool vec)
{
    auto at = [&](auto arr) {
        switch (L.arrays) {
        case 1: gather_lanes<1>(arr, L, g.lo, g.hi, g.q, g.G, vec); break;
        case 2: gather_lanes<2>(arr, L, g.lo, g.hi, g.q, g.G, vec); break;
        case 3: gather_lanes<3>(arr, L, g.lo, g.hi, g.q, g.G, vec); break;
        case 4: gather_lanes<4>(arr, L, g.lo, g.hi, g.q, g.G, vec); break;
        default: gather_lanes<0>(arr, L, g.lo, g.hi, g.q, g.G, vec); break;
        }
    };
    if (g.space == SPACE_LDS) at((const LDSQ int32_t *)(dsr_lds + cb_bytes(T.nw) + g.off));
    else at((const GLB int32_t *)((g.space == SPACE_IMAGE ? T.image : T.stack_hbm) + g.off));
}

__device__ __forceinline__ bool gather_vec4(const dsr_dloop &L, span_t sp) { return !((L.len & 3u) || (sp.lo & 3u)); }

/* A nested fork or join inside one wave: the leader lanes' frame and
 * descriptor writes (LDS, or the global part of a member stack) become
 * visible to the wave's other lanes.  Workgroup scope covers both memories
 * (the wave's own CU). */
__device__ __forceinline__ void nest_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ uint32_t pack_place(frame_t f) { return (f.space << 24) | f.off; }

/* Nested levels below the team's fork (section 3.1.2; section 7's sharing
 * at worker level).  Level 1: this wave is member `member` of `members`
 * and takes its piece of the team's range.  It pushes the frame {lo, hi,
 * team frame's space, offset} on its own member stack, publishes it in its
 * descriptor and forks its inner team, the four 16-lane groups.  Level 2:
 * each group reads the descriptor, then the frame, and takes its pieces.  At
 * depth 2 its lanes gather through the team frame the frame names.  At
 * depth 3 each group's leader lane pushes a frame {lo, hi, the wave frame's
 * space, offset} on the group's own member stack and forks the group's
 * inner team, four 4-lane groups, which reach the team frame by following
 * the two references.  The inner members take chunks of the wave's range in
 * turn (one group of outputs per lane, as a cyclic static schedule does), so
 * that the wave's stores cover consecutive elements: with one contiguous
 * piece per 4-lane member a store instruction had touched 16 cache lines a
 * quarter full or less.  Frames are popped in LIFO order after each inner
 * team joins.  A member stack's frame goes to its on-chip part, or to its
 * global part when the on-chip part is full or `nest_global` is set; each
 * global part holds several nested frames, so no nested push fails. */
__device__ __forceinline__ void body_gather_nested(team_t &T, frame_t outer, const dsr_dloop &L, span_t sp,
                                                   uint32_t member, uint32_t members, uint32_t &inner_pushes,
                                                   GLB uint32_t *tr)
{
    static_assert(DSR_NEST_WAVE_HBM >= DSR_NEST_FRAME && DSR_NEST_GROUP_HBM >= DSR_NEST_FRAME,
                  "a global part holds at least one nested frame");
    const uint32_t depth = uniform(L.depth);
    const bool vec = gather_vec4(L, sp);
    const uint32_t gran = vec ? 4u : 1u;
    const uint32_t lane = T.lane;
    uint32_t *desc = nest_desc(T, member);
    /* level 1: this wave's piece and its frame */
    uint64_t mlo, mhi;
    split_range(sp.lo, sp.hi, members, member, gran, mlo, mhi);
    mstack_t ws = mstack(member * DSR_NEST_WAVE_LDS, DSR_NEST_WAVE_LDS, member * DSR_NEST_WAVE_HBM,
                         DSR_NEST_WAVE_HBM);
    const frame_t f2 = mpush(ws, DSR_NEST_FRAME, T.nest_global != 0);
    uint32_t *p2 = nest_addr(T, f2.space, f2.off);
    if (lane == 0) {
        p2[0] = (uint32_t)mlo;
        p2[1] = (uint32_t)mhi;
        p2[2] = outer.space;
        p2[3] = outer.off;
        desc[0] = f2.space;
        desc[1] = f2.off;
        if (tr) tr[128 + 8 * member] = pack_place(f2);
    }
    inner_pushes += 1;
    nest_sync();
    /* level 2: lane group g reads the published frame; its first chunk is 16
     * lanes' outputs, the next one a wave's outputs further on */
    const uint32_t g = lane >> 4, l = lane & 15u;
    const uint32_t d2s = desc[0], d2o = desc[1];
    const uint32_t *q2 = nest_addr(T, d2s, d2o);
    gather_t leaf{q2[2], q2[3], q2[0] + g * 16u * gran, q2[1], l, 64u};
    mstack_t gs{};
    frame_t f3{SPACE_NONE, 0, 0};
    if (depth != 2) {
        const uint32_t k = member * DSR_NEST_GROUPS + g;
        gs = mstack(members * DSR_NEST_WAVE_LDS + k * DSR_NEST_GROUP_LDS, DSR_NEST_GROUP_LDS,
                    members * DSR_NEST_WAVE_HBM + k * DSR_NEST_GROUP_HBM, DSR_NEST_GROUP_HBM);
        f3 = mpush(gs, DSR_NEST_FRAME, T.nest_global != 0);
        uint32_t *p3 = nest_addr(T, f3.space, f3.off);
        if (l == 0) {
            p3[0] = leaf.lo;
            p3[1] = leaf.hi;
            p3[2] = d2s;
            p3[3] = d2o;
            desc[2 + 2 * g] = f3.space;
            desc[3 + 2 * g] = f3.off;
            if (tr) tr[129 + 8 * member + g] = pack_place(f3);
        }
        inner_pushes += DSR_NEST_GROUPS;
        nest_sync();
        /* level 3: 4-lane group s of group g */
        const uint32_t s = l >> 2, q = l & 3u;
        const uint32_t *q3 = nest_addr(T, desc[2 + 2 * g], desc[3 + 2 * g]);
        const uint32_t *pp = nest_addr(T, q3[2], q3[3]);      /* the wave's frame */
        leaf = gather_t{pp[2], pp[3], q3[0] + s * 4u * gran, q3[1], q, 64u};
    }
    /* every lane follows the same chain to the same team frame */
    leaf.space = uniform(leaf.space);
    leaf.off = uniform(leaf.off);
    gather_loop(T, L, leaf, vec);
    if (depth != 2) {
        nest_sync();                                            /* inner join */
        if (!mpop(gs, f3) && tr) tr[133 + 8 * member] = 1;
    }
    nest_sync();                                                /* inner join */
    if (!mpop(ws, f2) && tr && lane == 0) tr[133 + 8 * member] = 1;
    if (tr && lane == 0) tr[134 + 8 * member] = inner_pushes;
}

__device__ __forceinline__ void body_gather(const team_t &T, frame_t f, const dsr_dloop &L, span_t sp)
{
    gather_loop(T, L, gather_t{f.space, f.off, (uint32_t)sp.lo, (uint32_t)sp.hi, sp.p, sp.P}, gather_vec4(L, sp));
}

/* Cross-team traffic (partials, arrival counters, results) uses
 * device-scope relaxed atomics: on gfx950 these are performed at the
 * device's coherence point, past the per-XCD L2 (which is not coherent
 * across XCDs), so a team's partial needs no L2 write-back (what a
 * device-scope release costs every team).  The hardware assumption this
 * rests on: a team waits for its partial's stores to complete (s_waitcnt)
 * before issuing its arrival atomic, and a store to the coherence point
 * that has completed is seen by any later device-scope read.  The last
 * arriver of a group and of the region takes a device-scope acquire
 * before reading the partials, once per group. */
__device__ __forceinline__ void store_dev(uint64_t *p, uint64_t v)
{
    __hip_atomic_store((GLB uint64_t *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t load_dev(const uint64_t *p)
{
    return __hip_atomic_load((const GLB uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void drain_memory() { __builtin_amdgcn_s_waitcnt(0); }


/* ---- region execution ---------------------------------------------------- */
__device__ __forceinline__ const uint8_t *frame_ptr(const team_t &T, frame_t f)
{
    return f.space == SPACE_LDS ? frame_lds(T, f) : frame_hbm(T, f);
}

/* The general instances run every body (fma chains with run-time counts).
 * VARIANT -1 (workgroups above 512 threads, 128 registers per lane) takes
 * fewer element pairs per batch. */
template <int VARIANT>
__device__ __forceinline__ void run_body(team_t &T, uint32_t body, frame_t f, const dsr_dloop &L, span_t sp,
                                         lane_acc &A, uint32_t *claim, uint32_t member,
                                         uint32_t members, uint32_t &inner_pushes, GLB uint32_t *tr)
{
    constexpr int U = VARIANT < 0 ? 1 : 8;
    const uint32_t lane = T.lane;
    switch (body) {
    case DSR_BODY_AFFINE_XOR: {
        /* frame layout: [8 B int64 sum][a][b][c][d] */
        const uint32_t a = uniform_u32((const uint8_t *)slot<int32_t>(T, f, 8));
        const uint32_t b = uniform_u32((const uint8_t *)slot<int32_t>(T, f, 12));
        const uint32_t c = uniform_u32((const uint8_t *)slot<int32_t>(T, f, 16));
        const uint32_t d = uniform_u32((const uint8_t *)slot<int32_t>(T, f, 20));
        GLB int32_t *out = (GLB int32_t *)L.out;
        for_spans(L, sp, lane, claim, A, [&](span_t q) { affine_span(a, b, c, d, out, q, A); });
        break;
    }
    case DSR_BODY_FMA_CHAIN:
    case DSR_BODY_FMA_CHAIN_REFS:
        body_chain<U, false>(T, body == DSR_BODY_FMA_CHAIN_REFS, f, L, sp, deal_t{0, 0}, A, claim, lane);
        break;
    case DSR_BODY_GATHER:
        for_spans(L, sp, lane, claim, A, [&](span_t q) { body_gather(T, f, L, q); });
        break;
    case DSR_BODY_GATHER_NESTED:
        body_gather_nested(T, f, L, sp, member, members, inner_pushes, tr);
        break;
    default:
        break;
    }
}

__device__ __forceinline__ span_t team_span(const dsr_dloop &L, uint32_t team, uint32_t p, uint32_t P)
{
    span_t s;
    s.lo = min(L.dyn_start, (uint64_t)team * L.chunk);
    s.hi = min(L.dyn_start, s.lo + L.chunk);
    s.p = p;
    s.P = P;
    return s;
}

/* A participating wave leaves its partial and its range flag (one 32-byte
 * reduction slot) for the join. */
__device__ __forceinline__ void deposit(const team_t &T, i192 w, uint32_t bad)
{
    if (T.lane == 0) {
        LDSQ uint64_t *r = (LDSQ uint64_t *)(dsr_lds + red_slot_at(T.wave));
        r[0] = w.w0;
        r[1] = w.w1;
        r[2] = w.w2;
        r[3] = bad;
    }
}

/* Master wave, after the join: the sum of the `nwork` participating waves'
 * partials, one wave's slot per lane, and whether any of them flagged a value
 * outside the exact-sum window. */
__device__ __forceinline__ i192 joined_sum(uint32_t lane, uint32_t nwork, uint32_t &bad)
{
    const bool mine = lane < nwork;
    const LDSQ uint64_t *q = (const LDSQ uint64_t *)(dsr_lds + red_slot_at(mine ? lane : 0));
    const uint64_t q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
    bad = __any(mine && q3 != 0);
    return row_sum192(mine ? i192{q0, q1, q2} : i192{0, 0, 0});
}

/* Run one participating wave's share of a published body and join. */
template <int VARIANT>
__device__ __forceinline__ void participate(team_t &T, const dsr_dregion &R, const dsr_dconfig &C,
                                            uint32_t team, uint32_t body, frame_t f, uint32_t loop,
                                            const dsr_dloop &L, uint32_t &inner_pushes)
{
    const uint32_t nwork = C.master_joins ? T.nw : T.nw - 1;
    /* keeps the compiler from computing every body's lane offsets ahead of the
     * await loop and holding them in registers across all bodies */
    asm volatile("" : "+v"(T.lane));
    lane_acc A = acc_zero();
    GLB uint32_t *tr = (C.trace && R.trace) ? (GLB uint32_t *)(R.trace + (uint64_t)team * DSR_TRACE_WORDS) : nullptr;
    if (tr && T.lane == 0) tr[96 + 2 * T.wave] = (uint32_t)wall_clock64();
    run_body<VARIANT>(T, body, f, L, team_span(L, team, T.wave * 64 + T.lane, nwork * 64), A,
                      &R.result->claim[loop], T.wave, nwork, inner_pushes, tr);
    if (tr && T.lane == 0) tr[97 + 2 * T.wave] = (uint32_t)wall_clock64();
    /* served form: the request completes while the kernel keeps running,
     * so this wave's output stores must have reached L2 before the join
     * (the master then writes the L2 back before the team arrives) */
    if (C.serve) drain_memory();
    deposit(T, wave_sum192(widen(A)), __any(A.bad != 0));
    __syncthreads();
}

/* Bytes o .. o+3 of src as a little-endian word, zero from `lim` on. */
__device__ __forceinline__ uint32_t ragged_word(const uint8_t *src, uint32_t o, uint32_t lim)
{
    uint32_t w = 0;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q)
        if (o + q < lim) w |= (uint32_t)src[o + q] << (8 * q);
    return w;
}

/* The 16-byte vectors [first, full) of an LDS frame's image, in rounds of 64
 * (one per lane) that lie `step` apart, by loads that write LDS themselves;
 * the next round's first vector.  Lane i's vector lands 16 i bytes after the
 * wave's LDS address. */
__device__ __forceinline__ uint32_t direct_rounds(const team_t &T, uint32_t off, const uint8_t *src, uint32_t first,
                                                  uint32_t full, uint32_t step)
{
    const GLB uint8_t *g = (const GLB uint8_t *)src + 16u * T.lane;
    LDSQ uint8_t *l = (LDSQ uint8_t *)(dsr_lds + cb_bytes(T.nw) + off);
    for (; first + 64u <= full; first += step)
        __builtin_amdgcn_global_load_lds((const GLB uint32_t *)(g + 16u * first), (LDSQ uint32_t *)(l + 16u * first), 16, 0,
                                         0);
    return first;
}

/* Copy a frame's initial bytes (or zeros) with the whole master wave.  What
 * bounds it is the latency of a round of loads, so from global memory to LDS
 * the 16-byte vectors that lie wholly inside the initial bytes go by loads
 * that write LDS themselves: they hold no registers, and all those of a
 * 32 KiB frame are in flight together, where four rounds through registers
 * had followed each other (launch and wait of a chain over 2^20 outputs with
 * a 32 KiB frame 67.5 -> 65.7 us; of nested gathers over 2^26 outputs, 2048
 * teams with 32 KiB each, 63.3 -> 61.2 us).  To HBM, and from a served request's
 * copy in LDS (global = false), they go through registers in rounds of eight
 * per lane.  The first `under_way` vectors (whole rounds) are being copied
 * already.  The rest is zeros or a ragged edge. */
__device__ __forceinline__ void init_frame(team_t &T, frame_t f, const uint8_t *src, uint32_t init_bytes,
                                           uint32_t nbytes, bool global, uint32_t under_way = 0)
{
    uint8_t *dst = (uint8_t *)frame_ptr(T, f);
    const uint32_t nvec = nbytes >> 4;
    const bool src_aligned = (((uintptr_t)src) & 15u) == 0;
    const uint32_t full = src_aligned ? min(init_bytes, nbytes) >> 4 : 0;
    const uint4 *s4 = (const uint4 *)src;
    uint4 *d4 = (uint4 *)dst;
    uint32_t direct = under_way;
    if (global && f.space == SPACE_LDS && full >= 64u) {
        /* this wave's own writes to a popped frame here land first */
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        direct = direct_rounds(T, f.off, src, direct, full, 64u);
    }
    for (uint32_t k0 = direct + T.lane; k0 < full; k0 += 512) {
        const uint32_t k1 = k0 + 64, k2 = k0 + 128, k3 = k0 + 192, k4 = k0 + 256, k5 = k0 + 320,
                       k6 = k0 + 384, k7 = k0 + 448;
        /* indices past the end reload the last vector (always in bounds);
         * their stores are skipped */
        const uint32_t last = full - 1;
        const uint4 v0 = s4[k0];
        const uint4 v1 = s4[min(k1, last)], v2 = s4[min(k2, last)], v3 = s4[min(k3, last)];
        const uint4 v4 = s4[min(k4, last)], v5 = s4[min(k5, last)], v6 = s4[min(k6, last)];
        const uint4 v7 = s4[min(k7, last)];
        d4[k0] = v0;
        if (k1 < full) d4[k1] = v1;
        if (k2 < full) d4[k2] = v2;
        if (k3 < full) d4[k3] = v3;
        if (k4 < full) d4[k4] = v4;
        if (k5 < full) d4[k5] = v5;
        if (k6 < full) d4[k6] = v6;
        if (k7 < full) d4[k7] = v7;
    }
    for (uint32_t k = full + T.lane; k < nvec; k += 64) {
        const uint32_t o = k * 16;
        d4[k] = make_uint4(ragged_word(src, o, init_bytes), ragged_word(src, o + 4, init_bytes),
                           ragged_word(src, o + 8, init_bytes), ragged_word(src, o + 12, init_bytes));
    }
    for (uint32_t o = nvec * 16 + T.lane; o < nbytes; o += 64) dst[o] = o < init_bytes ? src[o] : 0;
    /* the workers read the frame after the hand-over barrier, which waits for
     * LDS operations but not for these loads */
    if (direct) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

/* The region's program, one op per lane of the master wave: all ops are
 * loaded in one round trip when the program starts, and each step takes
 * its op with readlanes, so no op load waits behind the parallel region. */
struct op_lanes {
    uint32_t w[10];
};

__device__ __forceinline__ op_lanes load_ops(const dsr_op *ops, uint32_t n, uint32_t lane)
{
    op_lanes o;
#pragma unroll
    for (int i = 0; i < 10; ++i) o.w[i] = 0;
    if (lane < n) {
        const uint4 *p = (const uint4 *)(ops + lane);
        const uint4 a = p[0], b = p[1], c = p[2];
        o.w[0] = a.x; o.w[1] = a.y; o.w[2] = a.z; o.w[3] = a.w;
        o.w[4] = b.x; o.w[5] = b.y; o.w[6] = b.z; o.w[7] = b.w;
        o.w[8] = c.x; o.w[9] = c.y;
    }
    return o;
}

__device__ __forceinline__ dsr_op op_at(const op_lanes &o, uint32_t k)
{
    dsr_op op;
    op.kind = __builtin_amdgcn_readlane(o.w[0], k);
    op.frame = __builtin_amdgcn_readlane(o.w[1], k);
    op.nbytes = __builtin_amdgcn_readlane(o.w[2], k);
    op.init_bytes = __builtin_amdgcn_readlane(o.w[3], k);
    op.init_stride = __builtin_amdgcn_readlane(o.w[4], k);
    op.body = __builtin_amdgcn_readlane(o.w[5], k);
    op.loop = __builtin_amdgcn_readlane(o.w[6], k);
    op.red = __builtin_amdgcn_readlane(o.w[7], k);
    op.init_off = (uint64_t)__builtin_amdgcn_readlane(o.w[8], k) |
                  ((uint64_t)__builtin_amdgcn_readlane(o.w[9], k) << 32);
    op.pad = 0;
    return op;
}

/* The region descriptor fields the arrival and the combine use, held in
 * registers: read once before the arrival atomics, so no fence between
 * them makes the last team reload the descriptor from memory. */
struct region_sums {
    uint64_t *partials;
    dsr_dresult *result;
    dsr_hred *out;
    int32_t *status;
    uint32_t teams, n_red, red_kind_mask;
};

__device__ __forceinline__ region_sums sums_of(const dsr_dregion &R)
{
    region_sums S;
    S.partials = R.partials;
    S.result = R.result;
    S.out = R.out;
    S.status = R.status;
    S.teams = uniform(R.teams);
    S.n_red = uniform(R.n_red);
    S.red_kind_mask = uniform(R.red_kind_mask);
    return S;
}

/* Master wave: this team's partial of one reduction, a word per lane. */
__device__ __forceinline__ void store_partial(uint64_t *pp, i192 sv, uint32_t lane)
{
    if (lane < DSR_PART_WORDS) store_dev(pp + lane, lane == 0 ? sv.w0 : (lane == 1 ? sv.w1 : sv.w2));
}

/* Master wave: add the join's total into the shared sum at c (an int64
 * for the integer body, else a 192-bit integer in 2^-75 units) and return
 * the new value as 192 bits. */
template <class P>
__device__ __forceinline__ i192 update_sum(P c, i192 tot, bool integer_sum, uint32_t lane)
{
    i192 sv;
    if (integer_sum) {
        const int64_t nv = (int64_t)(c[0] + tot.w0);
        sv = i192{(uint64_t)nv, (uint64_t)(nv >> 63), (uint64_t)(nv >> 63)};
        wave_sync();
        if (lane == 0) c[0] = (uint64_t)nv;
    } else {
        sv = add192(tot, i192{c[0], c[1], c[2]});
        wave_sync();
        if (lane == 0) {
            c[0] = sv.w0;
            c[1] = sv.w1;
            c[2] = sv.w2;
        }
    }
    return sv;
}

/* Master wave: the sequential code block of one region for one team
 * (Figure 2): pushes, publishes and pops.  Returns the team's error. */
template <int VARIANT>
__device__ __forceinline__ int32_t run_program(team_t &T, const dsr_dregion &R, const dsr_dconfig &C,
                                               uint32_t region, uint32_t team, uint32_t &barriers,
                                               uint32_t &inner_pushes)
{
    cb_header *h = header(T);
    /* trace words go through a global-space pointer: a generic store is
     * counted with the LDS accesses too, and the next LDS wait would wait
     * for the stamp to reach memory */
    GLB uint32_t *tr = (C.trace && R.trace) ? (GLB uint32_t *)(R.trace + (uint64_t)team * DSR_TRACE_WORDS) : nullptr;
    if (tr && T.lane == 0) tr[86] = (uint32_t)wall_clock64();
    wave_sync();
    int32_t err = 0;
    uint32_t npush = 0;
    bool stamped = false;
    const uint32_t nwork = C.master_joins ? T.nw : T.nw - 1;
    const uint32_t n_ops = min(uniform(R.n_ops), (uint32_t)DSR_MAX_OPS);
    /* read once, before any join: after a barrier the compiler would load
     * them from memory again, behind this wave's outstanding stores */
    const region_sums RS = sums_of(R);
    /* the 1024-thread instance has no registers to spare: it reads each op
     * when it gets to it */
    const op_lanes prog = load_ops(R.ops, VARIANT < 0 ? 0 : n_ops, T.lane);
    for (uint32_t k = 0; k < n_ops; ++k) {
        const dsr_op op = VARIANT < 0 ? R.ops[k] : op_at(prog, k);
        if (op.kind == DSR_OP_PUSH) {
            const frame_t f = push(T, op.nbytes);
            if (f.space == SPACE_NONE) { err = DSR_E_NOMEM; break; }
            if (tr && T.lane == 0 && npush < 16) {
                tr[1 + 3 * npush] = f.space;
                tr[2 + 3 * npush] = f.off;
                tr[3 + 3 * npush] = f.size;
            }
            npush++;
            init_frame(T, f, R.init + op.init_off + (uint64_t)team * op.init_stride, op.init_bytes, op.nbytes, !C.serve);
        } else if (op.kind == DSR_OP_PUBLISH) {
            frame_t f, lf{SPACE_NONE, 0, 0};
            if (op.body == DSR_BODY_FMA_CHAIN_REFS) {
                /* section 5.2: resolve each (frame, offset) reference to a
                 * stack address and write the list on chip, or to a list
                 * frame on the HBM stack when it is longer than the on-chip
                 * list (or global lists are asked for) */
                const uint32_t n = op.nbytes;
                const uint32_t *tab = (const uint32_t *)(R.init + op.init_off);
                const bool glist = n > DSR_REF_LIST || C.global_lists;
                uint32_t *dst = ref_list(T);
                if (glist) {
                    lf = push(T, 8 * n, true);
                    if (lf.space == SPACE_NONE) { err = DSR_E_NOMEM; break; }
                    dst = (uint32_t *)frame_hbm(T, lf);
                    f = frame_t{SPACE_HBM, lf.off, n};
                } else {
                    f = frame_t{SPACE_LIST, 0, n};
                }
                for (uint32_t k = T.lane; k < n; k += 64) {
                    const uint32_t *fte = frame_table(T) + 4 * tab[2 * k];
                    dst[2 * k] = fte[0];
                    dst[2 * k + 1] = fte[1] + tab[2 * k + 1];
                }
                if (tr && T.lane == 0) {
                    tr[89] = glist ? SPACE_HBM : SPACE_LIST;
                    tr[90] = f.off;
                    tr[91] = n;
                }
            } else {
                const uint32_t *ft = frame_table(T) + 4 * op.frame;
                f.space = uniform(ft[0]);
                f.off = uniform(ft[1]);
                f.size = uniform(ft[2]);
            }
            if (T.lane == 0) {
                h->region = region;
                h->team = team;
            }
            publish(T, f, op.body, op.loop);
            barriers++;
            if (tr && T.lane == 0 && !stamped) {
                const uint64_t t0 = wall_clock64();
                tr[82] = (uint32_t)t0;
                tr[83] = (uint32_t)(t0 >> 32);
            }
            stamped = true;
            /* the 1024-thread instance has no registers for a participating
             * master; the host never asks it to (teams above 512 threads) */
            if (VARIANT >= 0 && C.master_joins) {
                participate<VARIANT>(T, R, C, team, op.body, f, op.loop, R.loops[op.loop], inner_pushes);
            } else {
                __syncthreads();             /* the join (barrier 2) */
            }
            barriers++;
            if (tr && T.lane == 0) {
                const uint64_t t1 = wall_clock64();
                tr[84] = (uint32_t)t1;
                tr[85] = (uint32_t)(t1 >> 32);
            }
            /* join done: combine the participating waves' partials */
            uint32_t bad;
            const i192 tot = joined_sum(T.lane, nwork, bad);
            if (bad) err = DSR_E_RANGE;
            if (op.red != 0xffffffffu) {
                /* the shared sum: the frame's first bytes, or where reference
                 * 0 of the list points; read and written through a pointer
                 * of its own memory space (a generic access would also wait
                 * for this wave's outstanding loop stores) */
                uint32_t s_space = f.space, s_off = f.off;
                if (op.body == DSR_BODY_FMA_CHAIN_REFS) {
                    const uint32_t *lst = f.space == SPACE_LIST ? ref_list(T) : (const uint32_t *)frame_hbm(T, f);
                    s_space = uniform(lst[0]);
                    s_off = uniform(lst[1]);
                }
                const bool integer_sum = op.body == DSR_BODY_AFFINE_XOR;
                /* the team's partial is stored inside each branch: where the
                 * two would merge the compiler waits for every outstanding
                 * memory operation of the wave, its loop stores included */
                uint64_t *pp = RS.partials + ((uint64_t)op.red * RS.teams + team) * DSR_PART_WORDS;
                if (s_space == SPACE_LDS)
                    store_partial(pp, update_sum((LDSQ uint64_t *)(dsr_lds + cb_bytes(T.nw) + s_off), tot,
                                                 integer_sum, T.lane), T.lane);
                else
                    store_partial(pp, update_sum((GLB uint64_t *)(T.stack_hbm + s_off), tot, integer_sum, T.lane),
                                  T.lane);
            }
            wave_sync();
            /* a global reference list dies with its parallel region */
            if (lf.space == SPACE_HBM && !pop(T, lf)) err = DSR_E_ORDER;
            if (err) break;
        } else if (op.kind == DSR_OP_POP) {
            const uint32_t nf = uniform(h->nframes);
            if (nf == 0) { err = DSR_E_UNDERFLOW; break; }
            const uint32_t *ft = frame_table(T) + 4 * (nf - 1);
            frame_t f;
            f.space = uniform(ft[0]);
            f.off = uniform(ft[1]);
            f.size = uniform(ft[2]);
            if (!pop(T, f)) { err = DSR_E_ORDER; break; }
        }
    }
    if (tr && T.lane == 0) {
        tr[0] = npush;
        tr[81] = (uint32_t)err;
    }
    if (err && T.lane == 0) atomicCAS(&R.result->error, 0, err);
    return err;
}

/* Sum `cnt` 192-bit partials (three words each, `stride` partials apart)
 * with the whole wave: each lane takes up to eight partials per round, so up
 * to 512 cost one memory round trip. */
__device__ __forceinline__ i192 sum_partials(const uint64_t *base, uint32_t cnt, uint32_t stride, uint32_t lane)
{
    i192 s{0, 0, 0};
    if (cnt <= 64) {
        /* one load round of one partial per lane, a third of the instructions */
        if (lane < cnt) {
            const uint64_t *pp = base + (uint64_t)DSR_PART_WORDS * lane * stride;
            s = i192{load_dev(pp), load_dev(pp + 1), load_dev(pp + 2)};
        }
        return wave_sum192(s);
    }
    constexpr uint32_t PER = 8;
    for (uint32_t j0 = 0; j0 < cnt; j0 += 64 * PER) {
        uint64_t w[PER][3];
#pragma unroll
        for (uint32_t u = 0; u < PER; ++u) {
            const uint32_t j = j0 + 64u * u + lane;
            const uint64_t *pp = base + (uint64_t)DSR_PART_WORDS * j * stride;
            const bool in = j < cnt;
            w[u][0] = in ? load_dev(pp) : 0;
            w[u][1] = in ? load_dev(pp + 1) : 0;
            w[u][2] = in ? load_dev(pp + 2) : 0;
        }
#pragma unroll
        for (uint32_t u = 0; u < PER; ++u) s = add192(s, i192{w[u][0], w[u][1], w[u][2]});
    }
    return wave_sum192(s);
}

/* Last team: the region's reductions from the (group) partials, exact in
 * 192-bit integers, rounded once for fp64. */
__device__ __forceinline__ void combine_teams(const region_sums &R, uint32_t cnt, uint32_t stride, uint32_t lane,
                                              dsr_drec *rec, dsr_result_rec *pub)
{
    for (uint32_t r = 0; r < R.n_red; ++r) {
        const i192 s = sum_partials(R.partials + (uint64_t)r * R.teams * DSR_PART_WORDS, cnt, stride, lane);
        if (lane == 0) {
            GLB dsr_hred *out = (GLB dsr_hred *)R.out + r;
            const double f = ((R.red_kind_mask >> r) & 1u) ? fixed_to_double(s) : (double)(int64_t)s.w0;
            out->fixed[0] = s.w0;
            out->fixed[1] = s.w1;
            out->fixed[2] = s.w2;
            out->f64 = f;
            out->i64 = (int64_t)s.w0;
            /* served form: the completion record gets the same values */
            if (rec && r < DSR_MAX_RED) {
                rec->fixed[r][0] = s.w0;
                rec->fixed[r][1] = s.w1;
                rec->fixed[r][2] = s.w2;
                rec->i64[r] = (int64_t)s.w0;
                rec->f64[r] = f;
            }
            if (pub && r < DSR_MAX_RED) {
                GLB dsr_result_rec *p = (GLB dsr_result_rec *)pub;
                p->fixed[r][0] = s.w0;
                p->fixed[r][1] = s.w1;
                p->fixed[r][2] = s.w2;
                p->i64[r] = (int64_t)s.w0;
                p->f64[r] = f;
            }
        }
    }
}

/* Served form: finish a region's host-coherent completion record (its
 * sums are already there) and release the ticket; the system-scope release
 * also writes this XCD's L2 back, outputs included. */
__device__ __forceinline__ void publish_record(uint32_t n_red, uint64_t tag, dsr_drec *rec, int32_t err, uint32_t lane)
{
    if (lane != 0) return;
    rec->status = err;
    rec->n_red = n_red;
    rec->ticks = wall_clock64();
    __hip_atomic_store(&rec->seq, tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

/* Launch without allocation: the rest of the caller's public record. */
__device__ __forceinline__ void public_record(dsr_result_rec *pub, uint32_t n_red, int32_t err, uint32_t lane)
{
    GLB dsr_result_rec *p = (GLB dsr_result_rec *)pub;
    if (lane == 0) {
        p->status = err;
        p->n_red = (int32_t)n_red;
    }
    if (lane >= n_red && lane < DSR_MAX_RED) {
        p->f64[lane] = 0.0;
        p->i64[lane] = 0;
        for (int w = 0; w < 3; ++w) p->fixed[lane][w] = 0;
    }
}

/* A team's arrival after its program.  Arrivals go through a two-level
 * tree (groups of teams, then groups) so that no counter sees more than a
 * few dozen simultaneous atomics.  With up to 512 teams the last team
 * reads every partial in one round; with more, the last team of each group
 * first adds up its group's partials and leaves the sum in the group's
 * first partial slot, and the last team overall adds the group sums. */
__device__ __forceinline__ void finish_team(const region_sums &R, uint32_t team, uint32_t lane, uint64_t *done_ts,
                                            dsr_drec *rec, const dsr_dregion *served, dsr_result_rec *pub,
                                            GLB uint32_t *tr)
{
    uint32_t gsize = R.teams, ngroups = 1, g = 0, in_group = R.teams;
    if (R.teams > DSR_FLAT_TEAMS) {
        gsize = (R.teams + DSR_ARRIVE_GROUPS - 1) / DSR_ARRIVE_GROUPS;
        ngroups = (R.teams + gsize - 1) / gsize;
        g = team / gsize;
        in_group = min(gsize, R.teams - g * gsize);
    }
    const bool group_sums = R.teams > 512;
    drain_memory();                      /* this team's partials are stored */
    if (tr && lane == 0) tr[92] = (uint32_t)wall_clock64();
    GLB dsr_dresult *res = (GLB dsr_dresult *)R.result;
    uint32_t prev = 0;
    /* a region of one team has nothing to arrive at: this wave wrote every
     * partial and the error word itself */
    if (R.teams > 1) {
        if (lane == 0)
            prev = __hip_atomic_fetch_add(&res->group[g * 16], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        prev = uniform((uint32_t)__shfl((int)prev, 0, 64));
        if (tr && lane == 0) tr[93] = (uint32_t)wall_clock64();
        if (prev != in_group - 1) return;
        /* the last arriver of a group reads the others' partials: acquire */
        if (DSR_ARRIVE_FENCE) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (lane == 0) __hip_atomic_store(&res->group[g * 16], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (tr && lane == 0) {
        tr[93] = (uint32_t)wall_clock64();
    }
    if (ngroups > 1) {
        if (group_sums) {
            for (uint32_t r = 0; r < R.n_red; ++r) {
                uint64_t *gp = R.partials + ((uint64_t)r * R.teams + (uint64_t)g * gsize) * DSR_PART_WORDS;
                const i192 s = sum_partials(gp, in_group, 1, lane);
                if (lane == 0) {
                    store_dev(gp, s.w0);
                    store_dev(gp + 1, s.w1);
                    store_dev(gp + 2, s.w2);
                }
            }
            drain_memory();              /* the group sums are stored */
        }
        if (lane == 0)
            prev = __hip_atomic_fetch_add(&res->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        prev = uniform((uint32_t)__shfl((int)prev, 0, 64));
        if (prev != ngroups - 1) return;
        if (DSR_ARRIVE_FENCE) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (lane == 0) __hip_atomic_store(&res->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (tr && lane == 0) tr[94] = (uint32_t)wall_clock64();
    /* the error word, the partials and the counters are read and reset in
     * one round trip: nothing below waits on anything but the loads */
    int32_t err = 0;
    if (lane == 0) err = __hip_atomic_exchange(&res->error, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane < DSR_MAX_LOOPS) __hip_atomic_store(&res->claim[lane], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ngroups > 1 && group_sums) combine_teams(R, ngroups, gsize, lane, rec, pub);
    else combine_teams(R, R.teams, 1, lane, rec, pub);
    if (lane == 0) {
        *(GLB int32_t *)R.status = err;
        if (done_ts) *done_ts = wall_clock64();
        if (tr) tr[95] = (uint32_t)wall_clock64();
    }
    if (pub) public_record(pub, R.n_red, err, lane);
    if (rec) publish_record(R.n_red, served->tag, rec, err, lane);
}

/* Served form: close the server (one workgroup does it; see wait_item).
 * The device announces the close in host memory, then reads the host's
 * published count once more: the host publishes, then reads the closing
 * flag, so at least one side sees the other's write (both orders are
 * sequentially consistent at system scope, and a read from the device to
 * host memory does not pass the device's earlier write to it).  Every item
 * below the count read here is served; none above it is.  The count is
 * returned to the host, which takes back a request it published too late. */
__device__ __forceinline__ void close_server(const dsr_dlaunch &LP, uint32_t reason, uint32_t it, uint32_t pub,
                                             uint64_t idle)
{
    uint32_t *ctr = LP.counter;
    uint32_t open = 0;
    if (!__hip_atomic_compare_exchange_strong(ctr + DSR_SRV_STATE, &open, 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT))
        return;
    /* why, for the host's status: the reason (1 stop, 2 idle), the closing
     * workgroup, the item it waited for, the published count it saw and
     * the idle ticks it measured */
    uint32_t *why = LP.closing + 1;
    __hip_atomic_store(why, reason, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(why + 1, (uint32_t)blockIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(why + 2, it, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(why + 3, pub, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(why + 4, (uint32_t)idle, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(why + 5, (uint32_t)(idle >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(LP.closing, 1u, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_SYSTEM);
    __atomic_thread_fence(__ATOMIC_SEQ_CST);
    const uint32_t h = __hip_atomic_load(LP.published, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_fetch_max(ctr + DSR_SRV_PUB, h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(ctr + DSR_SRV_FINAL, h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(LP.final_items, h + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(ctr + DSR_SRV_STATE, 2u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

/* Served form: wait until item `it` is published (true: run it) or the
 * server has closed below it (false: leave).
 *
 * The host's published count lives in host memory, so polling it crosses
 * the host link; only the DSR_HOST_POLLERS workgroups holding the next
 * unpublished items poll the host, and they mirror what they see into
 * device memory, where every other waiting workgroup polls.  Polls are
 * relaxed (an acquire per poll would invalidate the L2 each time) and back
 * off with sleeps; once the item is seen, one agent-scope acquire makes
 * the request's device-memory inputs visible.
 *
 * Closing is one decision for the whole server, never a workgroup's own:
 * it happens when the host asks to stop, or when a waiting workgroup has
 * seen the device copy of the published count stay unchanged for
 * idle_limit ticks of its own clock.  The server then serves every item published before
 * the close and no other, so a workgroup leaves only while holding an
 * item nobody will publish to it, and no claimed item is lost.  Nothing
 * here waits for another workgroup, so the server does not rely on its
 * whole grid being resident at once. */
#define DSR_HOST_POLLERS 16u

__device__ __forceinline__ bool wait_item(const dsr_dlaunch &LP, uint32_t it, uint32_t lane, uint64_t &item)
{
    uint32_t ok = 0;
    const uint64_t *ring = (const uint64_t *)LP.items;
    if (lane == 0) {
        uint32_t *ctr = LP.counter;
        uint32_t nap = 0;
        /* idleness is timed on this wave's own clock from the last change
         * of the published count it saw: clocks of different workgroups
         * (other XCDs) are never compared */
        uint32_t seen = __hip_atomic_load(ctr + DSR_SRV_PUB, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint64_t seen_at = (uint64_t)wall_clock64();
        for (;;) {
            const uint32_t pub = __hip_atomic_load(ctr + DSR_SRV_PUB, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (it < pub) { ok = 1; break; }
            if (pub != seen) {
                seen = pub;
                seen_at = (uint64_t)wall_clock64();
            }
            const uint32_t st = __hip_atomic_load(ctr + DSR_SRV_STATE, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
            if (st == 2) {
                /* closed: items below the final count were made visible
                 * through the published copy above; this one is beyond it */
                if (it >= __hip_atomic_load(ctr + DSR_SRV_FINAL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
                continue;
            }
            if (st == 0) {
                if (it - pub < DSR_HOST_POLLERS) {
                    /* the workgroups holding the next items read the host's
                     * count themselves (a later team of a request need not
                     * wait for the device copy); the item is read in the same
                     * round, and its sequence field tells whether it is
                     * already this one */
                    const uint32_t h = __hip_atomic_load(LP.published, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    item = __hip_atomic_load(ring + (it & LP.ring_mask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    /* taken only while the server is still open: once a
                     * close has begun, items count as published up to the
                     * close's final count alone, which the closed branch
                     * above hands out */
                    if ((int32_t)(h - it) > 0 &&
                        __hip_atomic_load(ctr + DSR_SRV_STATE, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT) == 0) {
                        __hip_atomic_fetch_max(ctr + DSR_SRV_PUB, h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        ok = 1;
                        break;
                    }
                    if (it == pub && __hip_atomic_load(LP.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) {
                        close_server(LP, 1u, it, pub, 0);
                        continue;
                    }
                    nap = 0;
                }
                const uint64_t idle = (uint64_t)wall_clock64() - seen_at;
                if (idle > LP.idle_limit) {
                    close_server(LP, 2u, it, pub, idle);
                    continue;
                }
            }
            /* s_sleep takes an immediate (64 * n clocks); workgroups whose
             * item is far from the next one published sleep longest */
            if (it - pub >= 64) {
                __builtin_amdgcn_s_sleep(127);
                __builtin_amdgcn_s_sleep(127);
                __builtin_amdgcn_s_sleep(127);
                __builtin_amdgcn_s_sleep(127);
            } else {
                switch (nap) {
                case 0: __builtin_amdgcn_s_sleep(1); break;
                case 1: __builtin_amdgcn_s_sleep(2); break;
                case 2: __builtin_amdgcn_s_sleep(4); break;
                case 3: __builtin_amdgcn_s_sleep(8); break;
                case 4: __builtin_amdgcn_s_sleep(16); break;
                default: __builtin_amdgcn_s_sleep(32); break;
                }
                if (nap < 5) ++nap;
            }
        }
    }
    ok = __shfl((int)ok, 0, 64);
    if (ok) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (ok && lane == 0) {
        /* published before the count that was seen: a word still holding an
         * older sequence is read again (bounded, so a broken ring cannot
         * hold the workgroup).  Sequences start at 1: a word of the cleared
         * ring is no item, whichever item this workgroup waits for */
        for (uint32_t k = 0; (uint32_t)(item >> 32) != it + 1u && k < (1u << 22); ++k)
            item = __hip_atomic_load(ring + (it & LP.ring_mask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return ok != 0;
}

/* Served form: the request slot's descriptor, program and loop
 * descriptors live in host memory that the host rewrites between
 * requests; the master copies them into LDS with system-scope loads (never
 * through the scalar cache, which is not kept coherent with the host) and
 * points the copy's ops/loops at the LDS copies. */
__device__ __forceinline__ dsr_dregion *serve_area(const team_t &T)
{
    return (dsr_dregion *)(T.stack_lds + T.lds_cap);
}

/* Served form, large images: team 0 of the request copies the init blob
 * from the host slot into the slot's device buffer, and the other teams
 * wait for it there instead of each reading the whole blob across the
 * host link (64 teams of a 32 KiB image would move 2 MiB over it).  The
 * flag holds the ticket whose images the buffer holds; tickets are unique,
 * so it is never cleared.  A team that does not see its ticket within the
 * spin bound reads the host slot, which is always correct. */
__device__ __forceinline__ bool relay_images(const dsr_dregion *Rl, uint32_t team, uint32_t lane,
                                             uint32_t *count)
{
    GLB uint8_t *dst = (GLB uint8_t *)Rl->relay;
    GLB uint64_t *flag = (GLB uint64_t *)Rl->relay_flag;
    const uint64_t tag = Rl->tag;
    if (team == 0) {
        /* the slot is padded past the blob to a multiple of 256 bytes */
        const uint32_t nv = (Rl->init_size + 15u) >> 4;
        const i32x4 *src = (const i32x4 *)Rl->init;
        GLB i32x4 *d4 = (GLB i32x4 *)dst;
        for (uint32_t k0 = lane; k0 < nv; k0 += 512) {
            i32x4 v[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) {
                const uint32_t k = k0 + 64u * u;
                v[u] = src[min(k, nv - 1)];
            }
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u)
                if (k0 + 64u * u < nv) d4[k0 + 64u * u] = v[u];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (lane == 0) {
            __hip_atomic_store(flag, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (count) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return true;
    }
    uint32_t seen = 0;
    if (lane == 0) {
        for (uint32_t spin = 0; spin < (1u << 20); ++spin) {
            if (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag) {
                seen = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        if (!seen && count) __hip_atomic_fetch_add(count + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return __shfl((int)seen, 0, 64) != 0;
}

__device__ __forceinline__ const dsr_dregion &stage_request(team_t &T, const uint8_t *slot, uint32_t team,
                                                           uint32_t *relays)
{
    /* the slot's head has the layout of this LDS area: one round of loads
     * brings the descriptor, the ops and the loop descriptors together */
    dsr_dregion *Rl = serve_area(T);
    uint8_t *ops_l = (uint8_t *)Rl + DSR_SERVE_OPS_AT;
    uint8_t *loops_l = (uint8_t *)Rl + DSR_SERVE_LOOPS_AT;
    {
        /* every load issued before any store: one host round trip for the
         * head and the first DSR_SERVE_IMG_LDS bytes of the frame images */
        constexpr uint32_t NW = DSR_SERVE_AREA_BYTES / 8, PER = (NW + 63) / 64;
        const uint64_t *src = (const uint64_t *)slot;
        uint64_t *dst = (uint64_t *)Rl;
        uint64_t v[PER];
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r) {
            const uint32_t k = T.lane + 64u * r;
            v[r] = k < NW ? __hip_atomic_load(src + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) : 0ull;
        }
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r) {
            const uint32_t k = T.lane + 64u * r;
            if (k < NW) dst[k] = v[r];
        }
    }
    wave_sync();
    const uint32_t n_ops = min(uniform(Rl->n_ops), (uint32_t)DSR_SERVE_MAX_OPS);
    const bool img_here = uniform(Rl->init_size) <= DSR_SERVE_IMG_LDS;
    /* (the host asks for a relay only for blobs larger than the LDS copy) */
    const bool relayed = !img_here && Rl->relay != nullptr && relay_images(Rl, team, T.lane, relays);
    /* the relayed bytes are read with plain loads below: acquire */
    if (relayed) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    wave_sync();
    if (T.lane == 0) {
        Rl->ops = (const dsr_op *)ops_l;
        Rl->loops = (const dsr_dloop *)loops_l;
        Rl->n_ops = n_ops;
        if (img_here) Rl->init = (const uint8_t *)Rl + DSR_SERVE_SLOT_HEAD;
        if (relayed) Rl->init = Rl->relay;
    }
    wave_sync();
    return *Rl;
}

#if DSR_INST_VARIANT < DSR_LEAN_BASE
/* One kernel for both launch forms.  The master wave runs region programs
 * (one per workgroup for a single region; claimed items for a batch) and
 * then terminates the workers; worker waves sit in the await loop and take
 * the region and team of each published body from the control block. */
template <int MAXWG, int VARIANT>
__global__ __launch_bounds__(MAXWG) void dsr_region_kernel(dsr_dlaunch LP, dsr_dconfig C)
{
    team_t T = team_init(dsr_lds, C.nw, C.lds_cap, C.threshold,
                         C.hbm_base + (uint64_t)blockIdx.x * C.hbm_slot_bytes, (uint32_t)C.hbm_slot_bytes);
    T.nest_hbm = C.nest_base + (uint64_t)blockIdx.x * DSR_NEST_SLOT;
    T.nest_global = C.nest_global;
    const bool single = LP.items == nullptr;
    uint32_t barriers = 0, inner_pushes = 0;
    if (LP.published && T.wave == C.nw - 1 && T.lane == 0) {
        const uint64_t now = wall_clock64();
        if (blockIdx.x == 0 && LP.done_ts)
            __hip_atomic_store(LP.done_ts, now, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(LP.wg_started + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (LP.start_ts && blockIdx.x == 0 && T.wave == C.nw - 1 && T.lane == 0) *LP.start_ts = wall_clock64();
    if (T.wave == C.nw - 1) {
        for (uint32_t round = 0;; ++round) {
            uint32_t region, team;
            if (single) {
                if (round) break;
                region = 0;
                team = blockIdx.x;
            } else {
                uint32_t it = 0;
                if (T.lane == 0) it = atomicAdd(&LP.counter[DSR_SRV_CLAIM], 1u);
                it = uniform((uint32_t)__shfl((int)it, 0, 64));
                if (LP.published) {
                    /* served form: wait until the host has published item
                     * `it`; leave once the server has closed below it */
                    uint64_t item = 0;
                    if (!wait_item(LP, it, T.lane, item)) break;
                    const uint64_t w = (uint64_t)__shfl((long long)item, 0, 64);
                    region = uniform((uint32_t)(w >> 16) & 0xffffu);
                    team = uniform((uint32_t)w & 0xffffu);
                } else {
                    if (it >= LP.n_items) break;
                    if (it == 0 && LP.done_ts && T.lane == 0) LP.done_ts[LP.n_regions] = wall_clock64();
                    region = uniform(LP.items[2 * it]);
                    team = uniform(LP.items[2 * it + 1]);
                }
                team_reset(T);
            }
            const dsr_dregion &R = C.serve
                                       ? stage_request(T, (const uint8_t *)LP.regions + (uint64_t)region * LP.region_stride, team,
                                                   LP.relays)
                                       : LP.regions[region];
            run_program<VARIANT>(T, R, C, region, team, barriers, inner_pushes);
            GLB uint32_t *tr = (single && C.trace && R.trace) ? (GLB uint32_t *)(R.trace + (uint64_t)team * DSR_TRACE_WORDS) : nullptr;
            if (tr && T.lane == 0) tr[87] = (uint32_t)wall_clock64();
            /* outputs out of L2 before the arrival; a request of one team
             * has its completion record's system-scope release do it */
            if (C.serve && R.teams > 1) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            /* the 1024-thread instance reads fewer partials per round */
            finish_team(sums_of(R), team, T.lane, (LP.done_ts && !LP.published) ? LP.done_ts + region : nullptr,
                        LP.recs ? LP.recs + region : nullptr, &R, LP.pub, tr);
            if (tr && T.lane == 0) tr[88] = (uint32_t)wall_clock64();
        }
        if (LP.wg_exited && T.lane == 0)
            __hip_atomic_store(LP.wg_exited + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        /* terminate the workers (Figure 3's terminate branch) */
        frame_t none{SPACE_NONE, 0, 0};
        publish(T, none, DSR_BODY_TERMINATE, 0);
        barriers++;
        if (!single && !LP.published && T.lane == 0) {
            if (__hip_atomic_fetch_add(&LP.counter[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                gridDim.x - 1) {
                __hip_atomic_store(&LP.counter[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&LP.counter[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    } else {
        for (;;) {
            uint32_t body, loop;
            frame_t f;
            const bool go = await(T, &body, &f, &loop);
            barriers++;
            if (!go) break;
            const uint32_t region = uniform(header(T)->region), team = uniform(header(T)->team);
            const dsr_dregion &R = C.serve ? *serve_area(T) : LP.regions[region];
            participate<VARIANT>(T, R, C, team, body, f, loop, R.loops[loop], inner_pushes);
            barriers++;
        }
    }
    if (single && C.trace && LP.regions[0].trace && T.lane == 0) {
        GLB uint32_t *tr = (GLB uint32_t *)(LP.regions[0].trace + (uint64_t)blockIdx.x * DSR_TRACE_WORDS);
        tr[49 + T.wave] = barriers;
        tr[65 + T.wave] = inner_pushes;
    }
}

#else
/* ---- lean instances -----------------------------------------------------
 * Single-region launches with static schedules: the kernel holds the
 * single-region form only, and of the bodies what its variant is for
 * (DSR_LEAN_*).  A small
 * region's time is the chain of steps its master wave goes through one
 * after another (about 10 us of the 26 us launch-and-wait of a 64-team
 * region, and about 9 us of the 46 us of a 2^24-element one), so the steps
 * are short here: everything the launch needs comes in the kernel
 * arguments, whose cache lines are fetched together at the start; the
 * master keeps its stack pointers and top frame in registers and only
 * writes the control block; both roles run the body at one place, so its
 * code is fetched once; the waves' partials are combined across lanes; and
 * the workers are terminated before the team arrives.  Launch and wait
 * against the interpreter all instances shared before: 4-team affine loop
 * 26.1 -> 21.8 us, 64-team chain of 8 scalars 26.3 -> 24.6 us, the seven
 * 2^24-element regions of the sweep 455.8 -> 438.4 us. */
typedef __attribute__((address_space(4))) const uint32_t *kptr_t;

/* Touch every 64-byte line of the first BYTES of the kernel arguments: the
 * scalar loads that follow then hit, instead of missing one after another
 * as the code reaches them (0.8 us per launch). */
template <uint32_t BYTES>
__device__ __forceinline__ void touch_args()
{
    const kptr_t p = (kptr_t)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t v = 0;
#pragma unroll
    for (uint32_t k = 0; k < BYTES / 4; k += 16) v ^= p[k];
    asm volatile("" ::"s"(v));
}

/* A descriptor in global memory that no kernel writes, read with scalar
 * loads. */
template <class V>
__device__ __forceinline__ V load_const(const V *p)
{
    static_assert(sizeof(V) % 4 == 0, "whole words");
    union {
        V v;
        uint32_t w[sizeof(V) / 4];
    } u;
    const kptr_t q = (kptr_t)(uintptr_t)p;
#pragma unroll
    for (uint32_t k = 0; k < sizeof(V) / 4; ++k) u.w[k] = q[k];
    return u.v;
}

/* Fixed fma chain of a lean instance: the frame's scalars are read one word
 * per lane in one round and handed out with readlanes. */
template <int NI, int NF>
__device__ __forceinline__ void lean_chain(const team_t &T, frame_t f, const dsr_dloop &L, span_t sp, deal_t deal,
                                           lane_acc &A)
{
    constexpr uint32_t NWORDS = 2 * NF + NI;
    uint32_t w[2] = {0, 0};
#pragma unroll
    for (uint32_t h = 0; h < 2 && 64 * h < NWORDS; ++h) {
        const uint32_t k = T.lane + 64u * h;
        if (k < NWORDS)
            w[h] = f.space == SPACE_LDS
                       ? *(const LDSQ uint32_t *)(dsr_lds + cb_bytes(T.nw) + f.off + 24 + 4 * k)
                       : *(const GLB uint32_t *)(T.stack_hbm + f.off + 24 + 4 * k);
    }
    auto word = [&](int k) { return (uint32_t)__builtin_amdgcn_readlane(w[k >> 6], k & 63); };
    fixed_chain<NI, NF> ch;
#pragma unroll
    for (int k = 0; k < NF; ++k)
        ch.s[k] = __longlong_as_double((long long)((uint64_t)word(2 * k) | ((uint64_t)word(2 * k + 1) << 32)));
    /* all the scalars, one per lane, int32 ones first */
    double sv = 0.0;
    if constexpr (NI > 1) {
        const uint32_t at = T.lane < NI ? 2 * NF + T.lane : 2 * ((T.lane - NI) & 31u);
        auto pick = [&](uint32_t k) {
            const uint32_t lo = (uint32_t)__shfl((int)w[0], k & 63u, 64), hi = (uint32_t)__shfl((int)w[1], k & 63u, 64);
            return k < 64 ? lo : hi;
        };
        const uint32_t a = pick(at), b = pick(at + 1);
        sv = T.lane < NI ? (double)(int32_t)a : __longlong_as_double((long long)((uint64_t)a | ((uint64_t)b << 32)));
    } else {
        sv = (double)(int32_t)word(2 * NF);
    }
    ch.all = make_chain(sv, NI, NF, T.lane);
    chain_range<8, ARR_NONE, false>(ch, glb_array{nullptr}, 0, L, sp, deal, T.lane, A);
}

__device__ __forceinline__ void lean_affine(const team_t &T, frame_t f, const dsr_dloop &L, span_t sp, lane_acc &A)
{
    uint32_t w = 0;
    if (T.lane < 4)
        w = f.space == SPACE_LDS ? *(const LDSQ uint32_t *)(dsr_lds + cb_bytes(T.nw) + f.off + 8 + 4 * T.lane)
                                 : *(const GLB uint32_t *)(T.stack_hbm + f.off + 8 + 4 * T.lane);
    const uint32_t a = __builtin_amdgcn_readlane(w, 0), b = __builtin_amdgcn_readlane(w, 1);
    const uint32_t c = __builtin_amdgcn_readlane(w, 2), d = __builtin_amdgcn_readlane(w, 3);
    affine_span(a, b, c, d, (GLB int32_t *)L.out, sp, A);
}

/* Master wave, section 5.2: resolve each (frame, offset) reference of `tab` to
 * a stack address and write the list on chip, or to a list frame `lf` on the
 * HBM stack when it is longer than the on-chip list or `global` is set.  What
 * is published is the list's place; SPACE_NONE when it does not fit. */
__device__ __forceinline__ frame_t post_list(const team_t &T, stack_t &S, const uint32_t *tab, uint32_t n, uint32_t global,
                                             frame_t &lf)
{
    frame_t f{SPACE_LIST, 0, n};
    uint32_t *dst = ref_list(T);
    if (n > DSR_REF_LIST || global) {
        lf = push(T, S, 8 * n, true);
        if (lf.space == SPACE_NONE) return lf;
        dst = (uint32_t *)frame_hbm(T, lf);
        f = frame_t{SPACE_HBM, lf.off, n};
    }
    for (uint32_t q = T.lane; q < n; q += 64) {
        const uint32_t *fte = frame_table(T) + 4 * tab[2 * q];
        dst[2 * q] = fte[0];
        dst[2 * q + 1] = fte[1] + tab[2 * q + 1];
    }
    return f;
}

template <int MAXWG, int VARIANT>
__global__ __launch_bounds__(MAXWG) void dsr_region_kernel(dsr_lean A)
{
    constexpr bool gather = VARIANT == DSR_LEAN_GATHER, affine = VARIANT == DSR_LEAN_AFFINE;
    constexpr bool mixed = VARIANT == DSR_LEAN_MIXED, chains = VARIANT == DSR_LEAN_ANY_CHAIN || mixed;
    touch_args<offsetof(dsr_lean, image)>();
    const uint32_t team = blockIdx.x;
    team_t T = team_bind(dsr_lds, A.nw, A.lds_cap, A.threshold, A.hbm_base + (uint64_t)team * A.hbm_slot_bytes,
                         (uint32_t)A.hbm_slot_bytes);
    T.nest_hbm = A.nest_base + (uint64_t)team * DSR_NEST_SLOT;
    T.nest_global = A.nest_global;
    T.image = A.init;
    const bool master = T.wave == A.nw - 1;
    const uint32_t nwork = A.master_joins ? A.nw : A.nw - 1;
    GLB uint32_t *tr = A.trace ? (GLB uint32_t *)(A.trace + (uint64_t)team * DSR_TRACE_WORDS) : nullptr;
    const region_sums RS{A.partials, A.result, A.out, A.status, A.teams, A.n_red, A.red_kind_mask};
    uint32_t barriers = 0, inner_pushes = 0;
    /* the master's place in the program, and its stack */
    stack_t S = stack_empty();
    uint32_t k = 0, npush = 0;
    int32_t err = 0;
    bool stamped = false;
    if (tr && master && T.lane == 0) tr[86] = (uint32_t)wall_clock64();
    /* the first frame's image, 16 bytes a lane */
    i32x4 img = {0, 0, 0, 0};
    /* A first frame that goes to LDS is copied by all the team's waves, each
     * every nw-th round, from before the master looks at its program: its
     * place, at the bottom of the stack, is known.  Nothing orders the workers'
     * loads before a pop of that frame and a push in its place, so none may
     * come before the first publish; a program with both has five ops at least
     * and does not travel in the arguments.  (Fixed chains and affine loops have
     * small frames, whose image comes in the arguments.)  One wave has 64 loads
     * of 1 KiB in flight at most: 2^26 outputs of 2048 teams with 128 KiB each,
     * one team per CU, 76.5 -> 59.5 us per launch; the 2^20-element chain with
     * a 32 KiB frame 62.1 -> 61.2 us launch and wait. */
    uint32_t under_way = 0;
    static_assert(DSR_INLINE_OPS < 5, "push, pop, push, publish, pop");
    if ((gather || chains) && A.inl_ops && A.n_ops && A.inl_op[0].kind == DSR_OP_PUSH && !A.inl_img) {
        const dsr_op op = A.inl_op[0];
        const uint32_t size = (op.nbytes + DSR_ALIGN - 1) & ~(DSR_ALIGN - 1);
        const uint8_t *src = A.init + op.init_off + (uint64_t)team * op.init_stride;
        if (size <= T.threshold && size <= T.lds_cap && ((uintptr_t)src & 15u) == 0) {
            const uint32_t full = min(op.init_bytes, op.nbytes) >> 4;
            (void)direct_rounds(T, 0, src, 64u * T.wave, full, 64u * A.nw);
            under_way = full & ~63u;
            if (!master) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
    }
    if (master && 16u * T.lane < A.inl_img) img = *(const i32x4 *)(A.image + 16u * T.lane);
    for (;;) {
        uint32_t body = DSR_BODY_TERMINATE, loop = 0, red = 0xffffffffu;
        frame_t f{SPACE_NONE, 0, 0}, lf{SPACE_NONE, 0, 0};
        if (master) {
            while (k < A.n_ops && !err) {
                const dsr_op op = A.inl_ops ? A.inl_op[k] : load_const(A.ops + k);
                const uint32_t at = k++;
                if (op.kind == DSR_OP_PUSH) {
                    const frame_t p = push(T, S, op.nbytes);
                    if (p.space == SPACE_NONE) { err = DSR_E_NOMEM; break; }
                    if (tr && T.lane == 0 && npush < 16) {
                        tr[1 + 3 * npush] = p.space;
                        tr[2 + 3 * npush] = p.off;
                        tr[3 + 3 * npush] = p.size;
                    }
                    npush++;
                    static_assert(DSR_INLINE_FRAME == 16u * 64u && DSR_INLINE_FRAME % DSR_ALIGN == 0,
                                  "16 bytes a lane, whole after rounding");
                    if (at == 0 && A.inl_img && p.size <= DSR_INLINE_FRAME) {
                        /* the image (zero-padded to a multiple of 16 bytes)
                         * from registers, zeros after it */
                        if (16u * T.lane < p.size) {
                            if (p.space == SPACE_LDS)
                                *(LDSQ i32x4 *)(dsr_lds + cb_bytes(T.nw) + p.off + 16u * T.lane) = img;
                            else
                                *(GLB i32x4 *)(T.stack_hbm + p.off + 16u * T.lane) = img;
                        }
                    } else if (gather && p.space == SPACE_HBM && op.init_bytes == op.nbytes && A.init_in_place) {
                        /* no gather writes to a frame, so one that lies in
                         * global memory anyway is read where its image lies:
                         * every team's own copy of a 192 KiB frame had cost
                         * 384 MiB written and read back over 2048 teams, one
                         * wave of each at work (launch and wait of 2^26
                         * outputs, 3 x 16384: 232.8 -> 66.0 us) */
                        read_in_place(T, S, (uint32_t)(op.init_off + (uint64_t)team * op.init_stride));
                    } else {
                        init_frame(T, p, A.init + op.init_off + (uint64_t)team * op.init_stride, op.init_bytes,
                                   op.nbytes, true, at == 0 ? under_way : 0u);
                    }
                } else if (op.kind == DSR_OP_PUBLISH) {
                    if (chains && op.body == DSR_BODY_FMA_CHAIN_REFS) {
                        f = post_list(T, S, (const uint32_t *)(A.init + op.init_off), op.nbytes, A.global_lists, lf);
                        if (f.space == SPACE_NONE) { err = DSR_E_NOMEM; break; }
                        if (tr && T.lane == 0) {
                            tr[89] = f.space;
                            tr[90] = f.off;
                            tr[91] = op.nbytes;
                        }
                    } else {
                        f = frame_at(T, S, op.frame);
                    }
                    body = op.body;
                    loop = op.loop;
                    red = op.red;
                    break;
                } else if (op.kind == DSR_OP_POP) {
                    if (!pop(T, S)) err = DSR_E_UNDERFLOW;
                }
            }
            if (body == DSR_BODY_TERMINATE && tr && T.lane == 0) {
                tr[0] = npush;
                tr[81] = (uint32_t)err;
                tr[87] = (uint32_t)wall_clock64();
            }
            if (T.lane == 0) post(T, f, body, loop);
        }
        __syncthreads();                     /* hand-over (barrier 1) */
        barriers++;
        if (!master) take(T, body, f, loop);
        if (body == DSR_BODY_TERMINATE) break;
        if (tr && master && !stamped && T.lane == 0) {
            const uint64_t t0 = wall_clock64();
            tr[82] = (uint32_t)t0;
            tr[83] = (uint32_t)(t0 >> 32);
        }
        stamped = true;
        if (!master || A.master_joins) {
            const dsr_dloop L = loop == 0 ? A.loop0 : load_const(A.loops + loop);
            span_t sp = team_span(L, team, T.wave * 64 + T.lane, nwork * 64);
            deal_t deal{0, 0};
            const bool chain_body = !gather && !affine &&
                                    (!mixed || body == DSR_BODY_FMA_CHAIN || body == DSR_BODY_FMA_CHAIN_REFS);
            if (chain_body && L.deal) {
                sp = span_t{0, L.n, T.lane, 64u};
                deal = deal_t{team * nwork + T.wave, A.teams * nwork};
            }
            if (tr && T.lane == 0) tr[96 + 2 * T.wave] = (uint32_t)wall_clock64();
            lane_acc acc = acc_zero();
            if constexpr (gather) {
                if (body == DSR_BODY_GATHER) body_gather(T, f, L, sp);
                else body_gather_nested(T, f, L, sp, T.wave, nwork, inner_pushes, tr);
            } else if constexpr (affine) {
                lean_affine(T, f, L, sp, acc);
            } else if (mixed && !chain_body) {
                if (body == DSR_BODY_AFFINE_XOR) lean_affine(T, f, L, sp, acc);
                else if (body == DSR_BODY_GATHER) body_gather(T, f, L, sp);
                else body_gather_nested(T, f, L, sp, T.wave, nwork, inner_pushes, tr);
            } else if constexpr (chains) {
                body_chain<8, true>(T, body == DSR_BODY_FMA_CHAIN_REFS, f, L, sp, deal, acc, nullptr, T.lane);
            } else {
                lean_chain<DSR_LEAN_NI(VARIANT - DSR_LEAN_BASE), DSR_LEAN_NF(VARIANT - DSR_LEAN_BASE)>(T, f, L, sp, deal,
                                                                                                    acc);
            }
            if (tr && T.lane == 0) tr[97 + 2 * T.wave] = (uint32_t)wall_clock64();
            if constexpr (affine) {
                deposit(T, wave_sum192(from_i64(acc.i)), 0);
            } else if constexpr (!gather) {
                deposit(T, wave_sum192(widen(acc)), __any(acc.bad != 0));
            }
        }
        __syncthreads();                     /* the join (barrier 2) */
        barriers++;
        if (!master) continue;
        if (tr && T.lane == 0) {
            const uint64_t t1 = wall_clock64();
            tr[84] = (uint32_t)t1;
            tr[85] = (uint32_t)(t1 >> 32);
        }
        if constexpr (!gather) {
            uint32_t bad;
            const i192 tot = joined_sum(T.lane, nwork, bad);
            if (bad) err = DSR_E_RANGE;
            /* into the shared variable; the team's partial is stored inside
             * each branch: where the two would merge the compiler waits for
             * every outstanding memory operation of the wave, its loop stores
             * included */
            uint64_t *pp = A.partials + ((uint64_t)red * A.teams + team) * DSR_PART_WORDS;
            const bool whole = affine || (mixed && body == DSR_BODY_AFFINE_XOR);
            if (mixed && red == 0xffffffffu) continue;       /* a gather */
            if (chains && body == DSR_BODY_FMA_CHAIN_REFS) {
                /* the shared sum is where reference 0 points */
                const uint32_t *lst = f.space == SPACE_LIST ? ref_list(T) : (const uint32_t *)frame_hbm(T, f);
                f.space = uniform(lst[0]);
                f.off = uniform(lst[1]);
            }
            if (f.space == SPACE_LDS)
                store_partial(pp, update_sum((LDSQ uint64_t *)(dsr_lds + cb_bytes(T.nw) + f.off), tot, whole, T.lane),
                              T.lane);
            else
                store_partial(pp, update_sum((GLB uint64_t *)(T.stack_hbm + f.off), tot, whole, T.lane), T.lane);
            /* a global reference list dies with its parallel region */
            if (chains && lf.space == SPACE_HBM) pop(T, S);
        }
    }
    if (master) {
        if constexpr (gather) {
            /* nothing to combine, and every team meets the same error or none:
             * where a frame goes depends on sizes alone.  The first team tells
             * it; the others leave without arriving (a store, an atomic and a
             * fence less, about 1 us of each team's time) */
            if (tr && T.lane == 0) tr[92] = tr[93] = (uint32_t)wall_clock64();
            if (team == 0) {
                if (tr && T.lane == 0) tr[94] = (uint32_t)wall_clock64();
                if (T.lane == 0) *(GLB int32_t *)A.status = err;
                if (A.pub) public_record(A.pub, 0, err, T.lane);
                if (tr && T.lane == 0) tr[95] = (uint32_t)wall_clock64();
            }
        } else {
            if (err && T.lane == 0) atomicCAS(&A.result->error, 0, err);
            finish_team(RS, team, T.lane, nullptr, nullptr, nullptr, A.pub, tr);
        }
        if (tr && T.lane == 0) tr[88] = (uint32_t)wall_clock64();
    }
    if (tr && T.lane == 0) {
        tr[49 + T.wave] = barriers;
        tr[65 + T.wave] = inner_pushes;
    }
}
#endif

/* ---- this object's instance --------------------------------------------
 * The build compiles this file once per kernel instance, in parallel, with
 * DSR_INST_MAXWG, DSR_INST_VARIANT and DSR_INST_TAG defined; each object
 * exports its instance's launcher, occupancy and register queries under
 * names carrying the tag, and dsr_dispatch.cpp picks among them. */
#define DSR_INST_CAT2(a, b) a##b
#define DSR_INST_CAT(a, b) DSR_INST_CAT2(a, b)
#define DSR_INST_KERNEL dsr_region_kernel<DSR_INST_MAXWG, DSR_INST_VARIANT>

extern "C" int DSR_INST_CAT(dsr_inst_launch_, DSR_INST_TAG)(const void *args, const dsr_dconfig *cfg,
                                                            uint32_t grid, uint32_t wg_size, uint32_t lds_bytes,
                                                            void *stream)
{
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)DSR_INST_KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  160 * 1024);
        attr = true;
    }
#if DSR_INST_VARIANT < DSR_LEAN_BASE
    hipLaunchKernelGGL(DSR_INST_KERNEL, dim3(grid), dim3(wg_size), lds_bytes, (hipStream_t)stream,
                       *(const dsr_dlaunch *)args, *cfg);
#else
    (void)cfg;
    hipLaunchKernelGGL(DSR_INST_KERNEL, dim3(grid), dim3(wg_size), lds_bytes, (hipStream_t)stream,
                       *(const dsr_lean *)args);
#endif
    return (int)hipGetLastError();
}

extern "C" int DSR_INST_CAT(dsr_inst_occupancy_, DSR_INST_TAG)(uint32_t wg_size, uint32_t lds_bytes)
{
    (void)hipFuncSetAttribute((const void *)DSR_INST_KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024);
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)DSR_INST_KERNEL, (int)wg_size, lds_bytes) !=
        hipSuccess)
        return 0;
    return n;
}

extern "C" int DSR_INST_CAT(dsr_inst_regs_, DSR_INST_TAG)(void)
{
    hipFuncAttributes a{};
    if (hipFuncGetAttributes(&a, (const void *)DSR_INST_KERNEL) != hipSuccess) return 0;
    return a.numRegs;
}
