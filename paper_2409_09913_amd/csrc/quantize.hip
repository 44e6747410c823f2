// Algorithm 1 (Quantize) of Extended RaBitQ, Sec. 3.2.2, on gfx950.
//
// In the orthant of r' every coordinate has a magnitude a_i; level k_i in
// [0, K] (K = 2^{B-1}-1) means y_i = +-(k_i + 1/2).  Level k_i moves to m at
// the critical value t = m / a_i, an event of key d = a_i / m.  Algorithm 1
// takes the events in order (d descending, ties: dimension ascending) and
// keeps the first strict maximum of the objective
//     f = <y, r'> / ||y|| = S1 / sqrt(S2),  S1 += 2 a_i, S2 += 8 m per event,
// with S1 an int64 fixed point (a scaled by the power of two that puts max a
// in [1, 2), 40 fractional bits) and S2 = 4 ||y||^2 an exact integer.
//
// Sorting all dp K events (or enumerating them through a heap) is what the
// paper's algorithm does; here almost none are ever ordered:
//   1. Bins.  The key range is cut into NB bins with FP32 edges e_0 > e_1 >
//      ...; every event of the range is added (sum of 2a and of m, integer LDS
//      atomics, so the sums do not depend on the order) to its bin.  An event
//      belongs to the bin with e_{j+1} <= a/m < e_j, decided exactly (the sign
//      of the fused a - m e), so the prefix sums over the bins are the exact
//      states (S1, S2) of the enumeration at every edge.
//   2. Bound.  The best state at an edge is a lower bound of the maximum.
//      Inside a bin m = a/d with d in [e_{j+1}, e_j), so after a partial sum x
//      of its S1 increments D, S2 is at least both S2_start + 4x/e_j and
//      S2_end - 4(D - x)/e_{j+1}; (A + x)^2 over either line is quasi-convex
//      in x, so f^2 in the bin is at most its largest value at the two ends
//      and where the lines cross.  That exceeds the true maximum of the bin by
//      a relative (bin width)^2 / 8 only, so a handful of bins around the
//      maximum survive.
//   3. The range shrinks to the hull of the surviving bins and steps 1 and 2
//      repeat until at most kSortMax events are left (one pass for B <= 4 at
//      dp 768, two or three for B = 8).
//   4. Those are sorted by (key, dimension) and enumerated as Algorithm 1
//      does; the codes are the levels of the best event's state.
// A range that does not shrink (several far-apart maxima of nearly equal
// value) is enumerated in windows of at most `cap` events instead.
// Keys are compared exactly: for 24-bit magnitudes and levels below 2^7
// distinct ratios a/m differ by at least 2^-31 relative.
//
// What bounds it: vector ALU (about 4,000 instructions per wave at dp 768, B =
// 4, 14 per event of the first pass); the codes and rows alone are 0.14 ms of
// HBM traffic at 100,003 x 768.  Measured there, against one sorted window of
// all events per vector before: B = 4 15.8 -> 0.83 ms, B = 2 2.9 -> 0.55; 8,191
// x 1536, B = 8: 120 -> 1.8 ms.  Split: one wave per vector up to dp 768, two
// to 1536, four above, so that no barrier is needed at the widths in common
// use; the LDS (bins, magnitudes, levels: 8.2 KB at dp 768) lets 19 waves
// share a CU.  32 bins per octave for one wave: 64 cost 15% at B = 4 (12 KB of
// LDS and twice the bound tests) and gain nothing at B = 8.
#include <algorithm>

#include "erq_common.h"

namespace erq {

namespace {

// four floats and four codes at the alignment of their elements (the caller's
// arrays may start anywhere)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned u32u __attribute__((aligned(1)));

constexpr int kBinsPerThread = 4;    // 32 bins per octave of keys for one wave, 128 for four
constexpr int kWide = 4;             // first pass, many levels: the last bins are 1, 2, 4 octaves wide, and the rest
constexpr int kSortMax = 128;        // events left for the sort (else another pass of bins)
constexpr int kPasses = 6;           // passes of bins before the windows
// Events past t = S2/S1 (a <= S1 in units of max a in [1, 2)) cannot raise f:
// S2 (S1 + a) > 2 t S1^2 fails.  S2 <= kMaxDp * 255^2 < 2^28 and S1 >= 1, so no
// event with key below 2^-28 is ever the maximum.
constexpr unsigned kMinKey = 0x31800000u;    // bits of 2^-28f
static_assert((int64_t)kMaxDp * 255 * 255 < (1 << 28), "the bound on S2");
static_assert(kMaxDp <= 1 << 12, "event_key: the dimension takes 12 bits");

__device__ inline unsigned long long shfl_xor_u64(unsigned long long v, int o) {
    const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, o);
    const unsigned hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), o);
    return ((unsigned long long)hi << 32) | lo;
}

// v of another lane by a DPP control, `old` where the control has no source;
// 4- and 8-byte values
template <int CTRL, int ROWS, class T>
__device__ inline T dpp(T old, T v) {
    unsigned s[sizeof(T) / 4], o[sizeof(T) / 4];
    __builtin_memcpy(s, &v, sizeof(T));
    __builtin_memcpy(o, &old, sizeof(T));
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i)
        s[i] = (unsigned)__builtin_amdgcn_update_dpp((int)o[i], (int)s[i], CTRL, ROWS, 0xF, false);
    __builtin_memcpy(&v, s, sizeof(T));
    return v;
}
template <class T>
__device__ inline T last_lane(T v) {
    unsigned s[sizeof(T) / 4];
    __builtin_memcpy(s, &v, sizeof(T));
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) s[i] = (unsigned)__builtin_amdgcn_readlane((int)s[i], 63);
    __builtin_memcpy(&v, s, sizeof(T));
    return v;
}
// Inclusive scan over the wave without LDS: rows of 16 by shifts, then the
// last lanes of rows 0 and 2, then of the first half.  SUM: op is a sum (0
// where a lane has no source), else op is idempotent (the lane's own value).
template <bool SUM, class T, class F>
__device__ inline T wave_scan(T v, F op) {
    auto own = [&]() -> T { return SUM ? T(0) : v; };
    v = op(v, dpp<0x111, 0xF>(own(), v));
    v = op(v, dpp<0x112, 0xF>(own(), v));
    v = op(v, dpp<0x114, 0xF>(own(), v));
    v = op(v, dpp<0x118, 0xF>(own(), v));
    v = op(v, dpp<0x142, 0xA>(own(), v));
    v = op(v, dpp<0x143, 0xC>(own(), v));
    return v;
}

// Block-wide reduction over NT threads (every thread gets the result); red:
// NT/64 slots of 8 bytes.  One wave needs no LDS and no barrier.
template <int NT, bool SUM, class T, class F>
__device__ inline T block_reduce(T v, F op, unsigned long long* red) {
    static_assert(sizeof(T) == 8 || sizeof(T) == 4, "4- and 8-byte values");
    v = last_lane(wave_scan<SUM>(v, op));
    if constexpr (NT > 64) {
        __syncthreads();                             // the slots' last readers are done
        if ((threadIdx.x & 63) == 0) __builtin_memcpy(&red[threadIdx.x >> 6], &v, sizeof(T));
        __syncthreads();
        __builtin_memcpy(&v, &red[0], sizeof(T));
        for (int w = 1; w < NT / 64; ++w) {
            T u;
            __builtin_memcpy(&u, &red[w], sizeof(T));
            v = op(v, u);
        }
    }
    return v;
}
template <int NT, class T>
__device__ inline T block_sum(T v, unsigned long long* red) {
    return block_reduce<NT, true>(v, [](T x, T y) { return x + y; }, red);
}
template <int NT, class T>
__device__ inline T block_max(T v, unsigned long long* red) {
    return block_reduce<NT, false>(v, [](T x, T y) { return x > y ? x : y; }, red);
}
template <int NT, class T>
__device__ inline T block_min(T v, unsigned long long* red) {
    return block_reduce<NT, false>(v, [](T x, T y) { return x < y ? x : y; }, red);
}

// Block-wide exclusive prefix of (a, b); ta, tb: the totals.
template <int NT, class T, class U>
__device__ inline void block_scan2(T& a, U& b, T& ta, U& tb, unsigned long long* red) {
    const T ia = wave_scan<true>(a, [](T x, T y) { return x + y; });
    const U ib = wave_scan<true>(b, [](U x, U y) { return x + y; });
    T oa = 0;
    U ob = 0;
    if constexpr (NT > 64) {
        const int wid = threadIdx.x >> 6;
        __syncthreads();
        if ((threadIdx.x & 63) == 63) { red[2 * wid] = ia; red[2 * wid + 1] = ib; }
        __syncthreads();
        ta = 0;
        tb = 0;
        for (int w = 0; w < NT / 64; ++w) {
            if (w == wid) { oa = ta; ob = tb; }
            ta += (T)red[2 * w];
            tb += (U)red[2 * w + 1];
        }
    } else {
        ta = last_lane(ia);
        tb = last_lane(ib);
    }
    a = oa + ia - a;
    b = ob + ib - b;
}

// magnitude (max in [1, 2)) -> 40-bit fixed point, round half even: the low
// mantissa bits of a 2^40 + 1.5 2^52
__device__ inline unsigned long long fix40(float a) {
    const double v = __fma_rn((double)a, 0x1p40, 0x1.8p52);
    return (unsigned long long)(__double_as_longlong(v) & 0x0007FFFFFFFFFFFFll);
}

// the fixed point back in units of the magnitudes, FP32
__device__ inline float fix_f(unsigned long long s) {
    return __fmaf_rn((float)(unsigned)(s >> 32), 0x1p-8f, (float)(unsigned)s * 0x1p-40f);
}

// 1/x to about 2^-50 (bounds only)
__device__ inline double rcp_d(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __fma_rn(__fma_rn(-x, r, 1.0), r, r);
    return __fma_rn(__fma_rn(-x, r, 1.0), r, r);
}

// levels m <= K with a / m >= x, that is m x <= a, exactly; rx is about 1/x.
// a rx is off by less than 127 2^-21 where it is below 128, so only a value
// that close to an integer needs the test (the sign of a fused a - m x is exact).
constexpr float kNearLevel = 0x1p-13f;
__device__ inline int level_at(float a, float x, float rx, int K) {
    const float q = fminf((float)(K + 1), a * rx), f = floorf(q), d = q - f;
    int k = (int)f;
    if (d < kNearLevel || d > 1.0f - kNearLevel) {
        if (__fmaf_rn(-(float)k, x, a) < 0.0f) --k;
        else if (__fmaf_rn(-(float)(k + 1), x, a) >= 0.0f) ++k;
    }
    return min(k, K);
}

// Sort key of the event (m, dim): the order of (a/m descending, dim
// ascending) as an ascending integer, with the level in the low bits.  The
// correctly rounded quotient keeps 33 mantissa bits: equal ratios give equal
// quotients and distinct ones differ by 2^-31 or more.
__device__ inline unsigned long long event_key(float a, int m, int dim) {
    const unsigned long long q = (unsigned long long)__double_as_longlong((double)a / (double)m);
    return ((~q >> 19) << 19) | ((unsigned long long)dim << 7) | (unsigned long long)m;
}

__host__ __device__ inline size_t a16(size_t x) { return (x + 15) & ~(size_t)15; }

// LDS: the bins (sums of 2a and of m, one more slot each) share their space
// with the keys of the window being sorted; then the magnitudes and the levels
// at both ends of the range, by dimension
__host__ __device__ inline size_t quant_bins_bytes(int nb) { return a16((size_t)(nb + 2) * 12); }
__host__ __device__ inline size_t quant_union_bytes(int nb, int cap) {
    size_t u = quant_bins_bytes(nb);
    if (u < (size_t)kSortMax * 12) u = (size_t)kSortMax * 12;     // (dimension, level) and keys of a short sort
    if (u < (size_t)cap * 4) u = (size_t)cap * 4;                 // (dimension, level) of a window
    return a16(u);
}
__host__ __device__ inline size_t quant_smem(int nb, int cap, int dp) {
    return quant_union_bytes(nb, cap) + sizeof(float) * dp + sizeof(unsigned short) * dp;
}

}  // namespace

// NT threads per vector.  cap: events of a window, at
// least dp (a bin one FP32 step wide holds at most one event per coordinate, so
// windows always advance).
template <int NT>
__global__ __launch_bounds__(NT) void quantize_kernel(
    const float* __restrict__ rrot, int64_t n_vec, int dp, int bits, int cap,
    const float* __restrict__ norm2, uint8_t* __restrict__ codes, float* __restrict__ f_add,
    float* __restrict__ f_rescale, float* __restrict__ cos_oo, float2* __restrict__ fac)
{
    constexpr int NB = kBinsPerThread * NT;
    extern __shared__ __align__(16) char smem[];
    __shared__ unsigned long long red[2 * (NT / 64)];
    __shared__ float s_rm[128];                       // 1/m
    unsigned* const ev = (unsigned*)smem;                         // events: dimension << 7 | level
    unsigned long long* const keys = (unsigned long long*)(smem + 4 * kSortMax);
    unsigned long long* const b1 = (unsigned long long*)smem;     // NB + 1 sums of 2a, then states
    unsigned* const bm = (unsigned*)(smem + 8 * (NB + 2));        // NB + 1 sums of m
    float* const mag = (float*)(smem + quant_union_bytes(NB, cap));
    unsigned short* const lvl = (unsigned short*)(mag + dp);      // level at x_hi, and at x_lo in bits 8 up
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t row = blockIdx.x;
    if (row >= n_vec) return;
    const float* r = rrot + row * (int64_t)dp;
    const int K = (1 << (bits - 1)) - 1;
    const int half = 1 << (bits - 1);
    auto sync = [&]() {
        if constexpr (NT > 64) __syncthreads();
        else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    };

    // ---- load, magnitudes scaled so that the largest lies in [1, 2) --------
    float lmax = 0.0f;
    for (int i = 4 * tid; i < dp; i += 4 * NT) {
        const f4u v = *(const f4u*)(r + i);
        const float4 w = make_float4(fabsf(v.x), fabsf(v.y), fabsf(v.z), fabsf(v.w));
        lmax = fmaxf(fmaxf(fmaxf(lmax, w.x), fmaxf(w.y, w.z)), w.w);
        *(float4*)(mag + i) = w;
    }
    const float amax = block_max<NT>(lmax, red);
    int ex = 0;
    if (amax > 0.0f) { (void)frexpf(amax, &ex); ex -= 1; }
    const bool live = K > 0 && amax > 0.0f && amax < __builtin_huge_valf();
    unsigned long long s1 = 0, tiny = 0;
    unsigned nnz = 0;                 // coordinates with events
    sync();
    if (live) {
        for (int i = tid; i < dp; i += NT) {
            // coordinates below 2^-28 have no event in the range (and a NaN none at all)
            const float v = ldexpf(mag[i], -ex);
            const bool in = v >= __uint_as_float(kMinKey);
            const unsigned long long f = v > 0.0f ? fix40(v) : 0ull;
            s1 += f;
            tiny += in ? 0ull : f;
            nnz += in ? 1u : 0u;
            mag[i] = in ? v : 0.0f;
        }
        s1 = block_sum<NT>(s1, red);
        tiny = block_sum<NT>((unsigned)tiny, red);    // below 2^12 each
        nnz = block_sum<NT>(nnz, red);
    }
    // the state after all events: every coordinate that has any at level K
    const unsigned long long s1_all = 2ull * K * (s1 - tiny);
    const unsigned sm_all = nnz * (unsigned)(K * (K + 1) / 2);
    unsigned long long s2 = (unsigned long long)dp;

    double best_v = 0.0;              // strict improvement over 0 needed (v_max starts at 0)
    unsigned best_ev = 0;             // dimension and level of the best event
    unsigned long long best_s2 = (unsigned long long)dp;
    bool have = false;

    if (live) {
        for (int m = tid; m < 128; m += NT) s_rm[m] = m ? 1.0f / (float)m : 0.0f;

        // the range of keys [x_lo, x_hi) as bit patterns; set_range also sets the
        // levels of every coordinate at both ends and returns the number of
        // events between them
        unsigned bhi = __float_as_uint(ldexpf(amax, -ex)) + 1u, blo = kMinKey;
        unsigned mine = 0;                            // this thread's
        auto set_range = [&](unsigned hi, unsigned lo) {
            const float xh = __uint_as_float(hi), rh = __builtin_amdgcn_rcpf(xh);
            const float xl = __uint_as_float(lo), rl = __builtin_amdgcn_rcpf(xl);
            int n = 0;
            for (int i = tid; i < dp; i += NT) {
                const float av = mag[i];
                const int h = level_at(av, xh, rh, K), l = level_at(av, xl, rl, K);
                lvl[i] = (unsigned short)(h | (l << 8));
                n += l - h;
            }
            bhi = hi;
            blo = lo;
            mine = (unsigned)n;
            return block_sum<NT>(n, red);
        };
        // Enumerates the n <= cap events of the range from the state (s1, s2):
        // keys gathered, sorted, prefix sums, objective; keeps the first
        // strict maximum.  Advances the state past the range.
        auto enumerate = [&](int n) {
            unsigned pos = mine, zero = 0, tp_, tz_;
            block_scan2<NT>(pos, zero, tp_, tz_, red);
            sync();                                   // the bins (same LDS) have been read
            for (int i = tid; i < dp; i += NT)
                for (int m = (lvl[i] & 255) + 1; m <= (lvl[i] >> 8); ++m) ev[pos++] = (unsigned)(i << 7 | m);
            sync();
            auto key_of = [&](int t) -> unsigned long long {
                if (t >= n) return ~0ull;
                const unsigned e = ev[t];
                return event_key(mag[e >> 7], (int)(e & 127u), (int)(e >> 7));
            };
            if (n <= 64) {                            // one wave, in registers
                if (tid < 64) {
                    unsigned long long v = key_of(lane);
#pragma unroll
                    for (int k = 2; k <= 64; k <<= 1)
#pragma unroll
                        for (int j = k >> 1; j > 0; j >>= 1) {
                            const unsigned long long p = shfl_xor_u64(v, j);
                            const bool take_min = ((lane & j) == 0) == ((lane & k) == 0);
                            v = take_min ? (p < v ? p : v) : (p > v ? p : v);
                        }
                    ev[lane] = (unsigned)v & 0x7FFFFu;
                }
                sync();
            } else if (n <= kSortMax) {               // keys in LDS
                for (int t = tid; t < kSortMax; t += NT) keys[t] = key_of(t);
                sync();
                for (int k = 2; k <= kSortMax; k <<= 1)
                    for (int j = k >> 1; j > 0; j >>= 1) {
                        for (int t = tid; t < kSortMax / 2; t += NT) {
                            const int i = 2 * t - (t & (j - 1)), p = i + j;
                            const unsigned long long k0 = keys[i], k1 = keys[p];
                            if ((k0 < k1) != ((i & k) == 0)) { keys[i] = k1; keys[p] = k0; }
                        }
                        sync();
                    }
                for (int t = tid; t < kSortMax; t += NT) ev[t] = (unsigned)keys[t] & 0x7FFFFu;
                sync();
            } else {
                // a long tie group or window (rare): the events themselves, compared
                // by exact products; every comparison ascending, so the places past
                // n need no padding
                auto before = [&](unsigned e0, unsigned e1) {
                    const double x0 = (double)mag[e0 >> 7] * (double)(e1 & 127u);
                    const double x1 = (double)mag[e1 >> 7] * (double)(e0 & 127u);
                    return x0 > x1 || (x0 == x1 && e0 < e1);
                };
                int S = 2 * kSortMax;
                while (S < n) S <<= 1;
                for (int k = 2; k <= S; k <<= 1)
                    for (int j = k >> 1; j > 0; j >>= 1) {
                        for (int t = tid; t < S / 2; t += NT) {
                            const int i = 2 * t - (t & (j - 1));
                            const int p = j == k >> 1 ? (i | (k - 1)) - (t & (j - 1)) : i + j;
                            if (p < n) {
                                const unsigned e0 = ev[i], e1 = ev[p];
                                if (!before(e0, e1)) { ev[i] = e1; ev[p] = e0; }
                            }
                        }
                        sync();
                    }
            }
            double tv = 0.0;                          // this thread's best: value, position, event, S2
            int tp = 0x7FFFFFFF;
            unsigned te = 0;
            unsigned long long ts2 = 0;
            for (int p0 = 0; p0 < n; p0 += NT) {
                const int p = p0 + tid;
                const unsigned e = p < n ? ev[p] : 0u;
                unsigned long long i1 = p < n ? 2ull * fix40(mag[e >> 7]) : 0ull, t1;
                unsigned i2 = 8u * (e & 127u), t2;
                const unsigned long long d1 = i1;
                const unsigned d2 = i2;
                block_scan2<NT>(i1, i2, t1, t2, red);
                const unsigned long long c1 = s1 + i1 + d1, c2 = s2 + i2 + d2;
                const double v = (double)(long long)c1 / sqrt((double)(long long)c2);
                if (p < n && v > tv) { tv = v; tp = p; te = e; ts2 = c2; }
                s1 += t1;
                s2 += t2;
            }
            // largest value, earliest position
            const double bv = block_max<NT>(tv, red);
            const int bp = block_min<NT>(tv == bv ? tp : 0x7FFFFFFF, red);
            if (bp != 0x7FFFFFFF && bv > best_v) {
                sync();
                if (tp == bp) { red[0] = te; red[1] = ts2; }
                sync();
                best_v = bv;
                best_ev = (unsigned)red[0];
                best_s2 = red[1];
                have = true;
            }
            sync();                                   // the keys have been read
        };

        bool some = false;                            // an event lies before the range
        double lb = 0.0;                              // best squared objective at an edge
        bool first = true, done = false;
        // Few levels: the maximum lies well inside the first octaves and one bin
        // takes the rest of the range.  Many (K > 31): it can lie near their end
        // (t max a about K), so that end is bounded more finely.
        const int wide = K > 31 ? kWide : 1;
        sync();
        int n = dp * K;                               // an upper bound, enough for the first pass
        if (n <= kSortMax) n = set_range(bhi, blo);
        for (int pass = 0; n > kSortMax && pass < kPasses; ++pass) {
            // ---- bins: NF of 2^sh bit patterns, then wide ones (first pass) ----
            const int NF = first ? NB - wide : NB;
            int sh = first ? 26 - (31 - __clz(NB)) : 0;
            if (!first) while (((unsigned)NB << sh) < bhi - blo) ++sh;
            auto edge = [&](int j) -> unsigned {      // bits of e_j, at or above the end of the range
                const unsigned off = (unsigned)min(j, NF) << sh;
                const unsigned o = off + (j > NF ? ((1u << (j - NF)) - 1u) << 23 : 0u);
                return j == NB || o >= bhi - blo ? blo : bhi - o;
            };
            for (int t = tid; t < NB + 1; t += NT) { b1[t] = 0ull; bm[t] = 0u; }
            sync();
            // bin of an event by the rounded quotient d: d is within 1.5 steps of
            // a/m (half a step after a correction, taken where bins are narrower
            // than 4 steps), so only an event within two steps of an edge needs
            // the exact test at the two edges of its bin
            const unsigned low = (1u << sh) - 1u;
            auto add = [&](float av, unsigned long long inc, int m, float rm) {
                const float fm = (float)m;
                float d = av * rm;
                if (sh < 2) d = __fmaf_rn(__fmaf_rn(-fm, d, av), rm, d);
                const int off = (int)(bhi - 1u - __float_as_uint(d));
                int j = off >> sh;
                if (((unsigned)(off + 2) & low) < 4u || sh < 2) {
                    j = min(max(j, 0), NF - 1);
                    if (j + 1 < NF && __fmaf_rn(-fm, __uint_as_float(edge(j + 1)), av) < 0.0f) ++j;
                    else if (j > 0 && __fmaf_rn(-fm, __uint_as_float(edge(j)), av) >= 0.0f) --j;
                }
                j = min(max(j, 0), NF - 1);
                atomicAdd(&b1[j], inc);
                atomicAdd(&bm[j], (unsigned)m);
            };
            if (first) {
                const float xf = __uint_as_float(edge(NF)), rf = __builtin_amdgcn_rcpf(xf);
                for (int i = tid; i < dp; i += NT) {
                    const float av = mag[i];
                    const unsigned long long inc = 2ull * fix40(av);
                    const int mf = level_at(av, xf, rf, K);
                    lvl[i] = (unsigned short)mf;
                    for (int m = 1; m <= mf; ++m) add(av, inc, m, s_rm[m]);
                }
                // the wide bins from the levels at their edges (as atomics their many
                // events would all meet at the same few places); the last one is
                // what is left, so its end is the state after all events
                for (int c = 0; c < wide - 1; ++c) {
                    const float xc = __uint_as_float(edge(NF + c + 1)), rc = __builtin_amdgcn_rcpf(xc);
                    unsigned long long q1 = 0;
                    unsigned qm = 0;
                    for (int i = tid; i < dp; i += NT) {
                        const float av = mag[i];
                        const unsigned l = (unsigned)level_at(av, xc, rc, K), h = lvl[i];
                        lvl[i] = (unsigned short)l;
                        q1 += 2ull * fix40(av) * (l - h);
                        qm += (l * (l + 1) - h * (h + 1)) >> 1;
                    }
                    q1 = block_sum<NT>(q1, red);
                    qm = block_sum<NT>(qm, red);
                    if (tid == 0) { b1[NF + c] = q1; bm[NF + c] = qm; }
                }
            } else {
                for (int i = tid; i < dp; i += NT) {
                    const float av = mag[i];
                    const unsigned long long inc = 2ull * fix40(av);
                    for (int m = (lvl[i] & 255) + 1; m <= (lvl[i] >> 8); ++m) add(av, inc, m, s_rm[m]);
                }
            }
            sync();
            // ---- exact states at the edges: exclusive prefix over the bins ----
            {
                unsigned long long q1 = 0, t1;
                unsigned qm = 0, tm;
                unsigned long long e1[kBinsPerThread];
                unsigned em[kBinsPerThread];
#pragma unroll
                for (int k = 0; k < kBinsPerThread; ++k) {
                    e1[k] = b1[kBinsPerThread * tid + k];
                    em[k] = bm[kBinsPerThread * tid + k];
                    q1 += e1[k];
                    qm += em[k];
                }
                block_scan2<NT>(q1, qm, t1, tm, red);
#pragma unroll
                for (int k = 0; k < kBinsPerThread; ++k) {
                    b1[kBinsPerThread * tid + k] = q1;
                    bm[kBinsPerThread * tid + k] = qm;
                    q1 += e1[k];
                    qm += em[k];
                }
                if (tid == NT - 1) { b1[NB] = first ? s1_all : q1; bm[NB] = first ? sm_all : qm; }
            }
            sync();
            // ---- lower bound: the best state at an edge with an event before it ----
            // (found in FP32, evaluated in FP64)
            float fv = 0.0f;
            int fj = 0;
#pragma unroll
            for (int k = 0; k < kBinsPerThread; ++k) {
                const int j = tid + NT * k + 1;
                const float A = fix_f(s1 + b1[j]);
                const float v = A * A * __builtin_amdgcn_rcpf((float)((unsigned)s2 + 8u * bm[j]));
                if ((some || bm[j] > 0u) && v > fv) { fv = v; fj = j; }
            }
            const float bf = block_max<NT>(fv, red);
            fj = block_max<NT>(fv == bf ? fj : 0, red);
            if (fj > 0) {
                const double A = (double)(s1 + b1[fj]);
                lb = fmax(lb, A * A * rcp_d((double)(s2 + 8ull * bm[fj])));
            }
            const double thr = lb * (1.0 - 1e-12);    // covers the rounding of the bounds
            const float thrf = (float)(thr * 0x1p-80) * (1.0f - 0x1p-19f);
            // ---- surviving bins ------------------------------------------------
            int jmin = NB, jmax = -1;
#pragma unroll
            for (int k = 0; k < kBinsPerThread; ++k) {
                const int j = tid + NT * k;
                const unsigned dm = bm[j + 1] - bm[j];
                // no event, or S1 at the end with S2 at the start is below the bound already
                const float Ef = fix_f(s1 + b1[j + 1] + dm);
                if (dm == 0u || Ef * Ef < thrf * (float)((unsigned)s2 + 8u * bm[j])) continue;
                const double A = (double)(s1 + b1[j]), An = (double)(s1 + b1[j + 1]);
                const double B = (double)(s2 + 8ull * bm[j]), Bn = (double)(s2 + 8ull * bm[j + 1]);
                // dm: slack of the fixed point (at most one unit per event) in S1 against m
                const double nn = (double)dm, D = An - A;
                const unsigned eh = edge(j), el = edge(j + 1);
                const double c1 = 0x1p-38 * rcp_d((double)__uint_as_float(eh));   // S2 per unit of S1
                const double c2 = 0x1p-38 * rcp_d((double)__uint_as_float(el));
                bool keep = (A + nn) * (A + nn) >= thr * B || An * An >= thr * (Bn - c2 * nn);
                double xk = (B + c2 * D - Bn) * rcp_d(c2 - c1) + nn;  // where the two lines cross
                xk = fmin(fmax(xk, 0.0), D);
                const double low = fmax(B, B + c1 * (xk - nn));
                keep = keep || (A + xk) * (A + xk) >= thr * low;
                if (keep) { jmin = min(jmin, j); jmax = max(jmax, j); }
            }
            jmin = block_min<NT>(jmin, red);
            jmax = block_max<NT>(jmax, red);
            if (jmax < 0) break;                      // cannot happen (the lower bound's bin survives)
            const unsigned nhi = edge(jmin), nlo = edge(jmax + 1);
            s1 += b1[jmin];
            s2 += 8ull * bm[jmin];
            some = some || bm[jmin] > 0u;
            sync();                                   // the states have been read
            const bool stuck = !first && sh == 0;     // bins of one step: nothing finer
            first = false;
            n = set_range(nhi, nlo);
            if (stuck) break;
        }
        if (n <= cap) {
            enumerate(n);
        } else {
            // windows: the longest range from bhi that holds at most cap events
            const unsigned end = blo;
            while (!done) {
                const unsigned from = bhi;
                unsigned xb = end;
                n = set_range(from, end);
                if (n > cap) {
                    unsigned lo = end, hi = from - 1u;    // [lo, from) is too many, [hi, from) is not
                    while (hi - lo > 1u) {
                        const unsigned mid = lo + ((hi - lo) >> 1);
                        if (set_range(from, mid) > cap) lo = mid; else hi = mid;
                    }
                    xb = hi;
                    n = set_range(from, xb);
                }
                if (n > 0) enumerate(n);
                done = xb == end;
                bhi = xb;
            }
        }
    }

    // ---- replay: levels of the state at the best event ------------------------
    // level m of coordinate i belongs to it when a_i/m > a_b/m_b, or equal and
    // i <= b: a_i m_b against a_b m, exact in double
    const int bdim = (int)(best_ev >> 7);
    const double bm_ = (double)(best_ev & 127u);
    const double ba = have ? (double)mag[bdim] : 1.0;
    const float rb = have ? (float)bm_ / (float)ba : 0.0f;
    double ip = 0.0, nr = 0.0;
    uint8_t* crow = codes + row * (int64_t)dp;
    for (int i0 = 4 * tid; i0 < dp; i0 += 4 * NT) {
        const f4u rv = *(const f4u*)(r + i0);
        const float4 mv = *(const float4*)(mag + i0);
        const float av[4] = {mv.x, mv.y, mv.z, mv.w};
        unsigned out = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            int lev = 0;
            if (have) {
                const float x = fminf((float)(K + 1), av[u] * rb), f = floorf(x);
                lev = (int)f;
                if (x - f < kNearLevel || x - f > 1.0f - kNearLevel) {
                    const double q = (double)av[u] * bm_;
                    auto in = [&](int m) { return ba * (double)m < q || (ba * (double)m == q && i0 + u <= bdim); };
                    if (lev > 0 && !in(lev)) --lev;
                    else if (in(lev + 1)) ++lev;
                }
                lev = min(lev, K);
            }
            out |= (unsigned)(!(rv[u] < 0.0f) ? half + lev : half - 1 - lev) << (8 * u);
            ip += ((double)lev + 0.5) * (double)fabsf(rv[u]);
            if (norm2 == nullptr) nr += (double)rv[u] * (double)rv[u];
        }
        *(u32u*)(crow + i0) = out;
    }
    ip = block_sum<NT>(ip, red);
    if (norm2 == nullptr) nr = block_sum<NT>(nr, red);
    if (tid == 0) {
        const double nr2 = norm2 ? (double)norm2[row] : nr;
        const double ny = (double)(long long)best_s2 * 0.25;
        float fa = 0.0f, fr = 0.0f, co = 1.0f;
        if (nr2 > 0.0 && ip > 0.0) {
            fa = (float)nr2;
            fr = (float)(-2.0 * nr2 / ip);
            co = (float)(ip / (sqrt(ny) * sqrt(nr2)));
        }
        if (f_add) f_add[row] = fa;
        if (f_rescale) f_rescale[row] = fr;
        if (cos_oo) cos_oo[row] = co;
        if (fac) fac[row] = make_float2(fa, fr);
    }
}

template <int NT>
static hipError_t launch_quantize_t(const float* rrot, int64_t n, int dp, int bits, const float* norm2, uint8_t* codes,
                                    float* f_add, float* f_rescale, float* cos_oo, float2* fac, hipStream_t st)
{
    const int cap = dp > 2 * kSortMax ? dp : 2 * kSortMax;
    const size_t sm = quant_smem(kBinsPerThread * NT, cap, dp);
    constexpr int64_t rows = kLaunchRows * 64 / NT;
    for (int64_t r = 0; r < n; r += rows)
        hipLaunchKernelGGL(quantize_kernel<NT>, dim3((unsigned)std::min(rows, n - r)), dim3(NT), sm, st, rrot + r * dp,
                           std::min(rows, n - r), dp, bits, cap, norm2 ? norm2 + r : nullptr, codes + r * dp,
                           f_add ? f_add + r : nullptr, f_rescale ? f_rescale + r : nullptr,
                           cos_oo ? cos_oo + r : nullptr, fac ? fac + r : nullptr);
    return hipGetLastError();
}

hipError_t launch_quantize(const float* rrot, int64_t n, int dp, int bits, const float* norm2,
                           uint8_t* codes, float* f_add, float* f_rescale, float* cos_oo,
                           float2* fac, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    // Few vectors: four waves each, as long as the blocks leave CUs idle (two
    // or four per CU) and a wave alone would have many events (dp 768, B = 4:
    // 1 vector takes 15 us, 512 take 21).  Above, and at few events per wave,
    // the fewest waves that hold the vector.
    const bool few = n <= (bits >= 5 ? 1024 : 512) && (bits >= 5 || dp > 256);
    auto* launch = few || dp > 1536 ? launch_quantize_t<256> : dp > 768 ? launch_quantize_t<128> : launch_quantize_t<64>;
    return launch(rrot, n, dp, bits, norm2, codes, f_add, f_rescale, cos_oo, fac, st);
}

}  // namespace erq
