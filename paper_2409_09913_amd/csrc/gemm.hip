// Dense FP32 / BF16 matrix-core GEMM for the rotation by P (Sec. 3.4: the
// data and the queries are multiplied by P^{-1} = P^T) and for the squared
// distances of the coarse IVF probe (Sec. 4.1).
//
// Workgroup tile 128 x 128, 4 waves each owning 64 x 64 = 2 x 2 tiles of the
// 32 x 32 MFMA.  FP32: v_mfma_f32_32x32x2_f32, K staged 16 at a time.
// BF16: v_mfma_f32_32x32x16_bf16 with FP32 accumulation, K staged 32 at a
// time, inputs rounded to BF16 (nearest even) while staging.
#include <algorithm>

#include "erq_common.h"

namespace erq {

namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
constexpr int BM = 128, BN = 128;

// 32x32 MFMA output element (lane, reg) -> (row, col) within the tile
__device__ inline int out_row(int lane, int r) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

__device__ inline unsigned short f2bf(float f) {
    unsigned u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u) return (unsigned short)(u >> 16);   // inf / nan
    unsigned r = u + 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(r >> 16);
}

// EPI: 0 = store C; 1 = store ||a||^2 + ||b||^2 - 2 C
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(
    const float* __restrict__ A, int64_t n, int K, const float* __restrict__ B, int N, int b_trans,
    float* __restrict__ out, int64_t ldo, const float* __restrict__ an2, const float* __restrict__ bn2)
{
    constexpr int BK = 16;
    // two LDS buffers: the next K-tile is loaded into registers while the
    // current one is multiplied, then stored to the other buffer
    __shared__ float As[2][BK][BM + 4];
    __shared__ float Bs[2][BK][BN + 4];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.y * BM;
    const int col0 = blockIdx.x * BN;
    const int wm = (wid >> 1) * 64, wn = (wid & 1) * 64;
    v16f acc[2][2];
    for (int a = 0; a < 2; ++a) for (int b = 0; b < 2; ++b) for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;

    // 128 x 16 floats per operand = 2 float4 per thread
    float4 ra[2], rb[2];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = tid + 256 * i;
            const int m = e >> 2, kq = (e & 3) * 4;
            const int64_t gr = row0 + m;
            ra[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (gr < n && k0 + kq < K) ra[i] = *(const float4*)(A + gr * (int64_t)K + k0 + kq);
            if (!b_trans) {
                const int kk = e / (BN / 4), nq = (e % (BN / 4)) * 4;
                rb[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (k0 + kk < K && col0 + nq < N) rb[i] = *(const float4*)(B + (int64_t)(k0 + kk) * N + col0 + nq);
            } else {
                const int gc = col0 + m;
                rb[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (gc < N && k0 + kq < K) rb[i] = *(const float4*)(B + (int64_t)gc * K + k0 + kq);
            }
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = tid + 256 * i;
            const int m = e >> 2, kq = (e & 3) * 4;
            As[buf][kq + 0][m] = ra[i].x; As[buf][kq + 1][m] = ra[i].y;
            As[buf][kq + 2][m] = ra[i].z; As[buf][kq + 3][m] = ra[i].w;
            if (!b_trans) {
                const int kk = e / (BN / 4), nq = (e % (BN / 4)) * 4;
                *(float4*)&Bs[buf][kk][nq] = rb[i];
            } else {
                Bs[buf][kq + 0][m] = rb[i].x; Bs[buf][kq + 1][m] = rb[i].y;
                Bs[buf][kq + 2][m] = rb[i].z; Bs[buf][kq + 3][m] = rb[i].w;
            }
        }
    };
    load(0);
    store(0);
    __syncthreads();
    int cur = 0;
    for (int k0 = 0; k0 < K; k0 += BK) {
        const bool more = k0 + BK < K;
        if (more) load(k0 + BK);
#pragma unroll
        for (int ks = 0; ks < BK; ks += 2) {
            float a0 = As[cur][ks + (lane >> 5)][wm + (lane & 31)];
            float a1 = As[cur][ks + (lane >> 5)][wm + 32 + (lane & 31)];
            float b0 = Bs[cur][ks + (lane >> 5)][wn + (lane & 31)];
            float b1 = Bs[cur][ks + (lane >> 5)][wn + 32 + (lane & 31)];
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
        }
        if (more) store(cur ^ 1);
        __syncthreads();
        cur ^= 1;
    }
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) {
            const int gc = col0 + wn + 32 * b + (lane & 31);
            if (gc >= N) continue;
            for (int r = 0; r < 16; ++r) {
                const int64_t gr = row0 + wm + 32 * a + out_row(lane, r);
                if (gr >= n) continue;
                float v = acc[a][b][r];
                if (EPI == 1) v = (an2[gr] + bn2[gc]) - 2.0f * v;
                out[gr * ldo + gc] = v;
            }
        }
}

__global__ __launch_bounds__(256) void gemm_bf16_kernel(
    const float* __restrict__ A, int64_t n, int K, const float* __restrict__ B, int N, int b_trans,
    float* __restrict__ out, int64_t ldo)
{
    constexpr int BK = 32;
    // row-major by the contraction index so that a lane reads 8 consecutive k
    __shared__ unsigned short As[BM][BK + 8];
    __shared__ unsigned short Bs[BN][BK + 8];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.y * BM;
    const int col0 = blockIdx.x * BN;
    const int wm = (wid >> 1) * 64, wn = (wid & 1) * 64;
    v16f acc[2][2];
    for (int a = 0; a < 2; ++a) for (int b = 0; b < 2; ++b) for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
    for (int k0 = 0; k0 < K; k0 += BK) {
        for (int e = tid; e < BM * BK / 4; e += 256) {
            int m = e / (BK / 4), kq = (e % (BK / 4)) * 4;
            int64_t gr = row0 + m;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (gr < n && k0 + kq < K) v = *(const float4*)(A + gr * (int64_t)K + k0 + kq);
            As[m][kq + 0] = f2bf(v.x); As[m][kq + 1] = f2bf(v.y); As[m][kq + 2] = f2bf(v.z); As[m][kq + 3] = f2bf(v.w);
        }
        if (!b_trans) {
            for (int e = tid; e < BK * BN / 4; e += 256) {
                int kk = e / (BN / 4), nq = (e % (BN / 4)) * 4;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (k0 + kk < K && col0 + nq < N) v = *(const float4*)(B + (int64_t)(k0 + kk) * N + col0 + nq);
                Bs[nq + 0][kk] = f2bf(v.x); Bs[nq + 1][kk] = f2bf(v.y); Bs[nq + 2][kk] = f2bf(v.z); Bs[nq + 3][kk] = f2bf(v.w);
            }
        } else {
            for (int e = tid; e < BN * BK / 4; e += 256) {
                int nn = e / (BK / 4), kq = (e % (BK / 4)) * 4;
                int gc = col0 + nn;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (gc < N && k0 + kq < K) v = *(const float4*)(B + (int64_t)gc * K + k0 + kq);
                Bs[nn][kq + 0] = f2bf(v.x); Bs[nn][kq + 1] = f2bf(v.y); Bs[nn][kq + 2] = f2bf(v.z); Bs[nn][kq + 3] = f2bf(v.w);
            }
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < BK; ks += 16) {
            const int kk = ks + 8 * (lane >> 5);
            v8bf a0, a1, b0, b1;
            __builtin_memcpy(&a0, &As[wm + (lane & 31)][kk], 16);
            __builtin_memcpy(&a1, &As[wm + 32 + (lane & 31)][kk], 16);
            __builtin_memcpy(&b0, &Bs[wn + (lane & 31)][kk], 16);
            __builtin_memcpy(&b1, &Bs[wn + 32 + (lane & 31)][kk], 16);
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b1, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b0, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, acc[1][1], 0, 0, 0);
        }
        __syncthreads();
    }
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) {
            const int gc = col0 + wn + 32 * b + (lane & 31);
            if (gc >= N) continue;
            for (int r = 0; r < 16; ++r) {
                const int64_t gr = row0 + wm + 32 * a + out_row(lane, r);
                if (gr < n) out[gr * ldo + gc] = acc[a][b][r];
            }
        }
}

}  // namespace

hipError_t launch_gemm(const float* A, int64_t n, int K, const float* B, int N, int b_trans,
                       int precision, float* out, int64_t ldo, hipStream_t st)
{
    if (n <= 0 || N <= 0) return hipSuccess;
    dim3 grid((unsigned)((N + BN - 1) / BN), (unsigned)((n + BM - 1) / BM));
    if (precision == 1)
        hipLaunchKernelGGL(gemm_bf16_kernel, grid, dim3(256), 0, st, A, n, K, B, N, b_trans, out, ldo);
    else
        hipLaunchKernelGGL(gemm_f32_kernel<0>, grid, dim3(256), 0, st, A, n, K, B, N, b_trans, out, ldo,
                           (const float*)nullptr, (const float*)nullptr);
    return hipGetLastError();
}

// dist = ||a||^2 + ||b||^2 - 2 a.b, with norms an2 (n) and bn2 (N) precomputed
// FP32 -> two BF16 planes: hi = bf16(x) and lo = bf16(x - hi) (x - hi is
// exact, so x = hi + lo to 2^-17 relative); bit patterns, 4 elements per
// thread, n a multiple of 4.
__global__ __launch_bounds__(256) void split_bf16_kernel(const float* __restrict__ x, int64_t n,
                                                         unsigned short* __restrict__ hi,
                                                         unsigned short* __restrict__ lo)
{
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= n) return;
    const float4 v = *(const float4*)(x + i);
    const float xv[4] = {v.x, v.y, v.z, v.w};
    unsigned h[4], l[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        h[c] = f2bf(xv[c]);
        l[c] = f2bf(xv[c] - __uint_as_float(h[c] << 16));
    }
    *(uint2*)(hi + i) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    *(uint2*)(lo + i) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
}

__device__ inline uint4 ld16(const unsigned short* p, bool ok) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (ok) v = *(const uint4*)p;
    return v;
}

// EPI 1: squared distances ||a||^2 + ||b||^2 - 2 a.b of the coarse probe;
// EPI 2: negated inner products -a.b (the probe of the inner-product
// metrics); EPI 0: a.b (the query rotation).  Products on the BF16 matrix cores, from
// operands split beforehand into hi
// and lo BF16 planes (split_bf16_kernel): a.b = lo.hi + hi.lo + hi.hi per
// 16-wide K chunk, FP32 accumulation.  Each product is off by at most
// 2^-15 |a_i b_i| (the dropped lo.lo and the two split residuals), so a
// distance by at most 2^-14 sum|a_i b_i| plus FP32 accumulation: a few units
// in the 5th digit, enough to order centroids except near-ties.  A is n x K,
// B is N x K (row-major planes), K a multiple of 32.  Tile 128 x 128, K
// staged 32 at a time in one LDS buffer (40 KB, so several blocks share a
// CU); the next K-tile is loaded into registers while the current one is
// multiplied.
template <int EPI>
__global__ __launch_bounds__(256, 3) void sqdist_bf16x3_kernel(
    const unsigned short* __restrict__ Ahg, const unsigned short* __restrict__ Alg, int64_t n, int K,
    const unsigned short* __restrict__ Bhg, const unsigned short* __restrict__ Blg, int N,
    float* __restrict__ out, int64_t ldo, const float* __restrict__ an2, const float* __restrict__ bn2)
{
    constexpr int BK = 32, LD = BK + 8;
    __shared__ __align__(16) unsigned short Ah[BM][LD], Al[BM][LD], Bh[BN][LD], Bl[BN][LD];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.y * BM;
    const int col0 = blockIdx.x * BN;
    const int wm = (wid >> 1) * 64, wn = (wid & 1) * 64;
    v16f acc[2][2];
    for (int a = 0; a < 2; ++a) for (int b = 0; b < 2; ++b) for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
    // per K-tile and plane: 128 rows x 32 k = 512 chunks of 16 bytes; thread
    // tid moves chunks tid and tid + 256 (row m = e/4, k offset 8*(e%4))
    const int m0 = tid >> 2, m1 = m0 + 64, kq = (tid & 3) * 8;
    const bool a0 = row0 + m0 < n, a1 = row0 + m1 < n, b0 = col0 + m0 < N, b1 = col0 + m1 < N;
    const unsigned short* pa0h = Ahg + (row0 + m0) * K + kq;
    const unsigned short* pa1h = Ahg + (row0 + m1) * K + kq;
    const unsigned short* pa0l = Alg + (row0 + m0) * K + kq;
    const unsigned short* pa1l = Alg + (row0 + m1) * K + kq;
    const unsigned short* pb0h = Bhg + (int64_t)(col0 + m0) * K + kq;
    const unsigned short* pb1h = Bhg + (int64_t)(col0 + m1) * K + kq;
    const unsigned short* pb0l = Blg + (int64_t)(col0 + m0) * K + kq;
    const unsigned short* pb1l = Blg + (int64_t)(col0 + m1) * K + kq;
    uint4 r0 = ld16(pa0h, a0), r1 = ld16(pa1h, a1), r2 = ld16(pa0l, a0), r3 = ld16(pa1l, a1);
    uint4 r4 = ld16(pb0h, b0), r5 = ld16(pb1h, b1), r6 = ld16(pb0l, b0), r7 = ld16(pb1l, b1);
    *(uint4*)&Ah[m0][kq] = r0; *(uint4*)&Ah[m1][kq] = r1; *(uint4*)&Al[m0][kq] = r2; *(uint4*)&Al[m1][kq] = r3;
    *(uint4*)&Bh[m0][kq] = r4; *(uint4*)&Bh[m1][kq] = r5; *(uint4*)&Bl[m0][kq] = r6; *(uint4*)&Bl[m1][kq] = r7;
    __syncthreads();
    for (int k0 = 0; k0 < K; k0 += BK) {
        const bool more = k0 + BK < K;
        if (more) {                                 // next K-tile into registers while this one is multiplied
            const int k1 = k0 + BK;
            r0 = ld16(pa0h + k1, a0); r1 = ld16(pa1h + k1, a1); r2 = ld16(pa0l + k1, a0); r3 = ld16(pa1l + k1, a1);
            r4 = ld16(pb0h + k1, b0); r5 = ld16(pb1h + k1, b1); r6 = ld16(pb0l + k1, b0); r7 = ld16(pb1l + k1, b1);
        }
#pragma unroll
        for (int ks = 0; ks < BK; ks += 16) {
            const int kk = ks + 8 * (lane >> 5);
            v8bf ah[2], al[2], bh[2], bl[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                __builtin_memcpy(&ah[t], &Ah[wm + 32 * t + (lane & 31)][kk], 16);
                __builtin_memcpy(&al[t], &Al[wm + 32 * t + (lane & 31)][kk], 16);
                __builtin_memcpy(&bh[t], &Bh[wn + 32 * t + (lane & 31)][kk], 16);
                __builtin_memcpy(&bl[t], &Bl[wn + 32 * t + (lane & 31)][kk], 16);
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[a], bh[b], acc[a][b], 0, 0, 0);
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bl[b], acc[a][b], 0, 0, 0);
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bh[b], acc[a][b], 0, 0, 0);
                }
        }
        __syncthreads();                        // every read of this K-tile is done
        if (more) {
            *(uint4*)&Ah[m0][kq] = r0; *(uint4*)&Ah[m1][kq] = r1; *(uint4*)&Al[m0][kq] = r2; *(uint4*)&Al[m1][kq] = r3;
            *(uint4*)&Bh[m0][kq] = r4; *(uint4*)&Bh[m1][kq] = r5; *(uint4*)&Bl[m0][kq] = r6; *(uint4*)&Bl[m1][kq] = r7;
            __syncthreads();
        }
    }
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) {
            const int gc = col0 + wn + 32 * b + (lane & 31);
            if (gc >= N) continue;
            for (int r = 0; r < 16; ++r) {
                const int64_t gr = row0 + wm + 32 * a + out_row(lane, r);
                if (gr >= n) continue;
                if constexpr (EPI == 1) out[gr * ldo + gc] = (an2[gr] + bn2[gc]) - 2.0f * acc[a][b][r];
                else if constexpr (EPI == 2) out[gr * ldo + gc] = -acc[a][b][r];
                else out[gr * ldo + gc] = acc[a][b][r];
            }
        }
}

// Transposed split of a K x N row-major matrix: hi/lo planes of its
// transpose (N x K), for the B operand of sqdist_bf16x3_kernel.
__global__ __launch_bounds__(256) void split_bf16_t_kernel(const float* __restrict__ x, int K, int N,
                                                           unsigned short* __restrict__ hi,
                                                           unsigned short* __restrict__ lo)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;   // output index: row j of N, column k of K
    if (i >= (int64_t)K * N) return;
    const int64_t j = i / K, k = i - j * K;
    const float v = x[k * N + j];
    const unsigned h = f2bf(v);
    hi[i] = (unsigned short)h;
    lo[i] = f2bf(v - __uint_as_float(h << 16));
}

hipError_t launch_split_bf16_t(const float* x, int K, int N, unsigned short* hi, unsigned short* lo, hipStream_t st)
{
    const int64_t n = (int64_t)K * N;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_bf16_t_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, K, N, hi, lo);
    return hipGetLastError();
}

// out = A.B^T (n x N, leading dimension ldo) from the BF16 hi/lo planes of A
// (n x K) and B (N x K); same products and error as the probe's distances
hipError_t launch_gemm_bf16x3(const unsigned short* Ah, const unsigned short* Al, int64_t n,
                              const unsigned short* Bh, const unsigned short* Bl, int64_t N, int K,
                              float* out, int64_t ldo, hipStream_t st)
{
    if (n <= 0 || N <= 0) return hipSuccess;
    dim3 grid((unsigned)((N + BN - 1) / BN), (unsigned)((n + BM - 1) / BM));
    hipLaunchKernelGGL(sqdist_bf16x3_kernel<0>, grid, dim3(256), 0, st, Ah, Al, n, K, Bh, Bl, (int)N, out, ldo,
                       (const float*)nullptr, (const float*)nullptr);
    return hipGetLastError();
}

// Rows of X (n x K, K a multiple of 4) -> their BF16 hi/lo planes (as
// split_bf16_kernel; not with PLANES = false) and squared norms ||x||^2 (FP32);
// one wave per row, 4 consecutive elements per lane
template <bool PLANES>
__global__ __launch_bounds__(256) void split_norm_kernel(const float* __restrict__ X, int64_t n, int K,
                                                         unsigned short* __restrict__ hi,
                                                         unsigned short* __restrict__ lo, float* __restrict__ n2)
{
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= n) return;
    float s = 0.0f;
    for (int k = 4 * lane; k < K; k += 256) {
        const int64_t i = r * (int64_t)K + k;
        const float4 v = *(const float4*)(X + i);
        const float xv[4] = {v.x, v.y, v.z, v.w};
        unsigned h[4], l[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            s += xv[c] * xv[c];
            if constexpr (PLANES) {
                h[c] = f2bf(xv[c]);
                l[c] = f2bf(xv[c] - __uint_as_float(h[c] << 16));
            }
        }
        if constexpr (PLANES) {
            *(uint2*)(hi + i) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
            *(uint2*)(lo + i) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
        }
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) n2[r] = s;
}

hipError_t launch_split_norm(const float* X, int64_t n, int K, unsigned short* hi, unsigned short* lo, float* n2,
                             hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_norm_kernel<true>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, X, n, K, hi, lo, n2);
    return hipGetLastError();
}

// the squared norms alone (the same sums)
hipError_t launch_norm(const float* X, int64_t n, int K, float* n2, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_norm_kernel<false>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, X, n, K,
                       (unsigned short*)nullptr, (unsigned short*)nullptr, n2);
    return hipGetLastError();
}

hipError_t launch_split_bf16(const float* x, int64_t n, unsigned short* hi, unsigned short* lo, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_bf16_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, st, x, n, hi, lo);
    return hipGetLastError();
}

// Nearest column of every row (the assignment of rows to centroids): the
// smallest of the distances that sqdist_bf16x3_kernel<EPI> would write, ties to
// the lower column, without writing them.  A is read as FP32 and split into its
// BF16 planes on the way to LDS (the same values as split_bf16_kernel's).
//
// A workgroup takes 128 rows and a range of column tiles; every lane keeps the
// best of its columns for its 32 rows in registers over the whole range, so the
// cross-lane work is done once per workgroup.  best (n slots, all ones) holds
// (key of the distance, column) when the columns are split over gridDim.y > 1
// workgroups; with one, the columns go straight to out.
// Bound: LDS traffic and matrix cores, as the probe's GEMM (200,000 x 1024 x
// 768: 1.18 ms for the product, and the 0.8 GB of distances that the separate
// selection wrote, allocated and read back (0.84 ms) are gone).
template <int EPI>
__global__ __launch_bounds__(256, 2) void assign_bf16x3_kernel(
    const float* __restrict__ A, int64_t n, int K, const unsigned short* __restrict__ Bhg,
    const unsigned short* __restrict__ Blg, int N, const float* __restrict__ an2, const float* __restrict__ bn2,
    int tiles_per_block, unsigned long long* __restrict__ best, int32_t* __restrict__ out)
{
    constexpr int BK = 32, LD = BK + 8;
    __shared__ __align__(16) unsigned short Ah[BM][LD], Al[BM][LD], Bh[BN][LD], Bl[BN][LD];
    __shared__ float s_an[BM];
    __shared__ unsigned long long s_best[BM];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * BM;
    const int wm = (wid >> 1) * 64, wn = (wid & 1) * 64;
    if (tid < BM) {
        s_an[tid] = row0 + tid < n && EPI == 1 ? an2[row0 + tid] : 0.0f;
        s_best[tid] = ~0ull;
    }
    // per K-tile: thread tid moves k = 8 (tid % 4) .. + 8 of rows tid/4 and tid/4 + 64
    const int m0 = tid >> 2, m1 = m0 + 64, kq = (tid & 3) * 8;
    const bool a0 = row0 + m0 < n, a1 = row0 + m1 < n;
    const float* pa0 = A + (row0 + m0) * K + kq;
    const float* pa1 = A + (row0 + m1) * K + kq;
    const int tile0 = blockIdx.y * tiles_per_block, tile1 = min(tile0 + tiles_per_block, (N + BN - 1) / BN);
    float bv[2][16];
    int bc[2][16];                                   // column tile (32 wide) of the best
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) { bv[a][r] = __builtin_huge_valf(); bc[a][r] = (tile0 * BN + wn) >> 5; }
    auto ldf = [](const float* p, bool ok, float4& v0, float4& v1) {
        v0 = v1 = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ok) { v0 = *(const float4*)p; v1 = *(const float4*)(p + 4); }
    };
    auto put = [](unsigned short* ph, unsigned short* pl, const float4& v0, const float4& v1) {
        const float x[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        unsigned h[8], l[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            h[c] = f2bf(x[c]);
            l[c] = f2bf(x[c] - __uint_as_float(h[c] << 16));
        }
        *(uint4*)ph = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
        *(uint4*)pl = make_uint4(l[0] | (l[1] << 16), l[2] | (l[3] << 16), l[4] | (l[5] << 16), l[6] | (l[7] << 16));
    };
    for (int tile = tile0; tile < tile1; ++tile) {
        const int col0 = tile * BN;
        const bool b0 = col0 + m0 < N, b1 = col0 + m1 < N;
        const unsigned short* pb0h = Bhg + (int64_t)(col0 + m0) * K + kq;
        const unsigned short* pb1h = Bhg + (int64_t)(col0 + m1) * K + kq;
        const unsigned short* pb0l = Blg + (int64_t)(col0 + m0) * K + kq;
        const unsigned short* pb1l = Blg + (int64_t)(col0 + m1) * K + kq;
        v16f acc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
        float4 f0, f1, f2, f3;
        uint4 r4, r5, r6, r7;
        auto load = [&](int k) {
            ldf(pa0 + k, a0, f0, f1);
            ldf(pa1 + k, a1, f2, f3);
            r4 = ld16(pb0h + k, b0); r5 = ld16(pb1h + k, b1); r6 = ld16(pb0l + k, b0); r7 = ld16(pb1l + k, b1);
        };
        auto store = [&]() {
            put(&Ah[m0][kq], &Al[m0][kq], f0, f1);
            put(&Ah[m1][kq], &Al[m1][kq], f2, f3);
            *(uint4*)&Bh[m0][kq] = r4; *(uint4*)&Bh[m1][kq] = r5; *(uint4*)&Bl[m0][kq] = r6; *(uint4*)&Bl[m1][kq] = r7;
        };
        load(0);
        store();
        __syncthreads();
        for (int k0 = 0; k0 < K; k0 += BK) {
            const bool more = k0 + BK < K;
            if (more) load(k0 + BK);                // into registers while this K-tile is multiplied
#pragma unroll
            for (int ks = 0; ks < BK; ks += 16) {
                const int kk = ks + 8 * (lane >> 5);
                v8bf ah[2], al[2], bh[2], bl[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    __builtin_memcpy(&ah[t], &Ah[wm + 32 * t + (lane & 31)][kk], 16);
                    __builtin_memcpy(&al[t], &Al[wm + 32 * t + (lane & 31)][kk], 16);
                    __builtin_memcpy(&bh[t], &Bh[wn + 32 * t + (lane & 31)][kk], 16);
                    __builtin_memcpy(&bl[t], &Bl[wn + 32 * t + (lane & 31)][kk], 16);
                }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[a], bh[b], acc[a][b], 0, 0, 0);
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bl[b], acc[a][b], 0, 0, 0);
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bh[b], acc[a][b], 0, 0, 0);
                    }
            }
            __syncthreads();                        // every read of this K-tile is done
            if (more) {
                store();
                __syncthreads();
            }
        }
        // columns ascend over tiles and b, so a strict comparison keeps the lowest
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int gc = col0 + wn + 32 * b + (lane & 31);
            if (gc < N) {
                const float bn = EPI == 1 ? bn2[gc] : 0.0f;
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float v = EPI == 1 ? (s_an[wm + 32 * a + out_row(lane, r)] + bn) - 2.0f * acc[a][b][r]
                                                 : -acc[a][b][r];
                        const bool better = v < bv[a][r];
                        bv[a][r] = better ? v : bv[a][r];
                        bc[a][r] = better ? (col0 + wn + 32 * b) >> 5 : bc[a][r];
                    }
            }
        }
    }
    // over the 32 lanes of a row, then the two waves of a row
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const unsigned u = __float_as_uint(bv[a][r]);
            unsigned key = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
            unsigned col = (unsigned)(bc[a][r] * 32 + (lane & 31));
            if (col >= (unsigned)N) key = 0xFFFFFFFFu;              // a lane without columns
            for (int o = 16; o > 0; o >>= 1) {
                const unsigned ok = __shfl_xor(key, o), oc = __shfl_xor(col, o);
                const bool take = ok < key || (ok == key && oc < col);
                key = take ? ok : key;
                col = take ? oc : col;
            }
            if ((lane & 31) == 0)
                atomicMin(&s_best[wm + 32 * a + out_row(lane, r)], ((unsigned long long)key << 32) | col);
        }
    __syncthreads();
    if (tid < BM && row0 + tid < n) {
        if (gridDim.y == 1) out[row0 + tid] = (int32_t)(unsigned)s_best[tid];
        else atomicMin(&best[row0 + tid], s_best[tid]);
    }
}

namespace {
__global__ void fill_u64_kernel(unsigned long long* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = ~0ull;
}
__global__ void best_column_kernel(const unsigned long long* best, int64_t n, int32_t* out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (int32_t)(unsigned)best[i];
}
// Workgroups that share a row tile: enough for about three rounds of the
// resident ones (two per CU) where the rows alone do not give them.
int assign_split(int64_t n, int64_t N) {
    const int64_t rows = (n + BM - 1) / BM, tiles = (N + BN - 1) / BN;
    return (int)std::min<int64_t>(tiles, std::max<int64_t>(1, 1536 / rows));
}
}  // namespace

// scratch of launch_assign: the rows' (distance, column) slots when columns are split
size_t assign_scratch_bytes(int64_t n, int64_t N)
{
    return assign_split(n, N) > 1 ? sizeof(unsigned long long) * (size_t)n : 0;
}

hipError_t launch_assign(const float* A, int64_t n, int K, const unsigned short* Bh, const unsigned short* Bl,
                         int64_t N, const float* an2, const float* bn2, int neg_ip, int32_t* out, void* scratch,
                         hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    unsigned long long* best = (unsigned long long*)scratch;
    const int tiles = (int)((N + BN - 1) / BN), split = assign_split(n, N), per = (tiles + split - 1) / split;
    const dim3 grid((unsigned)((n + BM - 1) / BM), (unsigned)((tiles + per - 1) / per));
    const dim3 g1((unsigned)((n + 255) / 256));
    if (grid.y > 1) hipLaunchKernelGGL(fill_u64_kernel, g1, dim3(256), 0, st, best, n);
    if (neg_ip)
        hipLaunchKernelGGL(assign_bf16x3_kernel<2>, grid, dim3(256), 0, st, A, n, K, Bh, Bl, (int)N, an2, bn2, per,
                           best, out);
    else
        hipLaunchKernelGGL(assign_bf16x3_kernel<1>, grid, dim3(256), 0, st, A, n, K, Bh, Bl, (int)N, an2, bn2, per,
                           best, out);
    if (grid.y > 1) hipLaunchKernelGGL(best_column_kernel, g1, dim3(256), 0, st, best, n, out);
    return hipGetLastError();
}

hipError_t launch_sqdist_pre(const unsigned short* Ah, const unsigned short* Al, int64_t n,
                             const unsigned short* Bh, const unsigned short* Bl, int64_t N, int K,
                             const float* an2, const float* bn2, float* out, hipStream_t st, int neg_ip)
{
    if (n <= 0 || N <= 0) return hipSuccess;
    dim3 grid((unsigned)((N + BN - 1) / BN), (unsigned)((n + BM - 1) / BM));
    if (neg_ip)
        hipLaunchKernelGGL(sqdist_bf16x3_kernel<2>, grid, dim3(256), 0, st, Ah, Al, n, K, Bh, Bl, (int)N, out,
                           (int64_t)N, an2, bn2);
    else
        hipLaunchKernelGGL(sqdist_bf16x3_kernel<1>, grid, dim3(256), 0, st, Ah, Al, n, K, Bh, Bl, (int)N, out,
                           (int64_t)N, an2, bn2);
    return hipGetLastError();
}

}  // namespace erq
