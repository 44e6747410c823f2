// Matrix-core products: the rotation by P (Sec. 3.4: the data and the queries
// are multiplied by P^{-1} = P^T) in FP32, BF16 or BF16 hi/lo form, the
// distances of the coarse IVF probe (Sec. 4.1) and the assignment of rows to
// centroids in the hi/lo form.
//
// FP32 and BF16 (gemm_*): workgroup tile 128 x 128, 4 waves each owning 64 x 64
// = 2 x 2 tiles of the 32 x 32 MFMA.  FP32: v_mfma_f32_32x32x2_f32, K staged 16
// at a time.  BF16: v_mfma_f32_32x32x16_bf16 with FP32 accumulation, K staged
// 32 at a time, inputs rounded to BF16 (nearest even) while staging.
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

__global__ __launch_bounds__(256) void gemm_f32_kernel(
    const float* __restrict__ A, int64_t n, int K, const float* __restrict__ B, int N, int b_trans,
    float* __restrict__ out, int64_t ldo)
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
                out[gr * ldo + gc] = acc[a][b][r];
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

// out = A.B (B K x N row-major) for few rows, on v_mfma_f32_16x16x4_f32: a wave
// takes MT x NT tiles of 16 x 16 and loads its own operands, D steps of 4 k
// ahead, without LDS.  An FP32 matrix-core output is one chain of fused
// multiply-adds over k ascending whatever the tile shape, so a row gets the same
// bits here as from gemm_f32_kernel (tests compare them); the 16 x 16 x 4 form
// takes 32 cycles for 4 k where 32 x 32 x 2 takes 64 for 2, and a lone wave's
// time is that chain.
template <int MT, int NT, int D>
__global__ __launch_bounds__(64) void gemm_f32_small_kernel(const float* __restrict__ A, int64_t n, int K,
                                                            const float* __restrict__ B, int N,
                                                            float* __restrict__ out, int64_t ldo)
{
    const int lane = threadIdx.x, c = lane & 15, h = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.y * (16 * MT);
    const int col0 = blockIdx.x * (16 * NT);
    const float* pa[MT];
    const float* pb[NT];
#pragma unroll
    for (int a = 0; a < MT; ++a) {
        const int64_t r = row0 + 16 * a + c;
        pa[a] = A + (r < n ? r : n - 1) * K + h;
    }
#pragma unroll
    for (int b = 0; b < NT; ++b) {
        const int j = col0 + 16 * b + c;
        pb[b] = B + (int64_t)h * N + (j < N ? j : N - 1);
    }
    v4f acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.0f;
    float fa[D][MT], fb[D][NT];
    auto load = [&](int d, int s) {
#pragma unroll
        for (int a = 0; a < MT; ++a) fa[d][a] = pa[a][4 * s];
#pragma unroll
        for (int b = 0; b < NT; ++b) fb[d][b] = pb[b][(int64_t)4 * s * N];
    };
    const int S = K >> 2;                             // a multiple of 16, and D of 16's divisors
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, d);
    for (int s0 = 0; s0 < S; s0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[d][a], fb[d][b], acc[a][b], 0, 0, 0);
            load(d, s0 + D < S ? s0 + D + d : s0 + d);   // past the end the last steps again
        }
    }
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) {
            const int j = col0 + 16 * b + c;
            if (j >= N) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t i = row0 + 16 * a + 4 * h + r;
                if (i < n) out[i * ldo + j] = acc[a][b][r];
            }
        }
}

template <int MT, int NT, int D>
hipError_t launch_gemm_small(const float* A, int64_t n, int K, const float* B, int N, float* out, int64_t ldo,
                             hipStream_t st)
{
    const dim3 grid((unsigned)((N + 16 * NT - 1) / (16 * NT)), (unsigned)((n + 16 * MT - 1) / (16 * MT)));
    hipLaunchKernelGGL((gemm_f32_small_kernel<MT, NT, D>), grid, dim3(64), 0, st, A, n, K, B, N, out, ldo);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm(const float* A, int64_t n, int K, const float* B, int N, int b_trans,
                       int precision, float* out, int64_t ldo, hipStream_t st)
{
    if (n <= 0 || N <= 0) return hipSuccess;
    dim3 grid((unsigned)((N + BN - 1) / BN), (unsigned)((n + BM - 1) / BM));
    // Few 128 x 128 tiles leave CUs idle behind K / 16 staged steps.  768 x 768,
    // us against the tiles' 71: 1 row 8.5, 128 rows 14, 512 rows 36, 1000 rows 43,
    // 2,000 rows (96 tiles) 75.  Other widths, up to the last sizes under 96 tiles:
    // 128 x 128, 1 to 4,096 rows 7.8 against 15; 1536 x 1536, 100 rows 35, 800 rows
    // (84 tiles) 126 against 138; 3072 x 3072, 1 row 33, 100 rows 125, 380 rows (72)
    // 234 against 273; 4096 x 4096, 100 rows 193, 256 rows (64) 295 against 362.
    // 1 x 1 tiles of 16 up to two waves per SIMD.
    if (precision != 1 && !b_trans && (int64_t)grid.x * grid.y < 96) {
        if ((n + 15) / 16 * ((N + 15) / 16) < 2048) return launch_gemm_small<1, 1, 16>(A, n, K, B, N, out, ldo, st);
        return launch_gemm_small<2, 2, 8>(A, n, K, B, N, out, ldo, st);
    }
    if (precision == 1)
        hipLaunchKernelGGL(gemm_bf16_kernel, grid, dim3(256), 0, st, A, n, K, B, N, b_trans, out, ldo);
    else
        hipLaunchKernelGGL(gemm_f32_kernel, grid, dim3(256), 0, st, A, n, K, B, N, b_trans, out, ldo);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// BF16 hi/lo products.  An FP32 matrix of rows (queries, centroids, columns of
// P) is split into hi = bf16(x) and lo = bf16(x - hi) (x - hi is exact, so x =
// hi + lo to 2^-17 relative) and a.b is taken as lo.hi + hi.lo + hi.hi per
// 16-wide K chunk with FP32 accumulation: each product is off by at most 2^-15
// |a_i b_i| (the dropped lo.lo and the two split residuals), so a distance by
// at most 2^-14 sum|a_i b_i| plus FP32 accumulation: a few units in the 5th
// digit, enough to order centroids except near-ties.
//
// Plane layout ("fragments"): rows in tiles of 32, K in chunks of 16; a (tile,
// chunk) holds the hi fragment and then the lo fragment, 1 KB each, lane L's 16
// bytes being the 8 consecutive k = 16 chunk + 8 (L / 32) .. of row L % 32.
// That is the operand of v_mfma_f32_32x32x16_bf16, so every kernel below loads
// it with one coalesced 16-byte load per lane, straight to registers.  Rows are
// padded to a whole tile; what the padding holds does not matter (it only
// reaches rows and columns that are not stored).
// ---------------------------------------------------------------------------
size_t plane_elems(int64_t n, int K) { return (size_t)((n + 31) / 32 * 32) * (size_t)K * 2; }

namespace {

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// two floats -> packed hi and lo planes (round to nearest even)
__device__ inline void split2(float x, float y, unsigned& hi, unsigned& lo) {
    const v2bf h = __builtin_convertvector((v2f){x, y}, v2bf);
    __builtin_memcpy(&hi, &h, 4);
    const v2bf l = __builtin_convertvector((v2f){x - __uint_as_float(hi << 16), y - __uint_as_float(hi & 0xFFFF0000u)},
                                           v2bf);
    __builtin_memcpy(&lo, &l, 4);
}

// element offset of the hi plane of (row, k); the lo plane's is 512 further
__device__ inline int64_t plane_at(int64_t row, int k, int K) {
    return ((row >> 5) * (K >> 4) + (k >> 4)) * 1024 + (((row & 31) + 32 * ((k >> 3) & 1)) << 3) + (k & 7);
}

}  // namespace

// Rows of X (n x K, K a multiple of 64) -> their planes (when given) and
// squared norms ||x||^2 (FP32, when given); a lane has 4 consecutive elements
// of a row, 256 k a step.  RPW = 4: a workgroup takes 16 rows, 4 per wave, and
// puts a step's fragments together in LDS, so that the planes are written in
// runs of 256 bytes (the padding per chunk spreads the 16 chunks of a row over
// the banks).  RPW = 1, for few rows: one row per wave, 8-byte pieces written
// straight from registers (one row of 768: 2.5 us against 6.6; 10,000 rows: 25
// us against 13).
template <int RPW>
__global__ __launch_bounds__(256) void split_norm_kernel(const float* __restrict__ X, int64_t n, int K,
                                                         unsigned short* __restrict__ planes, float* __restrict__ n2)
{
    constexpr int RB = 4 * RPW, CS = 64 * RB + 16;    // rows of the workgroup, bytes of a chunk in LDS
    __shared__ __align__(16) char frag[RPW > 1 ? 16 * CS : 16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t rb = (int64_t)blockIdx.x * RB, r0 = rb + wid * RPW;
    float s[RPW];
#pragma unroll
    for (int u = 0; u < RPW; ++u) s[u] = 0.0f;
    for (int k0 = 0; k0 < K; k0 += 256) {
        const int k = k0 + 4 * lane, nch = min(16, (K - k0) >> 4);
        float4 v[RPW];
#pragma unroll
        for (int u = 0; u < RPW; ++u)
            v[u] = r0 + u < n && k < K ? *(const float4*)(X + (r0 + u) * K + k) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < RPW; ++u) {
            if (k < K) {
                s[u] += v[u].x * v[u].x;
                s[u] += v[u].y * v[u].y;
                s[u] += v[u].z * v[u].z;
                s[u] += v[u].w * v[u].w;
            }
            if (planes) {
                uint2 h, l;
                split2(v[u].x, v[u].y, h.x, l.x);
                split2(v[u].z, v[u].w, h.y, l.y);
                if constexpr (RPW > 1) {              // chunk: hi | lo, each half 0 | half 1 of RB rows
                    char* p = frag + (lane >> 2) * CS + (wid * RPW + u + RB * ((lane >> 1) & 1)) * 16 + 8 * (lane & 1);
                    *(uint2*)p = h;
                    *(uint2*)(p + 32 * RB) = l;
                } else if (r0 < n && k < K) {
                    unsigned short* p = planes + plane_at(r0, k, K);
                    *(uint2*)p = h;
                    *(uint2*)(p + 512) = l;
                }
            }
        }
        if (RPW > 1 && planes) {
            __syncthreads();
            uint4* o = (uint4*)planes + ((rb >> 5) * (K >> 4) + (k0 >> 4)) * 128 + (rb & 31);
            for (int t = tid; t < nch * 4 * RB; t += 256) {
                const int c = t / (4 * RB), i = t % (4 * RB);             // i: (plane, half) x row
                o[c * 128 + (i / RB) * 32 + i % RB] = *(const uint4*)(frag + c * CS + i * 16);
            }
            __syncthreads();
        }
    }
    if (n2) {
#pragma unroll
        for (int u = 0; u < RPW; ++u) {
            for (int o = 32; o > 0; o >>= 1) s[u] += __shfl_xor(s[u], o);
            if (lane == 0 && r0 + u < n) n2[r0 + u] = s[u];
        }
    }
}

hipError_t launch_split_norm(const float* X, int64_t n, int K, unsigned short* planes, float* n2, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    for (int64_t r0 = 0; r0 < n; r0 += kLaunchRows) {
        const int64_t m = std::min(kLaunchRows, n - r0);
        const float* x = X + r0 * K;
        unsigned short* pl = planes ? planes + 2 * r0 * K : nullptr;      // whole tiles: kLaunchRows is a multiple of 32
        float* nn = n2 ? n2 + r0 : nullptr;
        if (m <= 2048 || !planes)
            hipLaunchKernelGGL(split_norm_kernel<1>, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, st, x, m, K, pl, nn);
        else
            hipLaunchKernelGGL(split_norm_kernel<4>, dim3((unsigned)((m + 15) / 16)), dim3(256), 0, st, x, m, K, pl, nn);
    }
    return hipGetLastError();
}

// Planes of the transpose of N columns of a row-major matrix of K rows ld apart
// (rows j of N), 8 consecutive k per thread
__global__ __launch_bounds__(256) void split_t_kernel(const float* __restrict__ x, int K, int ld, int N,
                                                      unsigned short* __restrict__ planes)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)(K >> 3) * N) return;
    const int j = (int)(i % N), k = (int)(i / N) * 8;
    unsigned h[4], l[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
        split2(x[(int64_t)(k + 2 * c) * ld + j], x[(int64_t)(k + 2 * c + 1) * ld + j], h[c], l[c]);
    unsigned short* p = planes + plane_at(j, k, K);
    *(uint4*)p = make_uint4(h[0], h[1], h[2], h[3]);
    *(uint4*)(p + 512) = make_uint4(l[0], l[1], l[2], l[3]);
}

hipError_t launch_split_t(const float* x, int K, int ld, int N, unsigned short* planes, hipStream_t st)
{
    const int64_t n = (int64_t)(K >> 3) * N;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(split_t_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, K, ld, N, planes);
    return hipGetLastError();
}

namespace {

__device__ inline v8bf as_bf(const uint4& v) {
    v8bf r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

// One output of a product of A's rows with the rows of B (N of them): EPI 1
// squared distances ||a||^2 + ||b||^2 - 2 a.b, 2 negated inner products -a.b, 0 a.b
struct MmOut {
    const unsigned short* B;
    int N;
    int epi;
    float* out;
    int64_t ldo;
    const float* bn2;
};

// The outputs of row tile rt and NT column tiles from ct: the rows' norms are
// loaded together, and only the last row tile tests its rows.
template <int NT>
__device__ inline void store_tile(const v16f (&acc)[NT], const MmOut& o, const float* __restrict__ an2, int64_t n,
                                  int64_t rt, int ct, int lane)
{
    float rn[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int64_t gr = 32 * rt + out_row(lane, r);
        rn[r] = o.epi == 1 ? an2[gr < n ? gr : n - 1] : 0.0f;
    }
    const bool whole = 32 * rt + 32 <= n;
#pragma unroll
    for (int b = 0; b < NT; ++b) {
        const int gc = 32 * (ct + b) + (lane & 31);
        const float bn = o.epi == 1 && gc < o.N ? o.bn2[gc] : 0.0f;
        if (gc >= o.N) continue;
        float* p = o.out + (32 * rt + out_row(lane, 0)) * o.ldo + gc;
        auto value = [&](int r) {
            const float c = acc[b][r];
            return o.epi == 1 ? (rn[r] + bn) - 2.0f * c : o.epi == 2 ? -c : c;
        };
        if (whole) {
#pragma unroll
            for (int r = 0; r < 16; ++r) p[(8 * (r >> 2) + (r & 3)) * o.ldo] = value(r);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (32 * rt + out_row(lane, r) < n) p[(8 * (r >> 2) + (r & 3)) * o.ldo] = value(r);
        }
    }
}

// Products of A (n x K planes) with the rows of two matrices in one launch:
// the column blocks of o0, then those of o1 (the probe's distances and the
// query rotation share A).  A wave owns MT x NT tiles of 32 x 32, a workgroup
// 4 waves as WR x (4 / WR).  No LDS and no barrier: fragments go from L1/L2 to
// registers, D chunks of K ahead, in a ring that is consumed and refilled in
// place.  Workgroups are dealt to the 8 XCDs so that each takes a contiguous
// range of column blocks (its slice of B stays in its L2) over all rows.
template <int MT, int NT, int WR, int D>
__global__ __launch_bounds__(256, 2) void mm_bf16x3_kernel(const unsigned short* __restrict__ A, int64_t n, int K,
                                                           const float* __restrict__ an2, MmOut o0, MmOut o1,
                                                           int cb0, int64_t rb, int64_t nblk)
{
    constexpr int WC = 4 / WR;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t per = (nblk + 7) >> 3, blk = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per || blk >= nblk) return;
    int cb = (int)(blk / rb);
    const int64_t rt0 = ((blk - cb * rb) * WR + wid / WC) * MT;          // first row tile of the wave
    const bool second = cb >= cb0;
    const MmOut& o = second ? o1 : o0;
    if (second) cb -= cb0;
    const int ct0 = (cb * WC + wid % WC) * NT;                           // first column tile
    const int64_t rtn = (n + 31) >> 5;
    const int ctn = (o.N + 31) >> 5;
    if (rt0 >= rtn || ct0 >= ctn) return;
    const int S = K >> 4;                                                // chunks: a multiple of 4
    const uint4* pa[MT];
    const uint4* pb[NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
        pa[a] = (const uint4*)A + (rt0 + a < rtn ? rt0 + a : rtn - 1) * S * 128 + lane;
#pragma unroll
    for (int b = 0; b < NT; ++b)
        pb[b] = (const uint4*)o.B + (int64_t)(ct0 + b < ctn ? ct0 + b : ctn - 1) * S * 128 + lane;
    v16f acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
    uint4 fa[D][MT][2], fb[D][NT][2];
    auto load = [&](int d, int s) {
#pragma unroll
        for (int a = 0; a < MT; ++a) { fa[d][a][0] = pa[a][s * 128]; fa[d][a][1] = pa[a][s * 128 + 64]; }
#pragma unroll
        for (int b = 0; b < NT; ++b) { fb[d][b][0] = pb[b][s * 128]; fb[d][b][1] = pb[b][s * 128 + 64]; }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, D > 4 ? min(d, S - 1) : d);
    for (int s0 = 0; s0 < S; s0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (D > 4 && s0 + d >= S) break;         // wave-uniform (S is a multiple of 4)
            v8bf ah[MT], al[MT], bh[NT], bl[NT];
#pragma unroll
            for (int a = 0; a < MT; ++a) { ah[a] = as_bf(fa[d][a][0]); al[a] = as_bf(fa[d][a][1]); }
#pragma unroll
            for (int b = 0; b < NT; ++b) { bh[b] = as_bf(fb[d][b][0]); bl[b] = as_bf(fb[d][b][1]); }
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[a], bh[b], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bl[b], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int b = 0; b < NT; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bh[b], acc[a][b], 0, 0, 0);
            load(d, min(s0 + d + D, S - 1));         // past the end the last chunk again: no load is conditional
        }
    }
    __builtin_amdgcn_sched_barrier(0);                // the epilogue's loads hold no registers through the loop
#pragma unroll
    for (int a = 0; a < MT; ++a) store_tile<NT>(acc[a], o, an2, n, rt0 + a, ct0, lane);
}

template <int MT, int NT, int WR, int D>
hipError_t launch_mm_t(const unsigned short* A, int64_t n, int K, const float* an2, const MmOut& o0, const MmOut& o1,
                       hipStream_t st)
{
    constexpr int BR = 32 * MT * WR, BC = 32 * NT * (4 / WR);
    const int64_t rb = (n + BR - 1) / BR;
    const int cb0 = (o0.N + BC - 1) / BC, cb1 = (o1.N + BC - 1) / BC;
    const int64_t nblk = rb * (cb0 + cb1);
    hipLaunchKernelGGL((mm_bf16x3_kernel<MT, NT, WR, D>), dim3((unsigned)((nblk + 7) / 8 * 8)), dim3(256), 0, st, A, n,
                       K, an2, o0, o1, cb0, rb, nblk);
    return hipGetLastError();
}

// The same products with both operands in LDS, in two buffers of KC K chunks: 4
// waves take 32 BR x 128 outputs, BR / 2 x 2 tiles each.  BR = 8, KC = 1, for
// many rows (24 KB a buffer, so two workgroups share a CU and fill each other's
// waits); BR = 4, KC = 2 where 256 rows would be mostly padding or leave CUs
// idle.  The fragments are copied global -> LDS without registers; a wave has
// read a buffer's fragments before it issues the next copies, so the compiler's
// wait for copies in front of LDS reads never meets one in flight.  One barrier
// per buffer.
constexpr int kBigC = 4;                              // column tiles of 32 per workgroup

typedef const __attribute__((address_space(1))) void* gptr;
typedef __attribute__((address_space(3))) void* lptr;

// the 2 KB of a (tile, chunk) from global memory to LDS by one wave
__device__ inline void copy_chunk(const uint4* g, char* l) {
    __builtin_amdgcn_global_load_lds((gptr)g, (lptr)l, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((gptr)(g + 64), (lptr)(l + 1024), 16, 0, 0);
}

template <int BR, int KC>
__global__ __launch_bounds__(256, 2) void mm_big_kernel(const unsigned short* __restrict__ A, int64_t n, int K,
                                                        const float* __restrict__ an2, MmOut o0, MmOut o1, int cb0,
                                                        int64_t rb, int64_t nblk)
{
    constexpr int kChunk = (BR + kBigC) * 2048;       // bytes of a chunk: hi and lo fragment per tile
    constexpr int RW = BR / 2, RC = BR / 4;           // row tiles a wave multiplies and copies
    __shared__ __align__(16) char smem[2][KC * kChunk];
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t per = (nblk + 7) >> 3, blk = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per || blk >= nblk) return;
    int cb = (int)(blk / rb);
    const int64_t rt0 = (blk - cb * rb) * BR;
    const bool second = cb >= cb0;
    const MmOut& o = second ? o1 : o0;
    if (second) cb -= cb0;
    const int ct0 = cb * kBigC;
    const int64_t rtn = (n + 31) >> 5;
    const int ctn = (o.N + 31) >> 5;
    const int S = K >> 4;                                                // chunks: a multiple of 4
    // wave w copies row tiles RC w .. and column tile w
    const uint4* ga[RC];
#pragma unroll
    for (int u = 0; u < RC; ++u)
        ga[u] = (const uint4*)A + (rt0 + RC * wid + u < rtn ? rt0 + RC * wid + u : rtn - 1) * S * 128 + lane;
    const uint4* gb = (const uint4*)o.B + (int64_t)(ct0 + wid < ctn ? ct0 + wid : ctn - 1) * S * 128 + lane;
    auto copy = [&](int s, int buf) {
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            char* l = smem[buf] + c * kChunk;
#pragma unroll
            for (int u = 0; u < RC; ++u) copy_chunk(ga[u] + (s + c) * 128, l + (RC * wid + u) * 2048);
            copy_chunk(gb + (s + c) * 128, l + (BR + wid) * 2048);
        }
    };
    const int wr = (wid >> 1) * RW, wc = (wid & 1) * 2;
    v16f acc[RW][2];
#pragma unroll
    for (int a = 0; a < RW; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
    copy(0, 0);
    int buf = 0;
    for (int s = 0; s < S; s += KC, buf ^= 1) {
        const char* cur = smem[buf] + lane * 16;
        __syncthreads();                              // these chunks are in LDS; the other buffer's readers are done
        v8bf ah[KC][RW], al[KC][RW], bh[KC][2], bl[KC][2];
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            auto frag = [&](int tile, int plane) {
                v8bf v;
                __builtin_memcpy(&v, cur + c * kChunk + tile * 2048 + plane * 1024, 16);
                return v;
            };
#pragma unroll
            for (int b = 0; b < 2; ++b) { bh[c][b] = frag(BR + wc + b, 0); bl[c][b] = frag(BR + wc + b, 1); }
#pragma unroll
            for (int a = 0; a < RW; ++a) { ah[c][a] = frag(wr + a, 0); al[c][a] = frag(wr + a, 1); }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s + KC < S) copy(s + KC, buf ^ 1);
#pragma unroll
        for (int c = 0; c < KC; ++c) {
#pragma unroll
            for (int a = 0; a < RW; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[c][a], bh[c][b], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int a = 0; a < RW; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[c][a], bl[c][b], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int a = 0; a < RW; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[c][a], bh[c][b], acc[a][b], 0, 0, 0);
        }
    }
#pragma unroll
    for (int a = 0; a < RW; ++a) store_tile<2>(acc[a], o, an2, n, rt0 + wr + a, ct0 + wc, lane);
}

template <int BR, int KC>
hipError_t launch_mm_big(const unsigned short* A, int64_t n, int K, const float* an2, const MmOut& o0, const MmOut& o1,
                         hipStream_t st)
{
    const int64_t rb = (n + 32 * BR - 1) / (32 * BR);
    const int cb0 = (o0.N + 32 * kBigC - 1) / (32 * kBigC), cb1 = (o1.N + 32 * kBigC - 1) / (32 * kBigC);
    const int64_t nblk = rb * (cb0 + cb1);
    hipLaunchKernelGGL((mm_big_kernel<BR, KC>), dim3((unsigned)((nblk + 7) / 8 * 8)), dim3(256), 0, st, A, n, K, an2,
                       o0, o1, cb0, rb, nblk);
    return hipGetLastError();
}

// 256 x 128 tiles where they give every CU one (10,000 x 4,864 x 768: 199 us
// against 257 with 2 x 2 tiles per wave and no LDS, 270 with 128 x 128 tiles
// staged through registers; 2,000 rows: 56 against 61), unless a quarter of their
// rows or more would be padding: 128 x 128 tiles for 65 to 128 rows and for 257 to
// 384 (100 x 40,000 x 1536: 67 us against 105, 300 x 20,000 x 1536: 74 against 105),
// and up to 64 rows the waves' own loads (1 x 40,000 x 768: 24 us against 57).
// Else every wave loads its own fragments: 2 x 2 tiles where that leaves two
// waves for every SIMD, 2 x 1 down to one (1000 x 5056 x 960: 46 us against 62),
// below that 1 x 1 with the loads 8 chunks ahead, as the chain of one wave is what
// counts (1 x 1,792 x 768: 10 us against 51 with 128 x 128 tiles; 500 x 4,096 x
// 3072: 60 against 240).  Instead of 2 x 1, 128 x 128 tiles where there is one for
// every CU and K is long: each wave's reading of its fragments from L2 then costs
// more than the barriers (200 x 16,384 x 4096: 125 us against 221, x 1536: 42
// against 64).  Planes that are not 16-byte aligned (in a caller's workspace that
// is not) keep away from the direct LDS copies.
hipError_t launch_mm(const unsigned short* A, int64_t n, int K, const float* an2, const MmOut& o0, const MmOut& o1,
                     hipStream_t st)
{
    const int64_t waves = (n + 63) / 64 * ((o0.N + 63) / 64 + (o1.N + 63) / 64);
    const int64_t cols = (o0.N + 127) / 128 + (o1.N + 127) / 128, rows = (n + 127) / 128;
    const bool aligned = (((uintptr_t)A | (uintptr_t)o0.B | (uintptr_t)o1.B) & 15) == 0;
    if (aligned && (rows + 1) / 2 * cols >= 256) {
        if (n <= 32) return launch_mm_t<1, 1, 1, 8>(A, n, K, an2, o0, o1, st);
        if (n <= 64) return launch_mm_t<1, 1, 2, 8>(A, n, K, an2, o0, o1, st);
        if (rows == 1 || rows == 3) return launch_mm_big<4, 2>(A, n, K, an2, o0, o1, st);
        return launch_mm_big<8, 1>(A, n, K, an2, o0, o1, st);
    }
    if (waves >= 2048) return launch_mm_t<2, 2, 2, 2>(A, n, K, an2, o0, o1, st);
    if (n <= 32) return launch_mm_t<1, 1, 1, 8>(A, n, K, an2, o0, o1, st);
    if (aligned && waves >= 900 && K >= (waves >= 1024 ? 1536 : 3072) && rows * cols >= 256) return launch_mm_big<4, 2>(A, n, K, an2, o0, o1, st);
    if (waves >= 1024) return launch_mm_t<2, 1, 2, 2>(A, n, K, an2, o0, o1, st);
    return launch_mm_t<1, 1, 2, 8>(A, n, K, an2, o0, o1, st);
}

}  // namespace

// out = A.(B0 | B1)^T (n x (N0 + N1), leading dimension ldo) from the planes of A
// (n x K), B0 (N0 x K) and B1 (N1 x K; N1 may be 0)
hipError_t launch_gemm_bf16x3(const unsigned short* A, int64_t n, const unsigned short* B0, int N0,
                              const unsigned short* B1, int N1, int K, float* out, int64_t ldo, hipStream_t st)
{
    if (n <= 0 || N0 <= 0) return hipSuccess;
    return launch_mm(A, n, K, nullptr, MmOut{B0, N0, 0, out, ldo, nullptr}, MmOut{B1, N1, 0, out + N0, ldo, nullptr}, st);
}

// The probe's distances D (n x N; negated inner products with neg_ip) and,
// when R is given, the rotation rot = A.R^T (n x NR, leading dimension NR).
hipError_t launch_probe_products(const unsigned short* A, int64_t n, int K, const float* an2, const unsigned short* B,
                                 int64_t N, const float* bn2, int neg_ip, float* D, const unsigned short* R, int NR,
                                 float* rot, hipStream_t st)
{
    if (n <= 0 || N <= 0) return hipSuccess;
    return launch_mm(A, n, K, an2, MmOut{B, (int)N, neg_ip ? 2 : 1, D, N, bn2},
                     MmOut{R ? R : B, R ? NR : 0, 0, rot, NR, nullptr}, st);
}

// Nearest column of every row (the assignment of rows to centroids): the
// smallest of the distances that mm_bf16x3_kernel would write with this EPI (1
// or 2), ties to the lower column, without writing them.
//
// A workgroup takes 128 rows and a range of column tiles (128 wide).  A is read
// as FP32 and split into its planes on the way to LDS (two buffers, one barrier
// per 32 of K); B's fragments go straight to registers.  The product is taken
// transposed (MFMA rows: columns of B, lanes: rows of A), so a row's candidates
// lie in one lane's registers and the running minimum costs no cross-lane work;
// the two half-waves and the two waves of a row meet in LDS once per workgroup.
// 200,000 x 1024 x 768: 1.13 ms, 840 TFLOP/s (1.53 with B staged in LDS too and
// the rounding in integer arithmetic; 256 x 128 tiles spill and take 1.2-1.7).
// best (n slots, all ones) holds (key of the distance, column) when the columns
// are split over gridDim.y > 1 workgroups; with one, they go straight to out.
// The order is the probe selection's, that of the keys: a distance that is a NaN
// comes first or last by its sign.  Where a norm says that there may be one (not
// below kPlainNorm, so that |a.b| <= ||a|| ||b|| and the distance might overflow),
// the wave compares keys from that tile on; else the floats, which is the same
// (keys throughout would be 64 x 3 more instructions a tile).  Three workgroups
// per CU is what the launch bound asks for: left to itself the compiler takes 198
// registers for the second branch and two fit.
constexpr float kPlainNorm = 1e37f;

// order-preserving integer image of a float, and back
__device__ inline unsigned order_key(float v) {
    const unsigned u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float key_value(unsigned k) { return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k); }

template <int EPI>
__global__ __launch_bounds__(256, 3) void assign_bf16x3_kernel(
    const float* __restrict__ A, int64_t n, int K, const unsigned short* __restrict__ B, int N,
    const float* __restrict__ an2, const float* __restrict__ bn2, int tiles_per_block,
    unsigned long long* __restrict__ best, int32_t* __restrict__ out)
{
    constexpr int BK = 32;
    __shared__ __align__(16) unsigned short As[2][4][2][1024];           // buffer, row tile, chunk, hi | lo fragment
    __shared__ float s_bn[BN];
    __shared__ int s_odd[BN / 64];                                       // some norm of the tile's columns is not plain
    __shared__ unsigned long long s_best[BM];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * BM;
    const int wm = (wid >> 1) * 2, wn = (wid & 1) * 2;                   // first row / column tile of the wave
    if (tid < BM) s_best[tid] = ~0ull;
    // thread tid moves 4 k of row tid / 8 of every row tile: 8 lanes a row's 128
    // bytes of a stage
    const int m = tid >> 3, kq = 4 * (tid & 7);
    const float* pa = A + (row0 + m) * K + kq;
    unsigned short* const la = &As[0][0][kq >> 4][(m + 32 * ((kq >> 3) & 1)) * 8 + (kq & 7)];
    const int S = K >> 4, ctn = (N + 31) >> 5;
    const int tile0 = blockIdx.y * tiles_per_block, tile1 = min(tile0 + tiles_per_block, (N + BN - 1) / BN);
    float rn[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int64_t gr = row0 + 32 * (wm + a) + (lane & 31);
        rn[a] = gr < n ? an2[gr] : 0.0f;
    }
    bool odd = __any(!(rn[0] < kPlainNorm) || !(rn[1] < kPlainNorm));    // compare keys (the same in the whole wave)
    float bv[2] = {__builtin_huge_valf(), __builtin_huge_valf()};
    const int first = tile0 * BN + 32 * wn + out_row(lane, 0);
    int bc[2] = {first, first};
    float4 f[4];
    auto load_a = [&](int k) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            f[u] = row0 + m + 32 * u < n ? *(const float4*)(pa + (int64_t)32 * u * K + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    auto store_a = [&](int buf) {
        unsigned short* p = la + buf * (4 * 2 * 1024);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint2 h, l;
            split2(f[u].x, f[u].y, h.x, l.x);
            split2(f[u].z, f[u].w, h.y, l.y);
            *(uint2*)(p + u * 2048) = h;
            *(uint2*)(p + u * 2048 + 512) = l;
        }
    };
    for (int tile = tile0; tile < tile1; ++tile) {
        const uint4* pb[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) pb[b] = (const uint4*)B + (int64_t)min(4 * tile + wn + b, ctn - 1) * S * 128 + lane;
        uint4 fb[2][2][2];
        auto load_b = [&](int s, uint4 (&d)[2][2]) {
#pragma unroll
            for (int b = 0; b < 2; ++b) { d[b][0] = pb[b][s * 128]; d[b][1] = pb[b][s * 128 + 64]; }
        };
        v16f acc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;
        load_b(0, fb[0]);
        load_b(1, fb[1]);
        load_a(0);
        __syncthreads();                             // the last tile's reads of LDS are done
        store_a(0);
        if (tid < BN) {
            const float bn = tile * BN + tid < N ? bn2[tile * BN + tid] : 0.0f;
            s_bn[tid] = bn;
            const bool any = __any(!(bn < kPlainNorm));
            if (lane == 0) s_odd[wid] = any ? 1 : 0;
        }
        __syncthreads();
        int cur = 0;
        for (int k0 = 0; k0 < K; k0 += BK) {
            const bool more = k0 + BK < K;
            if (more) load_a(k0 + BK);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                v8bf ah[2], al[2], bh[2], bl[2];
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    __builtin_memcpy(&ah[a], &As[cur][wm + a][c][lane * 8], 16);
                    __builtin_memcpy(&al[a], &As[cur][wm + a][c][512 + lane * 8], 16);
                }
#pragma unroll
                for (int b = 0; b < 2; ++b) { bh[b] = as_bf(fb[c][b][0]); bl[b] = as_bf(fb[c][b][1]); }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bh[b], al[a], acc[a][b], 0, 0, 0);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bl[b], ah[a], acc[a][b], 0, 0, 0);
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bh[b], ah[a], acc[a][b], 0, 0, 0);
                load_b(min((k0 >> 4) + 2 + c, S - 1), fb[c]);
            }
            if (more) store_a(cur ^ 1);
            __syncthreads();
            cur ^= 1;
        }
        // columns ascend over tiles, b and r, so a strict comparison keeps the lowest
        auto value = [&](int a, int b, int r, float bn) {
            return EPI == 1 ? (rn[a] + bn) - 2.0f * acc[a][b][r] : -acc[a][b][r];
        };
        odd = odd || s_odd[0] != 0 || s_odd[1] != 0;
        if (!odd) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int lc = 32 * (wn + b) + out_row(lane, r), gc = tile * BN + lc;
                    const float bn = s_bn[lc];
                    if (gc < N) {
#pragma unroll
                        for (int a = 0; a < 2; ++a) {
                            const float v = value(a, b, r, bn);
                            const bool better = v < bv[a];
                            bv[a] = better ? v : bv[a];
                            bc[a] = better ? gc : bc[a];
                        }
                    }
                }
        } else {
            unsigned bk[2];                          // nothing yet: above every key but that of the last NaN
#pragma unroll
            for (int a = 0; a < 2; ++a) bk[a] = tile == tile0 ? 0xFFFFFFFFu : order_key(bv[a]);
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int lc = 32 * (wn + b) + out_row(lane, r), gc = tile * BN + lc;
                    const float bn = s_bn[lc];
                    if (gc < N) {
#pragma unroll
                        for (int a = 0; a < 2; ++a) {
                            // (of two NaNs in a sum either may come out: the row's)
                            const float v = EPI == 1 && rn[a] != rn[a] ? rn[a] : value(a, b, r, bn);
                            const unsigned k = order_key(v);
                            const bool better = k < bk[a];
                            bk[a] = better ? k : bk[a];
                            bc[a] = better ? gc : bc[a];
                        }
                    }
                }
#pragma unroll
            for (int a = 0; a < 2; ++a) bv[a] = key_value(bk[a]);
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        if (bc[a] < N)
            atomicMin(&s_best[32 * (wm + a) + (lane & 31)],
                      ((unsigned long long)order_key(bv[a]) << 32) | (unsigned)bc[a]);
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
// Column tiles per workgroup: few enough that there are some 4,000 workgroups
// (three are resident per CU; 200,000 x 1024 x 768: 1.13 ms, 300,000 x 7000 x
// 128: 2.0 against 2.2 with 2,000).
int assign_tiles(int64_t n, int64_t N) {
    const int64_t rows = (n + BM - 1) / BM, tiles = (N + BN - 1) / BN;
    return (int)std::min(tiles, std::max<int64_t>(1, rows * tiles / 4096));
}
}  // namespace

// scratch of launch_assign: the rows' (distance, column) slots when columns are split
size_t assign_scratch_bytes(int64_t n, int64_t N)
{
    return assign_tiles(n, N) < (N + BN - 1) / BN ? sizeof(unsigned long long) * (size_t)n : 0;
}

hipError_t launch_assign(const float* A, int64_t n, int K, const unsigned short* B, int64_t N, const float* an2,
                         const float* bn2, int neg_ip, int32_t* out, void* scratch, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    unsigned long long* best = (unsigned long long*)scratch;
    const int per = assign_tiles(n, N);
    const dim3 grid((unsigned)((n + BM - 1) / BM), (unsigned)(((N + BN - 1) / BN + per - 1) / per));
    const dim3 g1((unsigned)((n + 255) / 256));
    if (grid.y > 1) hipLaunchKernelGGL(fill_u64_kernel, g1, dim3(256), 0, st, best, n);
    auto* k = neg_ip ? assign_bf16x3_kernel<2> : assign_bf16x3_kernel<1>;
    hipLaunchKernelGGL(k, grid, dim3(256), 0, st, A, n, K, B, (int)N, an2, bn2, per, best, out);
    if (grid.y > 1) hipLaunchKernelGGL(best_column_kernel, g1, dim3(256), 0, st, best, n, out);
    return hipGetLastError();
}

}  // namespace erq
