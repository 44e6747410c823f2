// IVF list construction (Sec. 4.1: the lists come from k-means, each
// vector is centred on its own list's centroid, Sec. 5.1):
//  * a stable bucket sort of the rows by list (members of a list in
//    ascending row order), without atomics whose order could change a result;
//  * per-list means with FP64 sums in member order (the k-means update), so
//    the same input gives the same centroids bit for bit on every run;
//  * a row gather (the k-means initial centroids).
// Nothing here waits for the host: the list offsets and the chunks of the
// means are prefix sums on the device.
#include <algorithm>

#include "erq_common.h"

namespace erq {

namespace {

constexpr int kSortThreads = 256;
constexpr int kSortMaxBlocks = 512;
constexpr int kMeanChunk = 1024;      // members per partial sum

inline size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

// blocks of the bucket sort: at most kSortMaxBlocks (two per CU: 200,000 rows
// take 38 us of placement against 123 with 128), and at most 16M per-block
// list counters in total
int sort_blocks(int64_t n, int64_t nlist) {
    int64_t g = std::min<int64_t>(kSortMaxBlocks, std::max<int64_t>(1, ((int64_t)1 << 24) / std::max<int64_t>(nlist, 1)));
    g = std::min<int64_t>(g, std::max<int64_t>(1, (n + kSortThreads - 1) / kSortThreads));
    return (int)g;
}

// cnt2[b][l] = rows of block b's contiguous chunk in list l; bad (or null) is
// set when an id lies outside [0, nlist) (such rows are not counted)
__global__ __launch_bounds__(kSortThreads) void bucket_count_kernel(const int32_t* __restrict__ assign, int64_t n,
                                                                    int64_t nlist, int64_t chunk,
                                                                    int32_t* __restrict__ cnt2,
                                                                    int32_t* __restrict__ bad)
{
    const int64_t b = blockIdx.x;
    const int64_t r0 = b * chunk, r1 = min(n, r0 + chunk);
    for (int64_t r = r0 + threadIdx.x; r < r1; r += kSortThreads) {
        const int32_t l = assign[r];
        if (l < 0 || l >= nlist) {
            if (bad) atomicOr(bad, 1);
            continue;
        }
        atomicAdd(&cnt2[b * nlist + l], 1);
    }
}

// per list: exclusive prefix of cnt2 over the G blocks (in place) and the
// total.  32 lists per workgroup; thread (list, eighth) sums its eighth of the
// blocks, the eighths are combined in LDS
__global__ __launch_bounds__(256) void bucket_total_kernel(int32_t* __restrict__ cnt2, int64_t nlist, int G,
                                                           int32_t* __restrict__ cnt)
{
    __shared__ int32_t part[8][32];
    const int lq = threadIdx.x & 31, e = threadIdx.x >> 5;
    const int64_t l = (int64_t)blockIdx.x * 32 + lq;
    const int per = (G + 7) / 8, b0 = min(G, e * per), b1 = min(G, b0 + per);
    int32_t sum = 0;
    if (l < nlist)
#pragma unroll 8
        for (int b = b0; b < b1; ++b) sum += cnt2[(int64_t)b * nlist + l];
    part[e][lq] = sum;
    __syncthreads();
    if (l >= nlist) return;
    int32_t run = 0;
    for (int w = 0; w < e; ++w) run += part[w][lq];
    if (e == 7) cnt[l] = run + sum;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) {
        const int32_t c = cnt2[(int64_t)b * nlist + l];
        cnt2[(int64_t)b * nlist + l] = run;
        run += c;
    }
}

// One workgroup: list_off = exclusive prefix of the counts, chunk0 = exclusive
// prefix of their chunks of kMeanChunk members (nlist + 1 of each).
__global__ __launch_bounds__(1024) void list_prefix_kernel(const int32_t* __restrict__ cnt, int64_t nlist,
                                                           int64_t* __restrict__ list_off,
                                                           int32_t* __restrict__ chunk0)
{
    __shared__ long long s_n[16], s_c[16];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t per = (nlist + 1023) / 1024, l0 = min(nlist, tid * per), l1 = min(nlist, l0 + per);
    long long n = 0, c = 0;
    for (int64_t l = l0; l < l1; ++l) { n += cnt[l]; c += (cnt[l] + kMeanChunk - 1) / kMeanChunk; }
    long long in = n, ic = c;
    for (int o = 1; o < 64; o <<= 1) {
        const long long un = __shfl_up(in, o), uc = __shfl_up(ic, o);
        if (lane >= o) { in += un; ic += uc; }
    }
    if (lane == 63) { s_n[wid] = in; s_c[wid] = ic; }
    __syncthreads();
    long long rn = in - n, rc = ic - c;
    for (int w = 0; w < wid; ++w) { rn += s_n[w]; rc += s_c[w]; }
    for (int64_t l = l0; l < l1; ++l) {
        list_off[l] = rn;
        chunk0[l] = (int32_t)rc;
        rn += cnt[l];
        rc += (cnt[l] + kMeanChunk - 1) / kMeanChunk;
    }
    if (tid == 1023) { list_off[nlist] = rn; chunk0[nlist] = (int32_t)rc; }
}

// Block b places the rows of its chunk in rounds of kSortThreads rows: a row's
// rank among the round's earlier rows of the same list (LDS), then one atomic
// per list group of the round on the block's own counter, read back by the
// group through LDS.  Only block b touches its counters, and the rounds are
// ordered by barriers, so positions ascend with the row number.
__global__ __launch_bounds__(kSortThreads) void bucket_place_kernel(const int32_t* __restrict__ assign, int64_t n,
                                                                    int64_t nlist, int64_t chunk,
                                                                    const int64_t* __restrict__ list_off,
                                                                    int32_t* __restrict__ base2,
                                                                    int32_t* __restrict__ ids32)
{
    __shared__ int32_t s_l[kSortThreads];
    __shared__ int32_t s_base[kSortThreads];
    const int t = threadIdx.x;
    const int64_t b = blockIdx.x;
    const int64_t r0 = b * chunk, r1 = min(n, r0 + chunk);
    for (int64_t rb = r0; rb < r1; rb += kSortThreads) {
        const int64_t r = rb + t;
        const int32_t l = (r < r1) ? assign[r] : -1;
        s_l[t] = l;
        __syncthreads();
        int rank = 0, first = t, cnt = 0;
        if (l >= 0) {
            for (int u = 0; u < kSortThreads; ++u) {
                if (s_l[u] == l) {
                    if (u < t) { ++rank; first = min(first, u); }
                    ++cnt;
                }
            }
            if (first == t) s_base[t] = (int32_t)list_off[l] + atomicAdd(&base2[b * nlist + l], cnt);
        }
        __syncthreads();
        if (l >= 0) ids32[s_base[first] + rank] = (int32_t)r;
        __syncthreads();
    }
}

// partial FP64 sums of one (list, chunk of kMeanChunk members): thread t sums
// dimensions 4t .. 4t+3 (then those blockDim further) over the chunk's members
// in order, with the 16-byte loads of eight members in flight.  The grid is an
// upper bound of the number of chunks.
__global__ __launch_bounds__(256) void list_psum_kernel(const float* __restrict__ x, int dp,
                                                        const int32_t* __restrict__ ids32,
                                                        const int64_t* __restrict__ list_off, int64_t nlist,
                                                        const int32_t* __restrict__ chunk0,
                                                        double* __restrict__ psum)
{
    const int64_t c = blockIdx.x;
    if (c >= chunk0[nlist]) return;
    int64_t lo = 0, hi = nlist;                    // last list with chunk0[l] <= c: the one that holds c
    while (hi - lo > 1) { const int64_t mid = (lo + hi) >> 1; if (chunk0[mid] <= c) lo = mid; else hi = mid; }
    const int64_t m0 = list_off[lo] + (c - chunk0[lo]) * kMeanChunk;
    const int64_t m1 = min(list_off[lo + 1], m0 + kMeanChunk);
    for (int d = 4 * threadIdx.x; d < dp; d += 4 * blockDim.x) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
#pragma unroll 8
        for (int64_t v = m0; v < m1; ++v) {
            const float4 t = *(const float4*)(x + (int64_t)ids32[v] * dp + d);
            a0 += (double)t.x;
            a1 += (double)t.y;
            a2 += (double)t.z;
            a3 += (double)t.w;
        }
        double* o = psum + c * dp + d;
        o[0] = a0; o[1] = a1; o[2] = a2; o[3] = a3;
    }
}

// mean of list l from its chunks' partial sums in chunk order; an empty list keeps its centroid
__global__ __launch_bounds__(256) void list_mean_kernel(const double* __restrict__ psum, int dp,
                                                        const int64_t* __restrict__ list_off,
                                                        const int32_t* __restrict__ chunk0, float* __restrict__ cent)
{
    const int l = blockIdx.x;
    const int64_t cnt = list_off[l + 1] - list_off[l];
    if (cnt == 0) return;
    const int c0 = chunk0[l], c1 = chunk0[l + 1];
    for (int d = threadIdx.x; d < dp; d += 256) {
        double s = 0.0;
        for (int c = c0; c < c1; ++c) s += psum[(int64_t)c * dp + d];
        cent[(int64_t)l * dp + d] = (float)(s / (double)cnt);
    }
}

__global__ void gather_rows_kernel(const float* __restrict__ x, int dp, const int64_t* __restrict__ rows, int64_t m,
                                   float* __restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m * dp) return;
    const int64_t r = i / dp;
    out[i] = x[rows[r] * dp + (i - r * dp)];
}

}  // namespace

size_t bucket_scratch_bytes(int64_t n, int64_t nlist)
{
    return a256(sizeof(int32_t) * (size_t)sort_blocks(n, nlist) * (size_t)nlist);
}

hipError_t launch_bucket_count(const int32_t* assign, int64_t n, int64_t nlist, int32_t* cnt, int32_t* bad,
                               void* scratch, hipStream_t st)
{
    const int G = sort_blocks(n, nlist);
    const int64_t chunk = (n + G - 1) / G;
    int32_t* cnt2 = (int32_t*)scratch;
    hipError_t e = hipMemsetAsync(cnt2, 0, sizeof(int32_t) * (size_t)G * nlist, st);
    if (e != hipSuccess) return e;
    if (n > 0)
        hipLaunchKernelGGL(bucket_count_kernel, dim3(G), dim3(kSortThreads), 0, st, assign, n, nlist, chunk, cnt2, bad);
    hipLaunchKernelGGL(bucket_total_kernel, dim3((unsigned)((nlist + 31) / 32)), dim3(256), 0, st, cnt2, nlist, G, cnt);
    return hipGetLastError();
}

hipError_t launch_bucket_place(const int32_t* assign, int64_t n, int64_t nlist, const int64_t* list_off,
                               int32_t* ids32, void* scratch, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int G = sort_blocks(n, nlist);
    const int64_t chunk = (n + G - 1) / G;
    hipLaunchKernelGGL(bucket_place_kernel, dim3(G), dim3(kSortThreads), 0, st, assign, n, nlist, chunk, list_off,
                       (int32_t*)scratch, ids32);
    return hipGetLastError();
}

hipError_t launch_list_prefix(const int32_t* cnt, int64_t nlist, int64_t* list_off, int32_t* chunk0, hipStream_t st)
{
    hipLaunchKernelGGL(list_prefix_kernel, dim3(1), dim3(1024), 0, st, cnt, nlist, list_off, chunk0);
    return hipGetLastError();
}

// chunks of all lists: at most one per list beside the full ones
static int64_t mean_chunks(int64_t n, int64_t nlist) { return n / kMeanChunk + std::min(n, nlist); }

size_t list_mean_scratch_bytes(int64_t n, int64_t nlist, int dp)
{
    return a256(sizeof(double) * (size_t)std::max<int64_t>(mean_chunks(n, nlist), 1) * dp);
}

hipError_t launch_list_mean(const float* x, int64_t n, int dp, const int32_t* ids32, const int64_t* list_off,
                            int64_t nlist, const int32_t* chunk0, float* cent, void* scratch, hipStream_t st)
{
    double* psum = (double*)scratch;
    const int64_t nc = mean_chunks(n, nlist);
    const int th = std::min(256, (dp / 4 + 63) / 64 * 64);
    if (nc > 0)
        hipLaunchKernelGGL(list_psum_kernel, dim3((unsigned)nc), dim3(th), 0, st, x, dp, ids32, list_off, nlist, chunk0,
                           psum);
    hipLaunchKernelGGL(list_mean_kernel, dim3((unsigned)nlist), dim3(256), 0, st, psum, dp, list_off, chunk0, cent);
    return hipGetLastError();
}

hipError_t launch_gather_rows(const float* x, int dp, const int64_t* rows, int64_t m, float* out, hipStream_t st)
{
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((m * dp + 255) / 256)), dim3(256), 0, st, x, dp, rows, m, out);
    return hipGetLastError();
}

}  // namespace erq
