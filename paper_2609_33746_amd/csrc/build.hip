// Index build (Section 3.3; Appendix "Index build"): k-means over the keys of
// every (sequence, KV head) at once. The coarse problem clusters the
// directions u = k / ||k|| of R_b into n_list centers; each of the M subspace
// problems clusters the residual slices (u - c_a)^(m) into K codewords. One
// Lloyd iteration is:
//
//  * assign_kernel (coarse) or subspace_kernel: the nearest center of every
//    token, on the bf16 matrix cores; the near ties they leave go to
//    nearest_kernel or ties_kernel, on the 32-bit ones. The subspace kernels also
//    add the residuals to their codewords' sums.
//  * coarse: group_count / scan / place_kernel (group_kernel above 1024
//    lists), a stable counting sort of a KV head's tokens by list, so that
//    every mean adds its members in a fixed order, and centers_kernel, the
//    float64 mean of the members' directions (at the end of their values: the
//    list means). Subspaces: codewords_kernel, the sums over the counts.
//  * reseed_kernel: one workgroup per problem; a center without members
//    takes the point farthest from its assigned center (farthest first, ties
//    to the smaller token id; one point per empty center, in center order).
//
// init_centers_kernel: the starting centers, the direction or residual slice
// of caller-drawn tokens.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "pqhsa_internal.h"
#include "radix_select.h"

namespace pqhsa {

constexpr int kGroupThreads = 1024;
constexpr int kGroupScanPer = kMaxLists / kGroupThreads;

struct Problem {
    int bg, m, nkeys, dims;
};

__device__ __forceinline__ Problem problem_of(const Dims& D, int kind, int p) {
    const int M = D.pq_bits == 4 ? Pq4::M : Pq8::M;
    const int K = D.pq_bits == 4 ? Pq4::K : Pq8::K;
    if (kind == 1) return Problem{p / M, p % M, K, kHeadDim / M};
    return Problem{p, 0, D.n_list, kHeadDim};
}

// the vector of token t for a problem: its direction (kind 0) or the residual
// slice of subspace m (kind 1), element x
template <typename T>
__device__ __forceinline__ float token_elem(const Dims& D, int kind, const KV& kv, int bg, int m,
                                            int dims, int t, int x, const int32_t* ids_tm,
                                            const float* norms_tm, const float* centroids) {
    const int b = bg / D.Hkv, g = bg % D.Hkv;
    const int64_t row = b * kv.sb + g * kv.sh + static_cast<int64_t>(t) * kv.sn;
    const int col = m * dims + x;
    const float r = norms_tm[static_cast<int64_t>(bg) * D.rcap + t];
    const float u = r > 0.0f ? load1<T>(static_cast<const T*>(kv.k) + row + col) / r : 0.0f;
    if (kind == 0) return u;
    const int a = ids_tm[static_cast<int64_t>(bg) * D.rcap + t];
    return u - centroids[(static_cast<int64_t>(bg) * D.n_list + a) * kHeadDim + col];
}

__device__ __forceinline__ int64_t center_index(const Dims& D, int kind, const Problem& pr, int c,
                                                int x) {
    if (kind == 1) {
        const int M = kHeadDim / pr.dims;
        return ((static_cast<int64_t>(pr.bg) * M + pr.m) * pr.nkeys + c) * pr.dims + x;
    }
    return (static_cast<int64_t>(pr.bg) * D.n_list + c) * kHeadDim + x;
}

__global__ __launch_bounds__(kGroupThreads) void group_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                              const int32_t* ids_tm,
                                                              int32_t* order, int32_t* offs) {
    __shared__ int cnt[kMaxLists];
    __shared__ int placed[kMaxLists];
    __shared__ int chunk[kGroupThreads];
    __shared__ int wtot[kGroupThreads / kWave];
    const int p = blockIdx.x;   // (b, kv head)
    const int nk = D.n_list;
    const int b = p / D.Hkv;
    const int t0 = lo.v[b], t1 = hi.v[b];
    const int tid = threadIdx.x;
    const int64_t row = static_cast<int64_t>(p) * D.rcap;
    auto key = [&](int t) { return ids_tm[row + t]; };
    for (int j = tid; j < nk; j += kGroupThreads) {
        cnt[j] = 0;
        placed[j] = 0;
    }
    __syncthreads();
    for (int t = t0 + tid; t < t1; t += kGroupThreads) atomicAdd(&cnt[key(t)], 1);
    __syncthreads();
    lds_exclusive_scan<kGroupThreads, kGroupScanPer>(cnt, nk, wtot);
    int32_t* of = offs + static_cast<int64_t>(p) * (nk + 1);
    for (int j = tid; j <= nk; j += kGroupThreads) of[j] = j < nk ? cnt[j] : t1 - t0;
    int32_t* ord = order + static_cast<int64_t>(p) * D.rcap;
    for (int c0 = t0; c0 < t1; c0 += kGroupThreads) {
        const int t = c0 + tid;
        const int j = t < t1 ? key(t) : -1;
        chunk[tid] = j;
        __syncthreads();
        if (t < t1) {
            int r = 0;
            for (int i = 0; i < tid; ++i) r += chunk[i] == j;
            ord[cnt[j] + placed[j] + r] = t;
        }
        __syncthreads();
        if (t < t1) atomicAdd(&placed[j], 1);
        __syncthreads();
    }
}

// The same stable grouping for problems of at most kGroupFastKeys centers,
// spread over many workgroups and without the O(chunk^2) rank. A problem's
// tokens are cut into segments of kSegTok; three launches:
//  * group_count_kernel, one workgroup per (segment, problem): the
//    segment's key counts (LDS atomics) to seg_hist[problem][segment][key];
//  * group_scan_kernel, one workgroup per problem: the centers' offsets
//    (key-major, then segment order: a stable layout), and each segment's
//    first position per key in place of its counts;
//  * group_place_kernel, one workgroup per (segment, problem): wave w owns
//    the w-th sixteenth of the segment; the per-wave counts turn into each
//    wave's first position per key, and each wave places its tokens 64 at a
//    time, the rank among equal keys of a step coming from one ballot per bit
//    of the keys and its base from one LDS atomic of the key's first lane.
constexpr int kGroupWaves = kGroupThreads / kWave;
constexpr int kGroupFastKeys = 1024;
constexpr int kSegTok = kBuildSegTok;   // tokens per segment

__device__ __forceinline__ int group_key(const Dims& D, int64_t row, int t, const int32_t* ids_tm) {
    return min(max(ids_tm[row + t], 0), D.n_list - 1);
}

__global__ __launch_bounds__(kGroupThreads) void group_count_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                                    const int32_t* ids_tm,
                                                                    int32_t* seg_hist, int nseg) {
    __shared__ int hist[kGroupFastKeys];
    const int seg = blockIdx.x, p = blockIdx.y;
    const int nk = D.n_list;
    const int b = p / D.Hkv;
    const int s0 = lo.v[b] + seg * kSegTok, s1 = min(s0 + kSegTok, hi.v[b]);
    const int64_t row = static_cast<int64_t>(p) * D.rcap;
    for (int j = threadIdx.x; j < nk; j += kGroupThreads) hist[j] = 0;
    __syncthreads();
    for (int t = s0 + static_cast<int>(threadIdx.x); t < s1; t += kGroupThreads)
        atomicAdd(&hist[group_key(D, row, t, ids_tm)], 1);
    __syncthreads();
    int32_t* out = seg_hist + (static_cast<int64_t>(p) * nseg + seg) * nk;
    for (int j = threadIdx.x; j < nk; j += kGroupThreads) out[j] = hist[j];
}

__global__ __launch_bounds__(kGroupThreads) void group_scan_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                                   int32_t* seg_hist, int nseg,
                                                                   int32_t* offs) {
    __shared__ int tot[kGroupFastKeys];
    __shared__ int wtot[kGroupWaves];
    const int p = blockIdx.x;
    const int nk = D.n_list;
    const int b = p / D.Hkv;
    int32_t* h = seg_hist + static_cast<int64_t>(p) * nseg * nk;
    constexpr int kAtOnce = 8;   // segments' counts loaded at once (each is a round trip of its own otherwise)
    for (int j = threadIdx.x; j < nk; j += kGroupThreads) {
        int sum = 0;
        for (int s0 = 0; s0 < nseg; s0 += kAtOnce) {
            int c[kAtOnce];
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u)
                c[u] = s0 + u < nseg ? h[static_cast<int64_t>(s0 + u) * nk + j] : 0;
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u) sum += c[u];
        }
        tot[j] = sum;
    }
    __syncthreads();
    lds_exclusive_scan<kGroupThreads, 1>(tot, nk, wtot);
    int32_t* of = offs + static_cast<int64_t>(p) * (nk + 1);
    for (int j = threadIdx.x; j <= nk; j += kGroupThreads) of[j] = j < nk ? tot[j] : hi.v[b] - lo.v[b];
    for (int j = threadIdx.x; j < nk; j += kGroupThreads) {
        int at = tot[j];
        for (int s0 = 0; s0 < nseg; s0 += kAtOnce) {
            int c[kAtOnce];
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u)
                c[u] = s0 + u < nseg ? h[static_cast<int64_t>(s0 + u) * nk + j] : 0;
#pragma unroll
            for (int u = 0; u < kAtOnce; ++u) {
                if (s0 + u < nseg) h[static_cast<int64_t>(s0 + u) * nk + j] = at;
                at += c[u];
            }
        }
    }
}

__global__ __launch_bounds__(kGroupThreads) void group_place_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                                    const int32_t* ids_tm,
                                                                    const int32_t* seg_hist, int nseg,
                                                                    int32_t* order) {
    __shared__ int hist[kGroupWaves][kGroupFastKeys];
    const int seg = blockIdx.x, p = blockIdx.y;
    const int nk = D.n_list;
    const int b = p / D.Hkv;
    const int s0 = lo.v[b] + seg * kSegTok, s1 = min(s0 + kSegTok, hi.v[b]);
    if (s0 >= s1) return;
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    const int64_t row = static_cast<int64_t>(p) * D.rcap;
    // the wave's part of the segment
    const int n = s1 - s0;
    const int per = (n + kGroupWaves - 1) / kGroupWaves;
    const int w0 = s0 + min(wave * per, n), w1 = s0 + min(wave * per + per, n);
    for (int i = tid; i < kGroupWaves * kGroupFastKeys; i += kGroupThreads) (&hist[0][0])[i] = 0;
    __syncthreads();
    for (int t = w0 + lane; t < w1; t += kWave) atomicAdd(&hist[wave][group_key(D, row, t, ids_tm)], 1);
    __syncthreads();
    const int32_t* base_g = seg_hist + (static_cast<int64_t>(p) * nseg + seg) * nk;
    for (int j = tid; j < nk; j += kGroupThreads) {
        int at = base_g[j];
#pragma unroll
        for (int w = 0; w < kGroupWaves; ++w) {
            const int c = hist[w][j];
            hist[w][j] = at;
            at += c;
        }
    }
    __syncthreads();
    const int key_bits = nk > 1 ? 32 - __clz(nk - 1) : 0;
    int32_t* ord = order + static_cast<int64_t>(p) * D.rcap;
    for (int c0 = w0; c0 < w1; c0 += kWave) {
        const int t = c0 + lane;
        const bool valid = t < w1;
        const int k = valid ? group_key(D, row, t, ids_tm) : 0;
        // the lanes of an equal key from one ballot per bit of the keys (a step's
        // 64 keys are mostly distinct: a ballot per distinct key took 38 us in
        // place of 14 at 128K tokens x 8 KV heads x 1024 lists), then one
        // LDS atomic per distinct key, made by the key's first lane
        uint64_t same = __ballot(valid);
        for (int bit = 0; bit < key_bits; ++bit) {
            const bool one = (k >> bit) & 1;
            const uint64_t ones = __ballot(one);
            same &= one ? ones : ~ones;
        }
        const int leader_of = valid ? __ffsll(static_cast<long long>(same)) - 1 : lane;
        const int rank = lanes_below(same);
        const int cnt = __popcll(same);
        int base = 0;
        if (valid && lane == leader_of) base = atomicAdd(&hist[wave][k], cnt);
        base = __shfl(base, leader_of);
        if (valid) ord[base + rank] = t;
    }
}

// centers_kernel: the float64 mean of a center's members' directions (kind 0)
// or values (kind 2), 16 lanes of 8 dimensions per member row: stream si adds
// members si, si + 16, ... in order, kCenRows of them loaded at once, then the
// streams' sums are added in stream order (a fixed order: the build is
// deterministic). Bound by the gather of the rows: 128K tokens x 8 KV heads,
// 0.07 ms for the directions and 0.09 for the values (one thread per dimension
// and member: 0.45 and 0.30 ms).
constexpr int kCenThreads = 256;
constexpr int kCenStreams = kCenThreads / 16;
constexpr int kCenRows = 4;

template <typename T>
__global__ __launch_bounds__(kCenThreads) void centers_kernel(Dims D, int kind, KV kv,
                                                              const float* __restrict__ norms_tm,
                                                              const int32_t* __restrict__ order,
                                                              const int32_t* __restrict__ offs, float* __restrict__ out) {
    __shared__ double part[kCenStreams][kHeadDim];
    const int c = blockIdx.x;
    const int bg = blockIdx.y;
    const int b = bg / D.Hkv, g = bg % D.Hkv;
    const int si = threadIdx.x / 16;
    const int x0 = threadIdx.x % 16 * 8;
    const int32_t* of = offs + static_cast<int64_t>(bg) * (D.n_list + 1);
    const int o0 = of[c], o1 = of[c + 1];
    float* dst = out + (static_cast<int64_t>(bg) * D.n_list + c) * kHeadDim;
    if (o1 == o0) {   // empty: the list mean is 0; a center is re-seeded afterwards
        if (kind == 2 && si == 0)
#pragma unroll
            for (int e = 0; e < 8; ++e) dst[x0 + e] = 0.0f;
        return;
    }
    const T* src = static_cast<const T*>(kind == 2 ? kv.v : kv.k) + b * kv.sb + g * kv.sh + x0;
    const int64_t row = static_cast<int64_t>(bg) * D.rcap;
    double acc[8] = {};
    for (int i0 = o0 + si; i0 < o1; i0 += kCenStreams * kCenRows) {
        Raw8<T> raw[kCenRows];
        float r[kCenRows];
#pragma unroll
        for (int u = 0; u < kCenRows; ++u) {
            const int t = order[row + min(i0 + u * kCenStreams, o1 - 1)];   // past the end: the last again, unused
            raw[u].load(src + static_cast<int64_t>(t) * kv.sn);
            r[u] = kind == 2 ? 1.0f : norms_tm[row + t];
        }
#pragma unroll
        for (int u = 0; u < kCenRows; ++u) {
            if (i0 + u * kCenStreams >= o1) break;
            float x[8];
            raw[u].to(x);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                acc[e] += static_cast<double>(kind == 2 ? x[e] : r[u] > 0.0f ? x[e] / r[u] : 0.0f);
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[si][x0 + e] = acc[e];
    __syncthreads();
    if (threadIdx.x < kHeadDim) {
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < kCenStreams; ++w) sum += part[w][threadIdx.x];
        dst[threadIdx.x] = static_cast<float>(sum / (o1 - o0));
    }
}

template <typename T>
__global__ __launch_bounds__(kGroupThreads) void reseed_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                               int kind, KV kv,
                                                               const int32_t* ids_tm,
                                                               const float* norms_tm,
                                                               const float* centroids,
                                                               const int32_t* offs,
                                                               const uint32_t* counts,
                                                               const float* dist_c,
                                                               const float* dist_f, float* out) {
    __shared__ int empty[kMaxLists];   // the centers without members, in order
    __shared__ int wtot[kGroupThreads / kWave];
    __shared__ float wd[kGroupThreads / kWave];
    __shared__ int wt[kGroupThreads / kWave];
    __shared__ int pick;
    const int p = blockIdx.x;
    const Problem pr = problem_of(D, kind, p);
    const int b = pr.bg / D.Hkv;
    const int t0 = lo.v[b], t1 = hi.v[b];
    const int tid = threadIdx.x;
    const int32_t* of = offs + static_cast<int64_t>(p) * (pr.nkeys + 1);
    int n_empty = 0;
    for (int j0 = 0; j0 < pr.nkeys; j0 += kGroupThreads) {
        const int j = j0 + tid;
        const bool is = j < pr.nkeys &&
                        (kind == 1 ? counts[static_cast<int64_t>(p) * pr.nkeys + j] == 0u : of[j + 1] == of[j]);
        const uint64_t mask = __ballot(is);
        if (lane_id() == 0) wtot[tid / kWave] = __popcll(mask);
        __syncthreads();
        int at = n_empty;
        for (int w = 0; w < kGroupThreads / kWave; ++w) {
            if (w < tid / kWave) at += wtot[w];
            n_empty += wtot[w];
        }
        if (is) empty[at + lanes_below(mask)] = j;
        __syncthreads();
    }
    if (n_empty == 0) return;
    // distances of the problem's tokens: [B Hkv (M)][rcap]
    const float* dist_p = (kind == 1 ? dist_f : dist_c) + static_cast<int64_t>(p) * D.rcap;
    auto dist = [&](int t) { return dist_p[t]; };
    float pd = __builtin_huge_valf();   // the previous pick: points must order after it
    int pt = -1;
    for (int i = 0; i < n_empty; ++i) {
        const int c = empty[i];
        // the farthest point after (pd, pt) in the order (distance desc, token asc)
        float bd = -1.0f;
        int bt = -1;
        for (int t = t0 + tid; t < t1; t += kGroupThreads) {
            const float d = dist(t);
            const bool after = d < pd || (d == pd && t > pt);
            if (after && (d > bd || (d == bd && (bt < 0 || t < bt)))) {
                bd = d;
                bt = t;
            }
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const float od = __shfl_xor(bd, off);
            const int ot = __shfl_xor(bt, off);
            if (ot >= 0 && (bt < 0 || od > bd || (od == bd && ot < bt))) {
                bd = od;
                bt = ot;
            }
        }
        if (lane_id() == 0) {
            wd[tid / kWave] = bd;
            wt[tid / kWave] = bt;
        }
        __syncthreads();
        if (tid == 0) {
            float d = -1.0f;
            int t = -1;
            for (int w = 0; w < kGroupThreads / kWave; ++w)
                if (wt[w] >= 0 && (t < 0 || wd[w] > d || (wd[w] == d && wt[w] < t))) {
                    d = wd[w];
                    t = wt[w];
                }
            pick = t;
            wd[0] = d;
        }
        __syncthreads();
        const int t = pick;
        const float d = wd[0];
        __syncthreads();
        if (t < 0) break;   // no point left
        if (tid < pr.dims)
            out[center_index(D, kind, pr, c, tid)] =
                token_elem<T>(D, kind, kv, pr.bg, pr.m, pr.dims, t, tid, ids_tm, norms_tm, centroids);
        pd = d;
        pt = t;
    }
}

// ||k|| of the token row at p, over 16 lanes of 8 dimensions each: the same
// sum, in the same order, wherever the build takes a norm. x receives the
// lane's slice of the row.
template <typename T>
__device__ __forceinline__ float row_norm(const T* p, float (&x)[8]) {
    Load8<T>::run(p, x);
    float ss = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) ss += __shfl_xor(ss, off);
    return sqrtf(ss);
}

// The starting coarse centers are taken before any assignment pass has
// written the norms, so kind 0 takes the norm of its token itself.
template <typename T>
__global__ __launch_bounds__(kHeadDim) void init_centers_kernel(Dims D, int kind, KV kv,
                                                                const int32_t* init,
                                                                const int32_t* ids_tm,
                                                                const float* norms_tm,
                                                                const float* centroids,
                                                                float* out) {
    const int c = blockIdx.x;
    const int p = blockIdx.y;
    const Problem pr = problem_of(D, kind, p);
    const int x = threadIdx.x;
    if (c >= pr.nkeys) return;
    const int t = init[static_cast<int64_t>(p) * pr.nkeys + c];
    if (kind == 0) {
        if (x >= 16) return;
        const T* row = static_cast<const T*>(kv.k) + (pr.bg / D.Hkv) * kv.sb + (pr.bg % D.Hkv) * kv.sh +
                       static_cast<int64_t>(t) * kv.sn;
        float k[8];
        const float r = row_norm<T>(row + x * 8, k);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            out[center_index(D, kind, pr, c, x * 8 + e)] = r > 0.0f ? k[e] / r : 0.0f;
        return;
    }
    if (x >= pr.dims) return;
    out[center_index(D, kind, pr, c, x)] =
        token_elem<T>(D, kind, kv, pr.bg, pr.m, pr.dims, t, x, ids_tm, norms_tm, centroids);
}

__global__ __launch_bounds__(256) void check_starts_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                           const int32_t* __restrict__ coarse,
                                                           const int32_t* __restrict__ pq, int per_pq,
                                                           unsigned long long* bad) {
    const int64_t n_coarse = static_cast<int64_t>(D.B) * D.Hkv * D.n_list;
    const int64_t n = n_coarse + static_cast<int64_t>(D.B) * D.Hkv * per_pq;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t bg = i < n_coarse ? i / D.n_list : (i - n_coarse) / per_pq;
    const int t = i < n_coarse ? coarse[i] : pq[i - n_coarse];
    const int b = static_cast<int>(bg / D.Hkv);
    if (t < lo.v[b] || t >= hi.v[b]) atomicMin(bad, static_cast<unsigned long long>(i));
}

hipError_t launch_check_starts(const Dims& D, const BatchInts& lo, const BatchInts& hi, const int32_t* coarse,
                               const int32_t* pq, int per_pq, unsigned long long* bad, hipStream_t s) {
    const int64_t n = static_cast<int64_t>(D.B) * D.Hkv * (D.n_list + per_pq);
    hipLaunchKernelGGL(check_starts_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s, D, lo,
                       hi, coarse, pq, per_pq, bad);
    return hipGetLastError();
}

static int n_problems(const Dims& D, int kind) {
    return D.B * D.Hkv * (kind == 1 ? (D.pq_bits == 4 ? Pq4::M : Pq8::M) : 1);
}
static int n_keys(const Dims& D, int kind) {
    return kind == 1 ? (D.pq_bits == 4 ? Pq4::K : Pq8::K) : D.n_list;
}

hipError_t launch_group_segments(const Dims& D, const BatchInts& lo, const BatchInts& hi,
                                 const int32_t* ids_tm, int32_t* seg_hist, int32_t* order, int32_t* offs,
                                 hipStream_t s) {
    int max_n = 0;
    for (int b = 0; b < D.B; ++b) max_n = hi.v[b] - lo.v[b] > max_n ? hi.v[b] - lo.v[b] : max_n;
    const int nseg = (max_n + kSegTok - 1) / kSegTok;
    const dim3 grid(nseg, D.B * D.Hkv);
    if (nseg > 0) {
        hipLaunchKernelGGL(group_count_kernel, grid, dim3(kGroupThreads), 0, s, D, lo, hi, ids_tm,
                           seg_hist, nseg);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // also with no tokens: the offsets are written
    hipLaunchKernelGGL(group_scan_kernel, dim3(D.B * D.Hkv), dim3(kGroupThreads), 0, s, D, lo,
                       hi, seg_hist, nseg, offs);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nseg == 0) return e;
    hipLaunchKernelGGL(group_place_kernel, grid, dim3(kGroupThreads), 0, s, D, lo, hi, ids_tm,
                       seg_hist, nseg, order);
    return hipGetLastError();
}

hipError_t launch_group(const Dims& D, const BatchInts& lo, const BatchInts& hi, const int32_t* ids_tm,
                        const BuildBufs& bb, hipStream_t s) {
    if (D.n_list <= kGroupFastKeys && bb.seg_hist)
        return launch_group_segments(D, lo, hi, ids_tm, bb.seg_hist, bb.order, bb.offs, s);
    hipLaunchKernelGGL(group_kernel, dim3(D.B * D.Hkv), dim3(kGroupThreads), 0, s, D, lo, hi, ids_tm,
                       bb.order, bb.offs);
    return hipGetLastError();
}

hipError_t launch_centers(const Dims& D, int kind, const KV& kv, const float* norms_tm, const BuildBufs& bb,
                          float* out, hipStream_t s) {
    const dim3 grid(D.n_list, D.B * D.Hkv);
    if (kv.bf16)
        hipLaunchKernelGGL(centers_kernel<bf16_t>, grid, dim3(kCenThreads), 0, s, D, kind, kv, norms_tm,
                           bb.order, bb.offs, out);
    else
        hipLaunchKernelGGL(centers_kernel<float>, grid, dim3(kCenThreads), 0, s, D, kind, kv, norms_tm,
                           bb.order, bb.offs, out);
    return hipGetLastError();
}

hipError_t launch_reseed(const Dims& D, const BatchInts& lo, const BatchInts& hi, int kind,
                         const KV& kv, const int32_t* ids_tm, const float* norms_tm,
                         const float* centroids, const BuildBufs& bb, float* out, hipStream_t s) {
    const dim3 grid(n_problems(D, kind));
    if (kv.bf16)
        hipLaunchKernelGGL(reseed_kernel<bf16_t>, grid, dim3(kGroupThreads), 0, s, D, lo, hi, kind,
                           kv, ids_tm, norms_tm, centroids, bb.offs, bb.sums.counts, bb.dist_c, bb.dist_f, out);
    else
        hipLaunchKernelGGL(reseed_kernel<float>, grid, dim3(kGroupThreads), 0, s, D, lo, hi, kind,
                           kv, ids_tm, norms_tm, centroids, bb.offs, bb.sums.counts, bb.dist_c, bb.dist_f, out);
    return hipGetLastError();
}

hipError_t launch_init_centers(const Dims& D, int kind, const KV& kv, const int32_t* init,
                               const int32_t* ids_tm, const float* norms_tm, const float* centroids,
                               float* out, hipStream_t s) {
    const dim3 grid(n_keys(D, kind), n_problems(D, kind));
    if (kv.bf16)
        hipLaunchKernelGGL(init_centers_kernel<bf16_t>, grid, dim3(kHeadDim), 0, s, D, kind, kv,
                           init, ids_tm, norms_tm, centroids, out);
    else
        hipLaunchKernelGGL(init_centers_kernel<float>, grid, dim3(kHeadDim), 0, s, D, kind, kv, init,
                           ids_tm, norms_tm, centroids, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The searches of the build run on the bf16 matrix cores at the precision of
// 32-bit sums. A 32-bit x is the sum of three bf16 parts x1 + x2 + x3 (each
// part the rounding of what the earlier ones leave, 8 bits apiece), products
// of bf16 parts are exact in the matrix cores' 32-bit sums, and parts are
// added smallest first. Against float64 over random unit vectors of 128
// dimensions the dot products of a bf16 key with a split center are off by
// 6.2e-9 (rms; 7.0e-8 at most), those of v_mfma_f32_16x16x4f32 on the 32-bit
// direction by 1.8e-8 (1.7e-7).
// ---------------------------------------------------------------------------
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f16_t __attribute__((ext_vector_type(16)));

// N (2 or 4) consecutive elements of a row, from an address aligned to them.
template <typename T, int N>
__device__ __forceinline__ void load_slice(const T* p, float (&x)[N]) {
    static_assert(N == 2 || N == 4, "one load");
    if constexpr (std::is_same<T, float>::value && N == 4) {
        const float4 v = *reinterpret_cast<const float4*>(p);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else if constexpr (std::is_same<T, float>::value) {
        const float2 v = *reinterpret_cast<const float2*>(p);
        x[0] = v.x; x[1] = v.y;
    } else if constexpr (N == 4) {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        x[0] = bf16_lo(v.x); x[1] = bf16_hi(v.x); x[2] = bf16_lo(v.y); x[3] = bf16_hi(v.y);
    } else {
        const uint32_t v = *reinterpret_cast<const uint32_t*>(p);
        x[0] = bf16_lo(v); x[1] = bf16_hi(v);
    }
}

// The bf16 parts of x, largest first.
__device__ __forceinline__ void split_bf16(float x, __bf16 (&p)[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        p[i] = static_cast<__bf16>(x);
        x -= static_cast<float>(p[i]);
    }
}

// ---------------------------------------------------------------------------
// split_centers_kernel: the centers of each (b, kv head) as the A operands of
// assign_kernel, tiles of kTileCen centers in operand order: kSplitBlocks
// blocks of 64 lanes x 8 bf16, lane l of a block holding 8 consecutive
// dimensions (from 8 (l / 32)) of 16 of center l mod 32. Blocks 0-7 hold the
// third parts of dimensions 0-15, 16-31, ..., blocks 8-15 the second parts,
// 16-23 the first, and block 24 the parts of ||c||^2 / 2 in the slots that
// meet a token's norm parts (norm_slots below). Centers past the last stand
// farther than any real one.
// ---------------------------------------------------------------------------
constexpr int kTileCen = 32;
constexpr int kDimBlocks = kHeadDim / 16;             // 16-dimension blocks of a row: 8
constexpr int kSplitBlocks = 3 * kDimBlocks + 1;
constexpr int kTileBf16 = kSplitBlocks * kWave * 8;   // bf16 per tile: 25 KB
constexpr float kFarCenter = 1e15f;

static size_t split_center_count(const Dims& D) {
    const size_t tiles = (static_cast<size_t>(D.n_list) + kTileCen - 1) / kTileCen;
    return static_cast<size_t>(D.B) * D.Hkv * tiles * kTileBf16;
}
size_t split_center_bytes(const Dims& D) { return split_center_count(D) * sizeof(__bf16); }

// one workgroup per (tile, b g): 8 threads per center, 16 dimensions each
__global__ __launch_bounds__(kTileCen * 8) void split_centers_kernel(Dims D, const float* __restrict__ centroids,
                                                                     __bf16* __restrict__ split) {
    const int tile = blockIdx.x, n_tile = gridDim.x, bg = blockIdx.y;
    const int row = threadIdx.x / 8, kb = threadIdx.x % 8;
    const int c = tile * kTileCen + row;
    const bool real = c < D.n_list;
    const float* src = centroids + (static_cast<int64_t>(bg) * D.n_list + (real ? c : 0)) * kHeadDim + kb * 16;
    __bf16* out = split + (static_cast<int64_t>(bg) * n_tile + tile) * kTileBf16;
    double c2 = 0.0;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        float x[8];
        Load8<float>::run(src + half * 8, x);
        bf8_t v[3];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (!real) x[e] = 0.0f;
            c2 += static_cast<double>(x[e]) * x[e];
            __bf16 p[3];
            split_bf16(x[e], p);
#pragma unroll
            for (int i = 0; i < 3; ++i) v[i][e] = p[i];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
            *reinterpret_cast<bf8_t*>(out + (((2 - i) * kDimBlocks + kb) * kWave + half * 32 + row) * 8) = v[i];
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) c2 += __shfl_xor(c2, off);
    if (kb < 2) {
        __bf16 p[3];
        split_bf16(real ? static_cast<float>(0.5 * c2) : kFarCenter, p);
        bf8_t v = {};
        if (kb == 0) {   // against norm_slots: -(r3, r1, r2, r1, r2, r1, 0, 0)
            v[0] = p[0]; v[1] = p[2]; v[2] = p[1]; v[3] = p[1]; v[4] = p[0]; v[5] = p[0];
        }
        *reinterpret_cast<bf8_t*>(out + (3 * kDimBlocks * kWave + kb * 32 + row) * 8) = v;
    }
}

// The B operand that meets the ||c||^2 / 2 parts: minus the parts of r, paired
// so that the block adds -r ||c||^2 / 2 to 24 bits (lanes of the second 8 hold
// zeros).
__device__ __forceinline__ bf8_t norm_slots(float r, int half) {
    bf8_t v = {};
    if (half == 0) {
        __bf16 p[3];
        split_bf16(-r, p);
        v[0] = p[2]; v[1] = p[0]; v[2] = p[1]; v[3] = p[0]; v[4] = p[1]; v[5] = p[0];
    }
    return v;
}

// ---------------------------------------------------------------------------
// assign_kernel: the nearest center of every direction u = k / r, r = ||k||.
// Its distance is ||u||^2 - 2 (u . c - ||c||^2 / 2), so per token the largest
// r (u . c - ||c||^2 / 2) = k . c - r ||c||^2 / 2 decides: one product of the
// key, which in a bf16 cache is its own only part, with the center's parts,
// and a last 16-wide block that subtracts the center's half norm. So the
// accumulator is compared as it is: 3 VALU instructions per (token, center),
// which the next products hide. A 32-bit cache takes u itself, in three parts
// (6 products of parts; those left out are below 2^-24 of the terms).
//
// A workgroup of 4 waves holds 64 tokens (32 with a 32-bit cache) a wave as B
// operands in registers and streams the split centers through LDS, a tile of
// 32 (25 KB) at a time, the next tile's loads under the current one's
// products. v_mfma_f32_32x32x16_bf16: element i of lane l is center
// 8 (i / 4) + 4 (l / 32) + i mod 4 against token l mod 32. 128K tokens x 8 KV
// heads against 1024 lists: 0.71-0.76 ms (1.1-1.2 PFLOP/s of bf16 products, about what
// a large library product reaches here) in place of 3.19 ms with
// v_mfma_f32_16x16x4f32 and a distance and a two-key compare per pair.
// ---------------------------------------------------------------------------
// Squared distances closer than this are decided by nearest_kernel: two of the
// 32-bit matrix cores' are off by up to 9e-7 in their difference, two of
// assign_kernel's by 3e-7 (four times the largest error of a dot product, above,
// and a rounding).
constexpr float kNearGap = 4e-6f;
constexpr int kAsgThreads = 256;
constexpr int kAsgWaves = kAsgThreads / kWave;

template <typename T>
struct AsgTokens;
template <>
struct AsgTokens<bf16_t> {
    static constexpr int kTiles = 2, kParts = 1;   // token tiles of 32 per wave, bf16 parts per element
};
template <>
struct AsgTokens<float> {
    static constexpr int kTiles = 1, kParts = 3;
};

__device__ __forceinline__ void asg_fold(float& d, int& i, float od, int oi) {
    if (od > d || (od == d && oi < i)) {
        d = od;
        i = oi;
    }
}

// The operands of a token's row: lane half h holds dimensions 16 kb + 8 h ..
// + 7 of every block kb. Returns ||k|| (the sum in row_norm's order), in
// `scale` what the row stands multiplied by (r for the raw key, 1 for the
// direction), and in `unit2` ||u||^2. A zero row, or one whose norm
// overflows, is the zero direction; a row with a NaN or an infinity has the
// scale 0, so that all centers tie and nearest_kernel decides it.
template <typename T>
__device__ __forceinline__ float load_token(const T* p, bool present, int half,
                                            bf8_t (&v)[AsgTokens<T>::kParts][kDimBlocks], float& scale,
                                            float& unit2) {
    float ps[kDimBlocks];
    float x[std::is_same<T, float>::value ? kDimBlocks : 1][8];
    bool bad = false;
#pragma unroll
    for (int kb = 0; kb < kDimBlocks; ++kb) {
        float e8[8] = {};
        if constexpr (std::is_same<T, float>::value) {
            if (present) Load8<float>::run(p + kb * 16 + half * 8, x[kb]);
            else
#pragma unroll
                for (int e = 0; e < 8; ++e) x[kb][e] = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) e8[e] = x[kb][e];
        } else {
            uint4 w = make_uint4(0u, 0u, 0u, 0u);
            if (present) w = *reinterpret_cast<const uint4*>(p + kb * 16 + half * 8);
            v[0][kb] = __builtin_bit_cast(bf8_t, w);
#pragma unroll
            for (int e = 0; e < 8; ++e) e8[e] = static_cast<float>(v[0][kb][e]);
        }
        float ss = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            ss = fmaf(e8[e], e8[e], ss);
            bad = bad || !(fabsf(e8[e]) < __builtin_huge_valf());
        }
        ps[kb] = ss + __shfl_xor(ss, 32);
    }
    const float ss = ((ps[0] + ps[1]) + (ps[2] + ps[3])) + ((ps[4] + ps[5]) + (ps[6] + ps[7]));
    const float r = sqrtf(ss);
    bad = __shfl_xor(static_cast<int>(bad), 32) || bad;
    const bool live = !bad && r > 0.0f && r < __builtin_huge_valf();
    scale = bad ? 0.0f : live && !std::is_same<T, float>::value ? r : 1.0f;
    unit2 = live ? ss / (r * r) : 0.0f;
    if constexpr (std::is_same<T, float>::value) {
#pragma unroll
        for (int kb = 0; kb < kDimBlocks; ++kb)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                __bf16 q[3];
                split_bf16(live ? x[kb][e] / r : 0.0f, q);
#pragma unroll
                for (int i = 0; i < 3; ++i) v[i][kb][e] = q[i];
            }
    } else if (!live) {
#pragma unroll
        for (int kb = 0; kb < kDimBlocks; ++kb) v[0][kb] = bf8_t{};
    }
    return r;
}

template <typename T>
__global__ __launch_bounds__(kAsgThreads) void assign_kernel(Dims D, BatchInts lo, BatchInts hi, KV kv,
                                                             const __bf16* __restrict__ split, int n_tile,
                                                             int32_t* __restrict__ ids_tm,
                                                             float* __restrict__ norms_tm,
                                                             float* __restrict__ dist_c,
                                                             int32_t* __restrict__ near,
                                                             uint32_t* __restrict__ n_near) {
    constexpr int NT = AsgTokens<T>::kTiles, P = AsgTokens<T>::kParts;
    constexpr int kWgTok = kAsgWaves * NT * 32;
    __shared__ bf8_t cen[2][kSplitBlocks * kWave];
    const int b = blockIdx.z;
    const int g = blockIdx.y;
    const int t_base = lo.v[b] + static_cast<int>(blockIdx.x) * kWgTok;
    if (t_base >= hi.v[b]) return;
    const int nt = min(kWgTok, hi.v[b] - t_base);
    const int bg = b * D.Hkv + g;
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int col = lane % 32;
    const int half = lane / 32;

    // the tiles' staging: block wave, wave + 4, ... of a tile by each wave
    constexpr int kStage = (kSplitBlocks + kAsgWaves - 1) / kAsgWaves;
    const bf8_t* src = reinterpret_cast<const bf8_t*>(split) + static_cast<int64_t>(bg) * n_tile * kSplitBlocks * kWave;
    bf8_t st[kStage];
    auto fetch = [&](int tile) {
#pragma unroll
        for (int i = 0; i < kStage; ++i) {
            const int blk = min(i * kAsgWaves + wave, kSplitBlocks - 1);
            st[i] = src[(static_cast<int64_t>(tile) * kSplitBlocks + blk) * kWave + lane];
        }
    };
    auto put = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kStage; ++i)
            if (i * kAsgWaves + wave < kSplitBlocks) cen[buf][(i * kAsgWaves + wave) * kWave + lane] = st[i];
    };
    fetch(0);

    bf8_t tok[NT][P][kDimBlocks], nrm[NT];
    float unit2[NT], scale[NT];
    const T* kb = static_cast<const T*>(kv.k) + b * kv.sb + g * kv.sh;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
        const int tk = (wave * NT + tt) * 32 + col;
        const float r = load_token<T>(kb + static_cast<int64_t>(t_base + tk) * kv.sn, tk < nt, half, tok[tt],
                                      scale[tt], unit2[tt]);
        nrm[tt] = norm_slots(scale[tt], half);
        if (half == 0 && tk < nt) norms_tm[static_cast<int64_t>(bg) * D.rcap + t_base + tk] = r;
    }
    float best[NT], second[NT];
    int best_i[NT];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
        best[tt] = second[tt] = -__builtin_huge_valf();
        best_i[tt] = 0;   // a valid id whatever the values
    }
    put(0);
    __syncthreads();
    for (int tile = 0; tile < n_tile; ++tile) {
        if (tile + 1 < n_tile) fetch(tile + 1);
        const bf8_t* a = cen[tile & 1] + lane;
        f16_t acc[NT];
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) acc[tt] = f16_t{};
        // products of parts, smallest first: (center part, token part) with
        // the block of a center part p at (2 - p) kDimBlocks
        auto block = [&](int cp, int tp, int kd) {
            const bf8_t av = a[((2 - cp) * kDimBlocks + kd) * kWave];
#pragma unroll
            for (int tt = 0; tt < NT; ++tt)
                acc[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, tok[tt][tp][kd], acc[tt], 0, 0, 0);
        };
#pragma unroll
        for (int kd = 0; kd < kDimBlocks; ++kd) block(2, 0, kd);
        if constexpr (P == 3) {
#pragma unroll
            for (int kd = 0; kd < kDimBlocks; ++kd) block(1, 1, kd);
#pragma unroll
            for (int kd = 0; kd < kDimBlocks; ++kd) block(0, 2, kd);
        }
#pragma unroll
        for (int kd = 0; kd < kDimBlocks; ++kd) block(1, 0, kd);
        if constexpr (P == 3) {
#pragma unroll
            for (int kd = 0; kd < kDimBlocks; ++kd) block(0, 1, kd);
        }
#pragma unroll
        for (int kd = 0; kd < kDimBlocks; ++kd) block(0, 0, kd);
        const bf8_t av = a[3 * kDimBlocks * kWave];
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
            acc[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, nrm[tt], acc[tt], 0, 0, 0);
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
            // the lane's rows are in increasing center order: the first of
            // equal values stays (and a NaN, of a center that is one, never wins)
            float m = -__builtin_huge_valf(), m2 = m;
            int mi = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const bool up = acc[tt][i] > m;
                m2 = __builtin_amdgcn_fmed3f(acc[tt][i], m, m2);   // m2 <= m: the new second
                mi = up ? i : mi;
                m = up ? acc[tt][i] : m;
            }
            second[tt] = __builtin_amdgcn_fmed3f(best[tt], m, fmaxf(second[tt], m2));
            const bool up = m > best[tt];
            best[tt] = up ? m : best[tt];
            best_i[tt] = up ? tile * 16 + mi : best_i[tt];   // element 16 tile + i, until the end
        }
        if (tile + 1 < n_tile) put((tile + 1) & 1);   // its last readers passed the barrier below
        __syncthreads();
    }
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
        const int e = best_i[tt] % 16;
        best_i[tt] = best[tt] > -__builtin_huge_valf()
                         ? best_i[tt] / 16 * kTileCen + 8 * (e / 4) + 4 * half + e % 4 : 0;
        const float ob = __shfl_xor(best[tt], 32), os = __shfl_xor(second[tt], 32);
        second[tt] = __builtin_amdgcn_fmed3f(best[tt], ob, fmaxf(second[tt], os));
        asg_fold(best[tt], best_i[tt], ob, __shfl_xor(best_i[tt], 32));
        const int tk = (wave * NT + tt) * 32 + col;
        if (half == 0 && tk < nt) {
            const int64_t at = static_cast<int64_t>(bg) * D.rcap + t_base + tk;
            ids_tm[at] = min(best_i[tt], D.n_list - 1);
            if (dist_c) dist_c[at] = scale[tt] > 0.0f ? fmaxf(unit2[tt] - 2.0f * best[tt] / scale[tt], 0.0f) : 0.0f;
            if (!(best[tt] - second[tt] > 0.5f * kNearGap * scale[tt]))   // also with a NaN
                near[static_cast<int64_t>(bg) * D.rcap + atomicAdd(&n_near[bg], 1u)] = t_base + tk;
        }
    }
}

// ---------------------------------------------------------------------------
// nearest_kernel: the lists of the tokens that assign_kernel found nearly as
// close to a second center (near, n_near per KV head), by the distance the
// 32-bit matrix cores give (v_mfma_f32_16x16x4f32): which of two such centers is
// called the nearest is then the same as with those alone. One token in some
// thousands comes here (55 us at 128K tokens x 8 KV heads x 1024 lists); where
// centers coincide it can be all of them, which takes 5.3 ms there (6.9 with 32
// workgroups per KV head; the search with these instructions alone took 3.2).
//
// ||u - c||^2 = ||u||^2 + ||c||^2 - 2 u . c: 32 tokens per workgroup step (2
// tiles of 16), centers in chunks of 64 through LDS, the next chunk's loads
// under the current one's products; wave w takes the chunk's center tile w
// against both token tiles, since a KV head lists only some tens of tokens and a
// wave's chain of products is what a chunk waits for (8 tiles a wave: 0.16 ms in
// place of 0.06 ms). The 128 dimensions go as 32 steps: in step j, lane group q
// (lane / 16) contributes dimension 32 q + j, so each lane reads 32 contiguous
// floats of its row; rows are 132 floats apart in LDS, which puts the 16 rows of
// a read on distinct 16-byte bank groups.
// ---------------------------------------------------------------------------
constexpr int kNearThreads = 256;
constexpr int kNearTok = 32;                   // tokens per workgroup step
constexpr int kNearCen = 64;                   // centers per chunk, a tile per wave
constexpr int kNearLd = kHeadDim + 4;          // LDS row stride (floats)
constexpr int kNearWgs = 32;                   // workgroups per KV head, at least
constexpr int kNearPerCu = 3;                  // workgroups whose LDS a CU holds (51 KB each)
static_assert(kNearCen == kNearThreads / kWave * 16, "one center tile per wave");

__device__ __forceinline__ void near_fold(float& d, int& i, float od, int oi) {
    if (od < d || (od == d && oi < i)) {
        d = od;
        i = oi;
    }
}

template <typename T>
__global__ __launch_bounds__(kNearThreads) void nearest_kernel(Dims D, KV kv,
                                                               const float* __restrict__ centroids,
                                                               const int32_t* __restrict__ near,
                                                               const uint32_t* __restrict__ n_near,
                                                               int32_t* __restrict__ ids_tm,
                                                               float* __restrict__ dist_c) {
    __shared__ float4 tok4[kNearTok * kNearLd / 4];
    __shared__ float4 cen4[kNearCen * kNearLd / 4];
    __shared__ float cn[kNearCen];                    // ||c||^2 of the chunk's centers
    __shared__ float un[kNearTok];                    // ||u||^2 of the tokens
    __shared__ float wd[kNearThreads / kWave][kNearTok];
    __shared__ int wi[kNearThreads / kWave][kNearTok];
    float* tok = reinterpret_cast<float*>(tok4);
    float* rows = reinterpret_cast<float*>(cen4);
    // the KV heads along the grid's first dimension: the few workgroups that usually
    // have tokens come first, each on a CU of its own
    const int bg = blockIdx.x;
    const int b = bg / D.Hkv, g = bg % D.Hkv;
    const int n = static_cast<int>(n_near[bg]);
    const int32_t* list = near + static_cast<int64_t>(bg) * D.rcap;
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    const int col = lane % 16;   // the lane's token column (B) / center row (A) in a tile
    const int q = lane / 16;     // its lane group: dimensions 32 q .. 32 q + 31
    const T* kb = static_cast<const T*>(kv.k) + b * kv.sb + g * kv.sh;
    const float* cen = centroids + static_cast<int64_t>(bg) * D.n_list * kHeadDim;

    for (int base = static_cast<int>(blockIdx.y) * kNearTok; base < n;
         base += static_cast<int>(gridDim.y) * kNearTok) {
        const int nt = min(kNearTok, n - base);
        // the chunks' loads: 32 float4 per center row, zeros past the last center
        constexpr int kLoads = kNearCen * kHeadDim / 4 / kNearThreads;
        float4 next[kLoads];
        auto fetch = [&](int c0) {
#pragma unroll
            for (int it = 0; it < kLoads; ++it) {
                const int idx = it * kNearThreads + tid;
                const int c = c0 + idx / 32;
                next[it] = c < D.n_list
                               ? reinterpret_cast<const float4*>(cen + static_cast<int64_t>(c) * kHeadDim)[idx % 32]
                               : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        };
        fetch(0);
        // 1) the directions u = k / ||k|| of the workgroup's tokens into LDS:
        //    16 threads per token, 8 dimensions each
#pragma unroll
        for (int it = 0; it < kNearTok / 16; ++it) {
            const int tk = it * 16 + tid / 16;
            const int x0 = (tid % 16) * 8;
            float x[8];
            if (tk < nt) {
                Load8<T>::run(kb + static_cast<int64_t>(list[base + tk]) * kv.sn + x0, x);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = 0.0f;
            }
            float ss = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) ss = fmaf(x[e], x[e], ss);
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) ss += __shfl_xor(ss, off);
            const float r = sqrtf(ss);
            float uu = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                x[e] = r > 0.0f ? x[e] / r : 0.0f;
                uu = fmaf(x[e], x[e], uu);
            }
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) uu += __shfl_xor(uu, off);
            if (tid % 16 == 0) un[tk] = uu;
            float4* dst = reinterpret_cast<float4*>(tok + tk * kNearLd + x0);
            dst[0] = make_float4(x[0], x[1], x[2], x[3]);
            dst[1] = make_float4(x[4], x[5], x[6], x[7]);
        }
        __syncthreads();
        // 2) the B operands: token rows (2 tiles), 32 dimensions each
        float bv[2][32];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const float4* src = reinterpret_cast<const float4*>(tok + (tt * 16 + col) * kNearLd + 32 * q);
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const float4 f = src[v];
                bv[tt][4 * v] = f.x; bv[tt][4 * v + 1] = f.y; bv[tt][4 * v + 2] = f.z; bv[tt][4 * v + 3] = f.w;
            }
        }
        float best_d[2] = {__builtin_huge_valf(), __builtin_huge_valf()};
        int best_i[2] = {0, 0};   // a valid id even if every distance is NaN

        // 3) the centers, a chunk of 64 at a time
        for (int c0 = 0; c0 < D.n_list; c0 += kNearCen) {
#pragma unroll
            for (int it = 0; it < kLoads; ++it) {
                const int idx = it * kNearThreads + tid;
                const float4 v = next[it];
                float ss = fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(v.y, v.y, v.x * v.x)));   // this order, whatever the compiler contracts
#pragma unroll
                for (int off = 1; off < 32; off <<= 1) ss += __shfl_xor(ss, off);
                if (idx % 32 == 0) cn[idx / 32] = ss;
                reinterpret_cast<float4*>(rows + idx / 32 * kNearLd)[idx % 32] = v;
            }
            __syncthreads();
            if (c0 + kNearCen < D.n_list) fetch(c0 + kNearCen);
            f4_t acc[2] = {f4_t{0.0f, 0.0f, 0.0f, 0.0f}, f4_t{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
            for (int j4 = 0; j4 < 8; ++j4) {
                const float4 av = reinterpret_cast<const float4*>(rows + (wave * 16 + col) * kNearLd + 32 * q)[j4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const float a = jj == 0 ? av.x : jj == 1 ? av.y : jj == 2 ? av.z : av.w;
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt)
                        acc[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bv[tt][4 * j4 + jj], acc[tt], 0, 0, 0);
                }
            }
            // distances up to ||u||^2: row 4 q + i of tile w is center c0 + 16 w + 4 q + i
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int cl = wave * 16 + 4 * q + i;
                if (c0 + cl < D.n_list) {
                    const float c2 = cn[cl];
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt)
                        near_fold(best_d[tt], best_i[tt], fmaf(-2.0f, acc[tt][i], c2), c0 + cl);
                }
            }
            __syncthreads();   // the chunk is no longer read
        }
        // 4) the 4 lane groups of a token column, the waves, then the outputs
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
#pragma unroll
            for (int off = 16; off < kWave; off <<= 1) {
                const float od = __shfl_xor(best_d[tt], off);
                const int oi = __shfl_xor(best_i[tt], off);
                near_fold(best_d[tt], best_i[tt], od, oi);
            }
            if (q == 0) {
                wd[wave][tt * 16 + col] = best_d[tt];
                wi[wave][tt * 16 + col] = best_i[tt];
            }
        }
        __syncthreads();
        if (tid < nt) {
            float d = wd[0][tid];
            int i = wi[0][tid];
#pragma unroll
            for (int w = 1; w < kNearThreads / kWave; ++w) near_fold(d, i, wd[w][tid], wi[w][tid]);
            const int64_t at = static_cast<int64_t>(bg) * D.rcap + list[base + tid];
            ids_tm[at] = i;
            if (dist_c) dist_c[at] = fmaxf(d + un[tid], 0.0f);
        }
        __syncthreads();   // before the next tokens' rows
    }
}

// ---------------------------------------------------------------------------
// subspace_kernel: per token and subspace, the nearest codeword to the residual
// slice r = (u - c_a)^(m) (lists in ids_tm, norms in norms_tm), by half the
// squared distance, ||r||^2 / 2 - r . p + ||p||^2 / 2, again from products of
// bf16 parts: the six of a residual's and a codeword's parts that matter,
// v_mfma_f32_16x16x32_bf16 on 16 codewords x 16 tokens, started at the token's
// ||r||^2 / 2. These are never below 0 but for rounding, so their bits are
// compared as integers (a three-way minimum costs one instruction): the search
// is bound by the VALU, 16 instructions per 8 codewords, one of them for the
// second smallest value. A token whose two smallest are closer than the
// arithmetic tells apart (kTieGap below) is only marked, one bit per token and
// subspace, and ties_kernel decides it; so is one whose residual holds a NaN
// (all its values then do), and a codeword that holds one stands far away.
// Lane group q (lane / 16) owns DQ = DSUB / 4 consecutive
// dimensions of the subspace in both operands and holds every product of parts
// of these, so a lane computes, splits and later adds only its own slice of
// the residual, and no operand crosses lanes. Its 8 kBlocks slots, in order:
// products (codeword part, residual part) (3,1) (1,3) (2,2) (2,1) (1,2) of DQ
// dimensions each, the three parts of ||p||^2 / 2 (lane group 0) against 1,
// zeros, and product (1,1); the residual's parts are those of -r.
//
// A workgroup holds the operands of kSubs subspaces in LDS for all its tokens
// (one of Pq8's, all eight of Pq4's: 32 KB) and
// walks a slice of one KV head's tokens, 8 waves of kSubTiles x 16. In a
// training pass it also adds every residual to its codeword's sum, in LDS
// first, then with one global addition per workgroup. The sums are fixed
// point, so they don't depend on the order: 64 bits of 2^-41 (the slices are
// below 2 in size and at most 2^20 of them meet in a sum) and, for the
// remainder of the few residuals below 2^-17 that leave one, 64 bits of 2^-84.
// That replaces the grouping of every subspace's tokens and the gathers of
// their means.
// 128K tokens x 8 KV heads, Pq8: a training pass 0.85-0.90 ms, the final one
// 0.77-0.82 ms (1.9 ms with v_mfma_f32_16x16x4f32 and a two-key compare per pair;
// the grouping and gathers took another 1.3 ms a training pass). Two prompts of 40K, Pq4: 0.15 and 0.10 ms (0.20 ms, and 0.4 ms).
// ---------------------------------------------------------------------------
constexpr int kSubThreads = 512;
constexpr int kSubWaves = kSubThreads / kWave;
constexpr int kSubTiles = 2;                        // token tiles of 16 per wave and step
constexpr int kSubStep = kSubWaves * kSubTiles * 16;   // tokens per workgroup step
constexpr float kSumHi = 1048576.0f;                // 2^20: the fixed point's upper part
constexpr float kSumLo = 2199023255552.0f;          // 2^41
constexpr float kRestLo = 19342813113834066795298816.0f;   // 2^84: the remainders' fixed point

template <typename PQ>
struct SubLayout {
    static constexpr int kSubs = PQ::K >= 256 ? 1 : PQ::M;   // subspaces per workgroup
    static constexpr int kGroups = PQ::M / kSubs;            // workgroups that share a slice of tokens
    static constexpr int DQ = PQ::DSUB / 4;                  // dimensions per lane group
    static constexpr int kTiles = PQ::K / 16;                // codeword tiles per subspace
    static constexpr int kBlocks = DQ;                       // 32-slot blocks of an operand
    static constexpr int kNormSlot = 5 * DQ;
    static constexpr int kLastSlot = 8 * kBlocks - DQ;
    static constexpr int kPerCu = 2;                         // workgroups a CU's registers hold
    // Half squared distances closer than kTieGap (||r||^2 + D), D the smaller
    // squared distance, are a tie. With u = 2^-24, either sum's roundings and
    // ||p||^2 <= 2 (||r||^2 + D): one of the 32-bit matrix cores' is off by at
    // most (DSUB + 1) u (||r||^2 + 2 ||p||^2), one of the parts' by its 8 DSUB
    // slots' u (||r||^2 + ||p||^2), both for two codewords: below 54 DSUB u
    // (||r||^2 + D) in all. One (token, subspace) in some 2000 at 128K tokens
    // with Pq8, in 1200 at 40K with Pq4.
    static constexpr float kTieGap = 64.0f * PQ::DSUB / 16777216.0f;
    // the LDS sums, [subspace][dimension][codeword]: a row stride that puts
    // the four lane groups' dimensions 16 banks apart
    static constexpr int kSumLd = PQ::K + (PQ::K >= 256 ? 4 : 2);
    static_assert(2 * DQ * kSumLd % 64 == 16, "lane groups on distinct banks");
    static_assert(kNormSlot + 3 <= kLastSlot && PQ::K % 16 == 0 && PQ::M % kSubs == 0, "operand layout");
};

__device__ __forceinline__ uint32_t pack_bf16(__bf16 lo, __bf16 hi) {
    return static_cast<uint32_t>(__builtin_bit_cast(uint16_t, lo)) |
           (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, hi)) << 16);
}

// x (|x| < 2^10) in 2^-41 fixed point, to nearest, and in `rest` what that
// leaves of it, exactly.
__device__ __forceinline__ unsigned long long to_fixed(float x, float& rest) {
    const float hi = rintf(x * kSumHi);
    const float low = fmaf(hi, -1.0f / kSumHi, x);
    const float lo = rintf(low * kSumLo);
    rest = fmaf(lo, -1.0f / kSumLo, low);
    const long long v = static_cast<long long>(static_cast<int>(hi)) * static_cast<long long>(kSumLo / kSumHi) +
                        static_cast<int>(lo);
    return static_cast<unsigned long long>(v);
}
__device__ __forceinline__ unsigned long long rest_fixed(float rest) {
    return static_cast<unsigned long long>(static_cast<long long>(rest * kRestLo));
}

// The middle one of three.
__device__ __forceinline__ int med3(int a, int b, int c) { return max(min(a, b), min(max(a, b), c)); }

template <typename T, typename PQ, bool kTrain>
__global__ __launch_bounds__(kSubThreads) void subspace_kernel(
    Dims D, BatchInts lo, BatchInts hi, KV kv, const float* __restrict__ centroids,
    const float* __restrict__ codebooks, const int32_t* __restrict__ ids_tm,
    const float* __restrict__ norms_tm, int n_pair, int per, uint8_t* __restrict__ codes_tm,
    float* __restrict__ dist_f, SubSums out, uint32_t* __restrict__ ties, int tie_words) {
    using L = SubLayout<PQ>;
    constexpr int M = PQ::M, K = PQ::K, DS = PQ::DSUB, DQ = L::DQ, NB = L::kBlocks, CT = L::kTiles;
    constexpr int kSubs = L::kSubs;
    __shared__ uint4 op[kSubs * CT * NB * kWave];                  // codeword operands, in operand order
    __shared__ unsigned long long sum[kTrain ? kSubs * DS * L::kSumLd : 1];
    __shared__ unsigned long long rests[kTrain ? kSubs * DS * L::kSumLd : 1];
    __shared__ uint32_t cnt[kTrain ? kSubs * K : 1];
    // the kGroups workgroups of a slice have ids congruent mod 8: one XCD,
    // whose L2 then serves the slice's keys and lists to all of them
    const int j = blockIdx.x / 8;
    const int grp = j % L::kGroups;
    const int pair = j / L::kGroups * 8 + blockIdx.x % 8;
    if (pair >= n_pair) return;
    const int bg = pair % (D.B * D.Hkv);
    const int slice = pair / (D.B * D.Hkv);
    const int b = bg / D.Hkv, g = bg % D.Hkv;
    const int t0 = lo.v[b] + slice * per;
    const int t1 = min(t0 + per, hi.v[b]);
    if (t0 >= t1) return;
    const int m0 = grp * kSubs;
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    const int col = lane % 16;
    const int q = lane / 16;

    // 1) the codeword operands: one lane's slots of one codeword per thread
    const float* cb = codebooks + (static_cast<int64_t>(bg) * M + m0) * K * DS;
    for (int i = tid; i < kSubs * K * 4; i += kSubThreads) {
        const int z = i / 4 % K, sq = i % 4, ss = i / (4 * K);
        const float* p = cb + (ss * K + z) * DS;
        __bf16 part[3][DQ];
        double p2 = 0.0;
#pragma unroll
        for (int d = 0; d < DS; ++d) p2 += static_cast<double>(p[d]) * p[d];
        const bool real = p2 < static_cast<double>(kFarCenter);   // not a NaN
#pragma unroll
        for (int e = 0; e < DQ; ++e) {
            __bf16 x[3];
            split_bf16(real ? p[sq * DQ + e] : 0.0f, x);
#pragma unroll
            for (int u = 0; u < 3; ++u) part[u][e] = x[u];
        }
        __bf16 np[3];
        split_bf16(real ? static_cast<float>(0.5 * p2) : kFarCenter, np);
        __bf16 slot[8 * NB];
#pragma unroll
        for (int u = 0; u < 8 * NB; ++u) slot[u] = static_cast<__bf16>(0.0f);
        constexpr int kCodePart[5] = {2, 0, 1, 1, 0};
#pragma unroll
        for (int u = 0; u < 5; ++u)
#pragma unroll
            for (int e = 0; e < DQ; ++e) slot[u * DQ + e] = part[kCodePart[u]][e];
        if (sq == 0) {
#pragma unroll
            for (int u = 0; u < 3; ++u) slot[L::kNormSlot + u] = np[2 - u];
        }
#pragma unroll
        for (int e = 0; e < DQ; ++e) slot[L::kLastSlot + e] = part[0][e];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            uint32_t w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = pack_bf16(slot[nb * 8 + 2 * u], slot[nb * 8 + 2 * u + 1]);
            op[((ss * CT + z / 16) * NB + nb) * kWave + sq * 16 + z % 16] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    if constexpr (kTrain) {
        for (int i = tid; i < kSubs * DS * L::kSumLd; i += kSubThreads) sum[i] = rests[i] = 0ull;
        for (int i = tid; i < kSubs * K; i += kSubThreads) cnt[i] = 0u;
    }
    __syncthreads();

    // 2) the slice's tokens
    const T* kb = static_cast<const T*>(kv.k) + b * kv.sb + g * kv.sh;
    const float* cen = centroids + static_cast<int64_t>(bg) * D.n_list * kHeadDim;
    const int64_t row = static_cast<int64_t>(bg) * D.rcap;
    const __bf16 one = static_cast<__bf16>(1.0f), zero = static_cast<__bf16>(0.0f);
    for (int s0 = t0; s0 < t1; s0 += kSubStep) {
        int tk[kSubTiles], a[kSubTiles];
        float r[kSubTiles], inv[kSubTiles];
        bool none[kSubTiles];
#pragma unroll
        for (int tt = 0; tt < kSubTiles; ++tt) {
            tk[tt] = s0 + (wave * kSubTiles + tt) * 16 + col;
            const int t = min(tk[tt], t1 - 1);   // tokens past the slice repeat its last, unused
            a[tt] = min(max(ids_tm[row + t], 0), D.n_list - 1);
            // u = k / r: by the rounded reciprocal and one correction, which is the
            // rounded quotient (Markstein; above 2^-100, where no remainder
            // underflows); the zero direction for a zero norm or one that is no
            // number, 0 k for an infinite one
            const float n = norms_tm[row + t];
            none[tt] = !(n > 0.0f);
            const bool live = n > 0.0f && n < __builtin_huge_valf();
            const float y = __builtin_amdgcn_rcpf(n);
            r[tt] = live ? n : 0.0f;
            inv[tt] = live ? fmaf(fmaf(-n, y, 1.0f), y, y) : 0.0f;
        }
#pragma unroll 1
        for (int ss = 0; ss < kSubs; ++ss) {
            const int m = m0 + ss;
            float res[kSubTiles][DQ], r2[kSubTiles];
            bf8_t bv[kSubTiles][NB];
#pragma unroll
            for (int tt = 0; tt < kSubTiles; ++tt) {
                const int d0 = m * DS + q * DQ;
                const T* kp = kb + static_cast<int64_t>(min(tk[tt], t1 - 1)) * kv.sn + d0;
                const float* cp = cen + static_cast<int64_t>(a[tt]) * kHeadDim + d0;
                float x[DQ], c[DQ];
                load_slice<T, DQ>(kp, x);
                load_slice<float, DQ>(cp, c);
                r2[tt] = 0.0f;
                __bf16 part[3][DQ];
#pragma unroll
                for (int e = 0; e < DQ; ++e) {
                    const float xe = none[tt] ? 0.0f : x[e];
                    const float qt = xe * inv[tt];
                    res[tt][e] = fmaf(fmaf(-qt, r[tt], xe), inv[tt], qt) - c[e];
                    r2[tt] = fmaf(res[tt][e], res[tt][e], r2[tt]);
                    __bf16 y[3];
                    split_bf16(-res[tt][e], y);
#pragma unroll
                    for (int i = 0; i < 3; ++i) part[i][e] = y[i];
                }
                __bf16 slot[8 * NB];
#pragma unroll
                for (int u = 0; u < 8 * NB; ++u) slot[u] = zero;
                constexpr int kResPart[5] = {0, 2, 1, 0, 1};
#pragma unroll
                for (int u = 0; u < 5; ++u)
#pragma unroll
                    for (int e = 0; e < DQ; ++e) slot[u * DQ + e] = part[kResPart[u]][e];
#pragma unroll
                for (int u = 0; u < 3; ++u) slot[L::kNormSlot + u] = one;
#pragma unroll
                for (int e = 0; e < DQ; ++e) slot[L::kLastSlot + e] = part[0][e];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    uint32_t w[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) w[u] = pack_bf16(slot[nb * 8 + 2 * u], slot[nb * 8 + 2 * u + 1]);
                    bv[tt][nb] = __builtin_bit_cast(bf8_t, make_uint4(w[0], w[1], w[2], w[3]));
                }
            }
            // half squared distances (as bits) from here on
            f4_t half_r2[kSubTiles];
            constexpr int kAtOnce = CT < 2 ? CT : 2;   // codeword tiles per comparison
            constexpr int kOuts = 4 * kAtOnce;
            // keep: the best group's values; second: the second smallest of the groups' smallest
            int best[kSubTiles], second[kSubTiles], best_z[kSubTiles], keep[kSubTiles][kOuts];
#pragma unroll
            for (int tt = 0; tt < kSubTiles; ++tt) {
                r2[tt] += __shfl_xor(r2[tt], 16);
                r2[tt] += __shfl_xor(r2[tt], 32);
                const float h = 0.5f * r2[tt];
                half_r2[tt] = f4_t{h, h, h, h};
            }
            const uint4* ops = op + ss * CT * NB * kWave + lane;
            auto group = [&](int ct0, bool first) {
                f4_t acc[kAtOnce][kSubTiles];
#pragma unroll
                for (int ct = 0; ct < kAtOnce; ++ct)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const bf8_t av = __builtin_bit_cast(bf8_t, ops[((ct0 + ct) * NB + nb) * kWave]);
#pragma unroll
                        for (int tt = 0; tt < kSubTiles; ++tt)
                            acc[ct][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                av, bv[tt][nb], nb == 0 ? half_r2[tt] : acc[ct][tt], 0, 0, 0);
                    }
#pragma unroll
                for (int tt = 0; tt < kSubTiles; ++tt) {
                    int v[kOuts], m1 = __float_as_int(acc[0][tt][0]);
#pragma unroll
                    for (int u = 0; u < kOuts; ++u) v[u] = __float_as_int(acc[u / 4][tt][u % 4]);
#pragma unroll
                    for (int u = 1; u + 1 < kOuts; u += 2) m1 = min(min(v[u], v[u + 1]), m1);
                    m1 = min(m1, v[kOuts - 1]);
                    // strictly below: the first of equal groups stays
                    const bool down = first || m1 < best[tt];
                    second[tt] = first ? 0x7fffffff : med3(best[tt], m1, second[tt]);
                    best[tt] = first ? m1 : min(best[tt], m1);
                    best_z[tt] = down ? ct0 : best_z[tt];
#pragma unroll
                    for (int u = 0; u < kOuts; ++u) keep[tt][u] = down ? v[u] : keep[tt][u];
                }
            };
            group(0, true);
            // not unrolled: the compiler would keep the operands of every tile
            // in registers across the steps
#pragma unroll 1
            for (int ct0 = kAtOnce; ct0 < CT; ct0 += kAtOnce) group(ct0, false);
            uint64_t tied[kSubTiles];
            static_assert(kSubTiles == 2, "a word of ties per wave and step");
#pragma unroll
            for (int tt = 0; tt < kSubTiles; ++tt) {
                int e = 0;   // the first of the group's values that is the smallest
#pragma unroll
                for (int u = kOuts - 1; u >= 0; --u) e = keep[tt][u] == best[tt] ? u : e;
                int low = keep[tt][0], next = 0x7fffffff;   // and the second smallest
#pragma unroll
                for (int u = 1; u < kOuts; ++u) {
                    next = med3(low, keep[tt][u], next);
                    low = min(low, keep[tt][u]);
                }
                second[tt] = min(second[tt], next);
                best_z[tt] = (best_z[tt] + e / 4) * 16 + 4 * q + e % 4;
#pragma unroll
                for (int off = 16; off < kWave; off <<= 1) {
                    const int od = __shfl_xor(best[tt], off);
                    const int oz = __shfl_xor(best_z[tt], off);
                    second[tt] = min(max(best[tt], od), min(second[tt], __shfl_xor(second[tt], off)));
                    if (od < best[tt] || (od == best[tt] && oz < best_z[tt])) {
                        best[tt] = od;
                        best_z[tt] = oz;
                    }
                }
                const float h = __int_as_float(best[tt]);
                const bool tie = !(__int_as_float(second[tt]) - h > L::kTieGap * fmaf(2.0f, h, r2[tt]));   // also with a NaN
                tied[tt] = __ballot(tie && tk[tt] < t1);
                if (tie || tk[tt] >= t1) continue;
                if constexpr (kTrain) {
#pragma unroll
                    for (int e2 = 0; e2 < DQ; ++e2) {
                        const int at = (ss * DS + q * DQ + e2) * L::kSumLd + best_z[tt];
                        float rest;
                        atomicAdd(&sum[at], to_fixed(res[tt][e2], rest));
                        if (rest != 0.0f) atomicAdd(&rests[at], rest_fixed(rest));
                    }
                    if (q == 0) {
                        atomicAdd(&cnt[ss * K + best_z[tt]], 1u);
                        dist_f[(static_cast<int64_t>(bg) * M + m) * D.rcap + tk[tt]] = fmaxf(2.0f * h, 0.0f);
                    }
                } else {
                    if (q == 0) codes_tm[(row + tk[tt]) * M + m] = static_cast<uint8_t>(best_z[tt]);
                }
            }
            // the step's 32 tokens of the wave, a bit each (s0 - lo is a multiple of kSubStep)
            if (lane == 0)
                ties[(static_cast<int64_t>(bg) * M + m) * tie_words + (s0 - lo.v[b]) / 32 + wave] =
                    static_cast<uint32_t>(tied[0] & 0xffffu) | static_cast<uint32_t>(tied[1] & 0xffffu) << 16;
        }
    }
    if constexpr (kTrain) {
        __syncthreads();
        const int64_t pz = (static_cast<int64_t>(bg) * M + m0) * K;
        for (int i = tid; i < kSubs * K * DS; i += kSubThreads) {
            const int at = (i / (K * DS) * DS + i % DS) * L::kSumLd + i / DS % K;
            if (sum[at]) atomicAdd(&out.sums[pz * DS + i], sum[at]);
            if (rests[at]) atomicAdd(&out.rests[pz * DS + i], rests[at]);
        }
        for (int i = tid; i < kSubs * K; i += kSubThreads)
            if (cnt[i]) atomicAdd(&out.counts[pz + i], cnt[i]);
    }
}

// ---------------------------------------------------------------------------
// ties_kernel: the codewords of the tokens that subspace_kernel marked, by the
// distance the 32-bit matrix cores give (v_mfma_f32_16x16x4f32, lane group q with
// dimensions q DSUB / 4 + s in step s; ties to the smaller codeword), so the
// choice is the one that those alone would make. A residual that holds a NaN takes
// codeword 0 at distance 0. In training it also adds them to the sums; a
// residual that is a NaN marks its codeword's dimension in `nans`.
//
// One workgroup per problem and kTieWords words of marks, which it lists first;
// most find a few tokens or none, so each wave takes 16 of them against all the
// codewords: 22 us a pass at 128K tokens x 8 KV heads with Pq8 (2.2 ms where all
// codewords coincide). With it and the second smallest value subspace_kernel
// takes 0.85 and 0.77 ms there, 0.75 and 0.69 without.
// ---------------------------------------------------------------------------
constexpr int kTieThreads = 256;
constexpr int kTieWords = kTieThreads;

template <typename T, typename PQ, bool kTrain>
__global__ __launch_bounds__(kTieThreads) void ties_kernel(
    Dims D, BatchInts lo, BatchInts hi, KV kv, const float* __restrict__ centroids,
    const float* __restrict__ codebooks, const int32_t* __restrict__ ids_tm, const float* __restrict__ norms_tm,
    const uint32_t* __restrict__ ties, int tie_words, uint8_t* __restrict__ codes_tm, float* __restrict__ dist_f,
    SubSums out) {
    constexpr int M = PQ::M, K = PQ::K, DS = PQ::DSUB, S = DS / 4, LD = DS + 1;   // odd row stride: distinct banks
    __shared__ float rows[K * LD];
    __shared__ float pn[K];                        // ||p||^2
    __shared__ uint16_t list[kTieWords * 32];      // the marked tokens, from the first word's first
    __shared__ SelectScratch scan;
    static_assert(kTieWords * 32 <= 65536, "16-bit token offsets");
    const int p = blockIdx.x;
    const int bg = p / M, m = p % M;
    const int b = bg / D.Hkv, g = bg % D.Hkv;
    const int first = lo.v[b] + static_cast<int>(blockIdx.y) * kTieWords * 32;
    if (first >= hi.v[b]) return;
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    const int col = lane % 16;
    const int q = lane / 16;
    uint32_t bits = first + tid * 32 < hi.v[b]
                        ? ties[static_cast<int64_t>(p) * tie_words + blockIdx.y * kTieWords + tid] : 0u;
    int total = 0;
    int at = block_excl_scan<kTieThreads>(__popc(bits), total, scan);
    if (total == 0) return;
    for (; bits; bits &= bits - 1) list[at++] = static_cast<uint16_t>(tid * 32 + __ffs(bits) - 1);
    const float* cb = codebooks + static_cast<int64_t>(p) * K * DS;
    for (int i = tid; i < K * DS; i += kTieThreads) rows[i / DS * LD + i % DS] = cb[i];
    __syncthreads();
    for (int z = tid; z < K; z += kTieThreads) {
        float ss = 0.0f;
#pragma unroll
        for (int x = 0; x < DS; ++x) ss = fmaf(rows[z * LD + x], rows[z * LD + x], ss);
        pn[z] = ss;
    }
    __syncthreads();
    const int64_t row = static_cast<int64_t>(bg) * D.rcap;
    for (int i0 = wave * 16; i0 < total; i0 += kTieThreads / kWave * 16) {
        const bool present = i0 + col < total;
        const int t = first + list[min(i0 + col, total - 1)];
        const int a = min(max(ids_tm[row + t], 0), D.n_list - 1);
        const float r = norms_tm[row + t];
        const int d0 = m * DS + q * S;
        float x[S], c[S], res[S];
        load_slice<T, S>(static_cast<const T*>(kv.k) + b * kv.sb + g * kv.sh + static_cast<int64_t>(t) * kv.sn + d0, x);
        load_slice<float, S>(centroids + (static_cast<int64_t>(bg) * D.n_list + a) * kHeadDim + d0, c);
        float r2 = 0.0f;
#pragma unroll
        for (int s2 = 0; s2 < S; ++s2) {
            res[s2] = (r > 0.0f ? x[s2] / r : 0.0f) - c[s2];
            r2 = fmaf(res[s2], res[s2], r2);
        }
        float best_d = __builtin_huge_valf();
        int best_z = 0;   // a valid codeword even if every distance is NaN
#pragma unroll 2
        for (int ct = 0; ct < K / 16; ++ct) {
            f4_t acc = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s2 = 0; s2 < S; ++s2)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rows[(ct * 16 + col) * LD + q * S + s2], res[s2], acc, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int z = ct * 16 + 4 * q + i;
                near_fold(best_d, best_z, fmaf(-2.0f, acc[i], pn[z]), z);
            }
        }
#pragma unroll
        for (int off = 16; off < kWave; off <<= 1) {
            r2 += __shfl_xor(r2, off);
            const float od = __shfl_xor(best_d, off);
            const int oz = __shfl_xor(best_z, off);
            near_fold(best_d, best_z, od, oz);
        }
        if (!present) continue;
        if constexpr (kTrain) {
            const int64_t pz = static_cast<int64_t>(p) * K + best_z;
#pragma unroll
            for (int s2 = 0; s2 < S; ++s2) {
                const int d = q * S + s2;
                if (!(fabsf(res[s2]) < 1024.0f)) {   // a NaN
                    atomicOr(&out.nans[pz], 1u << d);
                    continue;
                }
                float rest;
                atomicAdd(&out.sums[pz * DS + d], to_fixed(res[s2], rest));
                if (rest != 0.0f) atomicAdd(&out.rests[pz * DS + d], rest_fixed(rest));
            }
            if (q == 0) {
                atomicAdd(&out.counts[pz], 1u);
                dist_f[static_cast<int64_t>(p) * D.rcap + t] = fmaxf(best_d + r2, 0.0f);
            }
        } else if (q == 0) {
            codes_tm[(row + t) * M + m] = static_cast<uint8_t>(best_z);
        }
    }
}

// The codewords from a training pass's sums: the mean of each one's members
// (an empty one keeps its value, the re-seeding replaces it).
__global__ __launch_bounds__(256) void codewords_kernel(int64_t n, int dims, SubSums in, float* __restrict__ out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t c = in.counts[i / dims];
    if (!c) return;
    const double s = static_cast<double>(static_cast<long long>(in.sums[i])) / static_cast<double>(kSumLo) +
                     static_cast<double>(static_cast<long long>(in.rests[i])) / static_cast<double>(kRestLo);
    out[i] = in.nans[i / dims] >> (i % dims) & 1u ? __builtin_nanf("") : static_cast<float>(s / c);
}

template <typename T, typename PQ>
static hipError_t launch_subspace_t(const Dims& D, const BatchInts& lo, const BatchInts& hi, int max_n,
                                    const KV& kv, const float* centroids, float* codebooks,
                                    const int32_t* ids_tm, uint8_t* codes_tm, const float* norms_tm,
                                    const BuildBufs& bb, bool train, hipStream_t s) {
    using L = SubLayout<PQ>;
    // slices of a KV head's tokens: one round of the workgroups a CU holds, but
    // no slice of fewer than four steps
    const int bgs = D.B * D.Hkv;
    const int n_cu = device_cu_count() > 0 ? device_cu_count() : 1;
    const int want = std::max(1, L::kPerCu * n_cu / (bgs * L::kGroups));
    const int most = (max_n + 4 * kSubStep - 1) / (4 * kSubStep);
    const int slices = std::min(want, most);
    const int per = ((max_n + slices - 1) / slices + kSubStep - 1) / kSubStep * kSubStep;
    const int n_pair = bgs * ((max_n + per - 1) / per);
    const dim3 grid((n_pair + 7) / 8 * 8 * L::kGroups);
    const int words = tie_words(D);
    const dim3 tie_grid(bgs * PQ::M, (max_n + kTieWords * 32 - 1) / (kTieWords * 32));
    const SubSums none{};
    if (!train) {
        hipLaunchKernelGGL((subspace_kernel<T, PQ, false>), grid, dim3(kSubThreads), 0, s, D, lo, hi, kv, centroids,
                           codebooks, ids_tm, norms_tm, n_pair, per, codes_tm, nullptr, none, bb.ties, words);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((ties_kernel<T, PQ, false>), tie_grid, dim3(kTieThreads), 0, s, D, lo, hi, kv, centroids,
                           codebooks, ids_tm, norms_tm, bb.ties, words, codes_tm, nullptr, none);
        return hipGetLastError();
    }
    const int64_t n = static_cast<int64_t>(bgs) * PQ::M * PQ::K;
    hipError_t e = hipMemsetAsync(bb.sums.sums, 0, sub_sums_bytes(n, PQ::DSUB), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((subspace_kernel<T, PQ, true>), grid, dim3(kSubThreads), 0, s, D, lo, hi, kv, centroids,
                       codebooks, ids_tm, norms_tm, n_pair, per, codes_tm, bb.dist_f, bb.sums, bb.ties, words);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ties_kernel<T, PQ, true>), tie_grid, dim3(kTieThreads), 0, s, D, lo, hi, kv, centroids,
                       codebooks, ids_tm, norms_tm, bb.ties, words, codes_tm, bb.dist_f, bb.sums);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(codewords_kernel, dim3(static_cast<unsigned>((n * PQ::DSUB + 255) / 256)), dim3(256), 0, s,
                       n * PQ::DSUB, PQ::DSUB, bb.sums, codebooks);
    return hipGetLastError();
}

hipError_t launch_subspace(const Dims& D, const BatchInts& lo, const BatchInts& hi, int max_n,
                           const KV& kv, const float* centroids, float* codebooks,
                           const int32_t* ids_tm, uint8_t* codes_tm, const float* norms_tm,
                           const BuildBufs& bb, bool train, hipStream_t s) {
    if (max_n <= 0) return hipSuccess;
#define PQHSA_SUB(TT, PQT)                                                                            \
    launch_subspace_t<TT, PQT>(D, lo, hi, max_n, kv, centroids, codebooks, ids_tm, codes_tm, norms_tm, bb, train, s)
    if (kv.bf16) return D.pq_bits == 4 ? PQHSA_SUB(bf16_t, Pq4) : PQHSA_SUB(bf16_t, Pq8);
    return D.pq_bits == 4 ? PQHSA_SUB(float, Pq4) : PQHSA_SUB(float, Pq8);
#undef PQHSA_SUB
}

hipError_t launch_assign(const Dims& D, const BatchInts& lo, const BatchInts& hi, int max_n,
                         const KV& kv, const float* centroids, const BuildBufs& bb, int32_t* ids_tm,
                         float* norms_tm, float* dist_c, hipStream_t s) {
    if (max_n <= 0) return hipSuccess;
    const int n_tile = (D.n_list + kTileCen - 1) / kTileCen;
    __bf16* parts = static_cast<__bf16*>(bb.split);
    hipLaunchKernelGGL(split_centers_kernel, dim3(n_tile, D.B * D.Hkv), dim3(kTileCen * 8), 0, s, D, centroids,
                       parts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = hipMemsetAsync(bb.n_near, 0, static_cast<size_t>(D.B) * D.Hkv * sizeof(uint32_t), s);
    if (e != hipSuccess) return e;
    const int tok = kAsgWaves * 32 * (kv.bf16 ? AsgTokens<bf16_t>::kTiles : AsgTokens<float>::kTiles);
    const dim3 grid((max_n + tok - 1) / tok, D.Hkv, D.B);
    const int n_cu = device_cu_count() > 0 ? device_cu_count() : 1;
    const int near_wgs = std::max(kNearWgs, kNearPerCu * n_cu / (D.B * D.Hkv));
    const dim3 near_grid(D.B * D.Hkv, std::min(near_wgs, (max_n + kNearTok - 1) / kNearTok));
#define PQHSA_ASSIGN(TT)                                                                                    \
    do {                                                                                                    \
        hipLaunchKernelGGL(assign_kernel<TT>, grid, dim3(kAsgThreads), 0, s, D, lo, hi, kv, parts, n_tile,  \
                           ids_tm, norms_tm, dist_c, bb.order, bb.n_near);                                  \
        e = hipGetLastError();                                                                              \
        if (e != hipSuccess) return e;                                                                      \
        hipLaunchKernelGGL(nearest_kernel<TT>, near_grid, dim3(kNearThreads), 0, s, D, kv, centroids,       \
                           bb.order, bb.n_near, ids_tm, dist_c);                                            \
    } while (0)
    if (kv.bf16) PQHSA_ASSIGN(bf16_t);
    else PQHSA_ASSIGN(float);
#undef PQHSA_ASSIGN
    return hipGetLastError();
}

}  // namespace pqhsa
