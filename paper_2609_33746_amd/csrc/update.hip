// Incremental index update (Section 3.3): tokens that leave the local window
// are encoded into the existing lists, without re-clustering, and the list
// means are refreshed over the grown lists.
//
//  * encode_coarse_kernel and encode_fine_kernel: the key is split into its norm
//    r and direction u (Section 3.1); u goes to the list with the nearest
//    centroid, and each slice of the residual u - c_a to its nearest codeword.
//    Squared Euclidean distances in fp32, summed in dimension order; ties go to
//    the smaller list id or codeword index. Write the token-major list id, codes
//    (one code per byte) and norm. (The build's passes over all of R use the
//    matrix-core search in the build's source.)
//  * means_update_kernel, after the merge below: one workgroup per (list,
//    kv head, sequence) adds the new members' values to the list's float64
//    value sum and writes the mean v_bar' = sum / (n_old + n_new) in fp32. The
//    sums start at |R_j| v_bar_j when an index is prepared or built, so the
//    fp32 means never feed back into later updates and do not drift.
//
// The list-major layout is then merged on the device (update_lists_kernel,
// shift_positions_kernel below) and codes and norms gathered into it.
#include <algorithm>

#include "device_common.h"
#include "pqhsa_internal.h"

namespace pqhsa {

constexpr int kEncThreads = 256;

// (d, i) < (od, oi) lexicographically: the smaller distance, then the smaller index
__device__ __forceinline__ void argmin_fold(float& d, int& i, float od, int oi) {
    if (od < d || (od == d && oi < i)) {
        d = od;
        i = oi;
    }
}

// encode_coarse_kernel: kEncTok tokens against chunks of kEncCen centroids
// staged in LDS; the workgroups of a token tile share the chunks out (gridDim.y
// of them, so that an update of a few hundred tokens fills the chip), and each
// writes its nearest centroid per token to part_d / part_i [B Hkv][token][share].
// A thread holds 2 tokens x 4 centroids and adds their squared differences in
// dimension order. Every centroid row then comes from L2 once per 32 tokens, not
// once per token (one workgroup per token: 139 us at 256 tokens x 8 KV heads x
// 1024 lists, against 33 + 12 us for the two kernels). Also writes the norms.
constexpr int kEncTok = 32;
constexpr int kEncCen = 64;
constexpr int kEncLd = kHeadDim + 4;   // LDS row stride: 16 rows on distinct 16-byte bank groups

template <typename T>
__global__ __launch_bounds__(kEncThreads) void encode_coarse_kernel(
    Dims D, BatchInts lo, BatchInts hi, const T* __restrict__ kcache, int64_t sb, int64_t sh, int64_t sn,
    const float* __restrict__ centroids, float* __restrict__ part_d, int32_t* __restrict__ part_i,
    int64_t part_stride, float* __restrict__ norms_tm) {
    __shared__ float4 us4[kEncTok * kEncLd / 4];
    __shared__ float4 cs4[kEncCen * kEncLd / 4];
    const int bg = blockIdx.z;
    const int b = bg / D.Hkv, g = bg % D.Hkv;
    const int t0 = lo.v[b] + static_cast<int>(blockIdx.x) * kEncTok;
    if (t0 >= hi.v[b]) return;
    const int nt = min(kEncTok, hi.v[b] - t0);
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    // r = ||k||, u = k / r (u = 0 for a zero key): one wave per token
    float* us = reinterpret_cast<float*>(us4);
    for (int i = wave; i < kEncTok; i += kEncThreads / kWave) {
        float k0 = 0.0f, k1 = 0.0f;
        if (i < nt) {
            const T* row = kcache + b * sb + g * sh + static_cast<int64_t>(t0 + i) * sn;
            k0 = load1<T>(row + lane);
            k1 = load1<T>(row + kWave + lane);
        }
        float s0 = k0 * k0, s1 = k1 * k1;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            s0 += __shfl_xor(s0, off);
            s1 += __shfl_xor(s1, off);
        }
        const float r = sqrtf(s0 + s1);
        us[i * kEncLd + lane] = r > 0.0f ? k0 / r : 0.0f;
        us[i * kEncLd + kWave + lane] = r > 0.0f ? k1 / r : 0.0f;
        if (lane == 0 && i < nt && blockIdx.y == 0) norms_tm[static_cast<int64_t>(bg) * D.rcap + t0 + i] = r;
    }
    const int tx = tid % 16;          // centroids tx, tx + 16, tx + 32, tx + 48 of a chunk
    const int ty = tid / 16 * 2;      // tokens ty, ty + 1
    const float* cen = centroids + static_cast<int64_t>(bg) * D.n_list * kHeadDim;
    float best_d[2] = {__builtin_huge_valf(), __builtin_huge_valf()};
    int best_i[2] = {0, 0};   // a valid id even if every distance is NaN
    for (int c0 = static_cast<int>(blockIdx.y) * kEncCen; c0 < D.n_list;
         c0 += static_cast<int>(gridDim.y) * kEncCen) {
        __syncthreads();   // the directions are written; the previous chunk is no longer read
#pragma unroll
        for (int it = 0; it < kEncCen * kHeadDim / 4 / kEncThreads; ++it) {
            const int idx = it * kEncThreads + tid;
            const int c = min(c0 + idx / 32, D.n_list - 1);   // 32 float4 per row; past the end unused
            cs4[idx / 32 * (kEncLd / 4) + idx % 32] =
                reinterpret_cast<const float4*>(cen + static_cast<int64_t>(c) * kHeadDim)[idx % 32];
        }
        __syncthreads();
        float acc[2][4] = {};
#pragma unroll 4
        for (int x = 0; x < kHeadDim / 4; ++x) {
            float4 u[2], c[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) u[i] = us4[(ty + i) * (kEncLd / 4) + x];
#pragma unroll
            for (int j = 0; j < 4; ++j) c[j] = cs4[(tx + 16 * j) * (kEncLd / 4) + x];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d0 = u[i].x - c[j].x, d1 = u[i].y - c[j].y;
                    const float d2 = u[i].z - c[j].z, d3 = u[i].w - c[j].w;
                    acc[i][j] = fmaf(d0, d0, acc[i][j]);
                    acc[i][j] = fmaf(d1, d1, acc[i][j]);
                    acc[i][j] = fmaf(d2, d2, acc[i][j]);
                    acc[i][j] = fmaf(d3, d3, acc[i][j]);
                }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (c0 + tx + 16 * j < D.n_list) argmin_fold(best_d[i], best_i[i], acc[i][j], c0 + tx + 16 * j);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const float od = __shfl_xor(best_d[i], off);
            const int oi = __shfl_xor(best_i[i], off);
            argmin_fold(best_d[i], best_i[i], od, oi);
        }
        if (tx == 0 && ty + i < nt) {
            const int64_t at = bg * part_stride +
                               static_cast<int64_t>(t0 + ty + i - lo.v[b]) * gridDim.y + blockIdx.y;
            part_d[at] = best_d[i];
            part_i[at] = best_i[i];
        }
    }
}

// encode_fine_kernel: 16 tokens x one subspace per workgroup, the subspace's
// codewords in LDS; 16 lanes share a token's codewords. Folds the token's nearest
// centroids of the coarse kernel's shares first (the first subspace's workgroups
// write the list ids).
template <typename T, typename PQ>
__global__ __launch_bounds__(kEncThreads) void encode_fine_kernel(
    Dims D, BatchInts lo, BatchInts hi, const T* __restrict__ kcache, int64_t sb, int64_t sh, int64_t sn,
    const float* __restrict__ centroids, const float* __restrict__ codebooks,
    const float* __restrict__ part_d, const int32_t* __restrict__ part_i, int64_t part_stride, int shares,
    const float* __restrict__ norms_tm, int32_t* __restrict__ ids_tm, uint8_t* __restrict__ codes_tm) {
    constexpr int K = PQ::K, DS = PQ::DSUB, kLd = DS + 1;   // odd row stride: lanes on distinct banks
    __shared__ float cb[K * kLd];
    __shared__ float res[kEncThreads / 16][DS];
    const int bg = blockIdx.z;
    const int b = bg / D.Hkv, g = bg % D.Hkv;
    const int m = blockIdx.y;
    const int t0 = lo.v[b] + static_cast<int>(blockIdx.x) * (kEncThreads / 16);
    if (t0 >= hi.v[b]) return;
    const int tl = threadIdx.x / 16;
    const int l16 = threadIdx.x % 16;
    const bool ok = t0 + tl < hi.v[b];
    const int t = ok ? t0 + tl : hi.v[b] - 1;
    const float* src = codebooks + (static_cast<int64_t>(bg) * PQ::M + m) * K * DS;
    for (int i = threadIdx.x; i < K * DS; i += kEncThreads) cb[i / DS * kLd + i % DS] = src[i];
    // the nearest centroid over the shares
    const int64_t at = bg * part_stride + static_cast<int64_t>(t - lo.v[b]) * shares;
    float bd = __builtin_huge_valf();
    int a = 0;
    for (int i = l16; i < shares; i += 16) argmin_fold(bd, a, part_d[at + i], part_i[at + i]);
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        const float od = __shfl_xor(bd, off);
        const int oi = __shfl_xor(a, off);
        argmin_fold(bd, a, od, oi);
    }
    const int64_t tok = static_cast<int64_t>(bg) * D.rcap + t;
    if (l16 < DS) {
        const int x = m * DS + l16;
        const float r = norms_tm[tok];
        const float k = load1<T>(kcache + b * sb + g * sh + static_cast<int64_t>(t) * sn + x);
        res[tl][l16] = (r > 0.0f ? k / r : 0.0f) - centroids[(static_cast<int64_t>(bg) * D.n_list + a) * kHeadDim + x];
    }
    __syncthreads();
    float ru[DS];
#pragma unroll
    for (int x = 0; x < DS; ++x) ru[x] = res[tl][x];
    float best = __builtin_huge_valf();
    int bz = 0;   // a valid id even if every distance is NaN
    for (int z = l16; z < K; z += 16) {
        float acc = 0.0f;
#pragma unroll
        for (int x = 0; x < DS; ++x) {
            const float dx = ru[x] - cb[z * kLd + x];
            acc = fmaf(dx, dx, acc);
        }
        argmin_fold(best, bz, acc, z);
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        const float od = __shfl_xor(best, off);
        const int oi = __shfl_xor(bz, off);
        argmin_fold(best, bz, od, oi);
    }
    if (ok && l16 == 0) {
        codes_tm[tok * PQ::M + m] = static_cast<uint8_t>(bz);
        if (m == 0) ids_tm[tok] = a;
    }
}

// One workgroup per (list j, kv head g, sequence b), one thread per dimension,
// after the merge: the list's new members are the last (new size - old size)
// positions of its new range, in token order.
template <typename T>
__global__ __launch_bounds__(kHeadDim) void means_update_kernel(
    Dims D, const T* __restrict__ vcache, int64_t sb, int64_t sh, int64_t sn,
    const int32_t* __restrict__ old_loff, const int32_t* __restrict__ new_loff,
    const int32_t* __restrict__ perm_new, float* __restrict__ means, double* __restrict__ sums) {
    const int j = blockIdx.x;
    const int g = blockIdx.y;
    const int b = blockIdx.z;
    const int bg = b * D.Hkv + g;
    const int64_t lo = static_cast<int64_t>(bg) * (D.n_list + 1) + j;
    const int n_old = old_loff[lo + 1] - old_loff[lo];
    const int end = new_loff[lo + 1];
    const int n_all = end - new_loff[lo];
    if (n_all == n_old) return;
    const int x = threadIdx.x;
    const int32_t* perm = perm_new + static_cast<int64_t>(bg) * D.rcap;
    const T* vb = vcache + b * sb + g * sh + x;
    const int64_t at = (static_cast<int64_t>(bg) * D.n_list + j) * kHeadDim + x;
    double s = sums[at];
    for (int p = end - (n_all - n_old); p < end; ++p)
        s += static_cast<double>(load1<T>(vb + static_cast<int64_t>(perm[p]) * sn));
    sums[at] = s;
    means[at] = static_cast<float>(s / static_cast<double>(n_all));
}

// The float64 value sums of the lists from the means of a prepared or built
// index: sum_j = |R_j| v_bar_j (0 for an empty list).
__global__ __launch_bounds__(kHeadDim) void init_sums_kernel(Dims D, const int32_t* __restrict__ loff,
                                                             const float* __restrict__ means,
                                                             double* __restrict__ sums) {
    const int j = blockIdx.x;
    const int bg = blockIdx.y;
    const int64_t lo = static_cast<int64_t>(bg) * (D.n_list + 1) + j;
    const int64_t at = (static_cast<int64_t>(bg) * D.n_list + j) * kHeadDim + threadIdx.x;
    sums[at] = static_cast<double>(loff[lo + 1] - loff[lo]) * static_cast<double>(means[at]);
}

hipError_t launch_init_sums(const Dims& D, const int32_t* loff, const float* means, double* sums,
                            hipStream_t s) {
    hipLaunchKernelGGL(init_sums_kernel, dim3(D.n_list, D.B * D.Hkv), dim3(kHeadDim), 0, s, D, loff,
                       means, sums);
    return hipGetLastError();
}

// List-major rebuild after an update, on the device. The new tokens of a
// (b, g) have larger ids than every indexed one, so each list keeps its old
// members in order and appends its new ones in increasing id: an old position
// p of list j moves to p + (new members of lists before j), and the r-th new
// member of list j lands at old_end(j) + (new members of lists before j) + r.
//
// update_lists_kernel: one workgroup per (b, g). Counts the new members per
// list (LDS atomics), scans the counts into the per-list shifts, writes the
// new list offsets, and places the new tokens chunk by chunk in id order
// (rank within a chunk = earlier lanes of the chunk with the same list).
constexpr int kListThreads = 1024;
constexpr int kScanPer = kMaxLists / kListThreads;   // list counts per thread in the scan

__global__ __launch_bounds__(kListThreads) void update_lists_kernel(
    Dims D, BatchInts lo, BatchInts hi, const int32_t* __restrict__ ids_tm,
    const int32_t* __restrict__ old_loff, int32_t* __restrict__ new_loff,
    int32_t* __restrict__ shift, int32_t* __restrict__ perm_new, uint32_t* __restrict__ pos_new,
    int32_t* __restrict__ n_r_dev, int32_t* __restrict__ n_seq_dev) {
    __shared__ int cnt[kMaxLists];     // new members per list, then the exclusive scan
    __shared__ int placed[kMaxLists];  // new members placed so far per list
    __shared__ int chunk[kListThreads];
    __shared__ int wtot[kListThreads / kWave];
    const int bg = blockIdx.x;
    const int b = bg / D.Hkv;
    const int tid = threadIdx.x;
    const int L = D.n_list;
    const int t0 = lo.v[b], t1 = hi.v[b];
    if (tid == 0 && bg % D.Hkv == 0) {
        n_r_dev[b] = t1 - D.n_sink;
        n_seq_dev[b] = t1 + D.n_local;
    }
    for (int j = tid; j < L; j += kListThreads) {
        cnt[j] = 0;
        placed[j] = 0;
    }
    __syncthreads();
    const int32_t* ids = ids_tm + static_cast<int64_t>(bg) * D.rcap;
    // list ids are clamped into [0, n_list): a prepare checks them separately
    // (check_ids_kernel) and fails the call, so an invalid id never indexes LDS
    auto list_of = [&](int t) { return min(max(ids[t], 0), L - 1); };
    for (int t = t0 + tid; t < t1; t += kListThreads) atomicAdd(&cnt[list_of(t)], 1);
    __syncthreads();
    lds_exclusive_scan<kListThreads, kScanPer>(cnt, L, wtot);
    const int32_t* ol = old_loff + static_cast<int64_t>(bg) * (L + 1);
    int32_t* nl = new_loff + static_cast<int64_t>(bg) * (L + 1);
    for (int j = tid; j <= L; j += kListThreads) nl[j] = ol[j] + (j < L ? cnt[j] : t1 - t0);
    for (int j = tid; j < L; j += kListThreads) shift[static_cast<int64_t>(bg) * L + j] = cnt[j];
    const int64_t row = static_cast<int64_t>(bg) * D.rcap;
    for (int c0 = t0; c0 < t1; c0 += kListThreads) {
        const int t = c0 + tid;
        const int j = t < t1 ? list_of(t) : -1;
        chunk[tid] = j;
        __syncthreads();
        if (t < t1) {
            int r = 0;
            for (int i = 0; i < tid; ++i) r += chunk[i] == j;
            const int pos = ol[j + 1] + cnt[j] + placed[j] + r;
            perm_new[row + pos] = t;
            pos_new[row + pos] = (static_cast<uint32_t>(j) << kPosBits) | static_cast<uint32_t>(t);
        }
        __syncthreads();
        if (t < t1) atomicAdd(&placed[j], 1);
        __syncthreads();
    }
}

// shift_positions_kernel: the old members move right by their list's shift;
// positions past the new |R_b| are cleared (perm -1).
__global__ __launch_bounds__(256) void shift_positions_kernel(
    Dims D, BatchInts lo, BatchInts hi, const int32_t* __restrict__ shift,
    const int32_t* __restrict__ perm_old, const uint32_t* __restrict__ pos_old,
    int32_t* __restrict__ perm_new, uint32_t* __restrict__ pos_new) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    const int bg = blockIdx.y;
    if (p >= D.rcap) return;
    const int b = bg / D.Hkv;
    const int old_nr = lo.v[b] - D.n_sink, new_nr = hi.v[b] - D.n_sink;
    const int64_t row = static_cast<int64_t>(bg) * D.rcap;
    if (p < old_nr) {
        const uint32_t w = pos_old[row + p];
        const int q = p + shift[static_cast<int64_t>(bg) * D.n_list + static_cast<int>(w >> kPosBits)];
        perm_new[row + q] = perm_old[row + p];
        pos_new[row + q] = w;
    } else if (p >= new_nr) {
        perm_new[row + p] = -1;
        pos_new[row + p] = 0u;
    }
}

// check_ids_kernel: the smallest flat index (b, g, token) of R whose list id
// lies outside [0, n_list), by atomicMin into `bad` (left at all ones when
// every id is valid).
__global__ __launch_bounds__(256) void check_ids_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                        const int32_t* __restrict__ ids_tm,
                                                        unsigned long long* bad) {
    const int bg = blockIdx.y;
    const int b = bg / D.Hkv;
    const int t = lo.v[b] + blockIdx.x * 256 + threadIdx.x;
    if (t >= hi.v[b]) return;
    const int64_t at = static_cast<int64_t>(bg) * D.rcap + t;
    const int32_t j = ids_tm[at];
    if (j < 0 || j >= D.n_list) atomicMin(bad, static_cast<unsigned long long>(at));
}

// finish_lists_kernel: after the grouping of R_b by list (perm, loff), the
// list word of every position and the cleared positions past |R_b|.
__global__ __launch_bounds__(256) void finish_lists_kernel(Dims D, BatchInts lo, BatchInts hi,
                                                           const int32_t* __restrict__ ids_tm,
                                                           int32_t* __restrict__ perm,
                                                           uint32_t* __restrict__ pos_word,
                                                           int32_t* __restrict__ n_r_dev,
                                                           int32_t* __restrict__ n_seq_dev) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    const int bg = blockIdx.y;
    const int b = bg / D.Hkv;
    if (p == 0 && bg % D.Hkv == 0) {
        n_r_dev[b] = hi.v[b] - D.n_sink;
        n_seq_dev[b] = hi.v[b] + D.n_local;
    }
    if (p >= D.rcap) return;
    const int64_t row = static_cast<int64_t>(bg) * D.rcap;
    if (p < hi.v[b] - lo.v[b]) {
        const int t = perm[row + p];
        const int j = min(max(ids_tm[row + t], 0), D.n_list - 1);
        pos_word[row + p] = (static_cast<uint32_t>(j) << kPosBits) | static_cast<uint32_t>(t);
    } else {
        perm[row + p] = -1;
        pos_word[row + p] = 0u;
    }
}

hipError_t launch_sort_lists(const Dims& D, const BatchInts& lo, const BatchInts& hi, int max_n,
                             const int32_t* ids_tm, const int32_t* zero_loff, int32_t* loff,
                             int32_t* shift, int32_t* perm, uint32_t* pos_word,
                             int32_t* n_r_dev, int32_t* n_seq_dev, unsigned long long* bad,
                             int32_t* scratch, size_t scratch_ints, hipStream_t s) {
    if (max_n > 0) {
        hipLaunchKernelGGL(check_ids_kernel, dim3((max_n + 255) / 256, D.B * D.Hkv), dim3(256), 0, s,
                           D, lo, hi, ids_tm, bad);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const size_t nseg = (static_cast<size_t>(max_n) + kBuildSegTok - 1) / kBuildSegTok;
    if (D.n_list <= 1024 && scratch &&
        nseg * static_cast<size_t>(D.B) * D.Hkv * D.n_list <= scratch_ints) {
        // the build's segmented grouping, many workgroups per (b, g)
        hipError_t e = launch_group_segments(D, lo, hi, ids_tm, scratch, perm, loff, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(finish_lists_kernel, dim3((D.rcap + 255) / 256, D.B * D.Hkv), dim3(256), 0, s,
                           D, lo, hi, ids_tm, perm, pos_word, n_r_dev, n_seq_dev);
        return hipGetLastError();
    }
    // a merge into an empty index: every token of R is new (old offsets all
    // zero, no old positions to move)
    hipLaunchKernelGGL(update_lists_kernel, dim3(D.B * D.Hkv), dim3(kListThreads), 0, s, D, lo, hi,
                       ids_tm, zero_loff, loff, shift, perm, pos_word, n_r_dev, n_seq_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // positions past |R_b| are cleared
    hipLaunchKernelGGL(shift_positions_kernel, dim3((D.rcap + 255) / 256, D.B * D.Hkv), dim3(256), 0,
                       s, D, lo, hi, shift, nullptr, nullptr, perm, pos_word);
    return hipGetLastError();
}

hipError_t launch_update_lists(const Dims& D, const BatchInts& lo, const BatchInts& hi,
                               const KV& kv, const int32_t* ids_tm, const int32_t* old_loff,
                               const int32_t* perm_old, const uint32_t* pos_old, int32_t* new_loff,
                               int32_t* shift, int32_t* perm_new, uint32_t* pos_new,
                               int32_t* n_r_dev, int32_t* n_seq_dev,
                               float* means, double* sums, hipStream_t s) {
    hipLaunchKernelGGL(update_lists_kernel, dim3(D.B * D.Hkv), dim3(kListThreads), 0, s, D, lo, hi,
                       ids_tm, old_loff, new_loff, shift, perm_new, pos_new, n_r_dev, n_seq_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(shift_positions_kernel, dim3((D.rcap + 255) / 256, D.B * D.Hkv), dim3(256), 0,
                       s, D, lo, hi, shift, perm_old, pos_old, perm_new, pos_new);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid(D.n_list, D.Hkv, D.B);
    if (kv.bf16)
        hipLaunchKernelGGL(means_update_kernel<bf16_t>, grid, dim3(kHeadDim), 0, s, D,
                           static_cast<const bf16_t*>(kv.v), kv.sb, kv.sh, kv.sn, old_loff, new_loff,
                           perm_new, means, sums);
    else
        hipLaunchKernelGGL(means_update_kernel<float>, grid, dim3(kHeadDim), 0, s, D,
                           static_cast<const float*>(kv.v), kv.sb, kv.sh, kv.sn, old_loff, new_loff,
                           perm_new, means, sums);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_encode_t(const Dims& D, const BatchInts& lo, const BatchInts& hi, int max_new,
                                  const KV& kv, const float* centroids, const float* codebooks,
                                  int32_t* ids_tm, uint8_t* codes_tm, float* norms_tm, float* part_d,
                                  int32_t* part_i, int64_t part_ints, hipStream_t s) {
    // shares of the centroids: about four workgroups per CU, one chunk of
    // centroids at least, and what the scratch holds per (b, kv head)
    const int bgs = D.B * D.Hkv;
    const int tiles = (max_new + kEncTok - 1) / kEncTok;
    const int chunks = (D.n_list + kEncCen - 1) / kEncCen;
    const int n_cu = device_cu_count() > 0 ? device_cu_count() : 1;
    int64_t shares = std::max<int64_t>(1, static_cast<int64_t>(4) * n_cu / (static_cast<int64_t>(tiles) * bgs));
    shares = std::min<int64_t>(std::min<int64_t>(shares, chunks), std::max<int64_t>(1, part_ints / bgs / max_new));
    const int64_t stride = shares * max_new;
    const T* k = static_cast<const T*>(kv.k);
    hipLaunchKernelGGL(encode_coarse_kernel<T>, dim3(tiles, static_cast<unsigned>(shares), bgs), dim3(kEncThreads),
                       0, s, D, lo, hi, k, kv.sb, kv.sh, kv.sn, centroids, part_d, part_i, stride, norms_tm);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int fine_tiles = (max_new + kEncThreads / 16 - 1) / (kEncThreads / 16);
#define PQHSA_FINE(PQT)                                                                                      \
    hipLaunchKernelGGL((encode_fine_kernel<T, PQT>), dim3(fine_tiles, PQT::M, bgs), dim3(kEncThreads), 0, s, \
                       D, lo, hi, k, kv.sb, kv.sh, kv.sn, centroids, codebooks, part_d, part_i, stride,      \
                       static_cast<int>(shares), norms_tm, ids_tm, codes_tm)
    if (D.pq_bits == 4) PQHSA_FINE(Pq4);
    else PQHSA_FINE(Pq8);
#undef PQHSA_FINE
    return hipGetLastError();
}

hipError_t launch_encode_update(const Dims& D, const BatchInts& lo, const BatchInts& hi,
                                int max_new, const KV& kv, const float* centroids,
                                const float* codebooks, int32_t* ids_tm, uint8_t* codes_tm,
                                float* norms_tm, float* part_d, int32_t* part_i, int64_t part_ints,
                                hipStream_t s) {
    if (max_new <= 0) return hipSuccess;
    return kv.bf16 ? launch_encode_t<bf16_t>(D, lo, hi, max_new, kv, centroids, codebooks, ids_tm, codes_tm,
                                             norms_tm, part_d, part_i, part_ints, s)
                   : launch_encode_t<float>(D, lo, hi, max_new, kv, centroids, codebooks, ids_tm, codes_tm,
                                            norms_tm, part_d, part_i, part_ints, s);
}

}  // namespace pqhsa
