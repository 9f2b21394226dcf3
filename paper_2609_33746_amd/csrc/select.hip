// Top-k selection (Section 3.2, Eq. 3): T = the k indexed tokens with the
// largest approximate logits, per (batch element, query head) row, ties to the
// smaller token id.
//
// One workgroup per row gathers the row's candidates (the tokens the scan
// found at or above the sampled threshold tau_lo, in list-major position
// order) into LDS, locates the k-th largest score with one histogram pass
// over monotone bins of the order keys, ranks the few candidates of the
// boundary bin exactly (score, then token id), writes T, and sums
// exp(l~ - shift) of the unselected candidates per list (in 64-bit fixed
// point, so the sums do not depend on the order of the atomic additions).
// If the threshold left fewer than k candidates (or none at all), the row is
// re-scanned in full from the LUT and every indexed token becomes a
// candidate; the below-threshold masses of the scan are then ignored for that
// row. Rows with more candidates than the LDS holds, or a very dense boundary
// bin, use a radix select instead. Every path gives the exact top-k.
//
// A thread loads the count of one region, each wave scans its own with DPP,
// candidate loads are issued in batches, and every workgroup-wide step is one
// scan or reduction, so the dependency chain stays short.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "hist_select.h"
#include "pq_score.h"
#include "pqhsa_internal.h"
#include "radix_select.h"

namespace pqhsa {

constexpr int kNW = kSelThreads / kWave;
constexpr int kRankCap = 128;
constexpr int kNzBits = 10;              // region bits of a nonempty-list entry
static_assert((1 << kNzBits) >= kSelMaxRegions, "region ids");
static_assert(kMaxSeq / kScanChunk <= kSelMaxRegions && kSelMaxRegions <= kSelThreads, "a region per thread");
constexpr float kMassScale = 1099511627776.0f;       // 2^40: fixed-point weights
constexpr float kMassUnscale = 1.0f / 1099511627776.0f;

// Bin of a key under bins fixed before the candidates are seen: keys from
// bkmin upward in steps of 2^bsh, everything above the last bin in it.
__device__ __forceinline__ uint32_t fixed_bin(uint32_t key, uint32_t bkmin, int bsh) {
    return key >= bkmin ? min((key - bkmin) >> bsh, static_cast<uint32_t>(kHistBins - 1)) : 0u;
}

// Rank the keys of one histogram bin exactly: key desc, then token id asc.
// The bin's keys are gathered into r_key / r_idx, then each wave ranks some of
// them against all the others with one ballot per 64 keys; token ids
// (tok_at) are read only when two keys of the bin are equal. Marks the `need`
// largest in the `chosen` bitmap and returns the need-th largest key in kth.
// Returns false without marking anything when the bin holds more than
// kRankCap keys. Must be called by the whole workgroup; flags[0] must be 0.
template <typename KeyAt, typename TokAt>
__device__ __forceinline__ bool rank_boundary_bin(KeyAt key_at, TokAt tok_at, int n, uint32_t kmin,
                                                  int sh, int bin, int m, int need, uint32_t* r_key,
                                                  int* r_idx, int* r_tok, int* counter, int* flags,
                                                  uint32_t* chosen, uint32_t& kth,
                                                  BlockScratch& bs) {
    if (m > kRankCap) return false;
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    for (int i0 = 0; i0 < n; i0 += kSelThreads) {
        const int i = i0 + tid;
        if (i < n) {
            const uint32_t kk = key_at(i);
            if (static_cast<int>(fixed_bin(kk, kmin, sh)) == bin) {
                const int slot = atomicAdd(counter, 1);
                r_key[slot] = kk;
                r_idx[slot] = i;
            }
        }
    }
    __syncthreads();
    // pass 1: rank by key alone, and look for equal keys
    for (int i = wave; i < m; i += kNW) {
        const uint32_t ki = r_key[i];
        int rank = 0;
        bool dup = false;
        for (int j0 = 0; j0 < m; j0 += kWave) {
            const int j = j0 + lane;
            const uint32_t kj = j < m ? r_key[j] : 0u;
            rank += __popcll(__ballot(j < m && kj > ki));
            dup |= __ballot(j < m && j != i && kj == ki) != 0ull;
        }
        if (dup) {
            if (lane == 0) flags[0] = 1;
        } else if (lane == 0 && rank < need) {
            const int idx = r_idx[i];
            atomicOr(&chosen[idx >> 5], 1u << (idx & 31));
            if (rank == need - 1) bs.bcast[2] = static_cast<int>(ki);
        }
    }
    __syncthreads();
    if (flags[0]) {
        // equal keys in the bin: rank again with the token ids
        if (tid < m) r_tok[tid] = tok_at(r_idx[tid]);
        __syncthreads();
        for (int i = wave; i < m; i += kNW) {
            const uint32_t ki = r_key[i];
            const int ti = r_tok[i];
            int rank = 0;
            bool dup = false;
            for (int j0 = 0; j0 < m; j0 += kWave) {
                const int j = j0 + lane;
                const uint32_t kj = j < m ? r_key[j] : 0u;
                const int tj = j < m ? r_tok[j] : 0;
                rank += __popcll(__ballot(j < m && (kj > ki || (kj == ki && tj < ti))));
                dup |= __ballot(j < m && j != i && kj == ki) != 0ull;
            }
            // keys that had no equal were marked by pass 1 already
            if (dup && lane == 0 && rank < need) {
                const int idx = r_idx[i];
                atomicOr(&chosen[idx >> 5], 1u << (idx & 31));
            }
            if (lane == 0 && rank == need - 1) bs.bcast[2] = static_cast<int>(ki);
        }
        __syncthreads();
    }
    kth = static_cast<uint32_t>(bs.bcast[2]);
    __syncthreads();
    return true;
}

// LDS layout of select_kernel (dynamic, 4-byte words), for kCap candidates:
//   keys [kCap] | cand [kCap] | hist [kHistBins] | rank_key [kRankCap] |
//   rank_idx [kRankCap] | rank_tok [kRankCap] | chosen bitmap [kCap / 32] |
//   counter, flags [4] | region offsets, or the nonempty regions, [kSelMaxRegions] |
//   mass (uint64) [n_list]
// The wide select keeps only the keys in LDS (the candidates' words go to
// global memory).
constexpr int kSelCapWide = 27648;
template <int kCap>
struct SelLayout {
    static constexpr bool kWide = kCap == kSelCapWide;
    static constexpr int kOffCand = kCap;
    static constexpr int kOffHist = kWide ? kCap : 2 * kCap;
    static constexpr int kOffRKey = kOffHist + kHistBins;
    static constexpr int kOffRIdx = kOffRKey + kRankCap;
    static constexpr int kOffRTok = kOffRIdx + kRankCap;
    static constexpr int kOffBits = kOffRTok + kRankCap;
    static constexpr int kOffCounter = kOffBits + kCap / 32;
    static constexpr int kOffRegion = kOffCounter + 4;
    static constexpr int kOffMass = (kOffRegion + kSelMaxRegions + 1) & ~1;   // 8-byte aligned
    static constexpr size_t bytes(int n_list) { return static_cast<size_t>(kOffMass + 2 * n_list) * 4; }
    static_assert(kCap % kSelThreads == 0 && kCap % 32 == 0, "whole copy tiers and bitmap words");
    static_assert(kOffCand % 4 == 0, "16-byte candidate stores");
    static_assert(kCap < (1 << (31 - kNzBits)), "first-candidate indices");
};
// Three capacities (select_cap below picks one per call): every row's
// candidates in LDS (one workgroup per CU); fewer (two workgroups per CU, for
// grids of more rows than CUs); and the wide one, keys alone, for rows likely to
// have more candidates than the first holds. Rows beyond the capacity take the
// global-memory path.
constexpr int kSelCapSmall = 7168;
constexpr size_t kLdsPerCu = 160 * 1024;
static_assert(SelLayout<kSelCapWide>::bytes(kMaxLists) + sizeof(SelectScratch) + sizeof(BlockScratch) <= kLdsPerCu,
              "the wide select fits a CU at the most lists");

// Read the candidates first + u kSelThreads + tid, u < N, of the row's
// `total` (>= 1) from their regions (one workgroup per CU):
// neighbouring lanes read neighbouring slots. Candidate i lives in the
// region c with pre[c] <= i < pre[c + 1] (the last of equal offsets, so
// empty regions never match). Every thread searches all of its indices
// together (top: half the power of two at or above nreg, 0 for one region) and
// issues all loads before using any, so the copy costs one search chain and one
// memory round trip (indices past the end repeat the last candidate's load).
template <int N>
__device__ __forceinline__ void read_candidates_search(const uint2* __restrict__ cand, const int* pre,
                                                       int nreg, int rshift, int top, int first, int total,
                                                       uint2 (&rec)[N]) {
    const int tid = threadIdx.x;
    // the N searches advance together, one step at a time, so their LDS
    // reads overlap instead of forming one long dependent chain
    int cs[N], ci[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        ci[u] = min(first + u * kSelThreads + tid, total - 1);
        cs[u] = 0;
    }
    for (int step = top; step > 0; step >>= 1) {
        int pv[N];
#pragma unroll
        for (int u = 0; u < N; ++u) pv[u] = pre[min(cs[u] + step, nreg - 1)];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int t = cs[u] + step;
            if (t < nreg && pv[u] <= ci[u]) cs[u] = t;
        }
    }
#pragma unroll
    for (int u = 0; u < N; ++u)   // slot in [0, count)
        rec[u] = cand[(static_cast<int64_t>(cs[u]) << rshift) + (ci[u] - pre[cs[u]])];
}

// Read the N consecutive candidates N tid + u, u < N. nzl lists the
// row's n_nz nonempty regions in position order, each as (index of its
// first candidate << kNzBits | region).
// One binary search over nzl finds the entry of the thread's first index, and
// since every listed region holds at least one candidate, index N tid + u
// lies at most u entries further, which one batch of N reads settles. All
// loads are issued before any is used, so the copy costs one search chain and
// one memory round trip (indices past the end repeat the last candidate's
// load).
template <int N>
__device__ __forceinline__ void read_candidates_runs(const uint2* __restrict__ cand, const int* nzl,
                                                     int n_nz, int rshift, int top, int total,
                                                     uint2 (&rec)[N]) {
    const int i0 = min(N * static_cast<int>(threadIdx.x), total - 1);
    int k = 0;   // the last entry whose first index is <= i0
    for (int step = top; step > 0; step >>= 1) {
        const int t = k + step;
        if (t < n_nz && (nzl[min(t, n_nz - 1)] >> kNzBits) <= i0) k = t;
    }
    int ent[N];   // entries k .. k + N - 1 (the last one repeated past the list)
#pragma unroll
    for (int v = 0; v < N; ++v) ent[v] = nzl[min(k + v, n_nz - 1)];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int i = min(N * static_cast<int>(threadIdx.x) + u, total - 1);
        int e = ent[0];
#pragma unroll
        for (int v = 1; v <= u && v < N; ++v)
            if ((ent[v] >> kNzBits) <= i) e = ent[v];
        const int c = e & ((1 << kNzBits) - 1);
        rec[u] = cand[(static_cast<int64_t>(c) << rshift) + (i - (e >> kNzBits))];
    }
}

// The copy of all candidates into LDS in position order: keys at lds[i], words
// (list << kPosBits | token) at lds[kOffCand + i], or for the wide select at
// words[i] in global memory. Tracks this thread's min / max key; with fixed bins
// (hist != nullptr), every candidate is also counted in hist at bin
// min((key - bkmin) >> bsh, kHistBins - 1), one LDS atomic per candidate (their
// bins are mostly distinct).
template <int N, int kCap>
__device__ __forceinline__ void copy_candidates_search(const uint2* __restrict__ cand, const int* pre,
                                                int nreg, int rshift, int top, int total, uint32_t* lds, int32_t* words,
                                                uint32_t& kmin, uint32_t& kmax, int* hist,
                                                uint32_t bkmin, int bsh) {
    using L = SelLayout<kCap>;
    uint2 rec[N];
    read_candidates_search<N>(cand, pre, nreg, rshift, top, 0, total, rec);
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int ci = u * kSelThreads + static_cast<int>(threadIdx.x);
        const uint32_t kk = float_key(__uint_as_float(rec[u].x));
        if (ci < total) {
            lds[ci] = kk;
            if constexpr (L::kWide) words[ci] = static_cast<int32_t>(rec[u].y);
            else lds[L::kOffCand + ci] = rec[u].y;
            kmin = min(kmin, kk);
            kmax = max(kmax, kk);
            if (hist) atomicAdd(&hist[fixed_bin(kk, bkmin, bsh)], 1);
        }
    }
}

template <int N, int kCap>
__device__ __forceinline__ void copy_candidates_runs(const uint2* __restrict__ cand, const int* nzl,
                                                int n_nz, int rshift, int top, int total, uint32_t* lds,
                                                uint32_t& kmin, uint32_t& kmax, int* hist,
                                                uint32_t bkmin, int bsh) {
    using L = SelLayout<kCap>;
    const int tid = threadIdx.x;
    uint2 rec[N];
    read_candidates_runs<N>(cand, nzl, n_nz, rshift, top, total, rec);
    uint32_t kk[N], cw[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        kk[u] = float_key(__uint_as_float(rec[u].x));
        cw[u] = rec[u].y;
    }
    // the thread's N slots (< N * kSelThreads <= the LDS capacity; slots past
    // total are never read), 16 bytes per store when N allows
    if constexpr (N % 4 == 0) {
#pragma unroll
        for (int u = 0; u < N; u += 4) {
            *reinterpret_cast<uint4*>(lds + N * tid + u) = make_uint4(kk[u], kk[u + 1], kk[u + 2], kk[u + 3]);
            *reinterpret_cast<uint4*>(lds + L::kOffCand + N * tid + u) =
                make_uint4(cw[u], cw[u + 1], cw[u + 2], cw[u + 3]);
        }
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            lds[N * tid + u] = kk[u];
            lds[L::kOffCand + N * tid + u] = cw[u];
        }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if (N * tid + u < total) {
            kmin = min(kmin, kk[u]);
            kmax = max(kmax, kk[u]);
            if (hist) atomicAdd(&hist[fixed_bin(kk[u], bkmin, bsh)], 1);
        }
    }
}

// Emit T as token ids in candidate order (each thread owns a contiguous
// range of candidate indices) and the per-list sums of exp(l~ - shift) over
// the unselected candidates (candidates are in list-major order, so a thread
// adds one partial per run of equal list ids).
// Variant Bx (Appendix B) in the top-k stage: the background value of list
// j is the mean of its unselected members, and its Eq. 4 term splits into
// W_j |R_j| v_bar_j minus W_j times the selected rows of the list, with
// W_j = M_j / |B n R_j|. The row forms W_j here, from the same masses as the
// background role (the scan's below-threshold segments of the list, scaled to
// the row's shift, plus its unselected candidates), and hands every entry of
// T its list's W_j. Thread t owns lists t + u * kSelThreads; their offsets are
// loaded when the row starts where one workgroup holds a CU (with two, the
// registers they would take cost the second workgroup its place), else with
// the masses.
constexpr int kBxPer = kMaxLists / kSelThreads;
static_assert(kMaxLists % kSelThreads == 0, "whole list strides");
struct BxRow {
    int lo[kBxPer], hi[kBxPer];   // the thread's lists in the list-major order (preloaded)
    const int32_t* loff;          // list starts of this head
    const float* segs;            // below-threshold masses of this head, stride G
    int seg_stride;
    float tlo;                    // the row's threshold tau_lo
    bool rescan;                  // the row took the re-scan path (no below-threshold masses)
    float* bx_w;                  // [n_list] W_j of the row
    float* bx_wsel;               // [max_topk] W of the list of each entry of T
};

// kBatch candidates' keys and words are read at once: 1 where both sit in LDS,
// 4 where they come from global memory (each read then waits for a round trip
// of its own, which the stores between them keep the compiler from overlapping).
template <bool kBx, bool kBxPre, int kBatch, typename KeyAt, typename CandAt, typename IsSel>
__device__ __forceinline__ void emit_selection(KeyAt key_at, CandAt cand_at, IsSel is_sel,
                                               int total, int k, int n_list,
                                               float shift, unsigned long long* mass,
                                               int32_t* sel_tok, float* cand_mass,
                                               const BxRow& bx, SelectScratch& ss) {
    const int tid = threadIdx.x;
    const int eper = (total + kSelThreads - 1) / kSelThreads;
    const int e0 = min(tid * eper, total);
    const int e1 = min(e0 + eper, total);
    // every candidate of the thread in order, kBatch read ahead
    auto each = [&](auto&& f) {
        for (int i0 = e0; i0 < e1; i0 += kBatch) {
            uint32_t kb[kBatch], cb[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                kb[u] = key_at(min(i0 + u, e1 - 1));
                cb[u] = cand_at(min(i0 + u, e1 - 1));
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (kBatch == 1 || i0 + u < e1) f(i0 + u, kb[u], cb[u]);
        }
    };
    int nsel = 0;
    each([&](int i, uint32_t key, uint32_t cand) { nsel += is_sel(i, key, cand) ? 1 : 0; });
    int tot = 0;
    int o = block_excl_scan<kSelThreads, false>(nsel, tot, ss);   // ss is not written before the barrier below
    const int o_first = o;
    int run_list = -1;
    unsigned long long run = 0ull;
    each([&](int i, uint32_t key, uint32_t cand) {
        const int lst = static_cast<int>(cand >> kPosBits);
        if (lst != run_list) {
            if (run) atomicAdd(&mass[run_list], run);
            run = 0ull;
            run_list = lst;
        }
        if (is_sel(i, key, cand)) {
            if (o < k) sel_tok[o] = static_cast<int32_t>(cand & kPosMask);
            ++o;
        } else {
            run += static_cast<unsigned long long>(__expf(key_float(key) - shift) * kMassScale);
        }
    });
    if (run) atomicAdd(&mass[run_list], run);
    __syncthreads();
    if constexpr (!kBx) {
        for (int j = tid; j < n_list; j += kSelThreads)
            cand_mass[j] = static_cast<float>(mass[j]) * kMassUnscale;
    } else {
        const float neg_inf = -__builtin_huge_valf();
        const bool live = shift != neg_inf;
        const bool use_below = live && bx.tlo != neg_inf && !bx.rescan;
        const float below_scale = use_below ? __expf(bx.tlo - shift) : 0.0f;
        float mj[kBxPer];
        int sz[kBxPer];
#pragma unroll
        for (int u = 0; u < kBxPer; ++u) {
            const int j = tid + u * kSelThreads;
            mj[u] = 0.0f;
            sz[u] = 0;
            if (j < n_list) {
                const float cm = static_cast<float>(mass[j]) * kMassUnscale;
                cand_mass[j] = cm;
                float below = 0.0f;
                const int lo = kBxPre ? bx.lo[u] : bx.loff[j];
                const int hi = kBxPre ? bx.hi[u] : bx.loff[j + 1];
                sz[u] = hi - lo;
                if (use_below && hi > lo)
                    for (int sg = j + lo / kSub; sg <= j + (hi - 1) / kSub; ++sg)
                        below += bx.segs[sg * bx.seg_stride];
                mj[u] = live ? below * below_scale + cm : 0.0f;
            }
        }
        // the masses are read: their words now hold |T n R_j| and then W_j
        __syncthreads();
        int* cnt = reinterpret_cast<int*>(mass);
        float* wl = reinterpret_cast<float*>(mass) + n_list;
        for (int j = tid; j < n_list; j += kSelThreads) cnt[j] = 0;
        __syncthreads();
        o = o_first;
        each([&](int i, uint32_t key, uint32_t cand) {
            if (is_sel(i, key, cand)) {
                if (o < k) atomicAdd(&cnt[cand >> kPosBits], 1);
                ++o;
            }
        });
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kBxPer; ++u) {
            const int j = tid + u * kSelThreads;
            if (j < n_list) {
                const int un = sz[u] - cnt[j];
                const float W = un > 0 ? mj[u] / static_cast<float>(un) : 0.0f;
                wl[j] = W;
                bx.bx_w[j] = W;
            }
        }
        __syncthreads();
        o = o_first;
        each([&](int i, uint32_t key, uint32_t cand) {
            if (is_sel(i, key, cand)) {
                if (o < k) bx.bx_wsel[o] = wl[cand >> kPosBits];
                ++o;
            }
        });
    }
}

// Score every indexed token of a row again from its head's LUT (the re-scan
// path): keys and words into comp_key / comp_pos in position order.
template <typename PQ>
__device__ __forceinline__ void rescan_row(const Dims& D, const Index& ix, const Work& w,
                                           float* lut_s, int bg, int hh, int n_r, int64_t base,
                                           int64_t rbase) {
    stage_head_lut<PQ, kSelThreads>(lut_s, w.lut + static_cast<int64_t>(bg) * PQ::LUT_ROW * D.G,
                                    D.G, hh);
    __syncthreads();
    const typename PQ::Code* codes = reinterpret_cast<const typename PQ::Code*>(ix.codes) + base;
    const float* coarse = w.coarse + static_cast<int64_t>(bg) * D.n_list * D.G;
    for (int pos = threadIdx.x; pos < n_r; pos += kSelThreads) {
        const uint32_t wd = ix.pos_word[base + pos];
        const int j = static_cast<int>(wd >> kPosBits);
        float fs[1];
        fine_sum<PQ, 1>(lut_s, codes[pos], fs);
        const float sc = pq_logit(ix.norms[base + pos], coarse[j * D.G + hh], fs[0]);
        w.comp_key[rbase + pos] = float_key(sc);
        w.comp_pos[rbase + pos] = static_cast<int32_t>(wd);
    }
}

template <bool kDev, int kCap, bool kBx>
__device__ __forceinline__ void select_row(const Dims& D, const BatchArgs& ba, const Index& ix,
                                           const Work& w, int force_fallback) {
    using L = SelLayout<kCap>;
    constexpr int kOffCand = L::kOffCand;
    extern __shared__ uint32_t lds[];
    unsigned long long* mass = reinterpret_cast<unsigned long long*>(lds + L::kOffMass);
    int* hist = reinterpret_cast<int*>(lds + L::kOffHist);
    uint32_t* r_key = lds + L::kOffRKey;
    int* r_idx = reinterpret_cast<int*>(lds + L::kOffRIdx);
    int* r_tok = reinterpret_cast<int*>(lds + L::kOffRTok);
    uint32_t* chosen = lds + L::kOffBits;
    int* counter = reinterpret_cast<int*>(lds + L::kOffCounter);
    // the copy by nonempty regions where two workgroups share a CU (1.2 us
    // faster at 512 rows), by a search of every index over the region
    // offsets with one workgroup per CU (0.4 us faster at 32 rows: its loads
    // of neighbouring lanes touch neighbouring slots)
    constexpr bool kWide = L::kWide;
    constexpr bool kRunsCopy = kCap == kSelCapSmall;
    int* regl = reinterpret_cast<int*>(lds + L::kOffRegion);
    __shared__ SelectScratch ss;
    __shared__ BlockScratch bs;
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = tid / kWave;
    const int row = blockIdx.x;
    const int b = row / D.Hq;
    const int h = row % D.Hq;
    const int g = h / D.G;
    const int hh = h % D.G;
    const int bg = b * D.Hkv + g;
    const int n_r = arg_n_r<kDev>(ba, w, b);
    const int k = arg_topk<kDev>(ba, w, b);
    const int rshift = w.region_shift;
    const int nreg = (n_r + (1 << rshift) - 1) >> rshift;   // <= kSelMaxRegions (scan_region_shift)
    const int64_t rbase = static_cast<int64_t>(row) * D.rcap;
    const int64_t base = static_cast<int64_t>(bg) * D.rcap;
    int32_t* sel_tok = w.sel_tok + static_cast<int64_t>(row) * D.max_topk;
    float* cand_mass = w.cand_mass + static_cast<int64_t>(row) * D.n_list;
    const float neg_inf = -__builtin_huge_valf();

    for (int j = tid; j < D.n_list; j += kSelThreads) mass[j] = 0ull;
    for (int i = tid; i < kHistBins; i += kSelThreads) hist[i] = 0;
    for (int i = tid; i < kCap / 32; i += kSelThreads) chosen[i] = 0u;
    if (tid < 4) counter[tid] = 0;   // counter[1] is the equal-key flag of the rank
    BxRow bx{};
    constexpr bool kBxPre = kCap == kSelCap;
    if constexpr (kBx) {
        bx.loff = ix.loff + static_cast<int64_t>(bg) * (D.n_list + 1);
        if constexpr (kBxPre) {
#pragma unroll
            for (int u = 0; u < kBxPer; ++u) {
                const int j = tid + u * kSelThreads;
                bx.lo[u] = j < D.n_list ? bx.loff[j] : 0;
                bx.hi[u] = j < D.n_list ? bx.loff[j + 1] : 0;
            }
        }
        bx.segs = w.seg_sum + static_cast<int64_t>(bg) * D.nseg_cap * D.G + hh;
        bx.seg_stride = D.G;
        bx.tlo = w.tau_lo[row];
        bx.bx_w = w.bx_w + static_cast<int64_t>(row) * D.n_list;
        bx.bx_wsel = w.bx_wsel + static_cast<int64_t>(row) * D.max_topk;
    }

    // 1) candidate counts, a region per thread
    const int c = tid < nreg ? w.cand_cnt[static_cast<int64_t>(row) * D.nsub_cap + tid] : 0;
    const int top = nreg > 1 ? 1 << (31 - __clz(nreg - 1)) : 0;   // the searches' first step
    int total = 0;
    int n_nz = 0;   // nonempty regions of the row
    {
        int incl = wave_incl_scan_i32(c);
        const uint64_t nzm = kRunsCopy ? __builtin_amdgcn_ballot_w64(c > 0) : 0ull;
        if (lane == kWave - 1) {
            ss.wave_tot[wave] = incl;
            ss.wave_aux[wave] = __popcll(nzm);
        }
        __syncthreads();
        constexpr int kCntWaves = kSelMaxRegions / kWave;   // the waves that hold counts
        int nzbase = 0, wbase = 0;
#pragma unroll
        for (int i = 0; i < kCntWaves; ++i) {
            const int t = ss.wave_tot[i];
            const int z = ss.wave_aux[i];
            wbase += i < wave ? t : 0;
            nzbase += i < wave ? z : 0;
            total += t;
            n_nz += z;
        }
        const int first = incl + wbase - c;   // row-wide index of the region's first candidate
        if constexpr (kRunsCopy) {
            // used while the indices fit beside the region bits (rows of more
            // candidates take the global-memory path)
            if (c > 0) regl[nzbase + lanes_below(nzm)] = (min(first, kCap) << kNzBits) | tid;
        } else {
            if (tid < nreg) regl[tid] = first;
        }
        __syncthreads();
    }
    const bool fallback = force_fallback || (n_r > 0 && total < (k > 0 ? k : 1));
    bx.rescan = fallback;
    float shift = neg_inf;

    if (!fallback && total <= kCap) {
        // ---- fast path: candidates in LDS, position order ----
        int32_t* words = w.comp_pos + rbase;   // the wide select's candidate words
        constexpr int kBatch = kWide ? 4 : 1;
        auto KEY = [&](int i) { return lds[i]; };
        auto CAND = [&](int i) {
            if constexpr (kWide) return static_cast<uint32_t>(words[i]);
            else return lds[kOffCand + i];
        };
        uint32_t kmin = 0xffffffffu, kmax = 0u, kcount = 0u;
        const uint2* cand = w.cand + rbase;
        // Bins fixed in advance from the sampled range [tau_lo, tau_hi] (every
        // candidate is >= tau_lo; those above tau_hi share the last bin), so
        // the histogram is built during the copy; otherwise from the
        // candidates' own min / max in a second pass.
        const float tlo = w.tau_lo[row], thi = w.tau_hi[row];
        const bool fixed = k > 0 && tlo > neg_inf && thi > tlo && thi < -neg_inf;
        uint32_t bkmin = fixed ? float_key(tlo) : 0u;
        int bsh = fixed ? bin_shift(bkmin, float_key(thi)) : 0;
        int* fh = fixed ? hist : nullptr;
        constexpr int kMid = kWide ? 16 : kCap / kSelThreads > 8 ? 8 : kCap / kSelThreads;
        constexpr int kLow = kWide ? 8 : 4;
        auto copy = [&](auto tier) {
            constexpr int N = decltype(tier)::value;
            if constexpr (kRunsCopy)
                copy_candidates_runs<N, kCap>(cand, regl, n_nz, rshift, top, total, lds, kmin, kmax, fh, bkmin, bsh);
            else
                copy_candidates_search<N, kCap>(cand, regl, nreg, rshift, top, total, lds, words, kmin, kmax, fh,
                                                bkmin, bsh);
        };
        if (total > kMid * kSelThreads)
            copy(std::integral_constant<int, kCap / kSelThreads>{});
        else if (total > kLow * kSelThreads)
            copy(std::integral_constant<int, kMid>{});
        else if (total > 0)
            copy(std::integral_constant<int, kLow>{});
        if (!fixed) block_min_max_count<kSelThreads>(kmin, kmax, kcount, bs);
        auto TOK = [&](int i) { return static_cast<int>(CAND(i) & kPosMask); };
        if (k == 0) {
            shift = total > 0 ? key_float(kmax) : neg_inf;
            emit_selection<kBx, kBxPre, kBatch>(
                KEY, CAND, [](int, uint32_t, uint32_t) { return false; }, total, 0, D.n_list, shift,
                mass, sel_tok, cand_mass, bx, ss);
        } else {
            if (!fixed) {
                bkmin = kmin;
                bsh = bin_shift(kmin, kmax);
                for (int i0 = 0; i0 < total; i0 += kSelThreads) {
                    const int i = i0 + tid;
                    const bool act = i < total;
                    if (act) atomicAdd(&hist[fixed_bin(KEY(i), bkmin, bsh)], 1);
                }
            }
            __syncthreads();
            // one wave finds the boundary bin and broadcasts it
            if (tid < kWave) {
                int ab = 0;
                const int bin = wave_find_bin_desc(hist, k, ab);
                if (tid == 0) {
                    bs.bcast[0] = bin;
                    bs.bcast[1] = ab;
                }
            }
            __syncthreads();
            const int bstar = bs.bcast[0];
            const int above = bs.bcast[1];
            uint32_t kth = 0u;
            const bool by_rank = rank_boundary_bin(KEY, TOK, total, bkmin, bsh, bstar, hist[bstar],
                                                   k - above, r_key, r_idx, r_tok, counter,
                                                   counter + 1, chosen, kth, bs);
            if (by_rank) {
                shift = key_float(kth);   // the k-th largest score
                emit_selection<kBx, kBxPre, kBatch>(
                    KEY, CAND,
                    [&](int i, uint32_t key, uint32_t) {
                        const int bn = static_cast<int>(fixed_bin(key, bkmin, bsh));
                        return bn > bstar || (bn == bstar && ((chosen[i >> 5] >> (i & 31)) & 1u));
                    },
                    total, k, D.n_list, shift, mass, sel_tok, cand_mass, bx, ss);
            } else {
                // very dense boundary bin: radix select
                const SelectResult r = block_select_desc<kSelThreads>(
                    KEY, [](int) { return true; }, total, k, ss);
                const uint32_t kk = r.key;
                const int need_r = k - r.count_above;
                int tok_cut = 0x7fffffff;
                if (r.count_equal > need_r) {
                    const SelectResult t = block_select_desc<kSelThreads>(
                        [&](int i) { return ~static_cast<uint32_t>(TOK(i)); },
                        [&](int i) { return KEY(i) == kk; }, total, need_r, ss);
                    tok_cut = static_cast<int>(~t.key);
                }
                shift = key_float(kk);
                emit_selection<kBx, kBxPre, kBatch>(
                    KEY, CAND,
                    [&](int, uint32_t key, uint32_t cw) {
                        return key > kk || (key == kk && static_cast<int>(cw & kPosMask) <= tok_cut);
                    },
                    total, k, D.n_list, shift, mass, sel_tok, cand_mass, bx, ss);
            }
        }
    } else {
        // ---- slow path: candidates in global memory (many, or the re-scan) ----
        if (!fallback) {
            // a batch of kSlowBatch candidates per thread and round trip, found
            // over the regions' first indices
            constexpr int kSlowBatch = 8;
            if constexpr (kRunsCopy) {
                // these are not the (clamped) entries of the nonempty regions
                __syncthreads();
                int first = wave_incl_scan_i32(c) - c;
                for (int i = 0; i < wave; ++i) first += ss.wave_tot[i];
                if (tid < nreg) regl[tid] = first;
                __syncthreads();
            }
            const uint2* __restrict__ src = w.cand + rbase;
            uint32_t* __restrict__ okey = w.comp_key + rbase;
            int32_t* __restrict__ oword = w.comp_pos + rbase;
            for (int first = 0; first < total; first += kSlowBatch * kSelThreads) {
                uint2 rec[kSlowBatch];
                read_candidates_search<kSlowBatch>(src, regl, nreg, rshift, top, first, total, rec);
#pragma unroll
                for (int u = 0; u < kSlowBatch; ++u) {
                    const int i = first + u * kSelThreads + tid;
                    if (i < total) {
                        okey[i] = float_key(__uint_as_float(rec[u].x));
                        oword[i] = static_cast<int32_t>(rec[u].y);
                    }
                }
            }
        } else {
            float* lut_s = reinterpret_cast<float*>(lds);   // at most 16 KB of the key area
            if (D.pq_bits == 4)
                rescan_row<Pq4>(D, ix, w, lut_s, bg, hh, n_r, base, rbase);
            else
                rescan_row<Pq8>(D, ix, w, lut_s, bg, hh, n_r, base, rbase);
            total = n_r;
        }
        __syncthreads();
        const uint32_t* ckey = w.comp_key + rbase;
        const uint32_t* ccand = reinterpret_cast<const uint32_t*>(w.comp_pos + rbase);
        auto KEY = [&](int i) { return ckey[i]; };
        auto CAND = [&](int i) { return ccand[i]; };
        if (total == 0) {
            shift = neg_inf;
            emit_selection<kBx, kBxPre, 4>(KEY, CAND, [](int, uint32_t, uint32_t) { return false; }, 0, 0,
                           D.n_list, shift, mass, sel_tok, cand_mass, bx, ss);
        } else {
            const SelectResult r = block_select_desc<kSelThreads>(
                KEY, [](int) { return true; }, total, k > 0 ? k : 1, ss);
            const uint32_t kth = k > 0 ? r.key : 0xffffffffu;
            int tok_cut = 0x7fffffff;
            if (k > 0 && r.count_equal > k - r.count_above) {
                const SelectResult t = block_select_desc<kSelThreads>(
                    [&](int i) { return ~(ccand[i] & kPosMask); },
                    [&](int i) { return ckey[i] == kth; }, total, k - r.count_above, ss);
                tok_cut = static_cast<int>(~t.key);
            }
            shift = key_float(r.key);   // k-th largest, or the maximum when k = 0
            emit_selection<kBx, kBxPre, 4>(
                KEY, CAND,
                [&](int, uint32_t key, uint32_t cand) {
                    return k > 0 && (key > kth || (key == kth && static_cast<int>(cand & kPosMask) <= tok_cut));
                },
                total, k, D.n_list, shift, mass, sel_tok, cand_mass, bx, ss);
        }
    }
    if (tid == 0) {
        w.row_shift[row] = shift;
        w.row_flag[row] = fallback ? 1 : 0;
    }
}

template <bool kDev, bool kBx>
__global__ __launch_bounds__(kSelThreads) void select_kernel(Dims D, BatchArgs ba, Index ix, Work w,
                                                             int force_fallback) {
    select_row<kDev, kSelCap, kBx>(D, ba, ix, w, force_fallback);
}

// Two of these share a CU only when each wave holds at most 80 SGPRs (the
// few beyond that spill to VGPR lanes).
template <bool kDev, bool kBx>
__global__ __launch_bounds__(kSelThreads) __attribute__((amdgpu_num_sgpr(80))) void select_small_kernel(
    Dims D, BatchArgs ba, Index ix, Work w, int force_fallback) {
    select_row<kDev, kSelCapSmall, kBx>(D, ba, ix, w, force_fallback);
}

template <bool kDev, bool kBx>
__global__ __launch_bounds__(kSelThreads) void select_wide_kernel(Dims D, BatchArgs ba, Index ix, Work w,
                                                                  int force_fallback) {
    select_row<kDev, kSelCapWide, kBx>(D, ba, ix, w, force_fallback);
}

// Candidates the sampled threshold is likely to leave, at most, for a row of
// n_r tokens and budget k: its rank c among the samples (see the prologue) in
// tokens, and 2.2 / sqrt(c) more for the spread of a sample's c-th largest. In
// units of that spread, the capacity that the rows of a call still fit lies
// between 1.9 and 2.3 above the rank: 32 to 288 rows of 64K to 512K tokens take
// fewer us with a capacity 2.3 above it (two workgroups per CU, 288 rows of
// 128K, 2%: 203 against 213 with one; one plain row set of 128K, 3.75%: 66 against
// 70 with the wide one) and more with one 1.9 above it (288 rows of 200K, 1.25%:
// 205 against 192; 32 rows of 512K, 0.7%: 81 against 76), where a row or two
// takes the global-memory path.
static int expected_candidates(int n_r, int k) {
    if (n_r <= 0) return 0;
    const SampleRuns sr = sample_runs(n_r);
    const double ns = static_cast<double>(sr.nrun) * sr.run_len;
    const double c = 2.0 * k * ns / n_r + 8.0;
    if (c > ns) return n_r;   // no threshold: every token
    return static_cast<int>(std::min<double>(n_r, (1.0 + 2.2 / std::sqrt(c)) * c * n_r / ns));
}

// The capacity of a call's select, by the row likely to have the most candidates:
//  * wide when that is more than the plain one holds: such rows took the
//    global-memory path (one sequence of 512K tokens, 1%: the select 189 -> 28 us);
//  * small when the rows outnumber the CUs, two of its workgroups fit in one
//    CU's LDS and that many candidates fit it.
// Budgets that are device data are unknown here, and the context's largest may
// be far above the step's: up to 1/64 of the tokens is provided for (rows of
// more take the global-memory path).
static int select_cap(const Dims& D, const int32_t* n_r, const int32_t* topk, bool dev_args) {
    int c_max = 0;
    for (int b = 0; b < D.B; ++b) {
        const int k = dev_args ? std::min(D.max_topk, n_r[b] / 64) : topk[b];
        c_max = std::max(c_max, expected_candidates(n_r[b], k));
    }
    if (c_max > kSelCap) return kSelCapWide;
    const int n_cu = device_cu_count();
    constexpr size_t kStatic = sizeof(SelectScratch) + sizeof(BlockScratch);
    if (n_cu > 0 && D.B * D.Hq > n_cu && c_max <= kSelCapSmall &&
        2 * (SelLayout<kSelCapSmall>::bytes(D.n_list) + kStatic) <= kLdsPerCu)
        return kSelCapSmall;
    return kSelCap;
}

// The tests' view of that rule: the capacity a call would take.
extern "C" int pqhsa_select_capacity(int batch, int n_q_heads, int n_list, int max_topk, const int32_t* n_r,
                                     const int32_t* topk, int dev_args) {
    Dims D{};
    D.B = batch;
    D.Hq = n_q_heads;
    D.n_list = n_list;
    D.max_topk = max_topk;
    return select_cap(D, n_r, topk, dev_args != 0);
}

template <bool kDev, bool kBx>
static void launch_select_d(const Dims& D, const BatchArgs& ba, const Index& ix, const Work& w,
                            int force_fallback, hipStream_t s, const KTiming& tm) {
    const dim3 grid(D.B * D.Hq), block(kSelThreads);
    switch (select_cap(D, ba.n_r, ba.topk, kDev)) {
        case kSelCapSmall:
            hipExtLaunchKernelGGL((select_small_kernel<kDev, kBx>), grid, block,
                                  SelLayout<kSelCapSmall>::bytes(D.n_list), s, tm.start, tm.stop, 0, D, ba,
                                  ix, w, force_fallback);
            break;
        case kSelCapWide:
            hipExtLaunchKernelGGL((select_wide_kernel<kDev, kBx>), grid, block,
                                  SelLayout<kSelCapWide>::bytes(D.n_list), s, tm.start, tm.stop, 0, D, ba,
                                  ix, w, force_fallback);
            break;
        default:
            hipExtLaunchKernelGGL((select_kernel<kDev, kBx>), grid, block, SelLayout<kSelCap>::bytes(D.n_list),
                                  s, tm.start, tm.stop, 0, D, ba, ix, w, force_fallback);
    }
}

hipError_t launch_select(const Dims& D, const BatchArgs& ba, const Index& ix, const Work& w,
                         int force_fallback, bool bx, hipStream_t s, const KTiming& tm) {
    if (w.ba_dev && bx)
        launch_select_d<true, true>(D, ba, ix, w, force_fallback, s, tm);
    else if (w.ba_dev)
        launch_select_d<true, false>(D, ba, ix, w, force_fallback, s, tm);
    else if (bx)
        launch_select_d<false, true>(D, ba, ix, w, force_fallback, s, tm);
    else
        launch_select_d<false, false>(D, ba, ix, w, force_fallback, s, tm);
    return hipGetLastError();
}

template <bool kDev, bool kBx>
static hipError_t configure_select_d() {
    const struct { const void* kernel; size_t bytes; } k[] = {
        {reinterpret_cast<const void*>(&select_kernel<kDev, kBx>), SelLayout<kSelCap>::bytes(kMaxLists)},
        {reinterpret_cast<const void*>(&select_small_kernel<kDev, kBx>), SelLayout<kSelCapSmall>::bytes(kMaxLists)},
        {reinterpret_cast<const void*>(&select_wide_kernel<kDev, kBx>), SelLayout<kSelCapWide>::bytes(kMaxLists)}};
    for (const auto& e : k) {
        const hipError_t r = hipFuncSetAttribute(e.kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(e.bytes));
        if (r != hipSuccess) return r;
    }
    return hipSuccess;
}

hipError_t configure_select() {
    hipError_t e = configure_select_d<false, false>();
    if (e == hipSuccess) e = configure_select_d<true, false>();
    if (e == hipSuccess) e = configure_select_d<false, true>();
    if (e == hipSuccess) e = configure_select_d<true, true>();
    return e;
}

}  // namespace pqhsa
