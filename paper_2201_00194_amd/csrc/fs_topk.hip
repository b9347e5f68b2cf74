// Per-family top-k: the k programs with the largest score, ordered by (score descending,
// index ascending) -- the cut that decides which candidates go on to measurement
// (Section 3.2 of the paper: sort by the estimate, keep the top k; Algorithm 1: k = g).
//
// Scores are mapped to unsigned keys whose integer order is the wanted order (-0 and +0
// share a key, NaN gets the lowest key).  One workgroup serves one request:
//   1. radix select (passes of 11, 11 and 10 bits, histogram in LDS) finds the key of the k-th
//      best entry and how many entries that tie with it still fit.  As soon as no more than
//      kRankMost entries can be among the best, each of these counts those above it and so knows
//      its place: steps 2 and 3 fall away (usually after the first pass);
//   2. every wavefront owns a contiguous slice of the scores; it counts the entries above
//      that key and the ties in its slice, the counts are scanned, and a second sweep places
//      every entry above the key plus the lowest-index ties as 64-bit composites
//      (key, ~index) in LDS;
//   3. the composites are sorted: runs of 64 by counting, then merges of two runs in which each
//      entry finds its place by bisection; all composites differ, so the result is unique.
// A long request (8192 entries, with small cuts 16384) is cut into up to 16 slices, one workgroup each, which
// leave their best k composites in scratch, best first; a second kernel merges the slices'
// lists pairwise in LDS, keeping the best k of every pair, and writes the answer.  The union
// of the slices' best k holds the request's best k, and composites order the same way
// everywhere, so nothing changes in the result.  Cuts wider than 4096 do not fit that merge:
// they are cut into slices of about 2048 entries (up to 128) whose sorted lists are merged
// eight at a time in global memory, level by level, each merge keeping the best k.
#include <algorithm>
#include <cstring>
#include <mutex>

#include "fs_internal.h"

namespace fs {

constexpr int kTopkThreads = 1024;

__device__ __forceinline__ uint32_t score_key(float s)
{
    if (s != s)
        return 0u;             // NaN: below every number
    s = s + 0.0f;              // -0 -> +0
    const uint32_t b = __float_as_uint(s);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

constexpr int kTopkWaves = kTopkThreads / 64;
// Entries a thread holds, all loads in flight at once: 16 where a workgroup has more than 8192 entries, as their keys are
// read once then (262 144 entries in 16 slices, cut of 64: 27.5 us with 8, so 17.5; cut of 1024 53.5 and 49.1), else 8.
// (A request alone whose cut falls among equal scores is the one that slices served better: all passes and sweeps over all
// entries are one workgroup's then.  16 of 16 384: random scores 11.2 us in slices and 7.9 whole, a tenth ones
// among zeros 12.1 and 18.6, seven values 16.1 and 19.9, all equal 17.8 and 18.2; 300 such requests of 64 79.6 and
// 29.2, 99 and 52 for seven values.  A wavefront's most frequent digit counted by ballots does not help: 18.6 -> 22.6,
// random 7.9 -> 9.5.)
constexpr int kTopkFew = 8, kTopkMany = kTopkAtOnce / kTopkThreads;

// Scores and keys of U consecutive 64-element pieces starting at `base`, this lane's element of
// each; pieces past `end` read a clamped address and are flagged invalid by the caller.
template <int U>
__device__ __forceinline__ void load_keys(const float *__restrict__ score, int base, int end,
                                          int lane, uint32_t (&key)[U], float (&v)[U])
{
#pragma unroll
    for (int u = 0; u < U; ++u)
        v[u] = score[min(base + u * 64 + lane, end - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
        key[u] = score_key(v[u]);
}

constexpr int kDigitBits = 11;     // of a pass of the radix select
constexpr int kBinsOf = 1 << kDigitBits;

// Entries are placed by counting those above each, which takes c^2 comparisons, where that is faster than what it saves:
//  - all of them, without a select, up to kRankAll: a cut of 256 entries 4.4 us, 4.7 with a select; of 320 5.4 and 4.8;
//  - what a pass of the select leaves, up to kRankSome.  4096 entries, cut of 64: 6.7 us (sorted: 14.0), of 180: 8.4 (16.4);
//  - up to kRankMost if another pass would leave nearly as many: cut of 300 9.6 us (10.6 always; sorted 19.2),
//    of 450 12.0 (17.4 with kRankSome only; sorted 19.4).
constexpr int kRankAll = 256, kRankSome = 320, kRankMost = 512;
static_assert(kRankMost * 16 <= kBinsOf * 4, "the entries, their scores and places lie where the histogram was");

__device__ __forceinline__ int wave_inclusive(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

// The digit whose bin holds the need-th best entry, by one wavefront: sel = {digit, place in the bin, entries of it}.
__device__ __forceinline__ void find_digit(const int *hist, int need, int lane, int *sel)
{
    constexpr int kPer = kBinsOf / 64;               // bins 32l .. 32l+31 of lane l, in an order that spreads over the banks
    int total = 0;
#pragma unroll
    for (int j = 0; j < kPer / 4; ++j) {
        const int4 c = *(const int4 *)&hist[kPer * lane + 4 * ((j + lane) & (kPer / 4 - 1))];
        total += c.x + c.y + c.z + c.w;
    }
    const int incl = wave_inclusive(total);
    const int above = __builtin_amdgcn_readlane(incl, 63) - incl;                 // entries in higher lanes' bins
    const unsigned long long here = __builtin_amdgcn_ballot_w64(above < need && above + total >= need);
    const int owner = __ffsll((long long)here) - 1;
    const int rest = need - __builtin_amdgcn_readlane(above, owner);
    const int digit = kPer * owner + kPer - 1 - (lane & (kPer - 1));              // downwards; both halves alike
    const int count = hist[digit], upto = wave_inclusive(lane < kPer ? count : 0);
    if (lane < kPer && upto >= rest && upto - count < rest) {
        sel[0] = digit;
        sel[1] = rest - (upto - count);
        sel[2] = count;
    }
}

// Merges the runs of LEN entries of c[0 .. n) pairwise, then those of 2 * LEN and so on (n a power of two, at most
// E * kTopkThreads; all entries differ).  An entry's place is its own in its run and that among the other run's
// entries, by bisection; a thread holds its entries in registers meanwhile.  Bound by instruction issue: four a probe.
template <int LEN, int E>
__device__ __forceinline__ void merge_runs(unsigned long long *c, int n, int tid)
{
    if constexpr (LEN < E * kTopkThreads) {
        if (LEN >= n)
            return;
        unsigned long long me[E];
        const unsigned long long *sib[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int at = tid + e * kTopkThreads;
            me[e] = c[at < n ? at : 0];
            sib[e] = c + (at < n ? (at & ~(LEN - 1)) ^ LEN : 0);
        }
#pragma unroll
        for (int step = LEN / 2; step > 0; step >>= 1) {
            unsigned long long o[E];
#pragma unroll
            for (int e = 0; e < E; ++e)
                o[e] = sib[e][step - 1];
#pragma unroll
            for (int e = 0; e < E; ++e)
                sib[e] += o[e] > me[e] ? step : 0;
        }
        int to[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int at = tid + e * kTopkThreads;
            const int above = (int)(sib[e] - c) - ((at & ~(LEN - 1)) ^ LEN) + (sib[e][0] > me[e] ? 1 : 0);
            to[e] = (at & ~(2 * LEN - 1)) + (at & (LEN - 1)) + above;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (tid + e * kTopkThreads < n)
                c[to[e]] = me[e];
        __syncthreads();
        merge_runs<2 * LEN, E>(c, n, tid);
    }
}

// Sorts c[0 .. n), largest first (n a power of two from 64 on, at most E * kTopkThreads; all entries differ).
// A bitonic sort has 66 rounds with a barrier each for 2048 entries: the whole cut 25.1 us, so 12.3; of 4000 of 8000
// entries 47 and 25, of 8000 78 and 37.
template <int E>
__device__ __forceinline__ void sort_descending(unsigned long long *c, int n, int tid)
{
    unsigned long long me[E];
    int to[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {                    // runs of 64, by counting
        const int at = tid + e * kTopkThreads, run = at < n ? at & ~63 : 0;
        me[e] = c[at < n ? at : 0];
        to[e] = run;
#pragma unroll 8
        for (int j = 0; j < 64; j += 2) {
            const ulonglong2 o = *(const ulonglong2 *)&c[run + j];
            to[e] += o.x > me[e] ? 1 : 0;
            to[e] += o.y > me[e] ? 1 : 0;
        }
    }
    // (a run is one wavefront's: nobody else reads or writes it)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (tid + e * kTopkThreads < n)
            c[to[e]] = me[e];
    __syncthreads();
    merge_runs<64, E>(c, n, tid);
}

// The same for 16384 entries: sixteen a thread would not fit its registers.
__device__ __forceinline__ void sort_bitonic(unsigned long long *c, int n, int tid)
{
    for (int size = 2; size <= n; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = tid; t < (n >> 1); t += kTopkThreads) {
                const int lo = ((t & ~(stride - 1)) << 1) | (t & (stride - 1));
                const int hi = lo | stride;
                const bool desc = (lo & size) == 0;
                const unsigned long long a = c[lo], b = c[hi];
                if ((a < b) == desc) {
                    c[lo] = b;
                    c[hi] = a;
                }
            }
            __syncthreads();
        }
    }
}

template <int U>
__global__ void __launch_bounds__(kTopkThreads)
topk_kernel(const TopkDesc *__restrict__ far, NearTopk)
{
    extern __shared__ unsigned long long cand[];   // [kpow2] then small scratch
    const TopkDesc d = where_descs(far, sizeof(far))[blockIdx.x];
    const int n = d.sub_end - d.sub_begin, k = d.k;   // this workgroup's entries
    const int kk = min(n, k);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *__restrict__ score = d.score + d.sub_begin;
    const uint32_t idx0 = (uint32_t)d.sub_begin;

    if (d.comp_out) {
        if (d.comp_pad)
            for (int j = kk + tid; j < k; j += kTopkThreads)
                d.comp_out[j] = 0ull;
    } else {
        for (int j = kk + tid; j < k; j += kTopkThreads) {
            d.out_idx[j] = -1;
            if (d.out_score)
                d.out_score[j] = -__builtin_inff();
        }
    }
    if (kk == 0)
        return;
    int kpow2 = 2;                        // at least 2: keeps the histogram 16-byte aligned
    while (kpow2 < kk)
        kpow2 <<= 1;
    int *hist = (int *)(cand + kpow2);    // kBinsOf ints
    int *wave_cnt = hist + kBinsOf;       // 2 x 16 ints: per-wavefront counts (above, equal)
    int *sel = wave_cnt + 2 * kTopkWaves; // [0] digit, [1] remaining need, [2] entries of the digit, [3] entries collected

    // Every wavefront owns a contiguous, 64-aligned slice of the scores: slices in wavefront
    // order are the scores in index order.
    const int per_wave = (((n + kTopkWaves - 1) / kTopkWaves) + 63) & ~63;
    const int w_begin = min(wave * per_wave, n), w_end = min(w_begin + per_wave, n);

    // A wavefront whose slice is a single round of loads (requests of up to 1024 * U entries)
    // fetches its keys once and keeps them in registers for all six sweeps below.
    const bool cached = per_wave <= 64 * U;
    uint32_t key[U];
    float v[U];
    if (cached && w_begin < w_end)
        load_keys(score, w_begin, w_end, lane, key, v);

    // ---- 1. key of the kk-th best entry ----
    uint32_t prefix = 0, mask = 0;
    int need = kk;
    int few = n <= kRankAll ? n : 0;     // entries that may be among the best, once there are few enough
    if (few == 0 && kk < n) {
        if (tid == 0)
            sel[3] = 0;
        for (int shift = 32 - kDigitBits;; shift = max(shift - kDigitBits, 0)) {
            for (int b = tid; b < kBinsOf; b += kTopkThreads)
                hist[b] = 0;
            __syncthreads();
            int run_digit = -1, run = 0;
            for (int base = w_begin; base < w_end; base += 64 * U) {
                if (!cached)
                    load_keys(score, base, w_end, lane, key, v);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool valid = base + u * 64 + lane < w_end;
                    if (valid && (key[u] & mask) == prefix) {
                        const int dg = (key[u] >> shift) & (kBinsOf - 1) & ~(mask >> shift);
                        if (dg != run_digit) {
                            if (run)
                                atomicAdd(&hist[run_digit], run);
                            run_digit = dg;
                            run = 0;
                        }
                        ++run;
                    }
                }
            }
            if (run)
                atomicAdd(&hist[run_digit], run);
            __syncthreads();
            if (wave == 0)
                find_digit(hist, need, lane, sel);
            __syncthreads();
            prefix |= (uint32_t)sel[0] << shift;
            mask = ~0u << shift;
            need = sel[1];
            const int may = kk - need + sel[2];
            if (cached && (may <= kRankSome || may <= min(kk + kk / 8, kRankMost))) {
                few = may;
                break;
            }
            if (shift == 0)
                break;
            __syncthreads();
        }
    } else {
        need = n;   // take everything; every key is >= 0
    }
    if (few > 0) {                        // entries of keys >= prefix
        unsigned long long *const all = (unsigned long long *)hist;
        float *const value = (float *)(all + kRankMost);
        int *const place = (int *)(value + kRankMost);
        int at = w_begin;
        if (n > kRankAll) {
            int mine = 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
                mine += __popcll(__builtin_amdgcn_ballot_w64(w_begin + u * 64 + lane < w_end && key[u] >= prefix));
            if (mine && lane == 0)
                at = atomicAdd(&sel[3], mine);
            at = __builtin_amdgcn_readfirstlane(at);
        }
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = w_begin + u * 64 + lane;
            const bool take = i < w_end && key[u] >= prefix;
            const unsigned long long who = __builtin_amdgcn_ballot_w64(take);
            if (take) {
                const int c = at + __popcll(who & below);
                all[c] = ((unsigned long long)key[u] << 32) | (unsigned long long)(0xFFFFFFFFu - (idx0 + (uint32_t)i));
                value[c] = v[u];
                place[c] = 0;
            }
            at += __popcll(who);
        }
        if (tid == 0 && (few & 1))
            all[few] = 0ull;              // (few < kRankMost then)
        __syncthreads();
        // 64 entries to a wavefront, and some of what each is compared with
        const int groups = (few + 63) >> 6, parts = kTopkWaves / groups, part = wave / groups;
        const int e = (wave - part * groups) * 64 + lane;
        if (part < parts) {
            const int per = ((few + parts - 1) / parts + 1) & ~1;
            const int end = min(part * per + per, few);
            const unsigned long long me = all[min(e, few - 1)];
            int above = 0;
#pragma unroll 8
            for (int j = part * per; j < end; j += 2) {
                const ulonglong2 o = *(const ulonglong2 *)&all[j];
                above += o.x > me ? 1 : 0;
                above += o.y > me ? 1 : 0;
            }
            if (e < few && above)
                atomicAdd(&place[e], above);
        }
        __syncthreads();
        if (tid < few && place[tid] < kk) {
            const int j = place[tid];
            if (d.comp_out) {
                d.comp_out[j] = all[tid];
            } else {
                d.out_idx[j] = (int32_t)(0xFFFFFFFFu - (uint32_t)all[tid]);
                if (d.out_score)
                    d.out_score[j] = value[tid];
            }
        }
        return;
    }
    const uint32_t tau = prefix;
    const int need_eq = need;
    const bool all = kk == n;
    const int sorted = max(kpow2, 64);                      // (room: the histogram is done with)

    // ---- 2. collect, in index order: count per wavefront, scan, then place ----
    int my_gt = 0, my_eq = 0;
    for (int base = w_begin; base < w_end && !all; base += 64 * U) {
        if (!cached)
            load_keys(score, base, w_end, lane, key, v);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool valid = base + u * 64 + lane < w_end;
            my_gt += __popcll(__ballot(valid && key[u] > tau));
            my_eq += __popcll(__ballot(valid && key[u] == tau));
        }
    }
    if (lane == 0) {
        wave_cnt[wave] = my_gt;
        wave_cnt[kTopkWaves + wave] = my_eq;
    }
    __syncthreads();
    int gt_before = all ? w_begin : 0, eq_before = 0;
    for (int w = 0; w < wave && !all; ++w) {
        gt_before += wave_cnt[w];
        eq_before += wave_cnt[kTopkWaves + w];
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int base = w_begin; base < w_end; base += 64 * U) {
        if (!cached)
            load_keys(score, base, w_end, lane, key, v);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * 64 + lane;
            const bool valid = i < w_end;
            const bool gt = valid && (all || key[u] > tau), eq = valid && !gt && key[u] == tau;
            const unsigned long long bg = __ballot(gt), be = __ballot(eq);
            const unsigned long long comp =
                ((unsigned long long)key[u] << 32) |
                (unsigned long long)(0xFFFFFFFFu - (idx0 + (uint32_t)i));
            if (gt) {
                cand[gt_before + __popcll(bg & below)] = comp;       // fewer than kk of these exist
            } else if (eq) {
                const int rank = eq_before + __popcll(be & below);   // index order among the ties
                if (rank < need_eq)
                    cand[kk - 1 - rank] = comp;
            }
            gt_before += __popcll(bg);
            eq_before += __popcll(be);
        }
    }
    // ---- 3. sort, descending ----
    for (int j = kk + tid; j < sorted; j += kTopkThreads)
        cand[j] = (unsigned long long)(sorted - j);         // below every real composite, and different
    __syncthreads();
    if (sorted <= kTopkThreads)
        sort_descending<1>(cand, sorted, tid);
    else if (sorted <= 2 * kTopkThreads)
        sort_descending<2>(cand, sorted, tid);
    else if (sorted <= 4 * kTopkThreads)
        sort_descending<4>(cand, sorted, tid);
    else if (sorted <= 8 * kTopkThreads)
        sort_descending<8>(cand, sorted, tid);
    else
        sort_bitonic(cand, sorted, tid);
    if (d.comp_out) {
        for (int j = tid; j < kk; j += kTopkThreads)
            d.comp_out[j] = cand[j];
        return;
    }
    for (int j = tid; j < kk; j += kTopkThreads) {
        const uint32_t idx = 0xFFFFFFFFu - (uint32_t)(cand[j] & 0xFFFFFFFFull);
        d.out_idx[j] = (int32_t)idx;
        if (d.out_score)
            d.out_score[j] = d.score[idx];
    }
}

// Second stage: the slices' sorted candidate lists into LDS (each padded to kp = 2^q >= k
// entries), then a tree of pairwise merges that each keep only the better kp entries:
// max(A[i], B[kp-1-i]) holds the best kp of two descending lists as a bitonic sequence, and
// q compare-exchange rounds sort it.  What is left in list 0 is the answer.
__global__ void __launch_bounds__(kTopkThreads)
topk_merge_kernel(const TopkMergeDesc *__restrict__ far, NearMerge)
{
    extern __shared__ unsigned long long cand[];
    const TopkMergeDesc d = where_descs(far, sizeof(far))[blockIdx.x];
    const int tid = threadIdx.x;
    const int k = d.k, lists = d.n_comp / k;
    int q = 0;
    while ((1 << q) < k)
        ++q;
    const int kp = 1 << q;
    for (int j = tid; j < lists * kp; j += kTopkThreads) {
        const int l = j >> q, i = j & (kp - 1);
        cand[j] = i < k ? d.comp_in[l * k + i] : 0ull;
    }
    __syncthreads();
    for (int step = 1; step < lists; step <<= 1) {
        const int groups = (lists + 2 * step - 1) / (2 * step);
        for (int t = tid; t < groups * kp; t += kTopkThreads) {
            const int a = (t >> q) * 2 * step, i = t & (kp - 1);
            if (a + step < lists) {
                const unsigned long long x = cand[a * kp + i], y = cand[(a + step) * kp + kp - 1 - i];
                if (x < y)
                    cand[a * kp + i] = y;
            }
        }
        __syncthreads();
        for (int stride = kp >> 1; stride > 0; stride >>= 1) {
            for (int t = tid; t < groups * (kp >> 1); t += kTopkThreads) {
                const int a = (t >> (q - 1)) * 2 * step, u = t & ((kp >> 1) - 1);
                if (a + step < lists) {
                    const int lo = a * kp + (((u & ~(stride - 1)) << 1) | (u & (stride - 1)));
                    const int hi = lo + stride;
                    const unsigned long long x = cand[lo], y = cand[hi];
                    if (x < y) {
                        cand[lo] = y;
                        cand[hi] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
    const int kk = min(d.n, k);
    for (int j = tid; j < k; j += kTopkThreads) {
        if (j < kk) {
            const uint32_t idx = 0xFFFFFFFFu - (uint32_t)(cand[j] & 0xFFFFFFFFull);
            d.out_idx[j] = (int32_t)idx;
            if (d.out_score)
                d.out_score[j] = d.score[idx];
        } else {
            d.out_idx[j] = -1;
            if (d.out_score)
                d.out_score[j] = -__builtin_inff();
        }
    }
}

// Merge of up to kTopkWays descending lists of composites that live in global memory, for cuts too wide
// for the LDS merge.  All composites differ, so an entry's place in the merged list is its own
// position plus the number of entries of the other lists that exceed it: one thread per entry
// finds these counts by bisection, side by side, and stores the entry if its place is among the best `lo`.
// blockIdx.y names the merge, blockIdx.x a run of kJoinThreads entries of its lists, one after the other.
// A chain of 12 to 16 loads from the L2 beside a launch's start and end, and bound by the lines that a compute unit's
// loads touch where its workgroup is large.  32 lists of 2048 entries, cut of 16384: 26.1 us two at a time, five
// launches of 1024 threads a workgroup; 18.2 four at a time with 256 (26.0 with 1024); 13.8 so.
constexpr int kJoinThreads = 256;

// Entries of the first W lists above v, of which `me` entries of list `mine` are known.
template <int W>
__device__ __forceinline__ int entries_above(const TopkJoinDesc &d, unsigned long long v, int mine, int me)
{
    int above[W], most[W], top = 1;
#pragma unroll
    for (int w = 0; w < W; ++w) {                        // counted no further than would push v out of the cut
        above[w] = 0;
        most[w] = w == mine ? 0 : min(d.len[w], d.lo - me);
    }
    while (2 * top <= d.longest)
        top <<= 1;
    for (int step = top; step > 0; step >>= 1) {
        unsigned long long o[W];
#pragma unroll
        for (int w = 0; w < W; ++w)
            o[w] = d.list[w][max(min(above[w] + step, most[w]), 1) - 1];
#pragma unroll
        for (int w = 0; w < W; ++w)
            above[w] += above[w] + step <= most[w] && o[w] > v ? step : 0;
    }
    int all = me;
#pragma unroll
    for (int w = 0; w < W; ++w)
        all += above[w];
    return all;
}

__global__ void __launch_bounds__(kJoinThreads)
topk_join_kernel(const TopkJoinDesc *__restrict__ far, NearJoins)
{
    const TopkJoinDesc d = where_descs(far, sizeof(far))[blockIdx.y];
    int me = blockIdx.x * kJoinThreads + threadIdx.x, mine = -1;
    const unsigned long long *self = nullptr;
#pragma unroll
    for (int w = 0; w < kTopkWays; ++w) {
        if (mine < 0 && me < d.len[w]) {
            mine = w;
            self = d.list[w];
        }
        me -= mine < 0 ? d.len[w] : 0;
    }
    if (mine >= 0 && me < d.lo) {
        const unsigned long long v = self[me];
        const int p = d.n <= 2   ? entries_above<2>(d, v, mine, me)
                      : d.n <= 4 ? entries_above<4>(d, v, mine, me)
                                 : entries_above<kTopkWays>(d, v, mine, me);
        if (p < d.lo) {
            if (d.out) {
                d.out[p] = v;
            } else {
                const uint32_t idx = 0xFFFFFFFFu - (uint32_t)(v & 0xFFFFFFFFull);
                d.out_idx[p] = (int32_t)idx;
                if (d.out_score)
                    d.out_score[p] = d.score[idx];
            }
        }
    }
    if (!d.out && blockIdx.x == 0) {
        for (int p = d.lo + threadIdx.x; p < d.k; p += kJoinThreads) {
            d.out_idx[p] = -1;
            if (d.out_score)
                d.out_score[p] = -__builtin_inff();
        }
    }
}

int launch_topk_joins(const Descs<TopkJoinDesc> &descs, int max_entries, hipStream_t stream)
{
    const int runs = max_entries > 0 ? (max_entries + kJoinThreads - 1) / kJoinThreads : 1;
    constexpr int kMaxY = 32768;             // merges per launch (grid.y)
    const NearJoins near = near_descs<NearJoins>(descs);
    for (int at = 0; at < descs.n; at += kMaxY) {
        const int cnt = descs.n - at < kMaxY ? descs.n - at : kMaxY;
        hipLaunchKernelGGL(topk_join_kernel, dim3(runs, cnt), dim3(kJoinThreads), 0, stream,
                           descs.far ? descs.far + at : nullptr, near);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return fail_hip(e, "topk_join_kernel launch");
    }
    return FS_OK;
}

int launch_topk_merge(const Descs<TopkMergeDesc> &descs, int max_padded, hipStream_t stream)
{
    if (max_padded > kTopkMergeCap)
        return fail(FS_EUNSUPPORTED, "top-k merge of %d candidates exceeds %d", max_padded, kTopkMergeCap);
    const size_t lds = (size_t)max_padded * 8;
    static size_t configured[16] = {0};
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    if (lds > 65536 && (dev < 0 || dev >= 16 || configured[dev] < lds)) {
        FS_HIP(hipFuncSetAttribute((const void *)topk_merge_kernel,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        if (dev >= 0 && dev < 16)
            configured[dev] = lds;
    }
    hipLaunchKernelGGL(topk_merge_kernel, dim3(descs.n), dim3(kTopkThreads), lds, stream, descs.far, near_descs<NearMerge>(descs));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_hip(e, "topk_merge_kernel launch");
    return FS_OK;
}

template <int U>
static int launch_topk_form(const Descs<TopkDesc> &descs, int max_k, hipStream_t stream)
{
    int kpow2 = 2;
    while (kpow2 < max_k)
        kpow2 <<= 1;
    const size_t lds = (size_t)kpow2 * 8 + (kBinsOf + 2 * kTopkWaves + 4) * sizeof(int);
    static size_t configured[16] = {0};
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    if (lds > 65536 && (dev < 0 || dev >= 16 || configured[dev] < lds)) {
        FS_HIP(hipFuncSetAttribute((const void *)topk_kernel<U>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        if (dev >= 0 && dev < 16)
            configured[dev] = lds;
    }
    hipLaunchKernelGGL(topk_kernel<U>, dim3(descs.n), dim3(kTopkThreads), lds, stream, descs.far, near_descs<NearTopk>(descs));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_hip(e, "topk_kernel launch");
    return FS_OK;
}

int launch_topk(const Descs<TopkDesc> &descs, int max_k, int max_entries, hipStream_t stream)
{
    return max_entries > kTopkFew * kTopkThreads ? launch_topk_form<kTopkMany>(descs, max_k, stream)
                                                 : launch_topk_form<kTopkFew>(descs, max_k, stream);
}

// ---- fs_topk_noalloc: the same cut for callers that cannot allocate -----------------------------
// Descriptors and the slices' candidate lists live in a fixed device array instead of grown
// library scratch; the descriptors travel as a kernel argument (no staging buffer, no copy).
constexpr size_t kNoAllocBytes = 1u << 20;        // the whole array
constexpr size_t kNoAllocDescBytes = 3584;        // its head: descriptors (one kernel argument)
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

struct DescBlob {
    uint32_t words[kNoAllocDescBytes / 4];
};

__global__ void __launch_bounds__(256)
topk_store_desc_kernel(DescBlob blob, uint32_t *dst, int n_words)
{
    for (int i = threadIdx.x; i < n_words; i += blockDim.x)
        dst[i] = blob.words[i];
}

static std::mutex g_noalloc_mu;
static unsigned char *g_noalloc_ptr[16] = {};     // device address of `scratch`, per device

}  // namespace fs

using namespace fs;

extern "C" int fs_topk_noalloc(int32_t n_requests, const fs_topk_req *reqs, void *stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (n_requests < 0)
        return fail(FS_EINVAL, "fs_topk_noalloc: n_requests %d is negative", n_requests);
    if (n_requests == 0)
        return FS_OK;
    if (!reqs)
        return fail(FS_EINVAL, "fs_topk_noalloc: reqs is NULL");
    size_t n_blocks = 0, n_merge = 0, comp_total = 0;
    int max_k = 0, max_comp = 0;
    bool whole = true;
    for (int i = 0; i < n_requests; ++i)
        whole &= topk_whole(reqs[i].n, reqs[i].k);
    for (int i = 0; i < n_requests; ++i) {
        const fs_topk_req &r = reqs[i];
        if (r.n < 0 || r.k < 0)
            return fail(FS_EINVAL, "fs_topk_noalloc: request %d: n=%d k=%d must be non-negative", i, r.n, r.k);
        if (r.k > FS_MAX_TOPK)
            return fail(FS_EUNSUPPORTED, "fs_topk_noalloc: request %d: k=%d exceeds FS_MAX_TOPK=%d", i,
                        r.k, FS_MAX_TOPK);
        if (r.n > 0 && !r.score)
            return fail(FS_EINVAL, "fs_topk_noalloc: request %d: score is NULL", i);
        if (r.k > 0 && !r.out_idx)
            return fail(FS_EINVAL, "fs_topk_noalloc: request %d: out_idx is NULL", i);
        const TopkPlan p = topk_plan(r.n, r.k, whole);
        if (p.mode == 2)
            return fail(FS_EUNSUPPORTED, "fs_topk_noalloc: request %d: cuts wider than 4096 of %d or "
                        "more entries are not served without allocation (use fs_topk)", i, kTopkSliceMin);
        n_blocks += (size_t)p.s;
        if (p.mode == 1) {
            ++n_merge;
            comp_total += (size_t)p.s * (size_t)r.k;
            int kp = 1;
            while (kp < r.k)
                kp <<= 1;
            if (p.s * kp > max_comp)
                max_comp = p.s * kp;
        }
        if (r.k > max_k)
            max_k = r.k;
    }
    if (max_k == 0)
        return FS_OK;
    const size_t merge_off = (sizeof(TopkDesc) * n_blocks + 15) & ~(size_t)15;
    const size_t desc_bytes = merge_off + sizeof(TopkMergeDesc) * n_merge;
    if (desc_bytes > kNoAllocDescBytes)
        return fail(FS_EUNSUPPORTED, "fs_topk_noalloc: %zu workgroups and %zu merges need %zu bytes of "
                    "descriptors, the limit is %zu (about 60 workgroups)", n_blocks, n_merge, desc_bytes,
                    kNoAllocDescBytes);
    if (comp_total * 8 > kNoAllocBytes - kNoAllocDescBytes)
        return fail(FS_EUNSUPPORTED, "fs_topk_noalloc: the sliced requests need %zu bytes of candidate "
                    "lists, the limit is %zu", comp_total * 8, kNoAllocBytes - kNoAllocDescBytes);

    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    int dev = 0;
    FS_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 16)
        return fail(FS_EUNSUPPORTED, "device ordinal %d not supported", dev);
    if (!g_noalloc_ptr[dev]) {
        // every device holds its own copy of the array, at its own address
        void *ptr = nullptr;
        FS_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr)
            return fail(FS_EDEVICE, "fs_topk_noalloc: no device address for the scratch array");
        g_noalloc_ptr[dev] = (unsigned char *)ptr;
    }
    unsigned char *base = g_noalloc_ptr[dev];

    DescBlob blob;
    memset(&blob, 0, sizeof(blob));
    TopkDesc *h = (TopkDesc *)blob.words;
    TopkMergeDesc *hm = (TopkMergeDesc *)((unsigned char *)blob.words + merge_off);
    unsigned long long *comp = (unsigned long long *)(base + kNoAllocDescBytes);
    size_t b = 0, m = 0;
    for (int i = 0; i < n_requests; ++i) {
        const fs_topk_req &r = reqs[i];
        const TopkPlan p = topk_plan(r.n, r.k, whole);
        for (int j = 0; j < p.s; ++j, ++b) {
            h[b].score = r.score;
            h[b].out_idx = r.out_idx;
            h[b].out_score = r.out_score;
            h[b].n = r.n;
            h[b].k = r.k;
            const long long lo = (long long)j * p.per, hi = lo + p.per;
            h[b].sub_begin = (int32_t)(lo < r.n ? lo : r.n);
            h[b].sub_end = (int32_t)(hi < r.n ? hi : r.n);
            h[b].comp_pad = p.mode == 1 ? 1 : 0;
            h[b].pad = 0;
            h[b].comp_out = p.mode == 1 ? comp + (size_t)j * (size_t)r.k : nullptr;
        }
        if (p.mode == 1) {
            hm[m].comp_in = comp;
            hm[m].score = r.score;
            hm[m].out_idx = r.out_idx;
            hm[m].out_score = r.out_score;
            hm[m].n_comp = p.s * r.k;
            hm[m].n = r.n;
            hm[m].k = r.k;
            hm[m].pad = 0;
            comp += (size_t)p.s * (size_t)r.k;
            ++m;
        }
    }
    // Nothing in the array has to start at zero: every workgroup writes its whole list (padding
    // included) before the merge reads it, and the descriptors are rewritten by every call.
    hipLaunchKernelGGL(topk_store_desc_kernel, dim3(1), dim3(256), 0, stream, blob, (uint32_t *)base,
                       (int)((desc_bytes + 3) / 4));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_hip(e, "topk_store_desc_kernel launch");
    prof_start(kKernTopk, stream);
    int max_entries = 0;
    for (size_t i = 0; i < n_blocks; ++i)
        max_entries = std::max(max_entries, h[i].sub_end - h[i].sub_begin);
    int rc = launch_topk({(const TopkDesc *)base, nullptr, (int)n_blocks}, max_k, max_entries, stream);
    if (rc == FS_OK && n_merge)
        rc = launch_topk_merge({(const TopkMergeDesc *)(base + merge_off), nullptr, (int)n_merge}, max_comp, stream);
    prof_stop(stream);
    return rc;
}
