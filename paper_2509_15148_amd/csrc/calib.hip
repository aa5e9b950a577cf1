// Online conformal calibration and ordinal classification (integer work, bit-exact).
//
// The calibration multiset is kept on the device as an ascending array of 32-bit keys; a key is
// an order-preserving image of the fp32 score (-0 folded onto +0, every NaN onto key 0, below
// -inf), so all comparisons are unsigned-integer comparisons that reproduce the IEEE ones.
//
//   append (Online Calibration):  keys of the new scores are sorted (sort.hip: sorted runs cut into buckets for
//       small batches, radix sort for large ones) and
//       merged with the resident array by a merge-path kernel into the other half of a ping-pong
//       buffer.  The same pass writes four sampled copies of its output (every 32nd, 1024th, 32768th,
//       2^20-th key), the levels of a static 32-ary search index: a node is one 128-byte line, the unit the L2
//       fills from memory.
//   classify (Eq. "p-value", Eq. "prediction_set"):  ranks = #{cal >= s} by one search per test
//       score: the coarsest index level sits in LDS, every further level costs one aligned 128-byte
//       line.  The class is an integer comparison of ranks + 1 with r_l = floor(alpha_l (N + 1));
//       the quantile thresholds of Eq. "quantile" are read straight from the sorted array.
//   conditional coverage (Proposition 2):  no state; one wavefront ranks the candidates of one input against
//       that input's own calibration scores.
#include "common.h"
#include "keys.h"
#include "block_sort.h"

#include <math.h>
#include <new>
#include <type_traits>

constexpr int kIndexLevels = 4;
constexpr int kFanBits = 5;                 // 32 keys per index node (one 128-byte line)
constexpr int kFan = 1 << kFanBits;

struct atts_calib {
    uint32_t* keys[2];                  // ping-pong sorted arrays, capacity each
    uint32_t* index[2][kIndexLevels];   // index[side][k][j] = keys[side][j * 32^(k+1)]
    uint32_t* runs;                     // the batch being appended: two buffers the sort alternates between
    uint32_t* batch;
    uint32_t* sort_scratch;             // samples of the sorted runs, or digit histograms of the radix sort
    int32_t* splits;                    // merge-path splits of one streaming merge launch
    int64_t splits_len;
    int64_t capacity;
    int64_t n;
    int cur;
};

namespace atts {
namespace {

constexpr int kMergeThreads = 256;
// outputs per merge workgroup: the shorter chain of 1024 while a workgroup a CU covers them (2048 and 1024, us: 1000 + 16 keys 6.8 and 6.4,
// 100,000 + 2000 with their sort 11.4 and 10.7, 250,000 + 2000 11.5 and 10.8, 500,000 + 2000 11.8 both, 3,000,000 + 100 13.4 and 13.5)
constexpr int kMergeSegTiny = 1024;
constexpr int64_t kMergeTinyTo = (int64_t)kMergeSegTiny * 256;
constexpr int kMergeSegSmall = 2048;   // ... cache-resident sizes (more workgroups)
constexpr int kMergeSegLarge = 4096;   // ... and streaming sizes (split search amortised over more keys; 8 workgroups per CU)
constexpr int64_t kMergeLargeFrom = (int64_t)1 << 22;
// Appends of up to kInlineMax scores into sets of up to kInlineTotal keys are sorted by the merge workgroups themselves, each for
// itself: one launch instead of two.  Up to kRankMax scores every thread ranks one against all others (its time grows with the
// square: 1000 + 16 scores 6.4 us, 48 7.7, 64 8.1, 256 13.3), more go through the register network of one wavefront (16: 7.3, 48: 7.8,
// 64: 7.8, 256: 8.2, 512: 8.4), a sort of its own ahead of the merge costs a launch (9.6, 10.1, 10.1, 10.4, 10.5).  Every workgroup repeats the
// sort, so sets whose merge has more than four workgroups a CU keep it apart (2,000,000 + 256: 10.6 inside, 12.0 apart; 4,000,000:
// 16.0 and 15.2).
constexpr int kInlineMax = kWaveKeys;
constexpr int kRankMax = 48;
constexpr int64_t kInlineTotal = (int64_t)kMergeSegSmall * 1024;

// first index in [0, n) with a[idx] >= x  (n if none)
__device__ __forceinline__ int64_t lower_bound(const uint32_t* __restrict__ a, int64_t n, uint32_t x) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}
// first index with a[idx] > x
__device__ __forceinline__ int64_t upper_bound(const uint32_t* __restrict__ a, int64_t n, uint32_t x) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// ---- merging two sorted arrays --------------------------------------------------------------------
struct MergeJob {
    const uint32_t* a;   // resident keys (first on ties)
    int64_t na;
    const uint32_t* b;   // the sorted batch
    int64_t nb;
    uint32_t* out;
    uint32_t* index[kIndexLevels];   // EMIT only: index[k][j] = out[j * 32^(k+1)]
    const float* scores;             // INLINE_SORT only: the unsorted batch, nb <= kInlineMax scores (b unused)
};

// LDS position of element i: one pad word per 32, so that the accesses "thread t, element t * PER + e" fall
// into distinct banks
__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 5); }

// For a streaming merge launch of `segs` workgroups: splits[x] = elements taken from a[] among the first
// min(x seg, total) outputs.  One thread per entry: the searches run in parallel here instead of serially in front of
// every workgroup's loads.
__global__ __launch_bounds__(256) void merge_split_kernel(MergeJob job, int seg, int segs, int32_t* __restrict__ splits) {
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (x > segs) return;
    const int64_t diag = min(x * (int64_t)seg, job.na + job.nb);
    splits[x] = (int32_t)merge_path<int64_t>(job.a, job.na, job.b, job.nb, diag);
}

// Each workgroup produces SEG consecutive outputs (out + segment start is 16-byte aligned).  PRESPLIT: the segment's
// merge-path splits come from merge_split_kernel.  INLINE_SORT: the batch is a few unsorted scores; every workgroup turns it
// into ascending keys in LDS first.
template <int SEG, bool EMIT, bool PRESPLIT, bool INLINE_SORT = false>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeJob job, const int32_t* __restrict__ splits) {
    constexpr int PER = SEG / kMergeThreads;
    const uint32_t* __restrict__ a = job.a;
    const uint32_t* __restrict__ b = job.b;
    uint32_t* __restrict__ out = job.out;
    const int64_t na = job.na, nb = job.nb;
    const int64_t total = na + nb;
    const int64_t o0 = (int64_t)blockIdx.x * SEG;
    if (o0 >= total) return;
    const int64_t o1 = min(o0 + SEG, total);

    __shared__ int64_t split[2];
    __shared__ __attribute__((aligned(16))) uint32_t buf[SEG + SEG / 32];
    __shared__ uint32_t batch[INLINE_SORT ? kInlineMax : 1];
    if constexpr (INLINE_SORT) {
        if (nb <= kRankMax) {
            // rank of every key among the batch (equal keys in batch order), then the key goes to its rank
            const int t = (int)threadIdx.x, m = (int)nb;
            const uint32_t mine = t < m ? score_to_key(job.scores[t]) : kPadKey;
            buf[t] = mine;
            __syncthreads();
            int rank = 0;
#pragma unroll 4
            for (int j = 0; j < m; j += 4) {                        // past the end: kPadKey, never below a key
                const uint4 q = *reinterpret_cast<const uint4*>(buf + j);
                rank += (q.x < mine || (q.x == mine && j < t) ? 1 : 0) + (q.y < mine || (q.y == mine && j + 1 < t) ? 1 : 0) +
                        (q.z < mine || (q.z == mine && j + 2 < t) ? 1 : 0) + (q.w < mine || (q.w == mine && j + 3 < t) ? 1 : 0);
            }
            if (t < m) batch[rank] = mine;
        } else if (threadIdx.x < 64) {
            float f[kPer];
#pragma unroll
            for (int e = 0; e < kPer; ++e) f[e] = job.scores[min((int64_t)(e * 64 + threadIdx.x), nb - 1)];
            uint32_t k[kPer];
#pragma unroll
            for (int e = 0; e < kPer; ++e) k[e] = e * 64 + threadIdx.x < nb ? score_to_key(f[e]) : kPadKey;
            sort_in_block<64>(k, kWaveKeys, nullptr);
#pragma unroll
            for (int e = 0; e < kPer; ++e) batch[kPer * threadIdx.x + e] = k[e];
        }
        __syncthreads();
    }
    auto batch_key = [&](int64_t i) { return INLINE_SORT ? batch[i] : b[i]; };
    if constexpr (PRESPLIT) {
        if (threadIdx.x < 2) split[threadIdx.x] = splits[blockIdx.x + threadIdx.x];
    } else
    // Merge-path split of both segment ends at once, one wavefront each: "a[i] <= b[diag - 1 - i]" is true below the split, and
    // every round probes 64 evenly spaced candidates of the range that is left, one a lane.  One load latency a round, three rounds
    // up to 2^18 candidates, and nothing to wait for but the wavefront's own loads: 2.2 us of a workgroup at 2^20 + 65,536 keys (128
    // candidates a round with counts and limits through LDS and three barriers 3.6; 512, eight a lane, keep the address unit busy
    // longer than the round that they save takes: the launch 11.8 -> 15.5).
    if (threadIdx.x < 128) {
        const int h = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
        const int64_t diag = h ? o1 : o0;
        int64_t lo = diag > nb ? diag - nb : 0, hi = diag < na ? diag : na;
        while (lo < hi) {
            const int64_t step = (hi - lo + 63) / 64, probe = lo + lane * step, i = min(probe, hi - 1);
            const int64_t below = __popcll(__ballot(a[i] <= batch_key(diag - 1 - i) && probe < hi));
            // the last true candidate and the one behind it (or the end) enclose the split
            hi = min(lo + below * step, hi);
            lo = below > 0 ? lo + (below - 1) * step + 1 : lo;
        }
        if (lane == 0) split[h] = lo;
    }
    __syncthreads();
    const int64_t i0 = split[0], i1 = split[1];
    const int64_t j0 = o0 - i0, j1 = o1 - i1;
    const int la = (int)(i1 - i0), lb = (int)(j1 - j0);
    const int len = la + lb;
    uint32_t k[PER];
    // all PER loads of a thread are issued before the first is consumed
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int i = (int)threadIdx.x + e * kMergeThreads;
        k[e] = kPadKey;
        if (i < la) k[e] = a[i0 + i];
        else if (i < len) k[e] = batch_key(j0 + (i - la));
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) buf[lds_pad((int)threadIdx.x + e * kMergeThreads)] = k[e];
    __syncthreads();

    // every thread merges PER consecutive outputs (its split by halving: three probes a step, with twice the reads, took 1.3 us
    // for 0.6 where several workgroups share a CU)
    const int d0 = min((int)threadIdx.x * PER, len);
    int ia;
    {
        int lo = d0 > lb ? d0 - lb : 0, hi = d0 < la ? d0 : la;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (buf[lds_pad(mid)] <= buf[lds_pad(la + d0 - 1 - mid)]) lo = mid + 1; else hi = mid;
        }
        ia = lo;
    }
    const int ib = d0 - ia;
    // The PER smallest of the next PER keys of both sides, all read together: min(a[e], b[PER - 1 - e]) is a bitonic sequence of
    // them, sorted by the last stages of a network (equal keys are alike, so which side one comes from does not matter).  Taken
    // one by one, each key waits for the LDS read that the choice before it made: 1.3 us a workgroup instead of 0.7.
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const uint32_t x = ia + e < la ? buf[lds_pad(ia + e)] : kPadKey;
        const int f = PER - 1 - e;
        const uint32_t y = ib + f < lb ? buf[lds_pad(la + ib + f)] : kPadKey;
        k[e] = min(x, y);
    }
#pragma unroll
    for (int stride = PER / 2; stride > 0; stride >>= 1)
#pragma unroll
        for (int e = 0; e < PER; ++e)
            if ((e & stride) == 0) cswap(k[e], k[e + stride]);
    uint32_t* o = out + o0;
    if constexpr (PER <= 8) {
        // straight from the registers: 16 or 32 bytes a lane
        if (d0 + PER <= len) {
#pragma unroll
            for (int e = 0; e < PER; e += 4) *reinterpret_cast<uint4*>(o + d0 + e) = make_uint4(k[e], k[e + 1], k[e + 2], k[e + 3]);
        } else {
#pragma unroll
            for (int e = 0; e < PER; ++e)
                if (d0 + e < len) o[d0 + e] = k[e];
        }
        if constexpr (EMIT) {                                    // an index entry is the first key of a thread
            if (d0 < len) {
#pragma unroll
                for (int lvl = 0; lvl < kIndexLevels; ++lvl) {
                    const int shift = kFanBits * (lvl + 1);
                    const int64_t at = o0 + d0;
                    if ((at & (((int64_t)1 << shift) - 1)) == 0) job.index[lvl][at >> shift] = k[0];
                }
            }
        }
        return;
    }
    __syncthreads();
    // through LDS again, so that the segment leaves in whole 16-byte pieces per lane
#pragma unroll
    for (int e = 0; e < PER; ++e) buf[lds_pad((int)threadIdx.x * PER + e)] = k[e];
    __syncthreads();
    for (int i = (int)threadIdx.x * 4; i < len; i += kMergeThreads * 4) {
        if (i + 4 <= len) {
            uint4 v;
            v.x = buf[lds_pad(i)];
            v.y = buf[lds_pad(i + 1)];
            v.z = buf[lds_pad(i + 2)];
            v.w = buf[lds_pad(i + 3)];
            *reinterpret_cast<uint4*>(o + i) = v;
        } else {
            for (int r = i; r < len; ++r) o[r] = buf[lds_pad(r)];
        }
    }
    if constexpr (EMIT) {
#pragma unroll
        for (int lvl = 0; lvl < kIndexLevels; ++lvl) {
            const int shift = kFanBits * (lvl + 1);
            if (((int64_t)1 << shift) <= SEG) {
                for (int t = threadIdx.x; (t << shift) < len; t += kMergeThreads)
                    job.index[lvl][(o0 >> shift) + t] = buf[lds_pad(t << shift)];
            } else if (threadIdx.x == 0 && (o0 & (((int64_t)1 << shift) - 1)) == 0) {
                job.index[lvl][o0 >> shift] = buf[lds_pad(0)];
            }
        }
    }
}

// (rank + 1) / (N + 1) as the binary64 quotient rounded once to fp32.  Whole numbers below 2^24 are exact in fp32 and its division
// is correctly rounded; the binary64 quotient has more than 2 x 24 + 2 bits, so rounding through it gives the same bits, and
// the fp32 sequence takes a fraction of the binary64 one.
__device__ __forceinline__ float p_value(int64_t c1, int64_t n1) {
    if (n1 < ((int64_t)1 << 24)) return (float)(int32_t)c1 / (float)(int32_t)n1;
    return (float)((double)c1 / (double)n1);
}

// ---- classification ----------------------------------------------------------------------------------
struct ClassifyLevels {
    int64_t r[ATTS_MAX_ALPHAS];   // reject ranks floor(alpha_l (N + 1))
    int32_t n_alpha;
};

constexpr int kTopEntries = 8192;   // LDS copy of the coarsest level (or of every 2^top_shift-th entry of it): 32 KB

struct SearchIndex {
    const uint32_t* lvl[kIndexLevels + 1];   // lvl[0] = the sorted keys, lvl[k][j] = keys[j * 32^k]
    int64_t len[kIndexLevels + 1];
    int32_t top_level;                       // the level staged in LDS
    int32_t top_shift;
    int32_t per_thread;                      // test scores per thread
};

// One level of the index for the four test keys of a quad of lanes (lane l of the quad owns key x_l and the count
// t_l of entries of the next coarser level below it).  Result for each lane: the same count for level L, whose
// candidates are the 32 entries of one aligned 128-byte line (the whole line the L2 fetches is used).  The quad
// shares its four keys: in round r all four lanes work on lane r's key, each loading and comparing a quarter
// (32 bytes) of its line, so that one load instruction of the wavefront touches 16 lines instead of 64 (the vector
// cache looks up one line per cycle: a lane-per-line load costs four times the tag look-ups).  Values move inside the
// quad by DPP, not through LDS.  Every lane of the quad must be active; a lane without work passes t = 0 and gets 0.
template <int CTRL>
__device__ __forceinline__ int quad_perm(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true); }

template <int ROUNDS>
__device__ __forceinline__ int quad_rounds(const uint32_t* __restrict__ L, int64_t len, int t, uint32_t x) {
    const int q = threadIdx.x & 3;
    // all four lines of the quad are requested together: taken one after the other, each waits out its own latency (16 lines of a
    // wavefront in flight instead of 64, twelve latencies in a search of three levels instead of three)
    const int tr[4] = {quad_perm<0x00>(t), quad_perm<0x55>(t), quad_perm<0xAA>(t), quad_perm<0xFF>(t)};
    const int xr[4] = {quad_perm<0x00>((int)x), quad_perm<0x55>((int)x), quad_perm<0xAA>((int)x), quad_perm<0xFF>((int)x)};
    uint4 v[ROUNDS][2];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint4* p = reinterpret_cast<const uint4*>(L + (max(tr[r] - 1, 0) << kFanBits) + 8 * q);      // a lane without work: any line
        v[r][0] = p[0];
        v[r][1] = p[1];
    }
    __builtin_amdgcn_sched_barrier(0);
    int out = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t k = (uint32_t)xr[r];
        const int base = (tr[r] - 1) << kFanBits;
        const int valid = (int)min((int64_t)kFan, len - base) - 8 * q;         // entries of this quarter that exist
        int c = ((valid > 0 && v[r][0].x < k) ? 1 : 0) + ((valid > 1 && v[r][0].y < k) ? 1 : 0) + ((valid > 2 && v[r][0].z < k) ? 1 : 0) +
                ((valid > 3 && v[r][0].w < k) ? 1 : 0) + ((valid > 4 && v[r][1].x < k) ? 1 : 0) + ((valid > 5 && v[r][1].y < k) ? 1 : 0) +
                ((valid > 6 && v[r][1].z < k) ? 1 : 0) + ((valid > 7 && v[r][1].w < k) ? 1 : 0);
        c += quad_perm<0xB1>(c);      // lanes (1, 0, 3, 2)
        c += quad_perm<0x4E>(c);      // lanes (2, 3, 0, 1)
        if (q == r) out = tr[r] > 0 ? base + c : 0;
    }
    return out;
}

// The same where the quads' upper lanes may all be without work (a call of one or two scores, the end of a batch): their rounds are
// left out.  One score against 10^6 3.7 us for 4.5, against 2^28 7.0 for 8.3.  Large batches take all four unasked (2^24 scores
// against 2^28 731 us with the question, 719 without).
__device__ __forceinline__ int quad_descend(const uint32_t* __restrict__ L, int64_t len, int t, uint32_t x) {
    const uint64_t work = __builtin_amdgcn_ballot_w64(t > 0);
    if ((work & 0xEEEEEEEEEEEEEEEEull) == 0) return quad_rounds<1>(L, len, t, x);
    if ((work & 0xCCCCCCCCCCCCCCCCull) == 0) return quad_rounds<2>(L, len, t, x);
    return quad_rounds<4>(L, len, t, x);
}

// Workgroups of 256 threads are for calls whose chain of latencies counts (kFew): the level staged in 16-byte pieces and searched by three probes
// a step.  512 threads want fewer LDS reads and no clamped loads instead (524,288 scores in 5000 keys 8.3 us, with the other form 10.5), and LDS
// and registers for 32 wavefronts a CU.  kOne: every thread has one score, which it requests ahead of the staged level (524,288 in 5000 keys
// 8.3 -> 6.0 us, in 2^23 25.9 -> 22.5); carried from round to round of a loop it costs the register that makes it 24 wavefronts.
template <int THREADS, bool kOne>
__global__ __launch_bounds__(THREADS) void classify_kernel(SearchIndex ix, const float* __restrict__ test, int64_t m,
                                                       ClassifyLevels lv, int32_t* __restrict__ ranks,
                                                       float* __restrict__ pvalues, uint8_t* __restrict__ classes,
                                                       float* __restrict__ thresholds) {
    constexpr bool kFew = THREADS == 256;
    static_assert(!kFew || kOne, "the levels and scores of a few are requested together");
    __shared__ __attribute__((aligned(16))) uint32_t top[kTopEntries + (kFew ? 4 : 0)];
    const uint32_t* __restrict__ T = ix.lvl[ix.top_level];
    const int64_t top_len = ix.len[ix.top_level], n = ix.len[0];
    const int s = ix.top_shift;
    const int n_top = (int)((top_len + ((int64_t)1 << s) - 1) >> s);
    const float none = __uint_as_float(0x7FC00000u);
    const bool quantile = blockIdx.x == 0 && thresholds && (int)threadIdx.x < lv.n_alpha;
    auto order_statistic = [&](int64_t kth) { return kth >= 1 && kth <= n ? ix.lvl[0][kth - 1] : 0u; };      // 1-indexed
    auto threshold = [&](int64_t kth, uint32_t key) { return kth > n ? INFINITY : (kth < 1 ? -INFINITY : key_to_score(key)); };
    float first = none;
    if constexpr (kOne) {
        const int64_t i = (int64_t)blockIdx.x * THREADS + threadIdx.x;
        if (i < m) first = test[i];
    }
    if constexpr (kFew) {
        // The thresholds are requested ahead of the staged level too, which comes in 16-byte pieces (its array is padded to whole lines): a small
        // call is nothing but this chain of latencies.  The first workgroup waits for the levels' ranks, read by index, in between; taken
        // from scalars by selects they cost every call 0.05 to 0.1 us.
        const int64_t kth = quantile ? n + 1 - lv.r[threadIdx.x] : 0;
        const uint32_t kth_key = quantile ? order_statistic(kth) : 0u;
        if (s == 0) {
            const int n4 = (n_top + 3) >> 2;
            for (int i0 = 0; i0 < n4; i0 += 4 * THREADS) {
                uint4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    v[u] = make_uint4(0, 0, 0, 0);               // (left undefined, the pieces go through scratch memory one by one)
                    if (i0 + u * THREADS < n4) v[u] = reinterpret_cast<const uint4*>(T)[min(i0 + u * THREADS + (int)threadIdx.x, n4 - 1)];   // block-uniform
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i0 + u * THREADS + (int)threadIdx.x < n4) reinterpret_cast<uint4*>(top)[i0 + u * THREADS + threadIdx.x] = v[u];
            }
        } else {
            for (int i = threadIdx.x; i < n_top; i += THREADS) top[i] = T[(int64_t)i << s];
        }
        __syncthreads();
        if (threadIdx.x == 0) top[n_top] = kPadKey;              // what the search below finds behind the last entry
        __syncthreads();
        if (quantile) thresholds[threadIdx.x] = threshold(kth, kth_key);
    } else {
        for (int i = threadIdx.x; i < n_top; i += THREADS) top[i] = T[(int64_t)i << s];
        __syncthreads();
        if (quantile) {
            const int64_t kth = n + 1 - lv.r[threadIdx.x];
            thresholds[threadIdx.x] = threshold(kth, order_statistic(kth));
        }
    }
    const int per_thread = kOne ? 1 : ix.per_thread;
    for (int j = 0; j < per_thread; ++j) {
        const int64_t i0 = ((int64_t)blockIdx.x * per_thread + j) * THREADS;      // block-uniform: whole quads stay in the loop
        if (i0 >= m) break;
        const int64_t i = i0 + threadIdx.x;
        const float sc = kOne ? first : (i < m ? test[i] : none);
        const bool searching = !score_is_nan(sc);
        const uint32_t x = score_to_key(sc);
        int t = 0;                                             // number of entries of the current level below x
        if (searching) {
            int lo = 0;                                        // number of staged entries < x
            if constexpr (kFew) {
                // three probes a step, read together: half the steps of a chain of LDS latencies (1024 entries 1.2 -> 0.9 us)
                for (int range = n_top + 1; range > 1;) {
                    const int q = (range + 3) >> 2;
                    int below = 0;
#pragma unroll
                    for (int u = 1; u <= 3; ++u) below += top[min(lo + u * q - 1, n_top)] < x ? 1 : 0;
                    lo += below * q;
                    range = q;
                }
            } else {
                int hi = n_top;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (top[mid] < x) lo = mid + 1; else hi = mid;
                }
            }
            t = lo;
            if (s > 0 && lo > 0) {
                const int64_t w0 = ((int64_t)(lo - 1) << s) + 1;
                const int64_t w1 = min(top_len, (int64_t)lo << s);
                t = (int)(w0 + lower_bound(T + w0, w1 - w0, x));
            }
        }
#pragma unroll
        for (int l = kIndexLevels - 1; l >= 0; --l)
            if (l < ix.top_level) {                            // a NaN or absent score carries t = 0 down
                if constexpr (THREADS == 256) t = quad_descend(ix.lvl[l], ix.len[l], t, x);
                else t = quad_rounds<4>(ix.lvl[l], ix.len[l], t, x);
            }
        if (i >= m) continue;
        const int64_t c = searching ? n - t : 0;
        ranks[i] = (int32_t)c;
        if (pvalues) pvalues[i] = kFew ? p_value(c + 1, n + 1) : (float)((double)(c + 1) / (double)(n + 1));     // alike; many scores hide the longer one
        int cls = 0;
        for (int l = 0; l < lv.n_alpha; ++l) cls += (c + 1 <= lv.r[l]) ? 1 : 0;
        classes[i] = (uint8_t)cls;
    }
}

// ---- classes only: the decision rule in its quantile form (Eq. "quantile") ------------------------------------
// ranks + 1 <= r_l  <=>  fewer than r_l calibration scores are >= s  <=>  s > the (N + 1 - r_l)-th smallest one.
// With the thresholds read from the sorted array once, a class costs n_alpha integer compares and no search:
// a pure streaming pass.  r_l = 0 never rejects, r_l > N always does; a NaN test score (rank 0) is rejected by
// every level with r_l >= 1.
__global__ __launch_bounds__(256) void classify_threshold_kernel(const uint32_t* __restrict__ keys, int64_t n,
                                                                 const float* __restrict__ test, int64_t m, ClassifyLevels lv,
                                                                 uint8_t* __restrict__ classes, float* __restrict__ thresholds) {
    __shared__ uint32_t q_key[ATTS_MAX_ALPHAS];
    if ((int)threadIdx.x < lv.n_alpha) {
        const int64_t kth = n + 1 - lv.r[threadIdx.x];        // 1-indexed order statistic
        const uint32_t qk = (kth >= 1 && kth <= n) ? keys[kth - 1] : 0u;
        q_key[threadIdx.x] = qk;
        if (blockIdx.x == 0 && thresholds)
            thresholds[threadIdx.x] = kth > n ? INFINITY : (kth < 1 ? -INFINITY : key_to_score(qk));
    }
    __syncthreads();
    auto classify_one = [&](float s) {
        const bool nan = score_is_nan(s);
        const uint32_t x = score_to_key(s);
        int cls = 0;
        for (int l = 0; l < lv.n_alpha; ++l) {
            const int64_t r = lv.r[l];
            const bool rej = r > n ? true : (r < 1 ? false : (nan ? true : x > q_key[l]));
            cls += rej ? 1 : 0;
        }
        return (uint32_t)cls;
    };
    // four scores per thread and step: one 16-byte load, one 4-byte store (both arrays are 16- / 4-byte aligned at
    // index 0 whenever the caller's pointers are; a misaligned pair or the tail goes one by one)
    const int64_t stride = (int64_t)gridDim.x * 256;
    const bool vec = ((reinterpret_cast<uintptr_t>(test) & 15) | (reinterpret_cast<uintptr_t>(classes) & 3)) == 0;
    const int64_t m4 = vec ? m / 4 : 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m4; i += stride) {
        const float4 s4 = reinterpret_cast<const float4*>(test)[i];
        const uint32_t packed = classify_one(s4.x) | (classify_one(s4.y) << 8) | (classify_one(s4.z) << 16) | (classify_one(s4.w) << 24);
        reinterpret_cast<uint32_t*>(classes)[i] = packed;
    }
    for (int64_t i = m4 * 4 + (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += stride) classes[i] = (uint8_t)classify_one(test[i]);
}

// ---- conditional coverage: one wavefront per input, its own calibration scores as the set ------------------
struct ConditionalLevels {
    double alpha[ATTS_MAX_ALPHAS];
    int32_t n_alpha;
};

// The work of an input is a few hundred instructions; what takes the time is its chain of loads (offsets, then scores), so both
// offset pairs are requested at once, then up to kCondHeld blocks of calibration scores and the first candidates.  The
// calibration scores go to the wavefront's own LDS and come back four to a read, the same for every lane, and are compared as
// they are (an IEEE comparison, sub-normals kept by the kernel's float mode, is what the rank counts): two vector instructions a
// pair, where a key passing by through a lane read made three, and no conversions.  What bounds it: the chain of loads, and from
// about 200 scores on those two instructions.  8192 inputs of about 400 and 100 scores 58.8 -> 30.7 us, of 200 and 32 17.2 -> 10.1;
// 4096 of 64 and 64 9.1 -> 5.9.
constexpr int kCondHeld = 8;                                     // blocks of 64 calibration scores a wavefront holds
__global__ __launch_bounds__(256) void conditional_kernel(const float* __restrict__ cal, const int64_t* __restrict__ cal_off,
                                                          const float* __restrict__ test, const int64_t* __restrict__ test_off,
                                                          int64_t n_inputs, int32_t* __restrict__ ranks, float* __restrict__ pvalues,
                                                          uint8_t* __restrict__ classes, ConditionalLevels lv) {
    constexpr int kChunk = 64 * kCondHeld;
    __shared__ __attribute__((aligned(16))) float lds[4][kChunk];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t x = (int64_t)blockIdx.x * 4 + wave, xl = min(x, n_inputs - 1);
    const int64_t c0 = cal_off[xl], c1 = cal_off[xl + 1], t0 = test_off[xl], t1 = test_off[xl + 1];
    // everything the wavefront reads as scalars is requested here, not one piece behind each branch
    asm volatile("" ::"s"(c0), "s"(c1), "s"(t0), "s"(t1), "s"(cal), "s"(test), "s"(ranks), "s"(pvalues), "s"(classes), "s"(lv.n_alpha));
    const int64_t m = max((int64_t)0, c1 - c0), k = max((int64_t)0, t1 - t0);
    if (x >= n_inputs || k == 0) return;                         // whole wavefronts leave together
    float* const set = lds[wave];
    const float none = __uint_as_float(0x7FC00000u);             // an absent score: never >= anything
    // calibration scores [at, at + kChunk) into LDS, whole blocks
    auto load_blocks = [&](const float* p, int here, auto count) __attribute__((always_inline)) {
        constexpr int kBlocks = decltype(count)::value;
        float f[kBlocks];
#pragma unroll
        for (int h = 0; h < kBlocks; ++h) f[h] = 64 * h + lane < here ? p[64 * h + lane] : none;
#pragma unroll
        for (int h = 0; h < kBlocks; ++h) set[64 * h + lane] = f[h];
    };
    auto load_chunk = [&](int64_t at) __attribute__((always_inline)) {
        const int here = (int)min(m - at, (int64_t)kChunk);
        if (here <= 128) load_blocks(cal + c0 + at, here, std::integral_constant<int, 2>{});
        else load_blocks(cal + c0 + at, here, std::integral_constant<int, kCondHeld>{});
    };
    float s = lane < k ? test[t0 + lane] : 0.f;
    if (m > 0) load_chunk(0);
    const double n1 = (double)(m + 1);
    for (int64_t tb = 0; tb < k; tb += 64) {
        const float next = tb + 64 + lane < k ? test[t0 + tb + 64 + lane] : 0.f;     // the next block's, in flight meanwhile
        int64_t c = 0;
        for (int64_t at = 0; at < m; at += kChunk) {
            if (m > kChunk && (at > 0 || tb > 0)) {              // every lane has read the chunk before: one wavefront, in order
                __builtin_amdgcn_wave_barrier();
                load_chunk(at);
            }
            __builtin_amdgcn_wave_barrier();
            const int pieces = (int)((min(m - at, (int64_t)kChunk) + 15) >> 4);
            int cnt = 0;
#pragma unroll 1
            for (int j = 0; j < pieces; ++j) {                   // in sixteens: a block is often partly filled
                float4 q[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) q[e] = reinterpret_cast<const float4*>(set)[4 * j + e];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // A comparison's result is added as a carry: four comparisons ahead of their additions, which may read a
                    // mask no sooner than two instructions behind its write (the compiler's pairs wait two slots each: 32.2 us for 30.7).
                    uint64_t b0, b1, b2, b3;
                    asm("v_cmp_ge_f32_e64 %1, %5, %9\n\t"
                        "v_cmp_ge_f32_e64 %2, %6, %9\n\t"
                        "v_cmp_ge_f32_e64 %3, %7, %9\n\t"
                        "v_cmp_ge_f32_e64 %4, %8, %9\n\t"
                        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\t"
                        "v_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
                        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\t"
                        "v_addc_co_u32_e64 %0, %4, 0, %0, %4"
                        : "+v"(cnt), "=&s"(b0), "=&s"(b1), "=&s"(b2), "=&s"(b3)
                        : "v"(q[e].x), "v"(q[e].y), "v"(q[e].z), "v"(q[e].w), "v"(s));
                }
            }
            c += cnt;                                            // a NaN candidate counts nothing
        }
        if (tb + lane < k) {
            const int64_t t = t0 + tb + lane;
            const double c1p = (double)(c + 1);
            ranks[t] = (int32_t)c;
            if (pvalues) pvalues[t] = p_value(c + 1, m + 1);
            int cls = 0;
            for (int l = 0; l < lv.n_alpha; ++l) cls += c1p <= floor(lv.alpha[l] * n1) ? 1 : 0;     // whole numbers below 2^53
            classes[t] = (uint8_t)cls;
        }
        s = next;
    }
}

__global__ void export_kernel(const uint32_t* __restrict__ keys, int64_t n, float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = key_to_score(keys[i]);
}

// keys and the four index levels of an array that is already in key order
struct ImportJob {
    uint32_t* keys;
    uint32_t* index[kIndexLevels];
};
__global__ void import_kernel(const float* __restrict__ scores, int64_t n, ImportJob job) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t k = score_to_key(scores[i]);
    job.keys[i] = k;
#pragma unroll
    for (int lvl = 0; lvl < kIndexLevels; ++lvl) {
        const int shift = kFanBits * (lvl + 1);
        if ((i & (((int64_t)1 << shift) - 1)) == 0) job.index[lvl][i >> shift] = k;
    }
}

// One merge launch producing `total` outputs.
template <bool EMIT>
int32_t launch_merge(atts_calib* c, const MergeJob& job, int64_t total, bool streaming, hipStream_t stream) {
    if (streaming) {
        const int64_t segs = ceil_div(total, kMergeSegLarge);
        if (segs + 1 <= c->splits_len) {
            hipLaunchKernelGGL(merge_split_kernel, dim3((unsigned)ceil_div(segs + 1, 256)), dim3(256), 0, stream, job,
                               kMergeSegLarge, (int)segs, c->splits);
            ATTS_LAUNCH_CHECK("merge_split_kernel");
            hipLaunchKernelGGL((merge_kernel<kMergeSegLarge, EMIT, true>), dim3((unsigned)segs), dim3(kMergeThreads), 0, stream, job, c->splits);
        } else {
            hipLaunchKernelGGL((merge_kernel<kMergeSegLarge, EMIT, false>), dim3((unsigned)segs), dim3(kMergeThreads), 0, stream, job, nullptr);
        }
    } else if (total <= kMergeTinyTo) {
        hipLaunchKernelGGL((merge_kernel<kMergeSegTiny, EMIT, false>), dim3((unsigned)ceil_div(total, kMergeSegTiny)), dim3(kMergeThreads), 0,
                           stream, job, nullptr);
    } else {
        hipLaunchKernelGGL((merge_kernel<kMergeSegSmall, EMIT, false>), dim3((unsigned)ceil_div(total, kMergeSegSmall)), dim3(kMergeThreads), 0,
                           stream, job, nullptr);
    }
    ATTS_LAUNCH_CHECK("merge_kernel");
    return ATTS_OK;
}

}  // namespace
}  // namespace atts

using namespace atts;

extern "C" {

int32_t atts_calib_create(int64_t capacity, atts_calib** out) {
    if (!out) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_create: out is NULL");
    *out = nullptr;
    if (capacity < 1 || capacity > ((int64_t)1 << 30))
        return fail(ATTS_ERR_INVALID_ARG, "atts_calib_create: capacity %lld outside [1, 2^30]", (long long)capacity);
    atts_calib* c = new (std::nothrow) atts_calib();
    if (!c) return fail(ATTS_ERR_HIP, "atts_calib_create: out of host memory");
    c->capacity = capacity;
    c->n = 0;
    c->cur = 0;
    // Every array is rounded up to whole 128-byte lines plus one: the index search reads whole lines (entries
    // past the fill are masked, not avoided), and the sort writes a batch's last run padded to 16 keys and reads the padding, in
    // `runs` and `batch`.
    uint32_t** bufs[5 + 2 * kIndexLevels] = {&c->keys[0], &c->keys[1], &c->runs, &c->batch, &c->sort_scratch};
    int64_t sizes[5 + 2 * kIndexLevels];
    for (int i = 0; i < 4; ++i) sizes[i] = capacity;
    sizes[4] = sort_scratch_words(capacity);
    for (int side = 0; side < 2; ++side)
        for (int k = 0; k < kIndexLevels; ++k) {
            bufs[5 + side * kIndexLevels + k] = &c->index[side][k];
            sizes[5 + side * kIndexLevels + k] = ceil_div(capacity, (int64_t)1 << (kFanBits * (k + 1)));
        }
    constexpr int n_bufs = 5 + 2 * kIndexLevels;
    for (int i = 0; i < n_bufs; ++i) *bufs[i] = nullptr;
    for (int i = 0; i < n_bufs; ++i) {
        const size_t bytes = ((size_t)ceil_div(sizes[i], kFan) * kFan + kFan) * sizeof(uint32_t);
        hipError_t e = hipMalloc(reinterpret_cast<void**>(bufs[i]), bytes);
        if (e != hipSuccess) {
            for (int j = 0; j < n_bufs; ++j)
                if (*bufs[j]) (void)hipFree(*bufs[j]);
            delete c;
            return fail(ATTS_ERR_HIP, "atts_calib_create: hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
        }
    }
    c->splits_len = capacity / kMergeSegLarge + 64;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&c->splits), (size_t)c->splits_len * sizeof(int32_t));
    if (e != hipSuccess) {
        for (int j = 0; j < n_bufs; ++j) (void)hipFree(*bufs[j]);
        delete c;
        return fail(ATTS_ERR_HIP, "atts_calib_create: hipMalloc of the split table failed: %s", hipGetErrorString(e));
    }
    *out = c;
    return ATTS_OK;
}

int32_t atts_calib_destroy(atts_calib* c) {
    if (!c) return ATTS_OK;
    (void)hipFree(c->splits);
    (void)hipFree(c->keys[0]);
    (void)hipFree(c->keys[1]);
    for (int side = 0; side < 2; ++side)
        for (int k = 0; k < kIndexLevels; ++k) (void)hipFree(c->index[side][k]);
    (void)hipFree(c->runs);
    (void)hipFree(c->batch);
    (void)hipFree(c->sort_scratch);
    delete c;
    return ATTS_OK;
}

int32_t atts_calib_size(const atts_calib* c, int64_t* out_n) {
    if (!c || !out_n) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_size: NULL argument");
    *out_n = c->n;
    return ATTS_OK;
}

int32_t atts_calib_reset(atts_calib* c) {
    if (!c) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_reset: NULL handle");
    c->n = 0;
    return ATTS_OK;
}

int32_t atts_calibrate_online(atts_calib* c, const float* new_scores, int64_t n_new, void* hip_stream) {
    if (!c) return fail(ATTS_ERR_INVALID_ARG, "atts_calibrate_online: NULL handle");
    if (n_new < 0) return fail(ATTS_ERR_INVALID_ARG, "atts_calibrate_online: n_new = %lld < 0", (long long)n_new);
    if (n_new == 0) return ATTS_OK;
    if (!new_scores) return fail(ATTS_ERR_INVALID_ARG, "atts_calibrate_online: new_scores is NULL");
    if (c->n + n_new > c->capacity)
        return fail(ATTS_ERR_CAPACITY, "atts_calibrate_online: %lld + %lld scores exceed the capacity %lld", (long long)c->n,
                    (long long)n_new, (long long)c->capacity);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);

    // 1. ascending keys of the new scores (a few scores and a small set: the merge does it itself)
    const int64_t total = c->n + n_new;
    const bool inline_sort = n_new <= kInlineMax && total <= kInlineTotal;
    const uint32_t* sorted = nullptr;
    if (!inline_sort) {
        StageTimer t_(ATTS_STAGE_CALIB_SORT, stream);
        int32_t rc = launch_sort_scores(new_scores, n_new, c->runs, c->batch, c->sort_scratch, &sorted, stream);
        if (rc != ATTS_OK) return rc;
    }

    // 2. merge with the resident array into the other half of the ping-pong buffer (+ its search index)
    const int to = c->cur ^ 1;
    MergeJob job{c->keys[c->cur], c->n, sorted, n_new, c->keys[to], {}, new_scores};
    for (int k = 0; k < kIndexLevels; ++k) job.index[k] = c->index[to][k];
    StageTimer t_(ATTS_STAGE_CALIB_MERGE, stream);
    if (inline_sort) {
        if (total <= kMergeTinyTo)
            hipLaunchKernelGGL((merge_kernel<kMergeSegTiny, true, false, true>), dim3((unsigned)ceil_div(total, kMergeSegTiny)), dim3(kMergeThreads),
                               0, stream, job, nullptr);
        else
            hipLaunchKernelGGL((merge_kernel<kMergeSegSmall, true, false, true>), dim3((unsigned)ceil_div(total, kMergeSegSmall)),
                               dim3(kMergeThreads), 0, stream, job, nullptr);
        ATTS_LAUNCH_CHECK("merge_kernel");
    } else {
        int32_t rc = launch_merge<true>(c, job, total, total >= kMergeLargeFrom, stream);
        if (rc != ATTS_OK) return rc;
    }
    c->cur ^= 1;
    c->n += n_new;
    return ATTS_OK;
}

int32_t atts_classify_ordinal(const atts_calib* c, const float* test_scores, int64_t M, const double* alphas, int32_t n_alpha,
                              int32_t* ranks, float* pvalues, uint8_t* classes, float* thresholds, void* hip_stream) {
    if (!c) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: NULL handle");
    if (M < 0) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: M = %lld < 0", (long long)M);
    if (!alphas || n_alpha < 1 || n_alpha > ATTS_MAX_ALPHAS)
        return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: need 1..%d alpha levels", ATTS_MAX_ALPHAS);
    for (int l = 0; l < n_alpha; ++l) {
        if (!(alphas[l] > 0.0 && alphas[l] < 1.0))
            return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: alpha[%d] = %g is not inside (0, 1)", l, alphas[l]);
        if (l > 0 && alphas[l] < alphas[l - 1])
            return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: alpha levels must be non-decreasing");
    }
    if (c->n < 1) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: the calibration set is empty");
    if (M > 0 && (!test_scores || !classes))
        return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: test_scores and classes must not be NULL");
    if (!ranks && pvalues) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: pvalues without ranks");
    if (M > ((int64_t)1 << 31) * 255) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_ordinal: M too large");
    ClassifyLevels lv;
    lv.n_alpha = n_alpha;
    for (int l = 0; l < ATTS_MAX_ALPHAS; ++l) lv.r[l] = 0;
    for (int l = 0; l < n_alpha; ++l) lv.r[l] = (int64_t)floor(alphas[l] * (double)(c->n + 1));
    if (M == 0 && !thresholds) return ATTS_OK;
    if (!ranks) {
        // decisions only: compare with the thresholds, no search
        const int64_t want = M > 0 ? ceil_div(M, (int64_t)256 * 16) : 1;
        const unsigned blocks = (unsigned)(want < 1 ? 1 : (want > 4096 ? 4096 : want));
        StageTimer t_(ATTS_STAGE_CLASSIFY, static_cast<hipStream_t>(hip_stream));
        hipLaunchKernelGGL(classify_threshold_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                           c->keys[c->cur], c->n, test_scores, M, lv, classes, thresholds);
        ATTS_LAUNCH_CHECK("classify_threshold_kernel");
        return ATTS_OK;
    }
    SearchIndex ix;
    ix.lvl[0] = c->keys[c->cur];
    ix.len[0] = c->n;
    for (int k = 1; k <= kIndexLevels; ++k) {
        ix.lvl[k] = c->index[c->cur][k - 1];
        ix.len[k] = ceil_div(c->n, (int64_t)1 << (kFanBits * k));
    }
    ix.top_level = 0;
    while (ix.top_level < kIndexLevels && ix.len[ix.top_level] > kTopEntries) ++ix.top_level;
    ix.top_shift = 0;
    while (ceil_div(ix.len[ix.top_level], (int64_t)1 << ix.top_shift) > kTopEntries) ++ix.top_shift;
    // Enough workgroups to fill the chip, few enough that staging the top level stays a small part of the work.  A search is a
    // chain of memory latencies, so many scores take workgroups of 512 threads: the staged 32 KB leave room for five workgroups on
    // a CU (four with kFew's spare entries, of which 2^19 scores take up to eight), which are 20 wavefronts of 32 with 256 threads.  With both
    // changes (quad_rounds) 2^24 scores against 2^28 keys take 713 us for 770 (5.0 GB of lines from beyond the L2 by the counters: 7 TB/s, bandwidth
    // now bounds it), with many ties 330 for 488, 2^22 against 2^26 153 for 174.  Fewer stay spread over more CUs, in the form for few at every
    // size: against halving and plain staging 65,536 scores in 8192 keys 3.6 and 6.5 us, in 2^20 4.75 and 4.9, 200,000 in 5000 4.2 and 5.3,
    // 524,287 in 2^23 18.9 and 34.9, in 500,000 10.6 and 10.5.
    const bool large = M >= (int64_t)256 * 2048;
    const int threads = large ? 512 : 256;
    int64_t per = M / ((int64_t)threads * 1024);
    ix.per_thread = (int32_t)(per < 1 ? 1 : (per > 16 ? 16 : per));
    const unsigned blocks = (unsigned)(M > 0 ? ceil_div(M, (int64_t)threads * ix.per_thread) : 1);
    StageTimer t_(ATTS_STAGE_CLASSIFY, static_cast<hipStream_t>(hip_stream));
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3((unsigned)threads), 0, static_cast<hipStream_t>(hip_stream), ix, test_scores, M, lv, ranks,
                           pvalues, classes, thresholds);
    };
    if (ix.per_thread > 1) launch(classify_kernel<512, false>);
    else if (large) launch(classify_kernel<512, true>);
    else launch(classify_kernel<256, true>);
    ATTS_LAUNCH_CHECK("classify_kernel");
    return ATTS_OK;
}

int32_t atts_classify_conditional(const float* cal_scores, const int64_t* cal_offsets, const float* test_scores,
                                  const int64_t* test_offsets, int64_t n_inputs, const double* alphas, int32_t n_alpha,
                                  int32_t* ranks, float* pvalues, uint8_t* classes, void* hip_stream) {
    if (n_inputs < 0) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_conditional: n_inputs = %lld < 0", (long long)n_inputs);
    if (!alphas || n_alpha < 1 || n_alpha > ATTS_MAX_ALPHAS)
        return fail(ATTS_ERR_INVALID_ARG, "atts_classify_conditional: need 1..%d alpha levels", ATTS_MAX_ALPHAS);
    ConditionalLevels lv;
    lv.n_alpha = n_alpha;
    for (int l = 0; l < ATTS_MAX_ALPHAS; ++l) lv.alpha[l] = 0.0;
    for (int l = 0; l < n_alpha; ++l) {
        if (!(alphas[l] > 0.0 && alphas[l] < 1.0))
            return fail(ATTS_ERR_INVALID_ARG, "atts_classify_conditional: alpha[%d] = %g is not inside (0, 1)", l, alphas[l]);
        if (l > 0 && alphas[l] < alphas[l - 1])
            return fail(ATTS_ERR_INVALID_ARG, "atts_classify_conditional: alpha levels must be non-decreasing");
        lv.alpha[l] = alphas[l];
    }
    if (n_inputs == 0) return ATTS_OK;
    if (!cal_offsets || !test_offsets) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_conditional: offsets must not be NULL");
    // score and output arrays may be NULL only if every range is empty, which the host cannot see: require them
    if (!cal_scores || !test_scores || !ranks || !classes)
        return fail(ATTS_ERR_INVALID_ARG, "atts_classify_conditional: cal_scores, test_scores, ranks and classes must not be NULL");
    if (n_inputs > ((int64_t)1 << 31) * 2) return fail(ATTS_ERR_INVALID_ARG, "atts_classify_conditional: too many inputs");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    StageTimer t_(ATTS_STAGE_CLASSIFY, stream);
    hipLaunchKernelGGL(conditional_kernel, dim3((unsigned)ceil_div(n_inputs, 4)), dim3(256), 0, stream, cal_scores, cal_offsets,
                       test_scores, test_offsets, n_inputs, ranks, pvalues, classes, lv);
    ATTS_LAUNCH_CHECK("conditional_kernel");
    return ATTS_OK;
}

int32_t atts_calib_export(const atts_calib* c, float* out, void* hip_stream) {
    if (!c) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_export: NULL handle");
    if (c->n == 0) return ATTS_OK;
    if (!out) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_export: out is NULL");
    hipLaunchKernelGGL(export_kernel, dim3((unsigned)ceil_div(c->n, 256)), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       c->keys[c->cur], c->n, out);
    ATTS_LAUNCH_CHECK("export_kernel");
    return ATTS_OK;
}

int32_t atts_calib_import(atts_calib* c, const float* scores, int64_t n, void* hip_stream) {
    if (!c) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_import: NULL handle");
    if (n < 0) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_import: n = %lld < 0", (long long)n);
    if (n > c->capacity)
        return fail(ATTS_ERR_CAPACITY, "atts_calib_import: %lld scores exceed the capacity %lld", (long long)n, (long long)c->capacity);
    if (n > 0 && !scores) return fail(ATTS_ERR_INVALID_ARG, "atts_calib_import: scores is NULL");
    if (n > 0) {
        ImportJob job{c->keys[c->cur], {}};
        for (int k = 0; k < kIndexLevels; ++k) job.index[k] = c->index[c->cur][k];
        hipLaunchKernelGGL(import_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, static_cast<hipStream_t>(hip_stream), scores, n, job);
        ATTS_LAUNCH_CHECK("import_kernel");
    }
    c->n = n;
    return ATTS_OK;
}

}  // extern "C"
