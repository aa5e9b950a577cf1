// Sorting a batch of new conformity scores into ascending keys (first half of "Online Calibration": the
// scores of newly pre-sampled outputs join the calibration multiset, which this library keeps sorted).
//
// Two regimes:
//   * up to kSmallSortMax scores (cache-resident, latency-bound): every workgroup sorts one run in registers
//     (block_sort_kernel), and where there are several, ONE further launch cuts them all at sampled keys and sorts the
//     buckets in between (bucket_sort_kernel).
//   * larger batches (bandwidth-bound): least-significant-digit radix sort, four passes of 8 bits.  A pass is
//     three launches: digit histograms of groups of tiles, a scan per digit over the groups, and a stable scatter (ranks
//     inside a tile by wavefront-wide digit matching, keys reordered through LDS so that each digit's keys of a
//     tile leave as one contiguous run).
// No inter-workgroup waiting anywhere.
#include "common.h"
#include "keys.h"
#include "block_sort.h"

namespace atts {
namespace {

// ------------------------------------------------------------------------------------------------------------
// small batches: sorted runs, then buckets between sampled keys
// ------------------------------------------------------------------------------------------------------------
constexpr int kRunMax = 8192;                // keys of the longest run: one workgroup of 1024 threads
constexpr int kSmallSortMax = 1 << 19;       // 64 runs of kRunMax
constexpr int kMaxRuns = 64;
constexpr int kSpacing = 64;                 // every 64th key of a run is a sample
constexpr int kSamplesMin = 8, kSamplesMax = 32;    // samples per bucket: about 512, 1024 or 2048 keys
constexpr int kBucketThreads = 1024;
constexpr int kBucketCap = kPer * kBucketThreads;
constexpr int kFewThreads = 512;             // ... and for few runs (of 2048 keys)
constexpr int kFewRuns = 32;
// a bucket's keys lie strictly between two splitters with at most q samples between them: at most kSpacing q keys, and from
// every run fewer than kSpacing more
static_assert(kSpacing * (kSamplesMax + kMaxRuns) <= kBucketCap && kSmallSortMax / kSpacing <= kBucketCap, "a workgroup holds a bucket, and all samples");
static_assert(kSpacing * (16 + kFewRuns) <= kPer * kFewThreads && kFewRuns * 16 <= kFewThreads && kMaxRuns * 16 <= kBucketThreads, "");
static_assert(kMaxRuns * kRunMax == kSmallSortMax && kSamplesMin % kPer == 0 && kSmallSortMax / kSpacing / kSamplesMax <= kBucketThreads, "");

// Every workgroup turns 8 THREADS scores into one ascending run; samples != NULL: every kSpacing-th key of it also goes there,
// run after run.  The last run is padded with kPadKey up to a multiple of 16 keys.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void block_sort_kernel(const float* __restrict__ scores, int64_t n, uint32_t* __restrict__ runs,
                                                             uint32_t* __restrict__ samples) {
    constexpr int kRun = kPer * THREADS;
    __shared__ __attribute__((aligned(16))) uint32_t buf[THREADS > 64 ? 2 * kRun : 4];
    const int64_t base = (int64_t)blockIdx.x * kRun;
    const int tid = threadIdx.x;
    float f[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) f[e] = scores[min(base + e * THREADS + tid, n - 1)];       // any order will do: coalesced
    uint32_t k[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) k[e] = base + e * THREADS + tid < n ? score_to_key(f[e]) : kPadKey;
    sort_in_block<THREADS>(k, kRun, buf);
    const int64_t at = base + tid * kPer, n16 = (n + 15) & ~(int64_t)15;
    if (at < n16) {                                                // whole groups of eight: n16 is a multiple
        reinterpret_cast<uint4*>(runs + at)[0] = make_uint4(k[0], k[1], k[2], k[3]);
        reinterpret_cast<uint4*>(runs + at)[1] = make_uint4(k[4], k[5], k[6], k[7]);
    }
    if (samples && at < n && tid % (kSpacing / kPer) == 0) samples[at / kSpacing] = k[0];
}

// Bucket b of the sorted batch: with S the sorted samples of all runs, the keys strictly between S[b q] and S[(b + 1) q] (no
// lower limit in the first bucket, no upper one in the last), and its share of the keys equal to S[b q], whose number is
// known without moving them.  Regular samples bound a bucket whatever the scores are (ties included: equal splitters share
// their value's range evenly), and no workgroup waits for another: each sorts the samples for itself, finds its limits in every
// run (the samples lead to one block of 64 keys, read in 16-byte pieces), gathers the segments between them and sorts those.
// What bounds it is its chain of steps (two sorts, the limits, the gathering), one bucket per CU: 65,536 scores 12 us behind
// 5.2 for the runs, where runs of 8192 keys merged through LDS and one pass that searched every key's place in the other runs took
// 25 + 14.  With the merge into an empty set 131,072 scores take 27 us, 262,144 33 and 524,288 47, by radix sort 65, 66 and 69 (which is why the
// line to it lies here: its launches are a floor, and 64 runs of one workgroup's keys end at 2^19).  Up to 32 runs by workgroups of 512
// threads: 0.6 us less.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void bucket_sort_kernel(const uint32_t* __restrict__ runs, int64_t n, int run_len, int n_runs,
                                                              const uint32_t* __restrict__ samples, int n_samples, int q,
                                                              uint32_t* __restrict__ out) {
    constexpr int kCap = kPer * THREADS, kRuns = THREADS / 16;
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    uint32_t* const buf = lds;                                     // 2 kCap: exchanges; then the gathered keys
    uint32_t* const smp = lds + 2 * kCap;                          // the samples, run after run
    __shared__ uint32_t splitter[kCap / kSamplesMin];
    __shared__ int below[3][kRuns];                                // keys of a run below / not above the lower limit, below the upper one
    __shared__ int seg_at[64 + 1];
    __shared__ int sum_lo[2];
    const int tid = threadIdx.x, b = blockIdx.x, n_buckets = gridDim.x;
    auto size_for = [](int m) {
        int size = kWaveKeys;
        while (size < m) size *= 2;
        return size;
    };
    uint32_t k[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) k[e] = samples[min(e * THREADS + tid, n_samples - 1)];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        const int i = e * THREADS + tid;
        if (i < n_samples) smp[i] = k[e];
        else k[e] = kPadKey;
    }
    // the network's places are thread-major: keep its first `size` places full when there are fewer samples than places
    if (n_samples <= kCap / 2) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kPer; ++e) k[e] = tid * kPer + e < n_samples ? smp[tid * kPer + e] : kPadKey;
    }
    sort_in_block<THREADS>(k, size_for(n_samples), buf);
    if (tid * kPer % q == 0) splitter[tid * kPer / q] = k[0];
    __syncthreads();
    const bool has_lo = b > 0, has_hi = b + 1 < n_buckets;
    const uint32_t lo = splitter[b], hi = splitter[has_hi ? b + 1 : b];
    // the splitters equal to lo, and those of them before this one
    const bool same = tid >= 1 && tid < n_buckets && splitter[tid] == lo;
    const int n_same = __syncthreads_count(same), my_same = __syncthreads_count(same && tid < b);
    {
        // Sixteen threads a run: the samples lead to one block of 64 keys for each of the three limits, of which every thread takes
        // 16 bytes; all three are requested before the first is counted (one thread a limit, with sixteen loads of its own: 3.2 us
        // of a workgroup's 11 at 65,536 scores, now 1.9).
        const int r = tid >> 4, l16 = tid & 15;
        if (r < n_runs) {
            const int len = (int)min((int64_t)run_len, n - (int64_t)r * run_len);
            const uint32_t* s = smp + r * (run_len / kSpacing);
            const uint32_t* run = runs + (int64_t)r * run_len;
            int first[3];                                          // -1: no sample lies below the limit, so no key does
            uint4 piece[3];
#pragma unroll
            for (int kind = 0; kind < 3; ++kind) {
                const uint32_t v = kind < 2 ? lo : hi;
                int x = 0, y = (len + kSpacing - 1) / kSpacing;    // samples below v
                while (x < y) {
                    const int mid = (x + y) >> 1;
                    if (s[mid] < v || (kind == 1 && s[mid] == v)) x = mid + 1; else y = mid;
                }
                first[kind] = (x - 1) * kSpacing;                  // the limit lies in the block of the last of them
                const int at = max(first[kind], 0) + 4 * l16;
                piece[kind] = reinterpret_cast<const uint4*>(run)[min(at, len - 1) >> 2];
            }
#pragma unroll
            for (int kind = 0; kind < 3; ++kind) {
                const uint32_t v = kind < 2 ? lo : hi;
                const int at = first[kind] + 4 * l16;
                auto goes = [&](uint32_t key, int i) { return (at + i < len && (key < v || (kind == 1 && key == v))) ? 1 : 0; };
                int count = goes(piece[kind].x, 0) + goes(piece[kind].y, 1) + goes(piece[kind].z, 2) + goes(piece[kind].w, 3);
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) count += __shfl_xor(count, o);
                count = first[kind] < 0 ? 0 : first[kind] + count;
                if (kind < 2 ? !has_lo : !has_hi) count = kind < 2 ? 0 : len;
                if (l16 == 0) below[kind][r] = count;
            }
        }
    }
    __syncthreads();
    if (tid < 64) {                                                // one lane per run: the segments side by side
        const int from = tid < n_runs ? below[1][tid] : 0;
        const int len = tid < n_runs ? max(below[2][tid] - from, 0) : 0;
        int at = len, s0 = tid < n_runs ? below[0][tid] : 0, s1 = from;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(at, o);
            if (tid >= o) at += up;
            s0 += __shfl_xor(s0, o);
            s1 += __shfl_xor(s1, o);
        }
        seg_at[tid + 1] = at;
        if (tid == 0) {
            seg_at[0] = 0;
            sum_lo[0] = s0;
            sum_lo[1] = s1;
        }
    }
    __syncthreads();
    const int m = seg_at[64];                                // at most kCap
    {
        const int r = tid >> 4;                                    // sixteen threads per run
        if (r < n_runs) {
            const int at = seg_at[r], len = seg_at[r + 1] - at;
            const uint32_t* src = runs + (int64_t)r * run_len + below[1][r];
            for (int i0 = tid & 15; i0 < len; i0 += 64) {          // four requested together
                uint32_t x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = src[min(i0 + 16 * u, len - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i0 + 16 * u < len) buf[at + i0 + 16 * u] = x[u];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPer; ++e) k[e] = tid * kPer + e < m ? buf[tid * kPer + e] : kPadKey;
    __syncthreads();
    sort_in_block<THREADS>(k, size_for(m), buf);
    __syncthreads();
    reinterpret_cast<uint4*>(buf)[2 * tid] = make_uint4(k[0], k[1], k[2], k[3]);
    reinterpret_cast<uint4*>(buf)[2 * tid + 1] = make_uint4(k[4], k[5], k[6], k[7]);
    __syncthreads();
    uint32_t* const o = out + sum_lo[1];
    for (int i = tid; i < m; i += THREADS) o[i] = buf[i];
    if (has_lo) {
        const int64_t width = sum_lo[1] - sum_lo[0];
        const int f0 = sum_lo[0] + (int)(width * my_same / n_same), f1 = sum_lo[0] + (int)(width * (my_same + 1) / n_same);
        for (int i = f0 + tid; i < f1; i += THREADS) out[i] = lo;
    }
}

// ------------------------------------------------------------------------------------------------------------
// large batches: LSD radix sort, 8 bits per pass
// ------------------------------------------------------------------------------------------------------------
constexpr int kRadixThreads = 256;
constexpr int kRadixItems = 16;                              // keys per thread
constexpr int kRadixTile = kRadixThreads * kRadixItems;      // 4096 keys per workgroup
constexpr int kRadixBins = 256;

// exclusive prefix of v over the 256 threads of the workgroup (thread order) and the total; red: 4 words of LDS
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* red, uint32_t& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    __syncthreads();
    if (lane == 63) red[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kRadixThreads / 64; ++w) {
        const uint32_t r = red[w];
        before += w < wave ? r : 0u;
        all += r;
    }
    total = all;
    return before + incl - v;
}

// key of element idx of the pass input: the first pass reads the scores themselves
template <bool FIRST>
__device__ __forceinline__ uint32_t load_key(const void* __restrict__ in, int64_t idx) {
    if constexpr (FIRST) return score_to_key(reinterpret_cast<const float*>(in)[idx]);
    else return reinterpret_cast<const uint32_t*>(in)[idx];
}

// Digit counts, [tile][digit].  A workgroup walks a group of `per_group` consecutive tiles and keeps one running histogram: the row of
// the group's first tile gets the group's totals (the scan turns them into the group's offsets), every other row the counts of the tiles
// before it in the group.  So the scan has at most 256 groups to add up, and all rows are written and read whole: a histogram per tile stored
// digit by digit cost a 4-byte access to 256 lines a tile here and in the scatter, and a scan over all tiles (2^24 keys, four passes:
// histograms 96 -> 59 us, scans 46 -> 20; the sort 350 -> 284, of one value 473 -> 294).  Four copies of the bins, 16 banks apart, lanes in turn: neighbouring keys often
// share a high digit, and an LDS atomic takes the lanes of one address one by one.
constexpr int kHistThreads = 1024, kHistCopies = 4, kHistPitch = kRadixBins + 16;
template <bool FIRST>
__global__ __launch_bounds__(kHistThreads) void radix_hist_kernel(const void* __restrict__ in, int64_t n, int shift, int n_tiles, int per_group,
                                                                  uint32_t* __restrict__ counts) {
    constexpr int kKeys = kRadixTile / kHistThreads;
    __shared__ uint32_t h[kHistCopies][kHistPitch];
    const int tid = threadIdx.x, first = blockIdx.x * per_group, last = min(first + per_group, n_tiles);
    if (tid < kRadixBins) {
#pragma unroll
        for (int c = 0; c < kHistCopies; ++c) h[c][tid] = 0;
    }
    auto sum = [&]() __attribute__((always_inline)) { return h[0][tid] + h[1][tid] + h[2][tid] + h[3][tid]; };
    auto load = [&](int tile, uint32_t (&k)[kKeys]) __attribute__((always_inline)) {
        const int64_t base = (int64_t)tile * kRadixTile;
#pragma unroll
        for (int i = 0; i < kKeys; ++i) k[i] = load_key<FIRST>(in, min(base + i * kHistThreads + tid, n - 1));
    };
    uint32_t key[kKeys], next[kKeys];
    load(first, key);
    for (int tile = first; tile < last; ++tile) {
        load(min(tile + 1, last - 1), next);
        __syncthreads();                                     // the tile before is counted (or the bins are clear)
        if (tile > first && tid < kRadixBins) counts[(int64_t)tile * kRadixBins + tid] = sum();
        __syncthreads();
        const int64_t base = (int64_t)tile * kRadixTile;
#pragma unroll
        for (int i = 0; i < kKeys; ++i) {
            if (base + i * kHistThreads + tid < n) atomicAdd(&h[tid & (kHistCopies - 1)][(key[i] >> shift) & 255u], 1u);
            key[i] = next[i];
        }
    }
    __syncthreads();
    if (tid < kRadixBins) counts[(int64_t)first * kRadixBins + tid] = sum();
}

// One workgroup per digit d: the groups' totals become their exclusive prefix over the groups (at most 256), digit_tot[d] the digit's total.
__global__ __launch_bounds__(kRadixThreads) void radix_scan_kernel(uint32_t* __restrict__ counts, int n_groups, int per_group,
                                                                   uint32_t* __restrict__ digit_tot) {
    __shared__ uint32_t red[4];
    uint32_t* const p = counts + (int64_t)threadIdx.x * per_group * kRadixBins + blockIdx.x;
    const uint32_t v = (int)threadIdx.x < n_groups ? *p : 0u;
    uint32_t total;
    const uint32_t ex = block_excl_scan(v, red, total);
    if ((int)threadIdx.x < n_groups) *p = ex;
    if (threadIdx.x == 0) digit_tot[blockIdx.x] = total;
}

// Stable scatter of one tile.  Order inside the tile: wavefront w owns a quarter of the tile (consecutive keys) and walks
// it in rounds of 64 consecutive keys.  In a round, the lanes that hold the same digit find each other with
// 8 ballots; a key's rank among its digit's keys of the wavefront = the digit's count so far (an LDS counter per
// wavefront and digit, read by all lanes of the group, advanced by its lowest lane) + the group's lanes below it.
// Prefixes over the wavefronts and digits then give every key its place in the tile's digit-sorted order; the
// keys go to that place in LDS and leave in tile order, so each digit's keys are written as one contiguous run.
template <bool FIRST>
__global__ __launch_bounds__(kRadixThreads) void radix_scatter_kernel(const void* __restrict__ in, int64_t n, int shift,
                                                                      int per_group, const uint32_t* __restrict__ counts,
                                                                      const uint32_t* __restrict__ digit_tot,
                                                                      uint32_t* __restrict__ out) {
    constexpr int kWaves = kRadixThreads / 64;
    __shared__ uint32_t wcnt[kWaves][kRadixBins];
    __shared__ uint32_t lkeys[kRadixTile];
    __shared__ uint32_t gdelta[kRadixBins];     // global position of a key = gdelta[digit] + its place in the tile (mod 2^32)
    __shared__ uint32_t lstart[kRadixBins];     // first place of the digit in the tile's digit-sorted order
    __shared__ uint32_t red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t base = (int64_t)blockIdx.x * kRadixTile + (int64_t)wave * (64 * kRadixItems);
    // keys of digit tid in the tiles before this one: its group's offset, and the tiles before it in the group
    const int group_first = (int)blockIdx.x / per_group * per_group;
    uint32_t before = counts[(int64_t)group_first * kRadixBins + tid];
    if ((int)blockIdx.x != group_first) before += counts[(int64_t)blockIdx.x * kRadixBins + tid];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) wcnt[w][tid] = 0;
    uint32_t key[kRadixItems];
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        const int64_t idx = base + i * 64 + lane;
        key[i] = idx < n ? load_key<FIRST>(in, idx) : kPadKey;
    }
    __syncthreads();
    volatile uint32_t* mine = wcnt[wave];
    const uint64_t below_me = ((uint64_t)1 << lane) - 1;
    uint32_t rank[kRadixItems];
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        const bool valid = base + i * 64 + lane < n;
        const uint32_t d = (key[i] >> shift) & 255u;
        const uint64_t live = __ballot(valid);
        uint32_t g_lo = (uint32_t)live, g_hi = (uint32_t)(live >> 32);     // lanes whose digit equals this lane's
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t mb = 0u - ((d >> b) & 1u);                       // all ones if the bit is set
            const uint64_t vote = __ballot(mb != 0u);
            g_lo &= ~((uint32_t)vote ^ mb);
            g_hi &= ~((uint32_t)(vote >> 32) ^ mb);
        }
        const uint32_t so_far = mine[d];
        const uint32_t lower = (uint32_t)(__popc(g_lo & (uint32_t)below_me) + __popc(g_hi & (uint32_t)(below_me >> 32)));
        rank[i] = so_far + lower;
        __builtin_amdgcn_wave_barrier();                      // every lane has read the counter before its group's leader advances it
        if (valid && lower == 0) mine[d] = so_far + (uint32_t)(__popc(g_lo) + __popc(g_hi));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread d: prefixes of digit d over the wavefronts, the digit's count in the tile, its global offset
    uint32_t cnt = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = wcnt[w][tid];
        wcnt[w][tid] = cnt;
        cnt += c;
    }
    uint32_t tile_total, all;
    const uint32_t first = block_excl_scan(cnt, red, tile_total);
    const uint32_t digit_base = block_excl_scan(digit_tot[tid], red, all);
    lstart[tid] = first;
    gdelta[tid] = digit_base + before - first;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRadixItems; ++i) {
        if (base + i * 64 + lane < n) {
            const uint32_t d = (key[i] >> shift) & 255u;
            lkeys[lstart[d] + wcnt[wave][d] + rank[i]] = key[i];
        }
    }
    __syncthreads();
    for (uint32_t j = tid; j < tile_total; j += kRadixThreads) {
        const uint32_t k = lkeys[j];
        out[gdelta[(k >> shift) & 255u] + j] = k;
    }
}

template <bool FIRST>
int32_t radix_pass(const void* in, int64_t n, int shift, int n_tiles, uint32_t* counts, uint32_t* out, hipStream_t stream) {
    uint32_t* digit_tot = counts + (int64_t)kRadixBins * n_tiles;
    const int per_group = (int)ceil_div(n_tiles, kRadixBins), n_groups = (int)ceil_div(n_tiles, per_group);
    hipLaunchKernelGGL(radix_hist_kernel<FIRST>, dim3((unsigned)n_groups), dim3(kHistThreads), 0, stream, in, n, shift, n_tiles, per_group, counts);
    ATTS_LAUNCH_CHECK("radix_hist_kernel");
    hipLaunchKernelGGL(radix_scan_kernel, dim3(kRadixBins), dim3(kRadixThreads), 0, stream, counts, n_groups, per_group, digit_tot);
    ATTS_LAUNCH_CHECK("radix_scan_kernel");
    hipLaunchKernelGGL(radix_scatter_kernel<FIRST>, dim3((unsigned)n_tiles), dim3(kRadixThreads), 0, stream, in, n, shift, per_group,
                       counts, digit_tot, out);
    ATTS_LAUNCH_CHECK("radix_scatter_kernel");
    return ATTS_OK;
}

}  // namespace

// radix sort: a digit histogram per tile + the digit totals; sorted runs: one sample in 64 keys, which is less
int64_t sort_scratch_words(int64_t n) { return (int64_t)kRadixBins * ceil_div(n > 0 ? n : 1, kRadixTile) + kRadixBins; }

int32_t launch_sort_scores(const float* scores, int64_t n, uint32_t* a, uint32_t* b, uint32_t* scratch, const uint32_t** sorted,
                           hipStream_t stream) {
    if (n <= kSmallSortMax) {
        // one run up to kRunMax scores; more: the shortest runs of which kMaxRuns hold the batch
        const int64_t run = n <= kRunMax ? kRunMax : (n <= 2048 * kMaxRuns ? 2048 : (n <= 4096 * kMaxRuns ? 4096 : 8192));
        const int n_runs = (int)ceil_div(n, run);
        uint32_t* samples = n_runs > 1 ? scratch : nullptr;
        const dim3 grid((unsigned)n_runs);
        if (n <= 512) hipLaunchKernelGGL(block_sort_kernel<64>, grid, dim3(64), 0, stream, scores, n, a, samples);
        else if (n <= 1024) hipLaunchKernelGGL(block_sort_kernel<128>, grid, dim3(128), 0, stream, scores, n, a, samples);
        else if (n <= 2048 || run == 2048) hipLaunchKernelGGL(block_sort_kernel<256>, grid, dim3(256), 0, stream, scores, n, a, samples);
        else if (n <= 4096 || run == 4096) hipLaunchKernelGGL(block_sort_kernel<512>, grid, dim3(512), 0, stream, scores, n, a, samples);
        else hipLaunchKernelGGL(block_sort_kernel<1024>, grid, dim3(1024), 0, stream, scores, n, a, samples);
        ATTS_LAUNCH_CHECK("block_sort_kernel");
        *sorted = a;
        if (n_runs > 1) {
            const int n_samples = (int)ceil_div(n, kSpacing);
            // a bucket takes a CU's LDS: at most 256.  Shorter ones while they are few: 20,000 scores 1.3 us less with 8 samples than
            // with 16, 65,536 the same
            const int q = n_samples <= 128 * kSamplesMin ? kSamplesMin : (n_samples <= 256 * 16 ? 16 : kSamplesMax);
            const int threads = n_runs <= kFewRuns ? kFewThreads : kBucketThreads;
            const size_t lds = (size_t)(2 * kPer * threads + align_up((size_t)n_samples, 4)) * sizeof(uint32_t);
            const dim3 buckets((unsigned)ceil_div(n_samples, q));
            if (threads == kFewThreads) {
                hipLaunchKernelGGL(bucket_sort_kernel<kFewThreads>, buckets, dim3(kFewThreads), lds, stream, a, n, (int)run, n_runs, samples, n_samples, q, b);
            } else {
                int32_t rc = allow_dynamic_lds<bucket_sort_kernel<kBucketThreads>>((size_t)3 * kBucketCap * sizeof(uint32_t));
                if (rc != ATTS_OK) return rc;
                hipLaunchKernelGGL(bucket_sort_kernel<kBucketThreads>, buckets, dim3(kBucketThreads), lds, stream, a, n, (int)run, n_runs, samples, n_samples, q, b);
            }
            ATTS_LAUNCH_CHECK("bucket_sort_kernel");
            *sorted = b;
        }
        return ATTS_OK;
    }
    const int n_tiles = (int)ceil_div(n, kRadixTile);
    int32_t rc = radix_pass<true>(scores, n, 0, n_tiles, scratch, a, stream);
    if (rc == ATTS_OK) rc = radix_pass<false>(a, n, 8, n_tiles, scratch, b, stream);
    if (rc == ATTS_OK) rc = radix_pass<false>(b, n, 16, n_tiles, scratch, a, stream);
    if (rc == ATTS_OK) rc = radix_pass<false>(a, n, 24, n_tiles, scratch, b, stream);
    *sorted = b;
    return rc;
}

}  // namespace atts
