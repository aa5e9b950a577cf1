// Shared-prefix (token-tree) attention.
//
// Rows of the call are laid out [prefix (P) | draft 0 (T) | ... | draft K-1 (T)].  All K drafts
// continue the same prompt, so the prefix keys/values exist once and every draft row attends
// to them ("shared-prefix mechanism", Introduction); a draft row additionally attends causally
// to the rows of its own draft.  With seg(r) = first row of r's draft (0 for a prefix row):
//     key j visible to query r   <=>   j <= r  and  (j < P  or  j >= seg(r)).
// This is exactly K independent causal sequences [prefix ; draft_k], evaluated without
// recomputing or re-storing the prefix.
//
// Four kernels:
//   * attn_mfma_kernel  bf16, head_dim 128: flash-style, 128 or 256 query rows of one head per
//     workgroup, key/value tiles of 64 rows staged in LDS and shared by its wavefronts.
//     Works on transposed products so that no register transpose is needed:
//        S^T = K Q^T   (32 keys x 32 queries per MFMA block; a lane owns ONE query column,
//                       so the online-softmax statistics are per lane)
//        O^T = V^T P^T (P^T is fed straight from the S^T accumulator registers; V^T tiles
//                       come from a [n_kv, hd, rows] copy of V written after the QKV GEMM)
//   * attn_split_kernel the same products for few query rows: 32 per workgroup, the keys divided among
//     its wavefronts.
//   * attn_rows_kernel  heads of 4 to 32 16-byte pieces: one wavefront per (row, head), in registers; used by the fp32 model.
//   * attn_simple_kernel any dtype / head_dim: one wavefront per (row, head).
#include "common.h"

#include <type_traits>

namespace atts {
namespace {

__device__ __forceinline__ int align_up_int(int x, int a) { return (x + a - 1) / a * a; }
__device__ __forceinline__ int seg_start(int r, int P, int T) { return r < P ? 0 : P + (r - P) / T * T; }

// ------------------------------------------------------------------------------------------
// Simple kernel
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(64) void attn_simple_kernel(const T* __restrict__ qkv, T* __restrict__ out, int row0, int P, int Tn,
                                                         int nq, int nkv, int hd, float scale) {
    extern __shared__ float sm[];           // [hd] query, then [n_keys] scores
    float* sq = sm;
    float* sp = sm + hd;
    const int r = row0 + blockIdx.x, head = blockIdx.y, lane = threadIdx.x;
    const int kvh = head / (nq / nkv);
    const int64_t ld = (int64_t)(nq + 2 * nkv) * hd;
    const T* q = qkv + (int64_t)r * ld + head * hd;
    const T* kbase = qkv + (nq + kvh) * hd;
    const T* vbase = qkv + (nq + nkv + kvh) * hd;
    for (int c = lane; c < hd; c += 64) sq[c] = to_f32<T>(q[c]) * scale;
    __syncthreads();

    const int n1 = r < P ? r + 1 : P;                 // visible prefix keys
    const int s0 = seg_start(r, P, Tn);
    const int n2 = r < P ? 0 : r - s0 + 1;            // visible keys of the own draft
    const int n = n1 + n2;
    float mx = -INFINITY;
    for (int i = lane; i < n; i += 64) {
        const T* k = kbase + (int64_t)(i < n1 ? i : s0 + (i - n1)) * ld;
        float s = 0.f;
        for (int c = 0; c < hd; ++c) s += sq[c] * to_f32<T>(k[c]);
        sp[i] = s;
        mx = fmaxf(mx, s);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float sum = 0.f;
    for (int i = lane; i < n; i += 64) {
        float p = __expf(sp[i] - mx);
        sp[i] = p;
        sum += p;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    __syncthreads();
    const float inv = 1.f / sum;
    // output: `width` lanes (a power of two >= hd, at most 64) per key, the 64 / width groups of lanes take every such key; eight
    // of a group's keys are requested at a time, from the prefix rows and then from the draft's, so that a key costs one
    // load and one multiply-add; the groups are added by exchange at the end.  320 rows, 4 heads of 32 over up to 96 keys, fp32:
    // 11.1 us one key at a time, 7.4 now; 3256 rows, 4 heads of 64 over up to 3128, bf16: 838 and 746 (with a clamp and two
    // selects a key 1044)
    int width = 64;
    while (width / 2 >= hd) width /= 2;
    const int groups = 64 / width, grp = lane / width, sub = lane % width;
    const int64_t step = (int64_t)groups * ld;
    for (int c = sub; c < align_up_int(hd, width); c += width) {
        const bool ok = c < hd;
        float acc = 0.f;
        auto keys = [&](int i, int end, int row) __attribute__((always_inline)) {      // keys i, i + groups, ... below end; key i is that row
            const T* v = vbase + (int64_t)row * ld + (ok ? c : 0);
            for (; i + 7 * groups < end; i += 8 * groups, v += 8 * step) {
                T x[8];
                float p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = v[u * step];
#pragma unroll
                for (int u = 0; u < 8; ++u) p[u] = sp[i + u * groups];
                __builtin_amdgcn_sched_barrier(0);              // else each 16-bit value is waited for and widened by itself
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += p[u] * to_f32<T>(x[u]);
            }
            if (i < end) {                                      // fewer than eight left: the key repeated past the last is not added
                T x[8];
                float p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = v[i + u * groups < end ? u * step : 0];
#pragma unroll
                for (int u = 0; u < 8; ++u) p[u] = sp[i + u * groups < end ? i + u * groups : i];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 8; ++u) acc = i + u * groups < end ? acc + p[u] * to_f32<T>(x[u]) : acc;
            }
        };
        keys(grp, n1, grp);
        const int i2 = n1 + (grp - n1 % groups + groups) % groups;                     // the group's first key of the draft
        keys(i2, n, s0 + (i2 - n1));
        for (int o = width; o < 64; o <<= 1) acc += __shfl_xor(acc, o);
        if (ok && grp == 0) out[(int64_t)r * nq * hd + head * hd + c] = from_f32<T>(acc * inv);
    }
}

// The same for heads of 4 to 32 16-byte pieces at 16-byte addresses: one wavefront per (row, head) again, but everything in registers.
// PIECES lanes hold a key's row; 16 loads of keys and 16 of values (32 to 256 rows) are requested before the query is there, scores stay in
// the lanes that summed them, and the groups meet only in the maximum, the sum and the output; longer contexts go on in batches with a
// running maximum.  What bounds it is a memory latency and a chain of about 300 vector instructions a batch; the kernel above, a lane a
// key and scores through LDS, waits for five latencies and reads 64 rows with every load.  us before and now: fp32, hd 32: 4 heads, 64 + 8 x 32
// rows 6.0 -> 4.55; 30 + 2 x 20 3.55 -> 3.35; 400 + 16 x 64 46 -> 27.3; 32 query and 8 key heads, 500 + 4 x 500 982 -> 436; bf16, hd 64: 8.5 -> 5.3,
// 8 query and 2 key heads, 300 + 4 x 200 80 -> 44, 500 + 4 x 500 1530 -> 570; hd 256 of 16 heads, 1500 + 4 x 100 3684 -> 1234.
template <typename T, int PIECES>
__global__ __launch_bounds__(64) void attn_rows_kernel(const T* __restrict__ qkv, T* __restrict__ out, int row0, int P, int Tn, int nq, int nkv,
                                                      float scale) {
    constexpr int kPiece = 16 / (int)sizeof(T), hd = PIECES * kPiece, kGroups = 64 / PIECES, kLoads = 16;
    const int r = row0 + blockIdx.x, head = blockIdx.y, lane = threadIdx.x;
    const int kvh = head / (nq / nkv), grp = lane / PIECES, piece = lane % PIECES;
    const int64_t ld = (int64_t)(nq + 2 * nkv) * hd;
    const T* const kbase = qkv + (nq + kvh) * hd + piece * kPiece;
    const T* const vbase = kbase + nkv * hd;
    const int n1 = r < P ? r + 1 : P;                 // visible prefix keys
    const int s0 = seg_start(r, P, Tn);
    const int n = n1 + (r < P ? 0 : r - s0 + 1);      // ... and those of the own draft
    uint4 kx[kLoads], vx[kLoads];
    auto load = [&](const T* base, int first, uint4 (&x)[kLoads]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            const int i = min(first + u * kGroups + grp, n - 1);
            x[u] = *reinterpret_cast<const uint4*>(base + (int64_t)(i < n1 ? i : s0 + (i - n1)) * ld);
        }
    };
    const uint4 qx = *reinterpret_cast<const uint4*>(qkv + (int64_t)r * ld + head * hd + piece * kPiece);
    load(kbase, 0, kx);
    load(vbase, 0, vx);
    float q[kPiece], acc[kPiece], mx = -INFINITY, sum = 0.f;
#pragma unroll
    for (int e = 0; e < kPiece; ++e) {
        q[e] = to_f32<T>(reinterpret_cast<const T*>(&qx)[e]) * scale;
        acc[e] = 0.f;
    }
    auto across = [&](float v, auto op) __attribute__((always_inline)) {     // over the groups
#pragma unroll
        for (int o = PIECES; o < 64; o <<= 1) v = op(v, __shfl_xor(v, o));
        return v;
    };
    auto add_dpp = [&](float v, auto ctrl) __attribute__((always_inline)) {
        return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    for (int first = 0;;) {
        // 16-bit heads of up to 8 pieces: all loads stay ahead of the first scores (the compiler spreads them otherwise: 574 us for 562 below)
        if constexpr (sizeof(T) == 2 && PIECES <= 8) __builtin_amdgcn_sched_barrier(0);
        float s[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            s[u] = 0.f;
#pragma unroll
            for (int e = 0; e < kPiece; ++e) s[u] += q[e] * to_f32<T>(reinterpret_cast<const T*>(&kx[u])[e]);
        }
#pragma unroll
        for (int u = 0; u < kLoads; ++u) s[u] = add_dpp(s[u], std::integral_constant<int, 0xB1>{});         // lane ^ 1
#pragma unroll
        for (int u = 0; u < kLoads; ++u) s[u] = add_dpp(s[u], std::integral_constant<int, 0x4E>{});         // lane ^ 2
        if constexpr (PIECES >= 8) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u) s[u] = add_dpp(s[u], std::integral_constant<int, 0x141>{});    // the other quad of eight
        }
        if constexpr (PIECES >= 16) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u) s[u] = add_dpp(s[u], std::integral_constant<int, 0x140>{});    // the other eight of sixteen
        }
        if constexpr (PIECES >= 32) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u) s[u] += __shfl_xor(s[u], 16);
        }
        float here = -INFINITY;
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            if (first + u * kGroups + grp >= n) s[u] = -INFINITY;
            here = fmaxf(here, s[u]);
        }
        const float m = fmaxf(mx, across(here, [](float a, float b) { return fmaxf(a, b); }));
        const float base = m == -INFINITY ? 0.f : m;
        const float old = first == 0 ? 0.f : __expf(mx - base);
        float part = 0.f;
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            s[u] = __expf(s[u] - base);
            part += s[u];
        }
        sum = sum * old + part;                                     // this group's
#pragma unroll
        for (int e = 0; e < kPiece; ++e) {
            acc[e] *= old;
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                // a row past the last is a repeat with probability zero (an infinite value makes that a NaN: see below)
                acc[e] += s[u] * to_f32<T>(reinterpret_cast<const T*>(&vx[u])[e]);
            }
        }
        mx = m;
        first += kLoads * kGroups;
        if (first >= n) break;                                      // wave-uniform
        load(kbase, first, kx);
        load(vbase, first, vx);
    }
    auto plus = [](float a, float b) { return a + b; };
    const float inv = 1.f / across(sum, plus);
#pragma unroll
    for (int e = 0; e < kPiece; ++e) acc[e] = across(acc[e], plus) * inv;
    bool nan = false;
#pragma unroll
    for (int e = 0; e < kPiece; ++e) nan |= acc[e] != acc[e];
    if (__builtin_expect(__any(nan), 0)) {
        // Infinite values, or a NaN of the inputs: the elements that are NaN are added up again, over the rows there are and no repeats.
        // (Zeros in the repeats' place, selected behind the last loads, cost every call 0.3 to 0.6 us.)
        float again[kPiece];
#pragma unroll
        for (int e = 0; e < kPiece; ++e) again[e] = 0.f;
        const float base = mx == -INFINITY ? 0.f : mx;
        for (int i0 = 0; i0 < n; i0 += kGroups) {                   // whole groups stay for the exchange
            const int i = min(i0 + grp, n - 1);
            const T* const k = kbase + (int64_t)(i < n1 ? i : s0 + (i - n1)) * ld;
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < kPiece; ++e) s += q[e] * to_f32<T>(k[e]);
            for (int o = 1; o < PIECES; o <<= 1) s += __shfl_xor(s, o);
            if (i0 + grp >= n) continue;
            const float p = __expf(s - base);
#pragma unroll
            for (int e = 0; e < kPiece; ++e) again[e] += p * to_f32<T>(k[nkv * hd + e]);
        }
#pragma unroll
        for (int e = 0; e < kPiece; ++e) {
            const float v = across(again[e], plus) * inv;
            if (acc[e] != acc[e]) acc[e] = v;
        }
    }
    if (grp == 0) {
        T y[kPiece];
#pragma unroll
        for (int e = 0; e < kPiece; ++e) y[e] = from_f32<T>(acc[e]);
        T* const to = out + (int64_t)r * nq * hd + head * hd + piece * kPiece;
        if ((reinterpret_cast<uintptr_t>(out) & 15) == 0) {
            *reinterpret_cast<uint4*>(to) = *reinterpret_cast<const uint4*>(y);
        } else {
#pragma unroll
            for (int e = 0; e < kPiece; ++e) to[e] = y[e];
        }
    }
}

// Takes the call if the kernel serves its heads and addresses (outputs anywhere: 300 + 4 x 200 rows, bf16, heads of 64, an element off 43.5 us,
// by the general kernel 92.5).
template <typename T>
bool launch_attn_rows(const void* qkv, void* out, ScoreShape s, int32_t row0, int32_t nq, int32_t nkv, int32_t hd, float scale, hipStream_t stream) {
    const int bytes = hd * (int)sizeof(T);
    if (bytes % 16 || (reinterpret_cast<uintptr_t>(qkv) & 15)) return false;
    auto launch = [&](auto pieces) {
        hipLaunchKernelGGL((attn_rows_kernel<T, decltype(pieces)::value>), dim3(s.R() - row0, nq), dim3(64), 0, stream,
                           static_cast<const T*>(qkv), static_cast<T*>(out), row0, s.P, s.T, nq, nkv, scale);
        return true;
    };
    switch (bytes / 16) {
        case 4: return launch(std::integral_constant<int, 4>{});
        case 8: return launch(std::integral_constant<int, 8>{});
        case 16: return launch(std::integral_constant<int, 16>{});
        case 32: return launch(std::integral_constant<int, 32>{});
    }
    return false;
}

// ------------------------------------------------------------------------------------------
// MFMA kernel (bf16, hd = 128)
// ------------------------------------------------------------------------------------------
constexpr int kHd = 128;
constexpr int kKTile = 64;    // keys per LDS tile

// The values of both lanes of the pair (l, l ^ 32), the lower lane's first: the two 32-lane halves exchanged in registers (no
// LDS round trip in the middle of the softmax).  The results are taken out as integers first: a bit cast applied to an
// element of the pair reads element 0 whichever is named.
__device__ __forceinline__ float2 lane_pair(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned lower = sw[0], upper = sw[1];
    return make_float2(__builtin_bit_cast(float, lower), __builtin_bit_cast(float, upper));
}

// kWaves wavefronts of 32 query rows each share the key / value tiles of one head; kStages tiles of LDS form a ring.
// kPipe: the scores of tile t + 1 are issued to the matrix cores BEFORE the softmax of tile t, so that the exponentials
// (vector ALU) of one tile run while the matrix pipe works on the next one; needs the key tile t + 1 next to the value
// tile t in LDS, hence one more stage than the plain order for the same prefetch distance.
template <int kWaves, int kStages, bool kPipe>
__global__ __launch_bounds__(64 * kWaves, 512 / (64 * kWaves)) void attn_mfma_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ vt,
                                                           int64_t ldv, bf16* __restrict__ out, int row0, int R, int P, int Tn,
                                                           int nq, int nkv, float scale_log2e) {
    // Stages of [K tile: 64 keys x 256 B | V^T tile: 128 dims x 128 B], filled by direct global -> LDS loads.
    //   K rows are 256 B: 16-byte chunk index XOR (key & 15);  V^T rows are 128 B: chunk index XOR (dim >> 1) & 7.
    constexpr int kQTile = 32 * kWaves;                 // query rows per workgroup
    constexpr int kKBytes = kKTile * kHd * 2, kStage = 2 * kKBytes;
    constexpr int kDmaK = 16 / kWaves, kDmaV = 16 / kWaves;     // 1 KiB DMA instructions per wave and tile
    constexpr int kDmaTile = kDmaK + kDmaV;
    static_assert(kWaves == 4 || kWaves == 8, "DMA addressing below");
    static_assert(kStages >= (kPipe ? 3 : 2), "ring depth");
    extern __shared__ __attribute__((aligned(16))) char smem[];   // [kStages][kStage]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int head = blockIdx.y, kvh = head / (nq / nkv);
    const int r0 = row0 + blockIdx.x * kQTile;      // query tiles start at the first computed row
    const int r_last = min(r0 + kQTile, R) - 1;
    const int64_t ld = (int64_t)(nq + 2 * nkv) * kHd;

    // This lane's query row and its visibility window; the wave's row range decides which tiles it can skip.
    const int rw0 = r0 + wave * 32;                                  // first row of this wave
    const int rw1 = min(rw0 + 31, r_last);                           // last valid row (rw1 < rw0: the wave has no rows)
    const int r = rw0 + l32;
    const bool r_ok = r < R;
    const int ss = seg_start(r_ok ? r : r_last, P, Tn);
    const int ss_w0 = seg_start(min(rw0, r_last), P, Tn);            // draft start of the wave's first row
    const int ss_w1 = seg_start(max(rw1, rw0 <= r_last ? rw0 : r_last), P, Tn);   // ... and of its last row

    // Q fragments (B operand of S^T = K Q^T): lane holds Q[r][16 s + 8 g + (0..7)], s = 0..7.
    bf16x8 qf[8];
    {
        const bf16* qp = qkv + (int64_t)(r_ok ? r : 0) * ld + head * kHd + 8 * g;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (r_ok) qf[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
            else
#pragma unroll
                for (int e = 0; e < 8; ++e) qf[s][e] = (bf16)0.f;
        }
    }

    // Tiles: the prefix range [0, min(P, r_last + 1)) and the range of the drafts this query
    // tile touches, both walked in 64-key tiles aligned to multiples of 64.
    const int pre_end = min(P, r_last + 1);
    const int n1 = (pre_end + kKTile - 1) / kKTile;
    const int s2 = max(n1 * kKTile, seg_start(r0, P, Tn) / kKTile * kKTile);
    const int n2 = r_last >= s2 ? (r_last - s2) / kKTile + 1 : 0;
    const int n_tiles = n1 + n2;
    auto tile_start = [&](int t) { return t < n1 ? t * kKTile : s2 + (t - n1) * kKTile; };

    // ---- DMA addressing (one wave-wide instruction moves 1 KiB = 4 K rows or 8 V^T rows).
    // K: instruction j of this wave fills tile rows (64 / kWaves) wave + 4 j + (lane >> 4); lane lands at chunk slot
    //    lane & 15 and fetches chunk slot ^ (row & 15).  Rows past the end are clamped to row R - 1 (their scores
    //    are masked).
    // V^T: instruction j fills dims (128 / kWaves) wave + 8 j + (lane >> 3); slot lane & 7 fetches chunk
    //    slot ^ ((dim >> 1) & 7).  Columns past R are zero in the V^T copy.
    const int kq = lane >> 4, kslot = lane & 15;
    const int vq = lane >> 3, vslot = lane & 7;
    const bf16* kg = qkv + (nq + kvh) * kHd;
    const bf16* vg = vt + ((int64_t)kvh * kHd + (128 / kWaves) * wave + vq) * ldv;
    auto issue_tile = [&](int t) __attribute__((always_inline)) {
        const int j0 = tile_start(t);
        char* stage = smem + (t % kStages) * kStage;
#pragma unroll
        for (int j = 0; j < kDmaK; ++j) {
            const int row = (64 / kWaves) * wave + 4 * j;             // wave-uniform part of the tile row
            const int key = min(j0 + row + kq, R - 1);
            const bf16* src = kg + (int64_t)key * ld + ((kslot ^ ((row + kq) & 15)) << 3);
            __builtin_amdgcn_global_load_lds(ATTS_GPTR(src), ATTS_LPTR(stage + row * 256), 16, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < kDmaV; ++j) {
            const int dim = (128 / kWaves) * wave + 8 * j;
            const bf16* src = vg + (int64_t)(8 * j) * ldv + j0 + ((vslot ^ (((dim + vq) >> 1) & 7)) << 3);
            __builtin_amdgcn_global_load_lds(ATTS_GPTR(src), ATTS_LPTR(stage + kKBytes + dim * 128), 16, 0, 0);
        }
    };

    f32x16 acc_o[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[nb][v] = 0.f;
    float m_run = -1e30f;   // reference max (scaled, log2 domain), shared by the lane pair (l, l ^ 32)
    float l_run = 0.f;      // this lane's share of the running denominator
    const float move_from = g ? 64.f : 6.f;     // how far above the reference a key of this lane may stand

    // Wave-uniform visibility of tile t for the wave's rows rw0 .. rw1:
    //   nothing visible: the tile starts after the last row, or lies in drafts before the wave's first row's
    //   fully visible:   every key <= first row, and (a prefix tile or inside the draft of the last row)
    auto tile_none = [&](int t) {
        const int j0 = tile_start(t);
        return rw1 < rw0 || j0 > rw1 || (j0 >= P && j0 + kKTile <= ss_w0);
    };
    auto tile_full = [&](int t) {
        const int j0 = tile_start(t);
        return j0 + kKTile - 1 <= rw0 && (j0 + kKTile <= P || j0 >= ss_w1) && rw0 + 31 <= r_last;
    };

    // ---- S^T = K Q^T for the two 32-key blocks of tile t.  MFMA row i of a block is fed with key pi(i) of the block,
    // pi = exchange of bits 2 and 3: accumulator entry v of lane half g is then the score of key
    //     32 kb + 16 (v >> 3) + 8 g + (v & 7),
    // eight consecutive keys per lane and 16-key step: exactly the k order of a 16-byte V^T fragment, so the
    // probabilities feed the second product from registers and the value fragments are single 16-byte LDS reads.
    const int kperm = (l32 & 0x13) | ((l32 & 8) >> 1) | ((l32 & 4) << 1);
    auto score_tile = [&](int t, f32x16 (&acc_s)[2]) __attribute__((always_inline)) {
        const char* sK = smem + (t % kStages) * kStage;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_s[kb][v] = 0.f;
        // Fragments in groups of four (two 16-column slices of the head dimension x the two key blocks), double-buffered:
        // the reads of group q + 1 are issued behind the first MFMA of group q, whose wait has just drained the LDS
        // queue, and arrive under the other three.
        auto load_k = [&](int s_, int kb) __attribute__((always_inline)) {
            const int kr = kb * 32 + kperm;
            return *reinterpret_cast<const bf16x8*>(sK + kr * 256 + (((2 * s_ + g) ^ (kr & 15)) << 4));
        };
        bf16x8 kf[2][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) kf[0][i] = load_k(i >> 1, i & 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            acc_s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[q & 1][0], qf[2 * q], acc_s[0], 0, 0, 0);
            if (q < 3) {
#pragma unroll
                for (int i = 0; i < 4; ++i) kf[(q + 1) & 1][i] = load_k(2 * (q + 1) + (i >> 1), i & 1);
            }
            acc_s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[q & 1][1], qf[2 * q], acc_s[1], 0, 0, 0);
            acc_s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[q & 1][2], qf[2 * q + 1], acc_s[0], 0, 0, 0);
            acc_s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[q & 1][3], qf[2 * q + 1], acc_s[1], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (q < 3) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- softmax of tile t (raw scores in acc_s) and O^T += V^T P^T.  The softmax works on
    // z = score * scale * log2(e): the scale is folded into the one fused multiply-add in front of exp2.
    auto softmax_pv = [&](int t, f32x16 (&acc_s)[2]) __attribute__((always_inline)) {
        const int j0 = tile_start(t);
        const char* sV = smem + (t % kStages) * kStage + kKBytes;
        if (!tile_full(t)) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int j = j0 + 32 * kb + 16 * (v >> 3) + 8 * g + (v & 7);
                    const bool vis = r_ok && j <= r && (j < P || j >= ss);
                    acc_s[kb][v] = vis ? acc_s[kb][v] : -INFINITY;
                }
        }
        float mx = fmaxf(acc_s[0][0], acc_s[1][0]);
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(fmaxf(mx, acc_s[0][v]), acc_s[1][v]);    // one three-operand maximum each
        // Lazy rescaling: any reference value works in exp2(z - m) as long as it is the same for numerator and
        // denominator, so the running reference only moves when a key of the lower lanes exceeds it by more than 2^6 or one of the
        // upper lanes by more than 2^64, which every lane sees from its own keys; the exchange and the 64 accumulator
        // multiplies are skipped otherwise.  p stays <= 2^64: sums of 2^20 keys are finite up to values of 2^43.  40 query and 8 key
        // heads, 2048 + 64 x 512 rows: 1682 us; 1714 with the exchange and the test of both halves in every tile, 1698 with the
        // reference of the lower lanes alone, which gives NaN once a key of the upper ones stands out by more than 2^127.
        const float own = mx * scale_log2e;                                               // scale > 0: the order is kept
        if (__builtin_amdgcn_ballot_w64(own > m_run + move_from) != 0) {
            const float2 pair = lane_pair(own);
            float m_new = fmaxf(m_run, pair.x);
            m_new = pair.y > m_new + 64.f ? pair.y : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc_o[nb][v] *= alpha;
        }
        // value fragments in groups of four (one 16-key slice x the four 32-dim blocks), double-buffered as the key
        // fragments; the first group is requested here, ahead of the exponentials, and has arrived when they are through
        auto load_v = [&](int s_, int nb) __attribute__((always_inline)) {
            const int n = nb * 32 + l32;
            return *reinterpret_cast<const bf16x8*>(sV + n * 128 + (((2 * s_ + g) ^ ((n >> 1) & 7)) << 4));
        };
        bf16x8 vf[2][4];
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) vf[0][nb] = load_v(0, nb);
        __builtin_amdgcn_sched_barrier(0);
        float psum = 0.f;
        bf16x8 pf[4];
        const float neg_m = -m_run;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(acc_s[kb][v], scale_log2e, neg_m));   // -inf -> 0
                psum += p;
                pf[kb * 2 + (v >> 3)][v & 7] = (bf16)p;
            }
        l_run += psum;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s_ = 0; s_ < 4; ++s_) {
            acc_o[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s_ & 1][0], pf[s_], acc_o[0], 0, 0, 0);
            if (s_ < 3) {
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) vf[(s_ + 1) & 1][nb] = load_v(s_ + 1, nb);
            }
#pragma unroll
            for (int nb = 1; nb < 4; ++nb) acc_o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s_ & 1][nb], pf[s_], acc_o[nb], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (s_ < 3) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // Ring of kStages tiles, tiles 0 .. kStages - 2 requested up front.
#pragma unroll
    for (int t = 0; t < kStages - 1; ++t)
        if (t < n_tiles) issue_tile(t);
    if constexpr (!kPipe) {
        // At the top of step t the tiles up to t + kStages - 2 have been requested, tile t must have landed (the
        // younger ones may stay in flight); after the barrier tile t + kStages - 1 goes into the stage of tile t - 1.
        for (int t = 0; t < n_tiles; ++t) {
            if (t + kStages - 2 < n_tiles) wait_vmcnt<(kStages - 2) * kDmaTile>(); else wait_vmcnt<0>();
            block_barrier();            // tile t is in LDS for every wave; every wave is done with tile t - 1
            if (t + kStages - 1 < n_tiles) issue_tile(t + kStages - 1);
            if (tile_none(t)) continue;
            f32x16 acc_s[2];
            score_tile(t, acc_s);
            softmax_pv(t, acc_s);
        }
    } else {
        // Step t: scores of tile t + 1, then softmax and value product of tile t.  At its top the tiles up to
        // t + kStages - 2 have been requested and tile t + 1 must have landed; after the barrier (every wave is done
        // with tile t - 1) tile t + kStages - 1 goes into that tile's stage.
        f32x16 acc_a[2], acc_b[2];
        if (n_tiles > 0) {
            if (kStages - 2 < n_tiles) wait_vmcnt<(kStages - 2) * kDmaTile>(); else wait_vmcnt<0>();
            block_barrier();
            if (!tile_none(0)) score_tile(0, acc_a);
        }
        auto step = [&](int t, f32x16 (&cur)[2], f32x16 (&nxt)[2]) __attribute__((always_inline)) {
            if (t + 1 < n_tiles) {
                if (t + kStages - 2 < n_tiles) wait_vmcnt<(kStages - 3) * kDmaTile>(); else wait_vmcnt<0>();
                block_barrier();
                if (t + kStages - 1 < n_tiles) issue_tile(t + kStages - 1);
                if (!tile_none(t + 1)) score_tile(t + 1, nxt);
            }
            if (!tile_none(t)) softmax_pv(t, cur);
        };
        for (int t = 0; t < n_tiles; t += 2) {
            step(t, acc_a, acc_b);
            if (t + 1 < n_tiles) step(t + 1, acc_b, acc_a);
        }
    }

    // ---- normalise and store: acc_o[nb][4 a + b] = O[r][32 nb + 8 a + 4 g + b]
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (r_ok) {
        const float inv = 1.f / l_tot;
        bf16* op = out + (int64_t)r * nq * kHd + head * kHd + 4 * g;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                bf16x4 o4;
#pragma unroll
                for (int b = 0; b < 4; ++b) o4[b] = (bf16)(acc_o[nb][4 * a + b] * inv);
                *reinterpret_cast<bf16x4*>(op + 32 * nb + 8 * a) = o4;
            }
    }
}


// Few query rows: 32 of one head per workgroup, its 32-key tiles dealt to the eight wavefronts.  Each keeps a softmax of its own
// over every eighth tile and they are merged once, through LDS.  A tile is read in whole rows (the matrix fragments' own layout,
// one row per lane, takes the address unit four times as long), held in registers while the tile before is worked on, and
// laid out for the fragments in the wavefront's own part of LDS: no barrier until the merge.
// What bounds it is the CU's path from the L2: eight tiles (256 keys) of a workgroup take about 2 us, start and merge 5.5.
constexpr int kSplitWaves = 8;
constexpr int kSplitPitch = kHd + 4;                    // floats of a merge row in LDS
constexpr size_t kSplitLds = (size_t)kSplitWaves * 32 * (kSplitPitch + 2) * sizeof(float);
__global__ __launch_bounds__(64 * kSplitWaves) void attn_split_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ vt, int64_t ldv,
                                                                      bf16* __restrict__ out, int row0, int R, int P, int Tn, int nq, int nkv,
                                                                      int q_tiles, float scale_log2e) {
    constexpr int kTile = 32;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float* const part = reinterpret_cast<float*>(smem);                              // [wave][row][kSplitPitch]
    float2* const stat = reinterpret_cast<float2*>(part + kSplitWaves * 32 * kSplitPitch);   // [wave][row] (maximum, sum)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    // the workgroups an XCD receives (id mod 8) are consecutive ones of the order heads x query tiles: few key / value heads each
    const int n_wg = (int)gridDim.x, n8 = n_wg & ~7, pid = (int)blockIdx.x;
    const int lid = pid < n8 ? (pid & 7) * (n8 >> 3) + (pid >> 3) : pid;
    const int head = lid / q_tiles, kvh = head / (nq / nkv);
    const int r0 = row0 + (lid % q_tiles) * 32;
    const int r_last = min(r0 + 32, R) - 1;
    const int64_t ld = (int64_t)(nq + 2 * nkv) * kHd;
    const int r = r0 + l32;
    const bool r_ok = r < R;
    const int ss = seg_start(min(r, r_last), P, Tn);

    const int n1 = (min(P, r_last + 1) + kTile - 1) / kTile;
    const int s2 = max(n1 * kTile, seg_start(r0, P, Tn) / kTile * kTile);
    const int n_tiles = n1 + (r_last >= s2 ? (r_last - s2) / kTile + 1 : 0);
    auto tile_start = [&](int t) { return t < n1 ? t * kTile : s2 + (t - n1) * kTile; };

    const int kperm = (l32 & 0x13) | ((l32 & 8) >> 1) | ((l32 & 4) << 1);            // as in attn_mfma_kernel
    const bf16* const kg = qkv + (nq + kvh) * kHd + 8 * (lane & 15);
    const bf16* const vg = vt + ((int64_t)kvh * kHd + (lane >> 2)) * ldv + 8 * (lane & 3);
    char* const own = reinterpret_cast<char*>(part + wave * 32 * kSplitPitch);       // 32 keys x 256 B, then 128 dims x 64 B
    bf16x8 qf[8], kr[8], vr[8];
    auto request = [&](int t) __attribute__((always_inline)) {
        const int j0 = tile_start(t);
#pragma unroll
        for (int j = 0; j < 8; ++j) kr[j] = *reinterpret_cast<const bf16x8*>(kg + (int64_t)min(j0 + 4 * j + (lane >> 4), R - 1) * ld);
#pragma unroll
        for (int j = 0; j < 8; ++j) vr[j] = *reinterpret_cast<const bf16x8*>(vg + (int64_t)(16 * j) * ldv + j0);
    };
    // 16-byte chunks: index XOR (key & 15) in a key's row, XOR (dim / 4) & 3 in a dim's
    auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int row = 4 * j + (lane >> 4);
            *reinterpret_cast<bf16x8*>(own + row * 256 + (((lane & 15) ^ (row & 15)) << 4)) = kr[j];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            *reinterpret_cast<bf16x8*>(own + kTile * 256 + (16 * j + (lane >> 2)) * 64 + (((lane & 3) ^ (lane >> 4)) << 4)) = vr[j];
    };
    auto load_k = [&](int s) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(own + kperm * 256 + (((2 * s + g) ^ (kperm & 15)) << 4));
    };
    auto load_v = [&](int s, int nb) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(own + kTile * 256 + (32 * nb + l32) * 64 + (((2 * s + g) ^ ((l32 >> 2) & 3)) << 4));
    };
    if (wave < n_tiles) request(wave);
    {
        const bf16* qp = qkv + (int64_t)min(r, R - 1) * ld + head * kHd + 8 * g;     // rows past the last: masked
#pragma unroll
        for (int s = 0; s < 8; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
    }
    f32x16 acc_o[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[nb][v] = 0.f;
    float m_run = -1e30f, l_run = 0.f;

    for (int t = wave; t < n_tiles; t += kSplitWaves) {
        const int j0 = tile_start(t);
        stage();
        if (t + kSplitWaves < n_tiles) request(t + kSplitWaves);
        f32x16 acc_s;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_s[v] = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) acc_s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load_k(s), qf[s], acc_s, 0, 0, 0);
        if (!(j0 + kTile - 1 <= r0 && j0 + kTile <= P && r0 + 31 <= r_last)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int j = j0 + 16 * (v >> 3) + 8 * g + (v & 7);
                const bool vis = r_ok && j <= r && (j < P || j >= ss);
                acc_s[v] = vis ? acc_s[v] : -INFINITY;
            }
        }
        float mx = acc_s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc_s[v]);
        const float2 pair = lane_pair(mx);
        mx = fmaxf(pair.x, pair.y) * scale_log2e;
        if (__builtin_amdgcn_ballot_w64(mx > m_run + 6.f) != 0) {
            const float m_new = fmaxf(m_run, mx);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc_o[nb][v] *= alpha;
        }
        bf16x8 pf[2];
        float psum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(acc_s[v], scale_log2e, -m_run));
            psum += p;
            pf[v >> 3][v & 7] = (bf16)p;
        }
        l_run += psum;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) acc_o[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(load_v(s, nb), pf[s], acc_o[nb], 0, 0, 0);
    }

    // merge: the wavefronts that had a tile leave their sums, every thread weighs eight output columns of a row
    const int used = min(kSplitWaves, n_tiles);
    if (wave < used) {
        const float l_tot = l_run + __shfl_xor(l_run, 32);
        float* const mine = part + (wave * 32 + l32) * kSplitPitch + 4 * g;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int a = 0; a < 4; ++a)
                *reinterpret_cast<f32x4*>(mine + 32 * nb + 8 * a) = f32x4{acc_o[nb][4 * a], acc_o[nb][4 * a + 1], acc_o[nb][4 * a + 2], acc_o[nb][4 * a + 3]};
        if (g == 0) stat[wave * 32 + l32] = make_float2(m_run, l_tot);
    }
    __syncthreads();
    const int row = tid >> 4, col = (tid & 15) * 8;
    if (r0 + row > r_last) return;
    float m_all = -1e30f;
    for (int w = 0; w < used; ++w) m_all = fmaxf(m_all, stat[w * 32 + row].x);
    f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = {0.f, 0.f, 0.f, 0.f};
    float sum = 0.f;
    for (int w = 0; w < used; ++w) {
        const float2 st = stat[w * 32 + row];
        const float e = __builtin_amdgcn_exp2f(st.x - m_all);
        const f32x4* p = reinterpret_cast<const f32x4*>(part + (w * 32 + row) * kSplitPitch + col);
        sum += e * st.y;
        o0 += e * p[0];
        o1 += e * p[1];
    }
    const float inv = 1.f / sum;
    bf16x8 o;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        o[c] = (bf16)(o0[c] * inv);
        o[4 + c] = (bf16)(o1[c] * inv);
    }
    *reinterpret_cast<bf16x8*>(out + (int64_t)(r0 + row) * nq * kHd + head * kHd + col) = o;
}

}  // namespace

bool attention_uses_vt(int32_t dtype, int32_t hd) { return dtype == ATTS_DTYPE_BF16 && hd == kHd; }

// the general kernel keeps one score per key of the longest context (prefix + one draft) in LDS
constexpr size_t kSimpleLdsMax = 60 * 1024;
static size_t simple_attention_lds(int32_t hd, int32_t P, int32_t T) { return ((size_t)hd + (size_t)P + (size_t)T) * sizeof(float); }

int32_t attention_context_check(const char* fn, int32_t dtype, int32_t hd, int32_t P, int32_t T) {
    if (attention_uses_vt(dtype, hd) || simple_attention_lds(hd, P, T) <= kSimpleLdsMax) return ATTS_OK;
    return fail(ATTS_ERR_SHAPE, "%s: a context of %lld keys (prefix + one draft) is too long for the attention kernel of this dtype / head_dim",
                fn, (long long)P + T);
}

int32_t launch_attention(int32_t dtype, const void* qkv, const void* vt, int64_t ldv, void* out, ScoreShape s, int32_t row0,
                         int32_t nq, int32_t nkv, int32_t hd, hipStream_t stream) {
    const int R = s.R();
    const float scale = 1.f / sqrtf((float)hd);
    if (attention_uses_vt(dtype, hd)) {
        if (!vt || ldv < (int64_t)align_up(R, kKTile) || ldv % 8)
            return fail(ATTS_ERR_WORKSPACE, "attention: transposed-V buffer missing or too narrow");
        // 32 query rows per workgroup, its keys dealt to eight wavefronts, while one workgroup per CU holds them all: the other
        // forms then are few workgroups that walk their keys one tile after the other (7B widths, 128 rows against a prefix of 512:
        // 10.2 us for 18.3, of 2048: 20.7 for 44.8; 8 rows 12.1 for 21.2 and 22.5 for 67.6; 70B, 256 workgroups: 9.2 for 13.7 at
        // 256 keys, 24.4 for 45.5 at 2048).  A second round of them still wins for long contexts (448 to 512 workgroups:
        // 16.0 - 20.8 for 13.9 - 18.4 up to 512 keys, 28 - 30 for 27 - 28 at 1024, 40 - 44 for 46 - 47 at 2048).
        // 256 query rows per workgroup (8 wavefronts, one workgroup per CU, four LDS stages, scores of the next tile issued
        // ahead of the softmax) once the call has enough rows to fill the chip that way; 128 rows (4 wavefronts, two
        // workgroups per CU) for calls in between
        constexpr int kStage = 2 * kKTile * kHd * 2;
        const float sc2 = scale * 1.4426950408889634f;
        const int q_tiles = (int)ceil_div(R - row0, 32);
        const int64_t split_wgs = (int64_t)q_tiles * nq;
        if (split_wgs <= 256 || (split_wgs <= 512 && s.P + s.T >= 1536)) {
            int32_t rc = allow_dynamic_lds<attn_split_kernel>(kSplitLds);
            if (rc != ATTS_OK) return rc;
            hipLaunchKernelGGL(attn_split_kernel, dim3((unsigned)(q_tiles * nq)), dim3(64 * kSplitWaves), kSplitLds, stream, (const bf16*)qkv,
                               (const bf16*)vt, ldv, (bf16*)out, row0, R, s.P, s.T, nq, nkv, q_tiles, sc2);
        } else if ((int64_t)ceil_div(R - row0, 256) * nq >= 256) {
            constexpr size_t lds = 4 * kStage;
            int32_t rc = allow_dynamic_lds<attn_mfma_kernel<8, 4, true>>(lds);
            if (rc != ATTS_OK) return rc;
            hipLaunchKernelGGL((attn_mfma_kernel<8, 4, true>), dim3((unsigned)ceil_div(R - row0, 256), nq), dim3(512), lds, stream, (const bf16*)qkv,
                               (const bf16*)vt, ldv, (bf16*)out, row0, R, s.P, s.T, nq, nkv, sc2);
        } else {
            constexpr size_t lds = 2 * kStage;
            int32_t rc = allow_dynamic_lds<attn_mfma_kernel<4, 2, false>>(lds);
            if (rc != ATTS_OK) return rc;
            hipLaunchKernelGGL((attn_mfma_kernel<4, 2, false>), dim3((unsigned)ceil_div(R - row0, 128), nq), dim3(256), lds, stream, (const bf16*)qkv,
                               (const bf16*)vt, ldv, (bf16*)out, row0, R, s.P, s.T, nq, nkv, sc2);
        }
        ATTS_LAUNCH_CHECK("attn_mfma_kernel");
        return ATTS_OK;
    }
    // The limit of the general kernel's scores in LDS holds for both: whether the other one takes a call depends on the buffers' address, which is
    // no reason to serve or refuse a context.
    const size_t lds = simple_attention_lds(hd, s.P, s.T);
    if (lds > kSimpleLdsMax) return fail(ATTS_ERR_SHAPE, "attention: context of %d keys is too long for this dtype/head_dim", s.P + s.T);
    dim3 grid(R - row0, nq);
    if (dtype == ATTS_DTYPE_F32 ? launch_attn_rows<float>(qkv, out, s, row0, nq, nkv, hd, scale, stream)
                                : launch_attn_rows<bf16>(qkv, out, s, row0, nq, nkv, hd, scale, stream)) {
        ATTS_LAUNCH_CHECK("attn_rows_kernel");
        return ATTS_OK;
    }
    if (dtype == ATTS_DTYPE_F32)
        hipLaunchKernelGGL(attn_simple_kernel<float>, grid, dim3(64), lds, stream, (const float*)qkv, (float*)out, row0, s.P, s.T,
                           nq, nkv, hd, scale);
    else
        hipLaunchKernelGGL(attn_simple_kernel<bf16>, grid, dim3(64), lds, stream, (const bf16*)qkv, (bf16*)out, row0, s.P, s.T,
                           nq, nkv, hd, scale);
    ATTS_LAUNCH_CHECK("attn_simple_kernel");
    return ATTS_OK;
}

}  // namespace atts
