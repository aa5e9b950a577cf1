// Memory-bound stages of the scoring path: embedding gather, RMSNorm, rotary embedding +
// V transpose, scoring-row gather + final norm, score reduction.
// All are HBM-bound and tiny next to the GEMMs; they are written for coalesced 16-byte
// accesses and fixed reduction orders (no float atomics, so results are run-to-run stable).
#include "common.h"

namespace atts {
namespace {

// ---- wave / block reductions -------------------------------------------------------------
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Sum over a block of kBlock threads (kBlock multiple of 64, <= 1024); result valid in all threads.
template <int kBlock>
__device__ __forceinline__ float block_sum(float v, float* red /* [kBlock / 64] */) {
    v = wave_sum(v);
    if constexpr (kBlock == 64) return v;
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < kBlock / 64; ++i) t += red[i];
    return t;
}

// Row of the token tree -> (is it a draft row, which draft, which position in the draft)
__device__ __forceinline__ int tree_position(int r, int P, int T) { return r < P ? r : P + (r - P) % T; }

// ---- S1: RMSNorm over rows of the fp32 residual stream ---------------------------------------
// One row per workgroup, 16-byte loads; up to 4 float4 per thread (d <= 4096) stay in registers between the
// sum-of-squares pass and the scaling pass, longer rows are read again (from L2).  d % 4 == 0.
template <typename T>
__device__ __forceinline__ void store4(T* dst, float4 v);
template <>
__device__ __forceinline__ void store4<float>(float* dst, float4 v) { *reinterpret_cast<float4*>(dst) = v; }
template <>
__device__ __forceinline__ void store4<bf16>(bf16* dst, float4 v) {
    bf16x4 o;
    o[0] = (bf16)v.x; o[1] = (bf16)v.y; o[2] = (bf16)v.z; o[3] = (bf16)v.w;
    *reinterpret_cast<bf16x4*>(dst) = o;
}
template <typename T>
__device__ __forceinline__ float4 load4(const T* src);
template <>
__device__ __forceinline__ float4 load4<float>(const float* src) { return *reinterpret_cast<const float4*>(src); }
template <>
__device__ __forceinline__ float4 load4<bf16>(const bf16* src) {
    const bf16x4 v = *reinterpret_cast<const bf16x4*>(src);
    return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
}

// The row's values come as pieces of four from `load`; `seen` gets each of them once, behind the loads that are requested
// together.  Embedding, norm kernel and scoring rows take the sum in this one order: the same row has the same norm in each.
template <typename T, typename Load, typename Seen>
__device__ __forceinline__ void rmsnorm_pieces(Load load, Seen seen, const float* __restrict__ gain, float eps, int d,
                                               T* __restrict__ o, float* red) {
    constexpr int kKeep = 4;
    const int n4 = d >> 2;
    const float4* g4 = reinterpret_cast<const float4*>(gain);
    float4 keep[kKeep], g[kKeep];
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < kKeep; ++q) {
        const int c = threadIdx.x + 256 * q;
        keep[q] = c < n4 ? load(c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (gain) {                                                 // on their way with the row, not behind its sum
#pragma unroll
        for (int q = 0; q < kKeep; ++q) {
            const int c = threadIdx.x + 256 * q;
            g[q] = c < n4 ? g4[c] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
#pragma unroll
    for (int q = 0; q < kKeep; ++q) {
        const int c = threadIdx.x + 256 * q;
        if (c < n4) seen(c, keep[q]);
        ss += keep[q].x * keep[q].x + keep[q].y * keep[q].y + keep[q].z * keep[q].z + keep[q].w * keep[q].w;
    }
    for (int c = threadIdx.x + 256 * kKeep; c < n4; c += 256) {
        const float4 v = load(c);
        seen(c, v);
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
    if (!gain) return;                                          // block-uniform
    ss = block_sum<256>(ss, red);
    const float inv = rsqrtf(ss / (float)d + eps);
#pragma unroll
    for (int q = 0; q < kKeep; ++q) {
        const int c = threadIdx.x + 256 * q;
        if (c < n4)
            store4<T>(o + 4 * c, make_float4(keep[q].x * inv * g[q].x, keep[q].y * inv * g[q].y, keep[q].z * inv * g[q].z,
                                             keep[q].w * inv * g[q].w));
    }
    for (int c = threadIdx.x + 256 * kKeep; c < n4; c += 256) {
        const float4 v = load(c), gc = g4[c];
        store4<T>(o + 4 * c, make_float4(v.x * inv * gc.x, v.y * inv * gc.y, v.z * inv * gc.z, v.w * inv * gc.w));
    }
}

template <typename T>
__device__ __forceinline__ void rmsnorm_row(const float* __restrict__ x, const float* __restrict__ gain, float eps, int d,
                                            T* __restrict__ o, float* red) {
    auto load = [&](int c) __attribute__((always_inline)) { return load4<float>(x + 4 * c); };
    rmsnorm_pieces<T>(load, [](int, const float4&) {}, gain, eps, d, o, red);
}

template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ h, const float* __restrict__ gain,
                                                      float eps, int d, T* __restrict__ out) {
    __shared__ float red[4];
    rmsnorm_row<T>(h + (int64_t)blockIdx.x * d, gain, eps, d, out + (int64_t)blockIdx.x * d, red);
}

// (cos, sin)(pos theta^(-2 i / hd)), in fp64, rounded once
__device__ __forceinline__ float2 rope_pair(int pos, int i, double log_theta_over_half) {
    double s, c;
    sincos((double)pos * exp(-(double)i * log_theta_over_half), &s, &c);
    return make_float2((float)c, (float)s);
}

// ---- S0: start of a pass: embedding gather + first norm, rotary table, tail of V^T ----------------------------
// h = embedding of id (an id outside the vocabulary is read as 0 by the caller) and, with a gain vector, xn = rmsnorm(h).
// Pieces of four elements (rows are multiples of 16 bytes), in the norm's own order: with pieces of eight, a sum of another
// order moved the bf16 roundings of the first layer, and with them the whole pass by 1.8e-4, for no gain in time.
template <typename T>
__device__ __forceinline__ void embed_norm_row(const T* __restrict__ src, int d, float* __restrict__ h, const float* __restrict__ gain,
                                               float eps, T* __restrict__ xn, float* red) {
    auto load = [&](int c) __attribute__((always_inline)) { return load4<T>(src + 4 * c); };
    auto seen = [&](int c, const float4& v) __attribute__((always_inline)) { store4<float>(h + 4 * c, v); };
    rmsnorm_pieces<T>(load, seen, gain, eps, d, xn, red);
}

// Everything a pass needs before its first projection, in one launch (each of these is a few microseconds by itself, most of
// it the launch): the first row_wgs workgroups embed a row each and apply the first layer's norm; the next rope_wgs fill the
// rotary table, (cos, sin)(pos(r) theta^(-2 i / hd)) in fp64, rounded once; the last zero columns [R, ldv) of V^T for a
// producer that writes only the R real ones.  128 rows of the 7B width: 5.9 us for 8.9 + 4.7 + 4.9 in three launches (each
// with element-wise loads of the embedding); 4608 rows 31.3.
struct StartDims {
    int32_t vocab, d, P, T, row0, R, half, row_wgs, rope_wgs;
    double log_theta_over_half;
    float eps;
    int64_t ldv, vt_rows;
};
template <typename T>
__global__ __launch_bounds__(256) void tree_start_kernel(const T* __restrict__ emb, const int32_t* __restrict__ prefix_ids,
                                                         const int32_t* __restrict__ draft_ids, const int32_t* __restrict__ draft_lens,
                                                         float* __restrict__ h, const float* __restrict__ gain, T* __restrict__ xn,
                                                         float2* __restrict__ cs, T* __restrict__ vt, int32_t* __restrict__ err_flag,
                                                         const StartDims s) {
    __shared__ float red[4];
    const int rows = s.R - s.row0;
    if ((int)blockIdx.x < s.row_wgs) {
        const int r = s.row0 + (int)blockIdx.x;
        int id;
        bool padding = false;
        if (r < s.P) {
            id = prefix_ids[r];
        } else {
            const int k = (r - s.P) / s.T, t = (r - s.P) % s.T;
            id = draft_ids[(int64_t)k * s.T + t];
            padding = draft_lens && t >= draft_lens[k];
        }
        if (id < 0 || id >= s.vocab) {
            if (!padding && threadIdx.x == 0) *err_flag = 1;
            id = 0;
        }
        embed_norm_row<T>(emb + (int64_t)id * s.d, s.d, h + (int64_t)r * s.d, gain, s.eps, xn + (int64_t)r * s.d, red);
    } else if ((int)blockIdx.x < s.row_wgs + s.rope_wgs) {
        const int64_t idx = (int64_t)((int)blockIdx.x - s.row_wgs) * 256 + threadIdx.x;     // up to 2^24 rows x 128 pairs
        if (idx >= (int64_t)rows * s.half) return;
        const int r = s.row0 + (int)(idx / s.half), i = (int)(idx % s.half);
        cs[(int64_t)r * s.half + i] = rope_pair(tree_position(r, s.P, s.T), i, s.log_theta_over_half);
    } else {
        const int tail = (int)(s.ldv - s.R);
        const int64_t i = (int64_t)((int)blockIdx.x - s.row_wgs - s.rope_wgs) * 256 + threadIdx.x;
        if (i < s.vt_rows * tail) vt[(i / tail) * s.ldv + s.R + (i % tail)] = from_f32<T>(0.f);
    }
}

// One decoding step's rows: h[j] = embedding of ids[j stride], xn[j] = rmsnorm(h[j]; gain)
template <typename T>
__global__ __launch_bounds__(256) void embed_norm_rows_kernel(const T* __restrict__ emb, int vocab, int d, const int32_t* __restrict__ ids,
                                                              int64_t stride, float* __restrict__ h, const float* __restrict__ gain,
                                                              float eps, T* __restrict__ xn, int32_t* __restrict__ err_flag) {
    __shared__ float red[4];
    const int j = blockIdx.x;
    int id = ids[(int64_t)j * stride];
    if (id < 0 || id >= vocab) {
        if (threadIdx.x == 0) *err_flag = 1;
        id = 0;
    }
    embed_norm_row<T>(emb + (int64_t)id * d, d, h + (int64_t)j * d, gain, eps, xn + (int64_t)j * d, red);
}

// (cos, sin) rows by absolute position, for decoding
__global__ void rope_table_kernel(float2* __restrict__ cs, int first, int rows, int half, double log_theta_over_half) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)rows * half) return;
    const int r = first + (int)(idx / half), i = (int)(idx % half);
    cs[(int64_t)r * half + i] = rope_pair(r, i, log_theta_over_half);
}

// ---- residual update from K-slice partial sums, fused with the next RMSNorm ------------------------------
// One row per workgroup: h[r] += part[0][r] + part[1][r] + ... (slice order, so the sum does not depend on which
// workgroup of the projection finished first), then, with a gain vector, out[r] = rmsnorm(h[r]).  Up to 4 float4 per
// thread stay in registers between the passes; longer rows are read back (each thread re-reads what it wrote itself).
// A call with few rows is a handful of workgroups whose time is the latency of their loads: kThreads = 1024 then, so that a
// thread has one float4 of the row and requests eight slices of it at once: 4 rows of 3584 with nine slices 6.3 -> 4.8 us,
// 128 rows 8.1 -> 6.2.  From 512 rows on the two are alike (512: 13.1 and 13.1, 776: 15.4 and 14.8, 1024: 16.5 and 17.4).
template <typename T, int kThreads>
__global__ __launch_bounds__(kThreads) void resid_norm_kernel(float* __restrict__ h, const float* __restrict__ part, int n_slices,
                                                              int64_t pitch, const float* __restrict__ gain, float eps, int d,
                                                              T* __restrict__ out) {
    __shared__ float red[kThreads / 64];
    constexpr int kKeep = kThreads == 1024 ? 1 : 4;
    const int n4 = d >> 2;
    float4* x4 = reinterpret_cast<float4*>(h + (int64_t)blockIdx.x * d);
    const float4* p4 = reinterpret_cast<const float4*>(part + (int64_t)blockIdx.x * d);
    const int64_t pitch4 = pitch >> 2;
    // the slices are requested kBatch at a time for all of the thread's chunks, then added in slice order; a slice past the
    // last one contributes +0
    float4 keep[kKeep];
    constexpr int kBatch = kThreads == 1024 ? 8 : 4;
#pragma unroll
    for (int q = 0; q < kKeep; ++q) {
        const int c = threadIdx.x + kThreads * q;
        keep[q] = c < n4 ? x4[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int s0 = 0; s0 < n_slices; s0 += kBatch) {
        float4 t[kBatch][kKeep];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
#pragma unroll
            for (int q = 0; q < kKeep; ++q) {
                const int c = threadIdx.x + kThreads * q;
                t[u][q] = (s0 + u < n_slices && c < n4) ? p4[(s0 + u) * pitch4 + c] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
#pragma unroll
            for (int q = 0; q < kKeep; ++q) {
                keep[q].x += t[u][q].x; keep[q].y += t[u][q].y; keep[q].z += t[u][q].z; keep[q].w += t[u][q].w;
            }
    }
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < kKeep; ++q) {
        const int c = threadIdx.x + kThreads * q;
        if (c < n4) x4[c] = keep[q];
        ss += keep[q].x * keep[q].x + keep[q].y * keep[q].y + keep[q].z * keep[q].z + keep[q].w * keep[q].w;
    }
    for (int c = threadIdx.x + kThreads * kKeep; c < n4; c += kThreads) {
        float4 v = x4[c];
        for (int s0 = 0; s0 < n_slices; s0 += kBatch) {
            float4 t[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) t[u] = s0 + u < n_slices ? p4[(s0 + u) * pitch4 + c] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) { v.x += t[u].x; v.y += t[u].y; v.z += t[u].z; v.w += t[u].w; }
        }
        x4[c] = v;
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
    if (!gain) return;                                          // block-uniform
    ss = block_sum<kThreads>(ss, red);
    const float inv = rsqrtf(ss / (float)d + eps);
    const float4* g4 = reinterpret_cast<const float4*>(gain);
    T* o = out + (int64_t)blockIdx.x * d;
#pragma unroll
    for (int q = 0; q < kKeep; ++q) {
        const int c = threadIdx.x + kThreads * q;
        if (c < n4) {
            const float4 g = g4[c];
            store4<T>(o + 4 * c, make_float4(keep[q].x * inv * g.x, keep[q].y * inv * g.y, keep[q].z * inv * g.z,
                                             keep[q].w * inv * g.w));
        }
    }
    for (int c = threadIdx.x + kThreads * kKeep; c < n4; c += kThreads) {
        const float4 v = x4[c], g = g4[c];
        store4<T>(o + 4 * c, make_float4(v.x * inv * g.x, v.y * inv * g.y, v.z * inv * g.z, v.w * inv * g.w));
    }
}

// ---- S2 epilogue (unfused): rotate q and k in place -------------------------------------------
// One thread per (row, head, pair).  Heads 0 .. nq + nkv - 1 of the qkv row are rotated.
template <typename T>
__global__ __launch_bounds__(256) void rope_kernel(T* __restrict__ qkv, const float2* __restrict__ cs, int R,
                                                   int n_rot_heads, int hd, int64_t ld) {
    const int half = hd >> 1;
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t total = (int64_t)R * n_rot_heads * half;
    if (idx >= total) return;
    int i = (int)(idx % half);
    int head = (int)((idx / half) % n_rot_heads);
    int r = (int)(idx / ((int64_t)half * n_rot_heads));
    float2 c_s = cs[(int64_t)r * half + i];
    T* p = qkv + (int64_t)r * ld + head * hd + i;
    float x1 = to_f32<T>(p[0]), x2 = to_f32<T>(p[half]);
    p[0] = from_f32<T>(x1 * c_s.x - x2 * c_s.y);
    p[half] = from_f32<T>(x2 * c_s.x + x1 * c_s.y);
}

// ---- V transpose: vt[kvh][c][r] = qkv[r][v_off + kvh hd + c] ------------------------------------
// 64 x 64 tiles through LDS so both the read and the write are coalesced.  Columns r in [R, ldv)
// are written as zero: the attention kernel loads whole 64-key tiles and multiplies the masked
// probabilities (exact zeros) with whatever it finds there.
template <typename T>
__global__ __launch_bounds__(256) void transpose_v_kernel(const T* __restrict__ qkv, int row0, int R, int64_t ld, int v_off,
                                                          int hd, T* __restrict__ vt, int64_t ldv) {
    __shared__ T tile[64][65];
    const int r0 = row0 / 64 * 64 + blockIdx.x * 64, c0 = blockIdx.y * 64, kvh = blockIdx.z;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int i = ty; i < 64; i += 4) {
        int r = r0 + i, c = c0 + tx;
        tile[i][tx] = (r < R && c < hd) ? qkv[(int64_t)r * ld + v_off + kvh * hd + c] : from_f32<T>(0.f);
    }
    __syncthreads();
    for (int i = ty; i < 64; i += 4) {
        int c = c0 + i, r = r0 + tx;
        if (c < hd && r >= row0 && r < ldv) vt[((int64_t)kvh * hd + c) * ldv + r] = tile[tx][i];
    }
}

// Up to CopyBlocks::kMax blocks of pitched arrays, dst[r][c] = src[r][c] (prefix cache <-> workspace), by workgroups 0, 1, ...
// of a launch or a part of one.  A block whose rows start at multiples of 16 bytes on both sides takes 16 bytes per thread (the
// end of its rows element by element); any other one element per thread, so that a wavefront's accesses stay together:
// V^T of an extension whose prefix length is not a multiple of 8.
template <typename T>
__device__ __forceinline__ void copy_blocks(const CopyBlocks& jobs, int wg) {
    constexpr int V = 16 / (int)sizeof(T);
    int64_t i = (int64_t)wg * 256 + threadIdx.x;
#pragma unroll
    for (int j = 0; j < CopyBlocks::kMax; ++j) {
        if (j >= jobs.n) return;
        const CopyBlock& b = jobs.b[j];
        const int64_t pieces = b.wide ? (b.cols + V - 1) / V : b.cols, total = b.rows * pieces;
        if (i < total) {
            const int64_t r = i / pieces, c = (i % pieces) * (b.wide ? V : 1);
            const T* src = reinterpret_cast<const T*>(b.src) + r * b.src_ld + c;
            T* dst = reinterpret_cast<T*>(b.dst) + r * b.dst_ld + c;
            if (!b.wide) {
                *dst = *src;
            } else if (c + V <= b.cols) {
                *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
            } else {
                for (int u = 0; c + u < b.cols; ++u) dst[u] = src[u];
            }
            return;
        }
        i -= total;
    }
}
template <typename T>
__global__ __launch_bounds__(256) void copy_blocks_kernel(const CopyBlocks jobs) {
    copy_blocks<T>(jobs, (int)blockIdx.x);
}

// Finish of a K-split QKV projection: acc [n_slices][rows, (nq + 2 nkv) hd] holds the fp32 partial sums of the K slices,
// added here in slice order.  One thread per (row, head, rotation pair i < hd / 2): q and k heads are rotated
// (rotate-half RoPE, table row cs[r]) and stored to the qkv row, v heads are stored to the transposed copy
// vt [nkv hd, ldv] at column r.  The workgroups from finish_wgs on put the cached prefix rows in place (other rows of the same
// buffers): one launch of 7.2 us where finish, key copy and value copy took
// 6.0 + 4.8 + 4.8 (128 rows, prefix 512, 7B width).
template <typename T>
__global__ __launch_bounds__(256) void qkv_finish_kernel(const float* __restrict__ acc, int n_slices, int64_t pitch,
                                                         const float2* __restrict__ cs, int rows, int nq, int nkv, int hd,
                                                         T* __restrict__ qkv, T* __restrict__ vt, int64_t ldv, int finish_wgs,
                                                         const CopyBlocks jobs) {
    if ((int)blockIdx.x >= finish_wgs) {
        copy_blocks<T>(jobs, (int)blockIdx.x - finish_wgs);
        return;
    }
    const int half = hd >> 1, heads = nq + 2 * nkv;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)rows * heads * half) return;
    const int i = (int)(idx % half);
    const int head = (int)((idx / half) % heads);
    const int r = (int)(idx / ((int64_t)half * heads));
    const int64_t ld = (int64_t)heads * hd;
    const float* a = acc + (int64_t)r * ld + head * hd + i;
    float x1 = 0.f, x2 = 0.f;
    for (int s0 = 0; s0 < n_slices; s0 += 4) {          // four slices' loads in flight, added in slice order
        float t1[4], t2[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            t1[u] = s0 + u < n_slices ? a[(s0 + u) * pitch] : 0.f;
            t2[u] = s0 + u < n_slices ? a[(s0 + u) * pitch + half] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x1 += t1[u];
            x2 += t2[u];
        }
    }
    if (head < nq + nkv) {
        const float2 c_s = cs[(int64_t)r * half + i];
        T* p = qkv + (int64_t)r * ld + head * hd + i;
        p[0] = from_f32<T>(x1 * c_s.x - x2 * c_s.y);
        p[half] = from_f32<T>(x2 * c_s.x + x1 * c_s.y);
    } else {
        T* p = vt + ((int64_t)(head - nq - nkv) * hd + i) * ldv + r;
        p[0] = from_f32<T>(x1);
        p[(int64_t)half * ldv] = from_f32<T>(x2);
    }
}

// ---- S6: gather the scoring rows, final RMSNorm, targets -----------------------------------------
// Scoring row b = k T + t reads the hidden state that predicts y^k_t: the last prefix row (`first`: in the tree, or kept with a cached
// prefix) for t = 0, else the row of y^k_{t-1}.
template <typename T>
__global__ __launch_bounds__(256) void gather_norm_kernel(const float* __restrict__ h, const float* __restrict__ first, const float* __restrict__ gain,
                                                          float eps, int d, const int32_t* __restrict__ draft_ids,
                                                          const int32_t* __restrict__ draft_lens, int vocab, int P,
                                                          int Tn, T* __restrict__ xs, int32_t* __restrict__ targets,
                                                          uint8_t* __restrict__ valid) {
    __shared__ float red[4];
    const int b = blockIdx.x;
    const int k = b / Tn, t = b % Tn;
    rmsnorm_row<T>(t == 0 ? first : h + (int64_t)(P + k * Tn + t - 1) * d, gain, eps, d, xs + (int64_t)b * d, red);
    if (threadIdx.x == 0) {
        int id = draft_ids[b];
        bool ok = !(draft_lens && t >= draft_lens[k]);
        if (id < 0 || id >= vocab) id = 0;   // flagged by the embedding kernel already
        targets[b] = id;
        valid[b] = ok ? 1 : 0;
    }
}

// ---- S8: conformity score per draft, fixed-order tree sum ------------------------------------------
__global__ __launch_bounds__(256) void score_reduce_kernel(const float* __restrict__ lp,
                                                           const int32_t* __restrict__ draft_lens, int Tn, int mode,
                                                           float* __restrict__ token_logprobs,
                                                           float* __restrict__ scores) {
    __shared__ float red[4];
    const int k = blockIdx.x;
    const int len = draft_lens ? min(max(draft_lens[k], 0), Tn) : Tn;
    float s = 0.f;
    for (int t = threadIdx.x; t < Tn; t += 256) {
        float v = t < len ? lp[(int64_t)k * Tn + t] : 0.f;
        if (token_logprobs) token_logprobs[(int64_t)k * Tn + t] = v;
        s += v;
    }
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) scores[k] = mode == ATTS_SCORE_MEAN_NLL ? -s / (float)max(len, 1) : -s;
}

}  // namespace

#define DISPATCH_T(dtype, ...)                       \
    if ((dtype) == ATTS_DTYPE_F32) {                 \
        typedef float T;                             \
        __VA_ARGS__                                  \
    } else {                                         \
        typedef bf16 T;                              \
        __VA_ARGS__                                  \
    }

int32_t launch_tree_start(int32_t dtype, const void* tok_embed, int32_t vocab, int32_t d, const int32_t* prefix_ids,
                          const int32_t* draft_ids, const int32_t* draft_lens, ScoreShape s, int32_t row0, float* h, const float* gain,
                          float eps, void* xn, float2* cs, int32_t hd, float theta, void* vt, int64_t vt_rows, int64_t ldv,
                          int32_t* err_flag, hipStream_t stream) {
    StartDims t{};
    t.vocab = vocab; t.d = d; t.P = s.P; t.T = s.T; t.row0 = row0; t.R = s.R(); t.half = hd / 2; t.eps = eps;
    t.log_theta_over_half = log((double)theta) / (double)t.half;
    t.ldv = ldv;
    t.vt_rows = vt ? vt_rows : 0;
    const int64_t rows = t.R - row0, rope = ceil_div(rows * t.half, 256), zero = vt ? ceil_div(vt_rows * (ldv - t.R), 256) : 0;
    auto launch = [&](int64_t row_wgs, int64_t rope_wgs, int64_t zero_wgs) {
        t.row_wgs = (int32_t)row_wgs;
        t.rope_wgs = (int32_t)rope_wgs;
        DISPATCH_T(dtype, hipLaunchKernelGGL(tree_start_kernel<T>, dim3((unsigned)(row_wgs + rope_wgs + zero_wgs)), dim3(256), 0, stream,
                                             (const T*)tok_embed, prefix_ids, draft_ids, draft_lens, h, gain, (T*)xn, cs, (T*)vt, err_flag, t);)
    };
    // a launch of 2^32 threads or more runs a part of them without an error: together the parts reach that at 11.2 million rows
    // (head_dim 256), by themselves none does below the 2^24 rows a call may have
    if (rows + rope + zero < (1 << 24)) {
        launch(rows, rope, zero);
    } else {
        launch(rows, 0, 0);
        ATTS_LAUNCH_CHECK("tree_start_kernel");
        launch(0, rope, zero);
    }
    ATTS_LAUNCH_CHECK("tree_start_kernel");
    return ATTS_OK;
}

int32_t launch_embed_norm_rows(int32_t dtype, const void* tok_embed, int32_t vocab, int32_t d, const int32_t* ids, int64_t stride,
                               int32_t rows, float* h, const float* gain, float eps, void* xn, int32_t* err_flag, hipStream_t stream) {
    DISPATCH_T(dtype, hipLaunchKernelGGL(embed_norm_rows_kernel<T>, dim3(rows), dim3(256), 0, stream, (const T*)tok_embed, vocab, d, ids,
                                         stride, h, gain, eps, (T*)xn, err_flag);)
    ATTS_LAUNCH_CHECK("embed_norm_rows_kernel");
    return ATTS_OK;
}

int32_t launch_rmsnorm(int32_t dtype, const float* h, const float* gain, float eps, int32_t rows, int32_t d, void* out,
                       hipStream_t stream) {
    DISPATCH_T(dtype, hipLaunchKernelGGL(rmsnorm_kernel<T>, dim3(rows), dim3(256), 0, stream, h, gain, eps, d, (T*)out);)
    ATTS_LAUNCH_CHECK("rmsnorm_kernel");
    return ATTS_OK;
}

int32_t launch_rope_table(float2* cs, int32_t first, int32_t rows, int32_t hd, float theta, hipStream_t stream) {
    const int half = hd / 2;
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)ceil_div((int64_t)rows * half, 256)), dim3(256), 0, stream, cs, first, rows, half,
                       log((double)theta) / (double)half);
    ATTS_LAUNCH_CHECK("rope_table_kernel");
    return ATTS_OK;
}

int32_t launch_transpose_v(int32_t dtype, const void* qkv, int32_t row0, int32_t R, int32_t nq, int32_t nkv, int32_t hd,
                           void* vt, int64_t ldv, hipStream_t stream) {
    const int64_t ld = (int64_t)(nq + 2 * nkv) * hd;
    dim3 grid((unsigned)ceil_div(ldv - row0 / 64 * 64, 64), (unsigned)ceil_div(hd, 64), nkv);
    DISPATCH_T(dtype, hipLaunchKernelGGL(transpose_v_kernel<T>, grid, dim3(256), 0, stream, (const T*)qkv, row0, R, ld,
                                         (nq + nkv) * hd, hd, (T*)vt, ldv);)
    ATTS_LAUNCH_CHECK("transpose_v_kernel");
    return ATTS_OK;
}

int32_t launch_rope_split(int32_t dtype, void* qkv, const float2* cs, ScoreShape s, int32_t row0, int32_t nq, int32_t nkv,
                          int32_t hd, void* vt, int64_t ldv, hipStream_t stream) {
    const int64_t ld = (int64_t)(nq + 2 * nkv) * hd;
    const int rows = s.R() - row0;
    const int64_t total = (int64_t)rows * (nq + nkv) * (hd / 2);
    DISPATCH_T(dtype, hipLaunchKernelGGL(rope_kernel<T>, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, stream,
                                         (T*)qkv + (int64_t)row0 * ld, cs + (int64_t)row0 * (hd / 2), rows, nq + nkv, hd, ld);)
    ATTS_LAUNCH_CHECK("rope_kernel");
    if (vt) return launch_transpose_v(dtype, qkv, row0, s.R(), nq, nkv, hd, vt, ldv, stream);
    return ATTS_OK;
}

int32_t launch_qkv_finish(int32_t dtype, const float* acc, int32_t n_slices, int64_t slice_pitch, const float2* cs, int32_t rows,
                          int32_t nq, int32_t nkv, int32_t hd, void* qkv, void* vt, int64_t ldv, const CopyBlocks& copies,
                          hipStream_t stream) {
    const int64_t finish = ceil_div((int64_t)rows * (nq + 2 * nkv) * (hd / 2), 256);
    DISPATCH_T(dtype, hipLaunchKernelGGL(qkv_finish_kernel<T>, dim3((unsigned)(finish + copy_workgroups(dtype, copies))), dim3(256), 0, stream,
                                         acc, n_slices, slice_pitch, cs, rows, nq, nkv, hd, (T*)qkv, (T*)vt, ldv, (int)finish, copies);)
    ATTS_LAUNCH_CHECK("qkv_finish_kernel");
    return ATTS_OK;
}

int32_t launch_resid_norm(int32_t dtype, float* h, const float* partials, int32_t n_slices, int64_t slice_pitch, const float* gain,
                          float eps, int32_t rows, int32_t d, void* xn, hipStream_t stream) {
    if (rows <= 0) return ATTS_OK;
    if (d % 4 || slice_pitch % 4) return fail(ATTS_ERR_SHAPE, "residual update: row length and slice pitch must be multiples of 4");
    DISPATCH_T(dtype, if (rows <= 512)
                          hipLaunchKernelGGL((resid_norm_kernel<T, 1024>), dim3(rows), dim3(1024), 0, stream, h, partials, n_slices, slice_pitch,
                                             gain, eps, d, (T*)xn);
                      else
                          hipLaunchKernelGGL((resid_norm_kernel<T, 256>), dim3(rows), dim3(256), 0, stream, h, partials, n_slices, slice_pitch,
                                             gain, eps, d, (T*)xn);)
    ATTS_LAUNCH_CHECK("resid_norm_kernel");
    return ATTS_OK;
}

void add_copy(int32_t dtype, CopyBlocks& jobs, const void* src, int64_t src_ld, void* dst, int64_t dst_ld, int64_t rows, int64_t cols) {
    if (rows <= 0 || cols <= 0) return;
    const int64_t es = (int64_t)dtype_size(dtype);
    const bool wide = ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst) | (uintptr_t)(src_ld * es) | (uintptr_t)(dst_ld * es)) & 15) == 0;
    jobs.b[jobs.n++] = CopyBlock{src, dst, src_ld, dst_ld, rows, cols, wide};
}
int64_t copy_workgroups(int32_t dtype, const CopyBlocks& jobs) {
    const int64_t v = 16 / (int64_t)dtype_size(dtype);
    int64_t pieces = 0;
    for (int j = 0; j < jobs.n; ++j) pieces += jobs.b[j].rows * (jobs.b[j].wide ? ceil_div(jobs.b[j].cols, v) : jobs.b[j].cols);
    return ceil_div(pieces, 256);
}
int32_t launch_copies(int32_t dtype, const CopyBlocks& jobs, hipStream_t stream) {
    if (jobs.n == 0) return ATTS_OK;
    DISPATCH_T(dtype, hipLaunchKernelGGL(copy_blocks_kernel<T>, dim3((unsigned)copy_workgroups(dtype, jobs)), dim3(256), 0, stream, jobs);)
    ATTS_LAUNCH_CHECK("copy_blocks_kernel");
    return ATTS_OK;
}

int32_t launch_gather_norm(int32_t dtype, const float* h, const float* first, const float* gain, float eps, int32_t d,
                           const int32_t* draft_ids, const int32_t* draft_lens, int32_t vocab, ScoreShape s, void* xs,
                           int32_t* targets, uint8_t* valid, hipStream_t stream) {
    DISPATCH_T(dtype, hipLaunchKernelGGL(gather_norm_kernel<T>, dim3(s.B()), dim3(256), 0, stream, h, first, gain, eps, d,
                                         draft_ids, draft_lens, vocab, s.P, s.T, (T*)xs, targets, valid);)
    ATTS_LAUNCH_CHECK("gather_norm_kernel");
    return ATTS_OK;
}

int32_t launch_score_reduce(const float* lp, const int32_t* draft_lens, int32_t K, int32_t T, int32_t mode,
                            float* token_logprobs, float* scores, hipStream_t stream) {
    hipLaunchKernelGGL(score_reduce_kernel, dim3(K), dim3(256), 0, stream, lp, draft_lens, T, mode, token_logprobs, scores);
    ATTS_LAUNCH_CHECK("score_reduce_kernel");
    return ATTS_OK;
}

}  // namespace atts
