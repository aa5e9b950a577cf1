// NT GEMM for products too small to fill the chip with 128 x 128 tiles:  acc[M, N] = A[M, Kd] . W[N, Kd]^T.
//
// A small model's projections (the fp32 one: 320 rows, 128 to 512 features) are 3 to 24 tiles of the general kernel, each
// walking the whole K range by itself: what bounds them is the chain of matrix instructions of one wavefront (an fp32
// 32 x 32 x 2 step occupies the matrix pipe for 64 cycles, 64 of them per 32-deep slab of a 64 x 64 wave tile), while most
// compute units idle.  Here a workgroup of four wavefronts owns one 32 x 32 tile (32 x 64 for SwiGLU and the LM head) and
// the four split its K range, each in a contiguous quarter:
//   * operands go global -> registers (16 bytes per lane and step, A and W rows alike; the operands of such products sit
//     in the L2s), kSmallUnroll steps requested ahead of their matrix instructions, two buffers; no LDS, no barrier in
//     the loop;
//   * the four partial sums meet once in LDS and are added in wavefront order (no atomics: bit-reproducible).
// Against 128 x 128 tiles: fp32 320 x 128 x 512 45.3 -> 7.1 us, 320 x 512 x 128 15.3 -> 3.7, 1024 x 512 x 512 45.6 -> 13.4,
// 64 x 4096 x 4096 330 -> 35; bf16 320 x 512 x 512 11.7 -> 4.4.  The scoring pass of the fp32 model (2 layers, 320 rows):
// 267 -> 104 us.
// A launch of such a product is itself a third of its time, so in fp32 the passes around it ride along (2 layers,
// 320 rows: 20 launches and 90.5 us -> 15 and 80.0, the old residual values requested with the operands included):
//   kNorm  A is the residual stream: its rows are multiplied by the norm's gain as they are read, their sums of squares are taken
//          on the way, and the finished sums are scaled by 1 / rms;
//          (LM head: the rows are the scoring rows, gathered from the token tree; the targets are the draft ids.)
//   EPI_QKV_ROPE  heads of at most 32 columns lie inside one tile: rotated with the partner column's value from the lane that
//          holds it (values stay rows of the output, there is no transposed copy here).
#include "common.h"

namespace atts {
namespace {

constexpr int kSmallWaves = 4;
constexpr int kSmallUnroll = 4;

struct SmallDims {
    int32_t M, N, Kd;
    int64_t lda, ldw, ldc;
    int32_t n_part, nt_m;
    float eps;                              // kNorm
    int32_t rot_cols, half_hd, cs_ld;       // EPI_QKV_ROPE: columns that are rotated, half a head's columns (a power of two), pitch of the table
    const float* first;                     // EPI_LMHEAD with kNorm: see GemmArgs
    int32_t tree_P, tree_T;
};

// One step: lane (row = l % 32, half = l / 32) holds 16 bytes of its row, at byte 32 step + 16 half.  bf16: the operand of
// one 32 x 32 x 16 product.  fp32: four floats = four 32 x 32 x 2 products (the k order inside a step is permuted alike for
// both operands, which leaves the dot product unchanged).
template <typename T> struct SmallMma;
template <> struct SmallMma<bf16> {
    static __device__ __forceinline__ void mma(const uint4& a, const uint4& w, f32x16& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, w), c, 0, 0, 0);
    }
};
template <> struct SmallMma<float> {
    static __device__ __forceinline__ void mma(const uint4& a, const uint4& w, f32x16& c) {
        const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, w);
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], c, 0, 0, 0);
    }
};

template <typename T, int EPI, int NI, bool kNorm = false>
__global__ __launch_bounds__(64 * kSmallWaves) void gemm_small_kernel(const char* __restrict__ gA, const char* __restrict__ gW,
                                                                      void* __restrict__ g_out, const int32_t* __restrict__ g_targets,
                                                                      float2* __restrict__ g_partials, float* __restrict__ g_target_logit,
                                                                      const float* __restrict__ g_gain, const float2* __restrict__ g_rope,
                                                                      const SmallDims d) {
    static_assert(!kNorm || sizeof(T) == 4, "the residual stream is fp32");
    constexpr int ES = (int)sizeof(T), N_OUT = EPI == EPI_SWIGLU ? 32 : 32 * NI;
    static_assert((EPI == EPI_SWIGLU || EPI == EPI_LMHEAD) == (NI == 2), "tile width");
    __shared__ float part[kSmallWaves][NI][16][64];
    __shared__ float squares[kNorm ? kSmallWaves : 1][32];
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));    // scalar: the K loop's branches must be too
    const int tm = (int)blockIdx.x % d.nt_m, tn = (int)blockIdx.x / d.nt_m;
    const int m0 = tm * 32, n0 = tn * N_OUT;

    // rows and columns past the end repeat the last one (their results are dropped); 16-byte pieces past the end are zero
    const int a_row = min(m0 + l32, d.M - 1);
    const char* ap = gA + (int64_t)a_row * d.lda * ES + 16 * half;
    if constexpr (EPI == EPI_LMHEAD && kNorm) {                             // the hidden state that predicts token a_row % T of its draft
        ap = gA + (int64_t)(d.tree_P + a_row - 1) * d.lda * ES + 16 * half;
        if (a_row % d.tree_T == 0) ap = reinterpret_cast<const char*>(d.first) + 16 * half;
    }
    const char* wp[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int row = EPI == EPI_SWIGLU ? min(n0 + l32, d.N - 1) + j * d.N : min(n0 + 32 * j + l32, d.N - 1);
        wp[j] = gW + (int64_t)row * d.ldw * ES + 16 * half;
    }
    const int k_bytes = d.Kd * ES;
    const int n_steps = (k_bytes + 31) / 32;
    const int s0 = wave * n_steps / kSmallWaves, s1 = (wave + 1) * n_steps / kSmallWaves;
    struct Frags {
        uint4 a[kSmallUnroll], w[NI][kSmallUnroll], gain[kNorm ? kSmallUnroll : 1];
    };
    auto load = [&](Frags& f, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kSmallUnroll; ++u) {
            const int64_t off = (int64_t)(s + u) * 32;
            const bool ok = s + u < s1 && off + 16 * half < k_bytes;
            f.a[u] = ok ? *reinterpret_cast<const uint4*>(ap + off) : make_uint4(0, 0, 0, 0);
            if constexpr (kNorm)
                f.gain[u] = ok ? *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(g_gain) + off + 16 * half) : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NI; ++j) f.w[j][u] = ok ? *reinterpret_cast<const uint4*>(wp[j] + off) : make_uint4(0, 0, 0, 0);
        }
    };
    // residual update: the old values are on their way with the operands, not waited for behind the sums
    const int row0 = m0 + 8 * wave + 4 * half, col = n0 + l32;
    float old[EPI == EPI_RESID_F32 ? 4 : 1];
    if constexpr (EPI == EPI_RESID_F32) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
            old[b] = reinterpret_cast<const float*>(g_out)[(int64_t)min(row0 + b, d.M - 1) * d.ldc + min(col, d.N - 1)];
    }
    // ... and the rotation's table and the targets likewise
    float2 cs[EPI == EPI_QKV_ROPE ? 4 : 1];
    if constexpr (EPI == EPI_QKV_ROPE) {
#pragma unroll
        for (int b = 0; b < 4; ++b) cs[b] = g_rope[(int64_t)min(row0 + b, d.M - 1) * d.cs_ld + (col & (d.half_hd - 1))];
    }
    int target[EPI == EPI_LMHEAD ? 4 : 1];
    if constexpr (EPI == EPI_LMHEAD) {
#pragma unroll
        for (int b = 0; b < 4; ++b) target[b] = g_targets[min(row0 + b, d.M - 1)];
    }
    f32x16 acc[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    float sq = 0.f;
    auto mma = [&](const Frags& f) __attribute__((always_inline)) {      // steps past the end multiply zeros
#pragma unroll
        for (int u = 0; u < kSmallUnroll; ++u) {
            uint4 a = f.a[u];
            if constexpr (kNorm) {
                f32x4 x = __builtin_bit_cast(f32x4, a);
                const f32x4 gain = __builtin_bit_cast(f32x4, f.gain[u]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sq += x[e] * x[e];
                    x[e] *= gain[e];
                }
                a = __builtin_bit_cast(uint4, x);
            }
#pragma unroll
            for (int j = 0; j < NI; ++j) SmallMma<T>::mma(a, f.w[j][u], acc[j]);
        }
    };
    Frags fa, fb;
    load(fa, s0);
    for (int s = s0; s < s1; s += 2 * kSmallUnroll) {
        load(fb, s + kSmallUnroll);
        mma(fa);
        if (s + kSmallUnroll < s1) {                                        // scalar
            load(fa, s + 2 * kSmallUnroll);
            mma(fb);
        }
    }
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) part[wave][j][v][lane] = acc[j][v];
    if constexpr (kNorm) {
        sq += __shfl_xor(sq, 32);
        if (half == 0) squares[wave][l32] = sq;
    }
    __syncthreads();

    // wavefront w finishes entries v = 4 w .. 4 w + 3 of every block: rows m0 + 8 w + 4 half + (v & 3), column l32
    float z[NI][4];
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float s = part[0][j][4 * wave + b][lane];
#pragma unroll
            for (int w = 1; w < kSmallWaves; ++w) s += part[w][j][4 * wave + b][lane];
            if constexpr (kNorm) {
                float sum = 0.f;
#pragma unroll
                for (int w = 0; w < kSmallWaves; ++w) sum += squares[w][8 * wave + 4 * half + b];
                s *= rsqrtf(sum / (float)d.Kd + d.eps);
            }
            z[j][b] = s;
        }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int row = row0 + b;
        if constexpr (EPI == EPI_LMHEAD) {
            const bool row_ok = row < d.M;                                  // uniform over the 32 lanes that share `half`
            int tcol = target[b];
            if constexpr (kNorm)
                if (tcol < 0 || tcol >= d.N) tcol = 0;                      // flagged by the embedding kernel already
            tcol = row_ok ? tcol - n0 : -1;
            float mx = -INFINITY;
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                if (col + 32 * j < d.N) mx = fmaxf(mx, z[j][b]);
                if (tcol == 32 * j + l32) g_target_logit[row] = z[j][b];
            }
#pragma unroll
            for (int o = 1; o < 32; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
            float sum = 0.f;
            if (mx > -INFINITY) {
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    if (col + 32 * j < d.N) sum += __expf(z[j][b] - mx);
            }
#pragma unroll
            for (int o = 1; o < 32; o <<= 1) sum += __shfl_xor(sum, o);
            if (row_ok && l32 == 0) g_partials[(int64_t)row * d.n_part + tn] = make_float2(mx, sum);
        } else {
            float rotated = 0.f;
            if constexpr (EPI == EPI_QKV_ROPE) {                            // every lane of the wavefront takes part in the exchange
                const float other = __shfl_xor(z[0][b], d.half_hd);
                rotated = (col & d.half_hd) ? z[0][b] * cs[b].x + other * cs[b].y : z[0][b] * cs[b].x - other * cs[b].y;
                if (col >= d.rot_cols) rotated = z[0][b];
            }
            if (row >= d.M || col >= d.N) continue;
            const int64_t idx = (int64_t)row * d.ldc + col;
            if constexpr (EPI == EPI_SWIGLU) {
                const float gate = z[0][b], up = z[1][b];
                // hardware reciprocal, as in the tiled kernels
                reinterpret_cast<T*>(g_out)[idx] = from_f32<T>(gate * __builtin_amdgcn_rcpf(1.f + __expf(-gate)) * up);
            } else if constexpr (EPI == EPI_QKV_ROPE) {
                reinterpret_cast<T*>(g_out)[idx] = from_f32<T>(rotated);
            } else if constexpr (EPI == EPI_STORE_ACT) {
                reinterpret_cast<T*>(g_out)[idx] = from_f32<T>(z[0][b]);
            } else if constexpr (EPI == EPI_RESID_F32) {
                reinterpret_cast<float*>(g_out)[idx] = old[b] + z[0][b];
            } else {
                reinterpret_cast<float*>(g_out)[idx] = z[0][b];
            }
        }
    }
}

// fp32 products of so few 32 x 32 tiles that most compute units would idle: 16 x 16 tiles, four times as many workgroups, each wavefront's
// chain of matrix instructions a quarter as long.  A step is 64 bytes of K a row: lane (r = l % 16, q = l / 16) holds floats 4 q .. 4 q + 3 of
// its row, the operand of four 16 x 16 x 4 products (the k order inside a step is permuted alike for both operands).  Eight steps are
// requested at once, so that K up to 512 waits for one latency.  us, 32 x 32 and 16 x 16 tiles: 320 x 128 x 512 (40 tiles) 6.9 and 4.9,
// 100 x 256 x 1024 (32) 10.4 and 6.2, 64 x 1024 x 4096 (64) 33.2 and 21.8, 1000 x 128 x 512 (128) 7.0 and 6.3, 100 x 768 x 768 (96) 8.6 both;
// 320 x 512 x 512 (160) 7.0 and 8.4, 300 x 768 x 3072 (240) 27.8 and 50.1: the operands are read twice as often.
constexpr int kSmall16Unroll = 8;
// Where the smaller tiles are taken: up to 128 tiles of 32 x 32 (80 above K = 1024), and of those with more than one small tile a compute unit
// only where the eight steps requested at once are mostly there, or a single one.  Small over large tiles, time: up to 256 small ones 0.55 (K = 4096) to
// 0.94 (K = 128); more of them K <= 32 0.87 .. 0.94, 36 .. 128 1.00 .. 1.18 (1000 x 100 x 128 3.4 and 4.1 us), 132 .. 800 0.80 .. 1.01, 832 .. 1024
// 1.00 .. 1.12 (1000 x 128 x 1024 10.6 and 11.6), above that 0.94 .. 1.01 up to 80 large tiles; 96 x 1024 x 2048 (96) 17.5 and 18.3, 64 x 2048 x 4096 (128) 33.6 and 37.4
static bool use_tiles_of_16(const GemmArgs& g) {
    if (ceil_div(g.M, 32) * ceil_div(g.N, 32) > (g.Kd <= 1024 ? 128 : 80)) return false;
    return ceil_div(g.M, 16) * ceil_div(g.N, 16) <= 256 || g.Kd <= 32 || (g.Kd > 128 && g.Kd <= 800) || g.Kd > 1024;
}
template <int EPI>
__global__ __launch_bounds__(64 * kSmallWaves) void gemm_small16_kernel(const char* __restrict__ gA, const char* __restrict__ gW, float* __restrict__ g_out,
                                                                        const SmallDims d) {
    __shared__ float part[kSmallWaves][4][64];
    const int lane = threadIdx.x & 63, l16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));    // scalar: the K loop's branches must be too
    const int m0 = (int)blockIdx.x % d.nt_m * 16, n0 = (int)blockIdx.x / d.nt_m * 16;
    // rows and columns past the end repeat the last one (their results are dropped); 16-byte pieces past the end are zero
    const char* const ap = gA + (int64_t)min(m0 + l16, d.M - 1) * d.lda * 4 + 16 * q;
    const char* const wp = gW + (int64_t)min(n0 + l16, d.N - 1) * d.ldw * 4 + 16 * q;
    const int k_bytes = d.Kd * 4, n_steps = (k_bytes + 63) / 64;
    const int s0 = wave * n_steps / kSmallWaves, s1 = (wave + 1) * n_steps / kSmallWaves;
    struct Frags {
        uint4 a[kSmall16Unroll], w[kSmall16Unroll];
    };
    auto load = [&](Frags& f, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kSmall16Unroll; ++u) {
            const int64_t off = (int64_t)(s + u) * 64;
            const bool ok = s + u < s1 && off + 16 * q < k_bytes;
            f.a[u] = ok ? *reinterpret_cast<const uint4*>(ap + off) : make_uint4(0, 0, 0, 0);
            f.w[u] = ok ? *reinterpret_cast<const uint4*>(wp + off) : make_uint4(0, 0, 0, 0);
        }
    };
    const int row = m0 + 4 * q + wave, col = n0 + l16;                 // the element this lane finishes
    const bool mine = row < d.M && col < d.N;
    float old = 0.f;
    if constexpr (EPI == EPI_RESID_F32) old = g_out[(int64_t)min(row, d.M - 1) * d.ldc + min(col, d.N - 1)];
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const Frags& f) __attribute__((always_inline)) {   // steps past the end multiply zeros
#pragma unroll
        for (int u = 0; u < kSmall16Unroll; ++u) {
            const f32x4 x = __builtin_bit_cast(f32x4, f.a[u]), y = __builtin_bit_cast(f32x4, f.w[u]);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], acc, 0, 0, 0);
        }
    };
    Frags fa, fb;
    load(fa, s0);
    for (int s = s0; s < s1; s += 2 * kSmall16Unroll) {
        if (s + kSmall16Unroll < s1) {                                  // scalar
            load(fb, s + kSmall16Unroll);
            mma(fa);
            if (s + 2 * kSmall16Unroll < s1) load(fa, s + 2 * kSmall16Unroll);
            mma(fb);
        } else {
            mma(fa);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][v][lane] = acc[v];
    __syncthreads();
    float z = part[0][wave][lane];
#pragma unroll
    for (int w = 1; w < kSmallWaves; ++w) z += part[w][wave][lane];
    if (mine) g_out[(int64_t)row * d.ldc + col] = old + z;
}

template <typename T, int EPI, bool kNorm = false>
int32_t launch_small_epi(const GemmArgs& g, hipStream_t stream) {
    constexpr int NI = EPI == EPI_SWIGLU || EPI == EPI_LMHEAD ? 2 : 1, N_OUT = EPI == EPI_LMHEAD ? 64 : 32;
    if constexpr (sizeof(T) == 4 && (EPI == EPI_STORE_ACT || EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32)) {
        if (use_tiles_of_16(g)) {
            SmallDims d{};
            d.M = g.M; d.N = g.N; d.Kd = g.Kd;
            d.lda = g.lda; d.ldw = g.ldw; d.ldc = g.ldc;
            d.nt_m = (int32_t)ceil_div(g.M, 16);
            hipLaunchKernelGGL(gemm_small16_kernel<EPI>, dim3((unsigned)(d.nt_m * ceil_div(g.N, 16))), dim3(64 * kSmallWaves), 0, stream,
                               reinterpret_cast<const char*>(g.a), reinterpret_cast<const char*>(g.w), reinterpret_cast<float*>(g.out), d);
            ATTS_LAUNCH_CHECK("gemm_small16_kernel");
            return ATTS_OK;
        }
    }
    SmallDims d{g.M, g.N, g.Kd, g.lda, g.ldw, g.ldc, g.n_part, (int32_t)ceil_div(g.M, 32), g.norm_eps,
                g.n_rot_heads * g.head_dim, g.head_dim / 2, g.head_dim / 2, g.first, g.tree_P, g.tree_T};
    hipLaunchKernelGGL((gemm_small_kernel<T, EPI, NI, kNorm>), dim3((unsigned)(d.nt_m * ceil_div(g.N, N_OUT))), dim3(64 * kSmallWaves), 0, stream,
                       reinterpret_cast<const char*>(g.a), reinterpret_cast<const char*>(g.w), g.out, g.targets, g.partials, g.target_logit, g.norm_gain, g.rope, d);
    ATTS_LAUNCH_CHECK("gemm_small_kernel");
    return ATTS_OK;
}

template <typename T>
int32_t launch_small_t(GemmEpilogue epi, const GemmArgs& g, hipStream_t stream) {
    switch (epi) {
        case EPI_STORE_ACT: return launch_small_epi<T, EPI_STORE_ACT>(g, stream);
        case EPI_STORE_F32: return launch_small_epi<T, EPI_STORE_F32>(g, stream);
        case EPI_RESID_F32: return launch_small_epi<T, EPI_RESID_F32>(g, stream);
        case EPI_SWIGLU: return launch_small_epi<T, EPI_SWIGLU>(g, stream);
        case EPI_LMHEAD: return launch_small_epi<T, EPI_LMHEAD>(g, stream);
        default: break;
    }
    return fail(ATTS_ERR_INVALID_ARG, "gemm (small product): epilogue %d is not served", (int)epi);
}

}  // namespace

int32_t launch_gemm_small_fused(GemmEpilogue epi, const GemmArgs& g, hipStream_t stream) {
    if ((g.Kd % 4) || (g.lda % 4) || (g.ldw % 4) || (((uintptr_t)g.a | (uintptr_t)g.w | (uintptr_t)g.norm_gain) & 15))
        return fail(ATTS_ERR_SHAPE, "gemm (small product): rows and gain must be multiples of 16 bytes at 16-byte addresses");
    if (gemm_route(ATTS_DTYPE_F32, epi == EPI_QKV_ROPE ? EPI_STORE_ACT : epi, g).kernel != ATTS_KERNEL_SMALL)
        return fail(ATTS_ERR_SHAPE, "gemm (small product): %d x %d x %d is not one", g.M, g.N, g.Kd);
    if (epi == EPI_QKV_ROPE && (!small_rope_fusable(g.head_dim) || !g.rope || g.N % g.head_dim || g.n_rot_heads < 1 || g.n_rot_heads * g.head_dim > g.N))
        return fail(ATTS_ERR_SHAPE, "gemm (small product): the rotation of %d heads of %d columns does not fit", g.n_rot_heads, g.head_dim);
    if (epi == EPI_QKV_ROPE) return g.norm_gain ? launch_small_epi<float, EPI_QKV_ROPE, true>(g, stream) : launch_small_epi<float, EPI_QKV_ROPE>(g, stream);
    if (epi == EPI_SWIGLU && g.norm_gain) return launch_small_epi<float, EPI_SWIGLU, true>(g, stream);
    if (epi == EPI_LMHEAD && g.norm_gain) {
        if (!g.first || ((uintptr_t)g.first & 15) || g.tree_T < 1 || g.M % g.tree_T || !g.targets || !g.partials || !g.target_logit ||
            g.n_part != small_lmhead_partials(g.N))
            return fail(ATTS_ERR_INVALID_ARG, "gemm (small product): LM head without its rows or buffers");
        return launch_small_epi<float, EPI_LMHEAD, true>(g, stream);
    }
    return fail(ATTS_ERR_INVALID_ARG, "gemm (small product): epilogue %d is not fused", (int)epi);
}

int32_t small_lmhead_partials(int32_t N) { return (int32_t)ceil_div(N, 64); }

int32_t launch_gemm_small(int32_t dtype, GemmEpilogue epi, const GemmArgs& g, hipStream_t stream) {
    return dtype == ATTS_DTYPE_F32 ? launch_small_t<float>(epi, g, stream) : launch_small_t<bf16>(epi, g, stream);
}

}  // namespace atts
