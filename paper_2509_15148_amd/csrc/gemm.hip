// NT GEMM on MFMA for gfx950:  acc[M, N] = A[M, Kd] . W[N, Kd]^T  with fused epilogues.
//
// Every linear map of the target model (QKV, attention output, SwiGLU feed-forward, LM head)
// goes through one of the kernels below; scoring the drafts is the compute-bound part of the
// method (Sec. "Q1"), so this is where the time goes.
//
//   gemm_bf16_wide_kernel   aligned bf16 shapes (the bf16 models' projections of more rows): 8 wavefronts,
//                           384 x 256, 256 x 256 or 128 x 256 output tiles, operand slabs of 128 bytes
//                           per row DMA-ed global -> LDS in whole 128-byte lines, explicit waits.
//   gemm_streamed_kernel    (streamed.hip) SwiGLU of at most 128 rows, narrow projections of at most 64 (bf16)
//   gemm_small_kernel       (small.hip) products of few tiles, any shape and dtype
//   gemm_nt_kernel          any shape, bf16 or fp32 (v_mfma_f32_32x32x2_f32): 4 wavefronts (2 x 2),
//                           tile BM x BN, 128-byte slabs through registers with bounds checks,
//                           double-buffered, one barrier per slab; LDS chunk index XOR (row >> 1) & 7.
// All share gemm_epilogue (store / fp32 residual add / SwiGLU / LM-head partials / QKV + RoPE) and the
// workgroup-id remap that hands each XCD (id mod 8) a compact block of tiles, so that its private L2
// re-uses A and W slabs.
#include "common.h"

#include <atomic>
#include <type_traits>

namespace atts {
namespace {

constexpr int kThreads = 256;
constexpr int kRowBytes = 128;  // bytes of K per LDS row per slab

template <typename T> struct Mma;

template <> struct Mma<bf16> {
    static constexpr int kSteps = 4;  // 16-wide k-steps per 64-element slab
    typedef bf16x8 Frag;
    // lane (row = l % 32, half = l / 32) holds k = 16 step + 8 half + [0, 8)
    static __device__ __forceinline__ Frag load(const char* row_ptr, int row, int step, int half) {
        int chunk = step * 2 + half;
        return *reinterpret_cast<const Frag*>(row_ptr + ((chunk ^ ((row >> 1) & 7)) << 4));
    }
    static __device__ __forceinline__ void mma(const Frag& a, const Frag& b, f32x16& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};

template <> struct Mma<float> {
    static constexpr int kSteps = 8;  // one 16-byte chunk (4 floats) per step, two MFMAs
    typedef float2 Frag;
    // half h of the wave takes floats 2h, 2h+1 of the chunk: the k-order inside a chunk is
    // permuted identically for A and W, which leaves the dot product unchanged.
    static __device__ __forceinline__ Frag load(const char* row_ptr, int row, int step, int half) {
        return *reinterpret_cast<const Frag*>(row_ptr + ((step ^ ((row >> 1) & 7)) << 4) + half * 8);
    }
    static __device__ __forceinline__ void mma(const Frag& a, const Frag& b, f32x16& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, c, 0, 0, 0);
    }
};

struct TileCoord {
    int tm, tn;
};

// XCD-aware, grouped tile order.
// round > 0: the launch has `round` workgroups that walk the tiles in rounds (pid = workgroup + i round); the tiles of
// one round are then `round` consecutive positions of the order, dealt to the XCDs in blocks, so that at any time the
// whole chip works inside one group of tile rows and its A rows stay in the Infinity Cache whatever the size of A
// (with the XCDs spread over the whole order instead, eight groups are live at once: 250 MB of A rows at the 32B
// workload, which the streaming W rows then push out; measured there 1993 -> 1881 ms per step, nothing at 7B).
template <int kGroupM = 8>
__device__ __forceinline__ TileCoord tile_of_block(int pid, int nt_m, int nt_n, int round = 0) {
    int n = nt_m * nt_n;
    int base = 0;
    if (round > 0) {
        base = pid / round * round;
        pid -= base;
        n = min(round, n - base);
    }
    int n8 = n & ~7;
    int lid = base + (pid < n8 ? (pid & 7) * (n8 >> 3) + (pid >> 3) : pid);
    int per_group = kGroupM * nt_n;
    int g = lid / per_group;
    int first_m = g * kGroupM;
    int gsz = min(kGroupM, nt_m - first_m);
    int in_g = lid - g * per_group;
    TileCoord t;
    t.tm = first_m + in_g % gsz;
    t.tn = in_g / gsz;
    return t;
}


// Scalars of one GEMM launch (pointers are passed as direct kernel arguments so that the compiler
// knows they are global addresses).
struct GemmDims {
    int32_t M, N, Kd;
    int64_t lda, ldw, ldc;
    int32_t n_part, nt_m, nt_n;
    int32_t round;          // workgroups of a tile-walking launch (0: one workgroup per tile)
    int64_t ldv;            // EPI_QKV_ROPE: row pitch of the transposed V
    int32_t n_rot_heads;    // EPI_QKV_ROPE: heads (128 columns each) that get rotated; later heads are V
    int32_t k_slices;       // EPI_PARTIAL_F32: the K range is split over this many workgroups per tile, slice s stores
    int64_t slice_pitch;    // its partial sums at out + s slice_pitch (floats); 1 for every other epilogue
    int32_t v0;             // EPI_LMHEAD_T: vocabulary entry of row 0
};


// Epilogue shared by both kernels.  acc[i][j][v] is element (row, col) of the tile with
//   row = wm WM + 32 i + 8 (v / 4) + 4 half + (v % 4),   col = wn WN + 32 j + l32   (WM = 32 MI, WN = 32 NI).
// Start of a tile's accumulators: zero, or (EPI_RESID_F32) the old values of the output tile, so that the residual update
// out += A W^T is the accumulation itself and the epilogue is a plain store.  The old values are then requested while the
// first slabs are still on their way, instead of at the end of the tile, where every workgroup of a one-round launch
// would wait for them at once (7B step: O and down projections 1.9 ms faster than with a load / add / store epilogue);
// no atomics, one writer per element.
template <int MI, int NI, int EPI, bool kWide = false>
__device__ __forceinline__ void start_accumulators(f32x16 (&acc)[MI][NI], int m0, int n0, int wm, int wn, int l32, int half,
                                                   const void* __restrict__ g_out, const GemmDims& g) {
    constexpr int WM = 32 * MI, WN = 32 * NI;
    if constexpr (kWide && EPI == EPI_RESID_F32) {
        // aligned kernel: whole tiles in the column direction; addresses as wave-uniform base + lane offset, rows of a
        // last, partial tile row clamped to the last existing one (only when the wave-uniform test says there are any)
        const int rows_left = g.M - (m0 + wm * WM);
        const char* const wave_base = reinterpret_cast<const char*>(g_out) + ((int64_t)(m0 + wm * WM) * g.ldc + n0 + wn * WN) * 4;
        const uint32_t lane_off = (uint32_t)((4 * half * g.ldc + l32) * 4);
        auto rows = [&](auto checked) __attribute__((always_inline)) {
            constexpr bool kChecked = decltype(checked)::value;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = 32 * i + 8 * (v >> 2) + (v & 3);
                    const char* p = wave_base + (int64_t)r * g.ldc * 4 + lane_off;
                    if (kChecked) {     // this lane's row, clamped to the last row of the output (what it starts from is never stored)
                        const int row = min(m0 + wm * WM + r + 4 * half, g.M - 1);
                        p = reinterpret_cast<const char*>(g_out) + ((int64_t)row * g.ldc + n0 + wn * WN + l32) * 4;
                    }
#pragma unroll
                    for (int j = 0; j < NI; ++j) acc[i][j][v] = *reinterpret_cast<const float*>(p + 32 * j * 4);
                }
        };
        if (rows_left >= WM) rows(std::false_type{}); else rows(std::true_type{});
        return;
    }
    const int row_base = m0 + wm * WM + 4 * half, col_base = n0 + wn * WN + l32;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][j][v] = 0.f;
                if (EPI == EPI_RESID_F32) {
                    // rows and columns past the end are clamped, not skipped (no branches: the loads go out back to
                    // back); what they start from is never stored
                    const int row = min(row_base + 32 * i + 8 * (v >> 2) + (v & 3), g.M - 1);
                    const int col = min(col_base + 32 * j, g.N - 1);
                    acc[i][j][v] = reinterpret_cast<const float*>(g_out)[(int64_t)row * g.ldc + col];
                }
            }
}

// kWide: called by the aligned kernel, whose tiles are whole in the column direction.  The plain stores and the SwiGLU
// then go without per-element checks (one wave-uniform test tells whether the tile is whole in the row direction too) and
// address each element as a wave-uniform base (scalar arithmetic) plus one 32-bit lane offset: the checked form costs
// about 25 instructions and a branch or two per element, which at 96 - 192 elements per lane and tile was a tenth of the
// gate/up tile's time with the matrix pipe idle.
template <typename T, int MI, int NI, int EPI, bool kWide = false, bool kRaggedB = false>
__device__ __forceinline__ void gemm_epilogue_impl(f32x16 (&acc)[MI][NI], int m0, int n0, int wm, int wn, int l32, int half,
                                                   int tn, void* __restrict__ g_out, const int32_t* __restrict__ g_targets,
                                                   float2* __restrict__ g_partials, float* __restrict__ g_target_logit,
                                                   const float2* __restrict__ g_rope, void* __restrict__ g_vt,
                                                   const GemmDims& g) {
    constexpr int WM = 32 * MI, WN = 32 * NI;
    const int row_base = m0 + wm * WM + 4 * half;

    constexpr bool kPlain = EPI == EPI_STORE_ACT || EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32 || EPI == EPI_PARTIAL_F32;
    if constexpr (kWide && (kPlain || EPI == EPI_SWIGLU)) {
        constexpr int kOutCols = EPI == EPI_SWIGLU ? WN / 2 : WN;      // output columns of this wave
        constexpr int kJ = EPI == EPI_SWIGLU ? NI / 2 : NI;
        constexpr int ES = (EPI == EPI_STORE_ACT || EPI == EPI_SWIGLU) ? (int)sizeof(T) : 4;
        const int rows_left = g.M - (m0 + wm * WM);                     // wave-uniform; >= WM: every row of the wave exists
        char* const wave_base = reinterpret_cast<char*>(g_out) + ((int64_t)(m0 + wm * WM) * g.ldc + n0 + wn * kOutCols) * ES;
        const uint32_t lane_off = (uint32_t)((4 * half * g.ldc + l32) * ES);
        auto value = [&](int i, int j, int v) __attribute__((always_inline)) {
            if constexpr (EPI == EPI_SWIGLU) {
                // blocks j < NI/2 hold gate, j + NI/2 the matching up columns; silu(gate) up with the hardware reciprocal
                // (1 ulp) instead of an IEEE division and its ten-instruction expansion
                const float gate = acc[i][j][v], up = acc[i][j + NI / 2][v];
                return gate * __builtin_amdgcn_rcpf(1.f + __expf(-gate)) * up;
            } else {
                return acc[i][j][v];
            }
        };
        auto rows = [&](auto checked) __attribute__((always_inline)) {
            constexpr bool kChecked = decltype(checked)::value;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = 32 * i + 8 * (v >> 2) + (v & 3);     // + 4 half: in lane_off
                    if (kChecked && r + 4 * half >= rows_left) continue;
                    char* const p = wave_base + (int64_t)r * g.ldc * ES + lane_off;
#pragma unroll
                    for (int j = 0; j < kJ; ++j) {
                        const float y = value(i, j, v);
                        if (ES == (int)sizeof(T) && ES != 4) *reinterpret_cast<T*>(p + 32 * j * ES) = from_f32<T>(y);
                        else *reinterpret_cast<float*>(p + 32 * j * ES) = y;
                    }
                }
        };
        if (rows_left >= WM) rows(std::false_type{}); else rows(std::true_type{});
    } else if constexpr (kPlain) {
        const int col_base = n0 + wn * WN + l32;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int row = row_base + 32 * i + 8 * (v >> 2) + (v & 3);
                if (row >= g.M) continue;
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    int col = col_base + 32 * j;
                    if (col >= g.N) continue;
                    int64_t idx = (int64_t)row * g.ldc + col;
                    if (EPI == EPI_STORE_ACT) reinterpret_cast<T*>(g_out)[idx] = from_f32<T>(acc[i][j][v]);
                    // (EPI_PARTIAL_F32: slice base in g_out; EPI_RESID_F32: the accumulators started from the old values)
                    if (EPI == EPI_STORE_F32 || EPI == EPI_PARTIAL_F32 || EPI == EPI_RESID_F32) reinterpret_cast<float*>(g_out)[idx] = acc[i][j][v];
                }
            }
    } else if constexpr (EPI == EPI_SWIGLU) {
        // blocks j < NI/2 hold gate, j + NI/2 the matching up columns
        const int col_base = n0 + wn * (WN / 2) + l32;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int row = row_base + 32 * i + 8 * (v >> 2) + (v & 3);
                if (row >= g.M) continue;
#pragma unroll
                for (int j = 0; j < NI / 2; ++j) {
                    int col = col_base + 32 * j;
                    if (col >= g.N) continue;
                    float gate = acc[i][j][v], up = acc[i][j + NI / 2][v];
                    // silu(gate) up with the hardware reciprocal (1 ulp) instead of an IEEE division, whose ten-instruction
                    // expansion per element made this epilogue cost about as much again as its exponentials
                    float y = gate * __builtin_amdgcn_rcpf(1.f + __expf(-gate)) * up;
                    reinterpret_cast<T*>(g_out)[(int64_t)row * g.ldc + col] = from_f32<T>(y);
                }
            }
    } else if constexpr (EPI == EPI_QKV_ROPE) {
        // The wave's 128 columns are exactly one head (head_dim 128): blocks j = 0, 1 hold dims 0..63 and blocks
        // j + 2 the partner dims 64..127 of the rotate-half pairing, in the same lane.
        static_assert(NI == 4 && sizeof(T) == 2, "QKV epilogue needs 128-column bf16 wave tiles");
        const int col0 = n0 + wn * WN;
        const int head = col0 / 128;                                  // wave-uniform
        // Addresses as a wave-uniform base plus one lane offset, and one wave-uniform test for "every row of the wave
        // exists" instead of a test per element (as in the plain stores above).
        const int wrow0 = m0 + wm * WM;                               // first row of the wave
        const int rows_left = g.M - wrow0;
        if (head < g.n_rot_heads) {
            char* const obase = reinterpret_cast<char*>(g_out) + ((int64_t)wrow0 * g.ldc + col0) * sizeof(T);
            const char* const cbase = reinterpret_cast<const char*>(g_rope + (int64_t)wrow0 * 64);
            const uint32_t o_lane = (uint32_t)((4 * half * g.ldc + l32) * sizeof(T));
            const uint32_t c_lane = (uint32_t)((4 * half * 64 + l32) * sizeof(float2));
            // The (cos, sin) pairs of eight rows are requested together and only then used: the compiler keeps every load
            // behind the stores in front of it, so one row at a time means one exposed L2 round trip per row.
            auto rows = [&](auto checked) __attribute__((always_inline)) {
                constexpr bool kChecked = decltype(checked)::value;
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int a2 = 0; a2 < 2; ++a2) {
                        float2 cs[8][2];
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const int r = 32 * i + 8 * (2 * a2 + (q >> 2)) + (q & 3);
                            // a row that exists: at most M - 1, also for a wave wholly past it (rc is negative there)
                            const int rc = kChecked ? min(r, rows_left - 1 - 4 * half) : r;
                            const float2* crow = reinterpret_cast<const float2*>(cbase + (int64_t)rc * (64 * (int)sizeof(float2)) + c_lane);
                            cs[q][0] = crow[0];
                            cs[q][1] = crow[32];
                        }
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const int v = 4 * (2 * a2 + (q >> 2)) + (q & 3);
                            const int r = 32 * i + 8 * (v >> 2) + (v & 3);
                            if (kChecked && r + 4 * half >= rows_left) continue;
                            T* orow = reinterpret_cast<T*>(obase + (int64_t)r * g.ldc * sizeof(T) + o_lane);
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                const float x1 = acc[i][j][v], x2 = acc[i][j + 2][v];
                                orow[32 * j] = from_f32<T>(x1 * cs[q][j].x - x2 * cs[q][j].y);
                                orow[32 * j + 64] = from_f32<T>(x2 * cs[q][j].x + x1 * cs[q][j].y);
                            }
                        }
                    }
            };
            if (rows_left >= WM) rows(std::false_type{}); else rows(std::true_type{});
        } else {
            // V head: lane holds 4 consecutive rows (v % 4) of one head dim -> one 8-byte store into V^T
            typedef T T4 __attribute__((ext_vector_type(4)));
            char* const vbase = reinterpret_cast<char*>(g_vt) + ((int64_t)(head - g.n_rot_heads) * 128 * g.ldv + wrow0) * sizeof(T);
            const uint32_t v_lane = (uint32_t)(((int64_t)l32 * g.ldv + 4 * half) * sizeof(T));
            auto rows = [&](auto checked) __attribute__((always_inline)) {
                constexpr bool kChecked = decltype(checked)::value;
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        const int r0 = 32 * i + 8 * a + 4 * half;     // first of the lane's 4 consecutive rows, relative to the wave
                        if (kChecked && r0 >= rows_left) continue;
#pragma unroll
                        for (int j = 0; j < NI; ++j) {
                            T4 o4;
#pragma unroll
                            for (int b = 0; b < 4; ++b) o4[b] = from_f32<T>(acc[i][j][4 * a + b]);
                            T* dst = reinterpret_cast<T*>(vbase + ((int64_t)(32 * j) * g.ldv + 32 * i + 8 * a) * sizeof(T) + v_lane);
                            if (!kChecked || r0 + 4 <= rows_left) {
                                *reinterpret_cast<T4*>(dst) = o4;
                            } else {
#pragma unroll
                                for (int b = 0; b < 4; ++b)
                                    if (r0 + b < rows_left) dst[b] = o4[b];
                            }
                        }
                    }
            };
            if (rows_left >= WM) rows(std::false_type{}); else rows(std::true_type{});
        }
    } else if constexpr (EPI == EPI_LMHEAD) {
        // One (max, sum exp) partial per row for this wave's WN columns, plus the target logit.
        const int col0 = n0 + wn * WN;            // first column of this wave's slab
        const int part = tn * 2 + wn;
        bool col_ok[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) col_ok[j] = col0 + 32 * j + l32 < g.N;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int row = row_base + 32 * i + 8 * (v >> 2) + (v & 3);
                bool row_ok = row < g.M;          // uniform over the 32 lanes that share `half`
                int tcol = row_ok ? g_targets[row] - col0 : -1;
                float mx = -INFINITY;
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    float z = acc[i][j][v];
                    if (col_ok[j]) mx = fmaxf(mx, z);
                    if (tcol == 32 * j + l32) g_target_logit[row] = z;
                }
#pragma unroll
                for (int o = 1; o < 32; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
                float sum = 0.f;
                if (mx > -INFINITY) {
#pragma unroll
                    for (int j = 0; j < NI; ++j)
                        if (col_ok[j]) sum += __expf(acc[i][j][v] - mx);
                }
#pragma unroll
                for (int o = 1; o < 32; o <<= 1) sum += __shfl_xor(sum, o);
                if (row_ok && l32 == 0) g_partials[(int64_t)row * g.n_part + part] = make_float2(mx, sum);
            }
    } else if constexpr (EPI == EPI_LMHEAD_T) {
        // Operands exchanged: the rows of this product are vocabulary entries (g.M of them), its columns the scoring rows.
        // A lane holds, for each of its NI scoring rows, the logits of the 16 MI vocabulary entries of its wave's row
        // block: maximum and sum of exponentials are taken inside the lane (no cross-lane reduction per scoring row, where
        // the other orientation needs ten), the two lane halves are merged with one exchange, and the wave's partial goes to
        // slot (tile row, wave row).  The target logit is stored by the lane that holds the target's vocabulary entry.
        const int part = (m0 / (4 * WM)) * 4 + wm;
        const int vrow0 = g.v0 + m0 + wm * WM + 4 * half;     // every vocabulary row of the tile exists (whole tiles, checked on the host)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int col = n0 + wn * WN + 32 * j + l32;              // scoring row; < g.N unless kRaggedB
            float mx = acc[0][j][0];
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int v = (i == 0 ? 1 : 0); v < 16; ++v) mx = fmaxf(mx, acc[i][j][v]);
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum += __expf(acc[i][j][v] - mx);
            // The target's vocabulary entry relative to this lane's first one: the lane holds entries 32 i + 8 a + b
            // (b < 4).  Only about one wave in twelve holds any of its 128 scoring rows' targets, so the selection of the
            // accumulator entry sits behind a branch that is mostly not taken.
            const int trel = !kRaggedB || col < g.N ? g_targets[col] - vrow0 : -1;
            if (trel >= 0 && trel < WM && (trel & 4) == 0) {
                const int ti = trel >> 5, tv = ((trel >> 3) & 3) * 4 + (trel & 3);
                float z = 0.f;
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) z = (ti == i && tv == v) ? acc[i][j][v] : z;
                g_target_logit[col] = z;
            }
            // merge with the other half of the lane pair (l, l ^ 32): same scoring row, the rows in between
            const float mx_o = __shfl_xor(mx, 32), sum_o = __shfl_xor(sum, 32);
            const float m = fmaxf(mx, mx_o);
            float tot = 0.f;
            if (m > -INFINITY) tot = sum * __expf(mx - m) + sum_o * __expf(mx_o - m);   // a half with no entry: 0 * exp(-inf) = 0
            if (half == 0 && (!kRaggedB || col < g.N)) g_partials[(int64_t)col * g.n_part + part] = make_float2(m, tot);
        }
    }
}

// EPI_LMHEAD_T with any number of scoring rows (columns; those past g.N are dropped) and one partial per row and tile: the
// wavefronts that share columns merge theirs in LDS (free by now), in wavefront order.
template <int MI, int NI>
__device__ __forceinline__ void lmhead_tile_epilogue(f32x16 (&acc)[MI][NI], int m0, int n0, int wm, int wn, int l32, int half,
                                                     char* smem, const int32_t* __restrict__ g_targets,
                                                     float2* __restrict__ g_partials, float* __restrict__ g_target_logit,
                                                     const GemmDims& g) {
    constexpr int WM = 32 * MI, WN = 32 * NI, BN = 2 * WN, kWm = 4;
    float2* red = reinterpret_cast<float2*>(smem);                    // [kWm][BN] (max, sum of exponentials)
    const int vrow0 = g.v0 + m0 + wm * WM + 4 * half;
    block_barrier();                                                  // every wave is through with the last slab
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int c = wn * WN + 32 * j + l32, col = n0 + c;
        float mx = acc[0][j][0];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int v = (i == 0 ? 1 : 0); v < 16; ++v) mx = fmaxf(mx, acc[i][j][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));                           // the other half of the lane pair: the rows in between
        float sum = 0.f;
        if (mx > -INFINITY) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum += __expf(acc[i][j][v] - mx);
        }
        sum += __shfl_xor(sum, 32);
        // the target's vocabulary entry relative to this lane's first one: the lane holds entries 32 i + 8 a + b (b < 4)
        const int trel = col < g.N ? g_targets[col] - vrow0 : -1;
        if (trel >= 0 && trel < WM && (trel & 4) == 0) {
            const int ti = trel >> 5, tv = ((trel >> 3) & 3) * 4 + (trel & 3);
            float z = 0.f;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) z = (ti == i && tv == v) ? acc[i][j][v] : z;
            g_target_logit[col] = z;
        }
        if (half == 0) red[wm * BN + c] = make_float2(mx, sum);
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < BN && n0 + c < g.N) {
        float mx = red[c].x;
#pragma unroll
        for (int w = 1; w < kWm; ++w) mx = fmaxf(mx, red[w * BN + c].x);
        float sum = 0.f;
        if (mx > -INFINITY) {
#pragma unroll
            for (int w = 0; w < kWm; ++w) sum += red[w * BN + c].y * __expf(red[w * BN + c].x - mx);
        }
        g_partials[(int64_t)(n0 + c) * g.n_part + m0 / (kWm * WM)] = make_float2(mx, sum);
    }
}

template <typename T, int MI, int NI, int EPI>
__device__ __forceinline__ void gemm_epilogue(f32x16 (&acc)[MI][NI], int m0, int n0, int wm, int wn, int l32, int half,
                                              int tn, void* __restrict__ g_out, const int32_t* __restrict__ g_targets,
                                              float2* __restrict__ g_partials, float* __restrict__ g_target_logit,
                                              const float2* __restrict__ g_rope, void* __restrict__ g_vt,
                                              const GemmDims& g) {
    gemm_epilogue_impl<T, MI, NI, EPI>(acc, m0, n0, wm, wn, l32, half, tn, g_out, g_targets, g_partials, g_target_logit, g_rope,
                                       g_vt, g);
}

template <typename T, int BM, int BN, int EPI>
__global__ __launch_bounds__(kThreads) void gemm_nt_kernel(const char* __restrict__ gA, const char* __restrict__ gW,
                                                           void* __restrict__ g_out,
                                                           const int32_t* __restrict__ g_targets,
                                                           float2* __restrict__ g_partials,
                                                           float* __restrict__ g_target_logit,
                                                           const float2* __restrict__ g_rope, void* __restrict__ g_vt,
                                                           const GemmDims g) {
    constexpr int MI = BM / 64, NI = BN / 64;   // 32x32 blocks per wave along M / N
    constexpr int WM = BM / 2, WN = BN / 2;     // wave tile
    constexpr int kElemsPerChunk = 16 / (int)sizeof(T);
    constexpr int kSlabElems = kRowBytes / (int)sizeof(T);
    constexpr int A_CHUNKS = BM * 8 / kThreads, B_CHUNKS = BN * 8 / kThreads;
    constexpr int N_OUT = (EPI == EPI_SWIGLU) ? BN / 2 : BN;   // output columns per tile

    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* sA = smem;                           // [2][BM][128 B]
    char* sB = smem + 2 * BM * kRowBytes;      // [2][BN][128 B]

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;

    const TileCoord tc = tile_of_block(blockIdx.x, g.nt_m, g.nt_n);
    const int m0 = tc.tm * BM;
    const int n0 = tc.tn * N_OUT;

    // Per-thread chunk coordinates: chunk c = tid + 256 i -> tile row (tid / 8) + 32 i, 16-byte
    // column tid % 8.  Row i of a thread differs from row 0 by a wave-uniform offset, so one base
    // pointer per operand is kept and the per-row offsets stay in scalar registers.
    const int crow = tid >> 3, ccol = tid & 7;
    const int64_t es = (int64_t)sizeof(T);
    const char* a_base = gA + ((int64_t)(m0 + crow) * g.lda + ccol * kElemsPerChunk) * es;
    const char* b_base = gW + ((int64_t)(n0 + crow) * g.ldw + ccol * kElemsPerChunk) * es;
    const int lds_off = crow * kRowBytes + ((ccol ^ ((crow >> 1) & 7)) << 4);  // + 32 i rows: swizzle term unchanged

    uint4 ra[A_CHUNKS], rb[B_CHUNKS];

    auto load_slab = [&](int k0) __attribute__((always_inline)) {
        const bool k_ok = k0 + ccol * kElemsPerChunk < g.Kd;
        const int64_t koff = (int64_t)k0 * es;
#pragma unroll
        for (int i = 0; i < A_CHUNKS; ++i) {
            const bool ok = k_ok && (m0 + crow + 32 * i < g.M);
            ra[i] = make_uint4(0, 0, 0, 0);
            if (ok) ra[i] = *reinterpret_cast<const uint4*>(a_base + koff + (int64_t)(32 * i) * g.lda * es);
        }
#pragma unroll
        for (int i = 0; i < B_CHUNKS; ++i) {
            // LDS row j = crow + 32 i of the W tile  <-  W row (n0 + crow) + row_off
            int64_t row_off;
            bool ok;
            if (EPI == EPI_SWIGLU) {
                // wave slab jw holds [gate | up] halves of WN / 2 features each
                constexpr int H = WN / 2;
                const int jw = (32 * i) / WN, jj = (32 * i) % WN;
                const int up = jj / H, feat_off = jw * H + jj % H;
                ok = n0 + crow + feat_off < g.N;
                row_off = (int64_t)up * g.N + feat_off;
            } else {
                ok = n0 + crow + 32 * i < g.N;
                row_off = 32 * i;
            }
            rb[i] = make_uint4(0, 0, 0, 0);
            if (ok && k_ok) rb[i] = *reinterpret_cast<const uint4*>(b_base + koff + row_off * g.ldw * es);
        }
    };
    auto store_slab = [&](int buf) __attribute__((always_inline)) {
        char* dA = sA + buf * BM * kRowBytes + lds_off;
        char* dB = sB + buf * BN * kRowBytes + lds_off;
#pragma unroll
        for (int i = 0; i < A_CHUNKS; ++i) *reinterpret_cast<uint4*>(dA + i * 32 * kRowBytes) = ra[i];
#pragma unroll
        for (int i = 0; i < B_CHUNKS; ++i) *reinterpret_cast<uint4*>(dB + i * 32 * kRowBytes) = rb[i];
    };

    f32x16 acc[MI][NI];
    start_accumulators<MI, NI, EPI>(acc, m0, n0, wm, wn, l32, half, g_out, g);

    const int nk = (g.Kd + kSlabElems - 1) / kSlabElems;
    load_slab(0);
    store_slab(0);
    __syncthreads();

    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load_slab((kt + 1) * kSlabElems);

        const char* pA = sA + buf * BM * kRowBytes + (wm * WM + l32) * kRowBytes;
        const char* pB = sB + buf * BN * kRowBytes + (wn * WN + l32) * kRowBytes;
#pragma unroll
        for (int s = 0; s < Mma<T>::kSteps; ++s) {
            typename Mma<T>::Frag fa[MI], fb[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[i] = Mma<T>::load(pA + i * 32 * kRowBytes, l32, s, half);
#pragma unroll
            for (int j = 0; j < NI; ++j) fb[j] = Mma<T>::load(pB + j * 32 * kRowBytes, l32, s, half);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) Mma<T>::mma(fa[i], fb[j], acc[i][j]);
        }

        if (kt + 1 < nk) store_slab(buf ^ 1);
        __syncthreads();
    }

    gemm_epilogue<T, MI, NI, EPI>(acc, m0, n0, wm, wn, l32, half, tc.tn, g_out, g_targets, g_partials, g_target_logit, g_rope, g_vt, g);
}

// ---------------------------------------------------------------------------------------------
// Wide-slab variant of the aligned kernel: 128 bytes of K per row and slab, so that every DMA instruction
// asks L2 for whole 128-byte lines (8 rows x 128 B instead of 16 rows x 64 B).  L2 -> LDS delivery, which bounds
// the 64-byte version, is ~1.4x faster that way; the price is LDS: 160 KB hold only 2.5 slabs of a 256 x 256 tile
// (a ring of five 32 KB units A0 W0 A1 W1 A2 ...: the A rows run two slabs ahead, the W rows one) or two slabs of
// a 384 x 256 tile.  A slab is four MFMA k-steps; the DMA of the following slabs is issued under the first two
// (under the first alone with two stages), one wait + barrier per slab at its end.
// ---------------------------------------------------------------------------------------------
// kRaggedB: any number of W rows (the last column tile is partly filled; its missing rows repeat existing ones and their
// columns are dropped).
template <int EPI, int kWavesM, int MI, int NI = 4 /* 32-column blocks per wave: 4 = 256-column tiles, 2 = 128-column tiles */,
          bool kRaggedB = false>
__global__ __launch_bounds__(128 * kWavesM) void gemm_bf16_wide_kernel(const char* __restrict__ gA,
                                                                       const char* __restrict__ gW,
                                                                       void* __restrict__ g_out,
                                                                       const int32_t* __restrict__ g_targets,
                                                                       float2* __restrict__ g_partials,
                                                                       float* __restrict__ g_target_logit,
                                                                       const float2* __restrict__ g_rope,
                                                                       void* __restrict__ g_vt, const GemmDims g) {
    constexpr int WN = 32 * NI, BN = 2 * WN;
    constexpr int WM = 32 * MI, BM = kWavesM * WM;
    constexpr int kWaves = 2 * kWavesM;
    constexpr int N_OUT = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
    constexpr int BKB = 128, BK = BKB / 2, CHUNKS = BKB / 16;   // four MFMA k-steps per slab
    constexpr int ROWS_PER_DMA = 1024 / BKB;                     // 8
    constexpr int DMA_A = BM / ROWS_PER_DMA / kWaves, DMA_B = BN / ROWS_PER_DMA / kWaves;
    static_assert(DMA_A % 2 == 0 && DMA_B % 2 == 0, "the swizzle parity of a DMA instruction must not depend on the wave");
    constexpr bool kDeep = BM == 256 && BN == 256;               // five-unit ring, A two slabs ahead
    constexpr int kStages = BM == 384 ? 2 : 3;                   // whole-slab stages otherwise (at most 160 KB of LDS)
    constexpr int UNIT_A = BM * BKB, UNIT_B = BN * BKB;
    static_assert(!kDeep || UNIT_A == UNIT_B, "ring units must have one size");

    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;

    const int n_tiles = g.nt_m * g.nt_n;
    const int slice = g.k_slices > 1 ? (int)blockIdx.x / n_tiles : 0;
    const int nk_all = g.Kd / BK;
    const int k_first = (int)((int64_t)slice * nk_all / g.k_slices);
    const int nk = (int)((int64_t)(slice + 1) * nk_all / g.k_slices) - k_first;   // >= 3 (checked on the host)
    // Two-stage form without a K split: a workgroup walks tiles blockIdx.x, blockIdx.x + gridDim.x, ... and requests
    // the first slab of the next tile under the last slab of the current one, so that the DMA ring never runs dry at a
    // tile boundary and the epilogue's stores overlap that request.  (The host launches one workgroup per CU then;
    // with a grid of n_tiles workgroups the loop body runs once.)
    constexpr bool kTileLoop = MI == 3;
    // Tile rows per group of the XCD-aware order.  The one-round calls of the 256-row tile do better with taller groups
    // (an XCD then touches fewer W columns, which come cold from HBM, at the price of more A rows, which the Infinity
    // Cache holds): O projection at 7B 3.79 -> 3.66 ms per step with 12 against 8, the other shapes within 0.5 %.
    constexpr int kGroup = kDeep ? 12 : 8;
    int tile = (int)blockIdx.x - slice * n_tiles;

    // LDS offsets of the operands of slab k
    auto a_slot = [&](int k) { return kDeep ? ((2 * k) % 5) * UNIT_A : (k % kStages) * (UNIT_A + UNIT_B); };
    auto b_slot = [&](int k) { return kDeep ? ((2 * k + 1) % 5) * UNIT_A : (k % kStages) * (UNIT_A + UNIT_B) + UNIT_A; };

    // ---- DMA addressing: instruction j of this wave fills LDS rows r0 = (wave DMA_x + j) 8 ... r0 + 7; lane i lands
    // at row r0 + i / 8, chunk slot i % 8 and fetches logical chunk slot ^ swz(row), swz(row) = (row >> 1) & 7.
    // r0 / 8 and j have the same parity, so two per-lane offsets per operand (even / odd j) serve every j.
    const int dq = lane / CHUNKS, dslot = lane % CHUNKS;
    uint32_t a_lane_off[2], b_lane_off[2];
    const char* a_base[DMA_A];
    const char* b_base[DMA_B];
    int b_split = -1;           // kRaggedB: this wave's instruction whose eight rows reach past the last W row, and what takes
    uint32_t b_back = 0;        // its lanes back to that row
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int sw = (4 * p + (dq >> 1)) & 7;
        a_lane_off[p] = (uint32_t)dq * (uint32_t)(g.lda * 2) + (uint32_t)((dslot ^ sw) * 16) + (uint32_t)k_first * BKB;
        b_lane_off[p] = (uint32_t)dq * (uint32_t)(g.ldw * 2) + (uint32_t)((dslot ^ sw) * 16) + (uint32_t)k_first * BKB;
    }
    // DMA sources of a tile: the row pointers of this wave's instructions
    auto aim_dma = [&](int m0, int n0) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < DMA_A; ++j) a_base[j] = gA + (int64_t)(m0 + (wave * DMA_A + j) * ROWS_PER_DMA) * g.lda * 2;
#pragma unroll
        for (int j = 0; j < DMA_B; ++j) {
            const int r0 = (wave * DMA_B + j) * ROWS_PER_DMA;
            int64_t wrow = r0;
            if (EPI == EPI_SWIGLU) {
                constexpr int H = WN / 2;                             // wave slab = [gate H | up H]
                const int jw = r0 / WN, jj = r0 % WN;
                wrow = (int64_t)(jj / H) * g.N + jw * H + jj % H;
            }
            if (kRaggedB) {
                if (j == 0) b_split = -1;
                const int last = g.N - 1 - (n0 + r0);                 // offset of the last W row from this instruction's first
                if (g.N < 8) {                                        // every instruction reads rows 0 .. N - 1
                    wrow = -n0;
                    b_back = (uint32_t)(dq - min(dq, g.N - 1)) * (uint32_t)(g.ldw * 2);
                } else if (last < 0) {                                // all past the end: any eight rows will do
                    wrow = g.N - 8 - n0;
                } else if (last < 7) {
                    b_split = j;
                    b_back = (uint32_t)(dq - min(dq, last)) * (uint32_t)(g.ldw * 2);
                }
            }
            b_base[j] = gW + (n0 + wrow) * g.ldw * 2;
        }
    };
    TileCoord tc = tile_of_block<kGroup>(tile, g.nt_m, g.nt_n, g.round);
    aim_dma(tc.tm * BM, tc.tn * N_OUT);
    auto issue_a = [&](int k) __attribute__((always_inline)) {
        char* dst = smem + a_slot(k);
#pragma unroll
        for (int j = 0; j < DMA_A; ++j)
            __builtin_amdgcn_global_load_lds(ATTS_GPTR(a_base[j] + a_lane_off[j & 1]),
                                             ATTS_LPTR(dst + (wave * DMA_A + j) * 1024), 16, 0, 0);
        a_lane_off[0] += BKB;
        a_lane_off[1] += BKB;
    };
    auto issue_b = [&](int k) __attribute__((always_inline)) {
        char* dst = smem + b_slot(k);
#pragma unroll
        for (int j = 0; j < DMA_B; ++j)
            __builtin_amdgcn_global_load_lds(ATTS_GPTR(b_base[j] + (b_lane_off[j & 1] - (kRaggedB && (j == b_split || g.N < 8) ? b_back : 0u))),
                                             ATTS_LPTR(dst + (wave * DMA_B + j) * 1024), 16, 0, 0);
        b_lane_off[0] += BKB;
        b_lane_off[1] += BKB;
    };

    // ---- fragments: rows wm WM + 32 i + l32 (A) / wn WN + 32 j + l32 (W); 32 i, WM, WN are multiples of 16, so the
    // swizzle term depends on l32 only
    const int frag_xor = (l32 >> 1) & 7;
    const int a_row_off = (wm * WM + l32) * BKB;
    const int b_row_off = (wn * WN + l32) * BKB;
    auto load_a = [&](int k, int s, bf16x8 (&fa)[MI]) __attribute__((always_inline)) {
        const char* pa = smem + a_slot(k) + a_row_off + (((2 * s + half) ^ frag_xor) << 4);
#pragma unroll
        for (int i = 0; i < MI; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(pa + i * 32 * BKB);
    };
    auto load_b1 = [&](int k, int s, int j) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(smem + b_slot(k) + b_row_off + j * 32 * BKB + (((2 * s + half) ^ frag_xor) << 4));
    };

    f32x16 acc[MI][NI];

    // One k-step, column by column: the MI MFMAs of column j, then the W fragment of column j is replaced in place
    // by the one of the next k-step (it is free as soon as those MFMAs have issued, and not needed again before the
    // other columns are through).  Only the A fragments are double-buffered.
    bf16x8 fa[2][MI], fb[NI];
    auto kstep = [&](int k, int s, auto cur_, auto reload_) __attribute__((always_inline)) {
        constexpr int cur = decltype(cur_)::value;
        constexpr bool reload = decltype(reload_)::value;   // fragments of k-step s + 1 of the same slab
        if (reload) load_a(k, s + 1, fa[cur ^ 1]);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
#pragma unroll
            for (int i = 0; i < MI; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[j], acc[i][j], 0, 0, 0);
            if (reload) fb[j] = load_b1(k, s + 1, j);
        }
    };
    // scheduling hint for one k-step with n_dma DMA issues: per column, MI MFMAs with one A read, the DMA issues and
    // the W reload placed among them
    auto kstep_hint = [&](auto reload_, auto n_dma_, auto sync_id) __attribute__((always_inline)) {
        constexpr int kId = decltype(sync_id)::value;
        constexpr bool reload = decltype(reload_)::value;
        constexpr int n_dma = decltype(n_dma_)::value;
        constexpr int per_col = (n_dma + NI - 1) / NI, a_per_col = (MI + NI - 1) / NI;
        if (MI < 3) return;   // measured: the 256-row tile does better with the compiler's own order
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, kId);                                           // MFMA
#pragma unroll
            for (int t = 0; t < a_per_col; ++t)
                if (reload && j * a_per_col + t < MI) __builtin_amdgcn_sched_group_barrier(0x100, 1, kId);  // DS read (A)
#pragma unroll
            for (int t = 0; t < per_col; ++t)
                if (j * per_col + t < n_dma) __builtin_amdgcn_sched_group_barrier(0x020, 1, kId);          // VMEM read (LDS DMA)
            __builtin_amdgcn_sched_group_barrier(0x008, MI - 1, kId);                                      // MFMA
            if (reload) __builtin_amdgcn_sched_group_barrier(0x100, 1, kId);                               // DS read (W)
        }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using CDmaA = std::integral_constant<int, DMA_A>;
    using CDmaB = std::integral_constant<int, DMA_B>;
    using CDmaAB = std::integral_constant<int, DMA_A + DMA_B>;
    // Two whole-slab stages: the stage a slab is fetched into is free for one slab's time only, so all of the next slab is
    // requested under k-step 0 (measured against A rows under k-step 0 and W rows under k-step 1: 2 % faster; all of it
    // ahead of the first MFMA: slower again)
    constexpr bool kEarly = !kDeep && kStages == 2;
    using T_ = std::true_type;
    using F_ = std::false_type;

    // ---- prologue (the accumulators' start values are requested first, so that they are on their way with the first slabs)
    start_accumulators<MI, NI, EPI, true>(acc, tc.tm * BM, tc.tn * N_OUT, wm, wn, l32, half, g_out, g);
    constexpr int kLook = kStages - 1;                 // whole-slab stages: slab k + kLook is issued during slab k
    constexpr int kSteadyWait = kDeep ? DMA_A : (kStages - 2) * (DMA_A + DMA_B);   // loads that may stay in flight
    issue_a(0);
    issue_b(0);
    if (kDeep) {
        issue_a(1);
    } else {
#pragma unroll
        for (int q = 1; q < kLook; ++q) {              // nk >= kStages (checked on the host)
            issue_a(q);
            issue_b(q);
        }
    }
    // slab k.  first / second: the DMA halves issued under k-steps 0 and 1:
    //   deep ring:         W rows of slab k + 1 (into the unit slab k - 1 freed), then A rows of slab k + 2
    //   whole-slab stages: A rows, then W rows of slab k + kLook
    // steady: the loads issued under this slab may stay in flight across its end (else everything is awaited).
    // Two-stage form, last slab of a tile (has_next false, first and second true): the DMA issued under this slab is
    // slab 0 of the next tile, whose sources aim_dma has already been pointed at; it lands in the stage slab k - 1
    // occupied and is awaited at the top of the tile loop.
    auto slab = [&](int k, auto has_next, auto first, auto second, auto steady) __attribute__((always_inline)) {
        // k-step 0
        if (first) { if (kDeep) issue_b(k + 1); else issue_a(k + kLook); }
        if (kEarly && second) issue_b(k + kLook);
        kstep(k, 0, C0{}, T_{});
        if (kEarly && first && second) kstep_hint(T_{}, CDmaAB{}, std::integral_constant<int, 0>{});
        else if (first) { if (kDeep) kstep_hint(T_{}, CDmaB{}, std::integral_constant<int, 0>{}); else kstep_hint(T_{}, CDmaA{}, std::integral_constant<int, 0>{}); }
        else kstep_hint(T_{}, C0{}, std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        // k-step 1
        if (!kEarly && second) { if (kDeep) issue_a(k + 2); else issue_b(k + kLook); }
        kstep(k, 1, C1{}, T_{});
        if (!kEarly && second) { if (kDeep) kstep_hint(T_{}, CDmaA{}, std::integral_constant<int, 1>{}); else kstep_hint(T_{}, CDmaB{}, std::integral_constant<int, 1>{}); }
        else kstep_hint(T_{}, C0{}, std::integral_constant<int, 1>{});
        __builtin_amdgcn_sched_barrier(0);
        // k-step 2
        kstep(k, 2, C0{}, T_{});
        kstep_hint(T_{}, C0{}, std::integral_constant<int, 2>{});
        __builtin_amdgcn_sched_barrier(0);
        // k-step 3, then the slab boundary: slab k + 1 has landed for every wave, every wave is done with slab k
        kstep(k, 3, C1{}, F_{});
        if (has_next) {
            if (steady) wait_vmcnt<kSteadyWait>(); else wait_vmcnt<0>();
            block_barrier();
            load_a(k + 1, 0, fa[0]);
#pragma unroll
            for (int j = 0; j < NI; ++j) fb[j] = load_b1(k + 1, 0, j);
        }
    };
    struct Yes { constexpr operator bool() const { return true; } };
    struct No { constexpr operator bool() const { return false; } };
    void* out = g_out;
    if (EPI == EPI_PARTIAL_F32) out = reinterpret_cast<float*>(g_out) + (int64_t)slice * g.slice_pitch;

    // kb: slabs this workgroup has walked in earlier tiles (the ring positions go on across tiles)
    for (int kb = 0;; kb += nk) {
        const int m0 = tc.tm * BM, n0 = tc.tn * N_OUT, tn = tc.tn;
        // slab 0 of this tile has landed for every wave (and every wave is through with the tile before)
        if (kb == 0) wait_vmcnt<kSteadyWait>(); else wait_vmcnt<0>();
        block_barrier();
        load_a(kb, 0, fa[0]);
#pragma unroll
        for (int j = 0; j < NI; ++j) fb[j] = load_b1(kb, 0, j);
        bool more = false;
        int k = 0;
        if (kDeep) {
            for (; k + 2 < nk; ++k) slab(k, Yes{}, Yes{}, Yes{}, Yes{});
            slab(k, Yes{}, Yes{}, No{}, No{});    // k = nk - 2: only the W rows of the last slab are left to issue
            slab(k + 1, No{}, No{}, No{}, No{});
        } else {
            for (; k + kLook < nk; ++k) slab(kb + k, Yes{}, Yes{}, Yes{}, Yes{});
            for (; k + 1 < nk; ++k) slab(kb + k, Yes{}, No{}, No{}, No{});
            if (kTileLoop) {
                // The last slab always carries a slab's worth of DMA, so that there is one code path: slab 0 of the next
                // tile, or (no tile left) slab 0 of this tile once more, into the free stage, awaited before leaving.
                tile += (int)gridDim.x;
                more = g.k_slices == 1 && tile < n_tiles;
                if (more) tc = tile_of_block<kGroup>(tile, g.nt_m, g.nt_n, g.round);
                aim_dma(tc.tm * BM, tc.tn * N_OUT);
#pragma unroll
                for (int p = 0; p < 2; ++p) {          // every slab of the tile has been issued: back to its first slab
                    a_lane_off[p] -= (uint32_t)nk * BKB;
                    b_lane_off[p] -= (uint32_t)nk * BKB;
                }
                slab(kb + k, No{}, Yes{}, Yes{}, No{});
            } else {
                slab(kb + k, No{}, No{}, No{}, No{});
            }
        }

        // the lane coordinates are handed over as values of this iteration, so that the epilogue's address arithmetic is
        // not hoisted out of the tile loop (it would sit in registers all through the main loop)
        int l32_e = l32, half_e = half;
        if (kTileLoop) asm volatile("" : "+v"(l32_e), "+v"(half_e));
        if constexpr (EPI == EPI_LMHEAD_T && !kTileLoop)
            lmhead_tile_epilogue<MI, NI>(acc, m0, n0, wm, wn, l32_e, half_e, smem, g_targets, g_partials, g_target_logit, g);
        else
            gemm_epilogue_impl<bf16, MI, NI, EPI, true, kRaggedB>(acc, m0, n0, wm, wn, l32_e, half_e, tn, out, g_targets, g_partials, g_target_logit,
                                                  g_rope, g_vt, g);
        if (!(kTileLoop && more)) break;
        start_accumulators<MI, NI, EPI, true>(acc, tc.tm * BM, tc.tn * N_OUT, wm, wn, l32_e, half_e, g_out, g);
    }
    if (kTileLoop) wait_vmcnt<0>();   // no DMA may still be writing this workgroup's LDS when it is given up
}

#define ATTS_TRY_RC(expr)                 \
    do {                                  \
        int32_t rc__ = (expr);            \
        if (rc__ != ATTS_OK) return rc__; \
    } while (0)

constexpr int kWideBK = 64;           // K elements per slab of the aligned kernel
constexpr int kWavesM = 4;            // wavefronts along M (2 along N)
constexpr int kMinSlabs = 12;         // every K slice must fill the DMA ring

// Shapes the aligned bf16 kernel takes: whole tiles (or padded A rows), K a multiple of the slab.
bool fast_path_ok(int32_t dtype, int epi, const GemmArgs& g) {
    const int n_out = epi == EPI_SWIGLU ? 128 : 256;
    return dtype == ATTS_DTYPE_BF16 && (g.M % 256 == 0 || g.a_rows_padded) && g.N % n_out == 0 && g.Kd % kWideBK == 0 &&
           g.Kd >= kMinSlabs * kWideBK && g.lda * 2 * 17 < (1ll << 31) && g.ldw * 2 * 17 < (1ll << 31);
}

// ---- tile shape and K split of an aligned call ----------------------------------------------------------------------
// Time of one tile of the aligned kernel, in microseconds: a slab of 64 k elements takes 0.86 / 1.53 / 2.05 for 128 / 256 /
// 384 rows of 256 W rows and 0.58 for 128 x 128, and about 5 go into start, first slabs and epilogue.  Fitted to QKV,
// gate/up and down projections of the 7B and 70B widths at 200 to 1494 rows (K = 3584, 8192, 18944; within 10 %).  At the 32B
// widths (K = 5120, 27648) measured times are above it: QKV 83 us for 74 with 128-row tiles and 132 for 127 with 256-row
// ones, gate/up and down 5 to 15 % from 1094 rows on, and 20 to 40 % at 200 to 516 rows, where the weights' one pass from memory
// (566 MB of gate/up) shows: 172 for 127, 208 for 169.  The heights compared share that, and the choices stand: 516 rows
// of gate/up in 384 + 256 rows 374 us, two rounds of 384 rows 371; 774 in 768 + 6 492, in three rounds of 384 540.  A launch
// takes its rounds of kPlanCus tiles; so the taller tile wins only where it does not add a partly filled round:
//   7B QKV     774 rows  128-row tiles  57 us (126 tiles), 256-row  90, 384-row 126
//   7B gate/up 516 rows  128-row tiles 174 us (3 rounds),  256-row 196, 384-row 250;  1094 rows 335, 305, 290
// Plans and sizes count the whole chip's compute units, whatever device is current or whether there is one: a workspace
// sized on the host must fit the launch.  (The launch itself asks the device, for the grid that walks the tiles.)
constexpr int kPlanCus = 256;
double fast_tile_us(int rows, bool narrow, int64_t slabs) {
    const double a = narrow ? 0.58 : (rows == 128 ? 0.86 : (rows == 256 ? 1.53 : 2.05));
    return a * (double)slabs + 5.0;
}
bool tile_rows_allowed(int rows, const GemmArgs& g) {
    if (rows == 128) return g.M % 128 == 0 || g.a_rows_padded;
    if (rows == 256) return g.M > 128;                           // whole tiles or padded rows: fast_path_ok
    return g.M > 256 && (g.M % 384 == 0 || g.a_rows_padded);
}

struct TilePlan {
    int rows, slices;        // slices > 1: partial sums per K slice (EPI_PARTIAL_F32; 128-row tiles are 128 columns wide there)
    double us;
    int head_m, tail_rows;   // tail_rows != 0: rows [0, head_m) in tiles of `rows`, the rest in a second launch of this height
    int head_n;              // ... or, != 0: columns [0, head_n) of all rows, and the rest
};

// Tile height of a call without a K split.  A last round of 384-row tiles that would leave most CUs idle (32B-class O and
// down projections: 1820 tiles = 7.1 rounds of 256) is avoided by giving the last tile rows to a second launch of smaller
// tiles: 89 tile rows in 7 full rounds, then 640 rows as 100 tiles of 128 rows; 5 % faster there.  With few tile rows the cut
// goes through the columns: whole rounds of tall tiles over the first columns, lower tiles over the last (776 rows of the 7B
// gate/up projection: 444 tiles of 384 rows are two rounds; 85 columns of them and 63 of 256-row tiles, 252, are one of each).
// Gate/up, us: 7B 776 rows 222 -> 209, 1300 330 -> 298, 1500 353 -> 310, 4096 846 -> 823; 32B 900 500 -> 456, 1024 498 -> 467,
// 4096 1737 -> 1673; 70B 1024 765 -> 722, 8192 5543 -> 5419; 70B 4608 rows, O 541 -> 490 and down 1844 -> 1598.  The residual epilogue,
// whose tiles wait for their old values, wants more than the model's 3 % (7B 8192 rows: O 199 -> 205 at 0.97).  384-row tiles with
// the rest in 128-row ones are up to 5 % slower than the model has them, so they want more: 5 % against 256-row tiles, whose partly
// filled last round is faster than its model, or rows cut already, and 7 % where the 128-row tiles take two rounds (us without and
// with them, model's ratio): against 256 rows 7B gate/up 644 - 740 rows 171 - 176 and 179 - 183 (0.976), 7B down 8068 - 8804 894 - 911
// and 901 - 920 (0.956), 32B down 5764 - 6372 1314 - 1393 and 1319 - 1347 (0.954), 70B gate/up 2436 1752 and 1762 (0.953), 32B down
// 15748 3390 and 3179 (0.918); two rounds 70B gate/up 1124 788 - 855 and 787 - 869 on two boxes (0.959), 70B 4868 O 545 and 551
// (0.938), down 1912 and 1840 (0.925).
TilePlan direct_plan(int epi, const GemmArgs& g) {
    const int n_out = epi == EPI_SWIGLU ? 128 : 256;
    const int64_t nt_n = g.N / n_out, slabs = g.Kd / kWideBK;
    auto rounds_us = [&](int rows, int64_t m) {
        return (double)ceil_div(ceil_div(m, rows) * nt_n, kPlanCus) * fast_tile_us(rows, false, slabs);
    };
    TilePlan best{};
    for (int rows : {384, 256, 128}) {
        if (!tile_rows_allowed(rows, g)) continue;
        // the LM head's epilogue reduces every row across lanes: with 128-row tiles it would take a third of the time
        if (rows == 128 && g.M > 128 && epi == EPI_LMHEAD) continue;
        const double us = rounds_us(rows, g.M);
        if (best.rows == 0 || us < best.us * 0.98) best = TilePlan{rows, 1, us, 0, 0, 0};
    }
    if (epi == EPI_QKV_ROPE) return best;                        // its V^T output is not addressed by row or column alone
    const int64_t nt_m = ceil_div(g.M, 384);
    for (int drop = 1; drop <= 3 && drop < nt_m && tile_rows_allowed(384, g); ++drop)
        for (int tail : {256, 128}) {
            const int head_m = (int)(nt_m - drop) * 384;
            // readable rows: the caller's, or up to the next multiple of 768
            if (head_m + ceil_div(g.M - head_m, tail) * tail > (int64_t)(g.a_rows_padded ? align_up((size_t)g.M, 768) : (size_t)g.M)) continue;
            const double us = rounds_us(384, head_m) + rounds_us(tail, g.M - head_m) + 4.0;     // a launch more
            if (us < best.us * 0.96) best = TilePlan{384, 1, us, head_m, tail, 0};
        }
    if (epi != EPI_LMHEAD)                                       // whose partials are counted in tiles of one width
        for (int rows : {384, 256}) {
            if (!tile_rows_allowed(rows, g)) continue;
            const int64_t tall = ceil_div(g.M, rows), full = tall * nt_n / kPlanCus, head = full * kPlanCus / tall;
            if (full == 0 || head == 0 || head >= nt_n) continue;    // both launches have columns
            for (int tail : {256, 128}) {
                if (tail >= rows || !tile_rows_allowed(tail, g)) continue;
                const int64_t tail_tiles = ceil_div(g.M, tail) * (nt_n - head);
                const double us = (double)full * fast_tile_us(rows, false, slabs) +
                                  (double)ceil_div(tail_tiles, kPlanCus) * fast_tile_us(tail, false, slabs) + 4.0;
                double need = epi == EPI_SWIGLU ? 0.985 : 0.96;
                if (rows == 384 && tail == 128) need = best.rows == 256 || best.head_m != 0 ? 0.95 : (tail_tiles > kPlanCus ? 0.93 : need);
                if (us < best.us * need) best = TilePlan{rows, 1, us, 0, tail, (int)head * n_out};
            }
        }
    return best;
}

// Tile height and K slices per tile for the partial-sum epilogue: where the tiles alone leave most of the chip idle
// (few rows, a narrow output), the K range is cut so that about one workgroup per CU runs; never more than CUs (no second
// round), and every slice still walks several slabs.  Every slice's sums are written and read once more (at the 4.5 TB/s
// a copy reaches), which at a few hundred rows weighs as much as the tiles: 7B O + down with their residual passes, 298 rows:
// 128 x 128 tiles, 3 slices 96 us; 256 x 256, 9 slices 105.  70B, 774 rows: 256-row tiles, 2 slices, 443 us against 785
// for the same 128 tiles unsplit.
TilePlan partial_plan(const GemmArgs& g) {
    const int64_t slabs = g.Kd / kWideBK, fitting = (int64_t)(g.room / ((size_t)g.M * g.N * sizeof(float)));
    const TilePlan none{0, 1, 0.0, 0, 0, 0};
    TilePlan best = none;
    for (int rows : {384, 256, 128}) {
        if (!tile_rows_allowed(rows, g)) continue;
        const bool narrow = rows == 128;
        const int64_t tiles = ceil_div(g.M, rows) * (g.N / (narrow ? 128 : 256));
        int64_t s = kPlanCus / tiles;
        if (s > slabs / 6) s = slabs / 6;
        if (s > fitting) s = fitting;
        if (s < 2) continue;
        const double us = fast_tile_us(rows, narrow, ceil_div(slabs, s)) + (double)s * g.M * g.N * 8 / 4.5e6 + 4.0;
        if (best.rows == 0 || us < best.us) best = TilePlan{rows, (int)s, us, 0, 0, 0};
    }
    // without the split the norm that follows is a pass of its own, which reads 4 and writes 2 bytes an element
    const double norm_us = 4.0 + (double)g.M * g.N * 6 / 4.5e6;
    if (best.rows == 0 || (g.M > 128 && direct_plan(EPI_RESID_F32, g).us + norm_us < best.us)) return none;
    return best;
}

// Compute units of the current device (asked once per device).
int32_t device_cu_count(int* out) {
    static std::atomic<int> cached[64];
    int dev = 0;
    ATTS_HIP_TRY(hipGetDevice(&dev));
    if (dev >= 0 && dev < 64 && cached[dev].load(std::memory_order_relaxed) > 0) {
        *out = cached[dev].load(std::memory_order_relaxed);
        return ATTS_OK;
    }
    int n = 0;
    ATTS_HIP_TRY(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
    if (n < 1) return fail(ATTS_ERR_HIP, "device %d reports %d compute units", dev, n);
    if (dev >= 0 && dev < 64) cached[dev].store(n, std::memory_order_relaxed);
    *out = n;
    return ATTS_OK;
}

template <int EPI, int MI, int NI = 4, bool kRaggedB = false>
int32_t launch_wide_tile(const GemmArgs& g, hipStream_t stream) {
    constexpr int n_out = (EPI == EPI_SWIGLU) ? 32 * NI : 64 * NI;
    constexpr int BM = kWavesM * MI * 32;
    GemmDims d{};
    d.M = g.M; d.N = g.N; d.Kd = g.Kd;
    d.lda = g.lda; d.ldw = g.ldw; d.ldc = g.ldc;
    d.n_part = g.n_part;
    d.ldv = g.ldv;
    d.n_rot_heads = g.n_rot_heads;
    d.nt_m = (int)ceil_div(g.M, BM);
    d.nt_n = (int)ceil_div(g.n_cols ? g.n_cols : g.N, n_out);     // whole tiles, except the columns of the exchanged LM head
    d.k_slices = EPI == EPI_PARTIAL_F32 ? g.n_slices : 1;
    d.slice_pitch = (int64_t)g.M * g.ldc;
    d.v0 = g.v0;
    const size_t lds = 160 * 1024;
    ATTS_TRY_RC((allow_dynamic_lds<gemm_bf16_wide_kernel<EPI, kWavesM, MI, NI, kRaggedB>>(lds)));
    // 384-row tiles without a K split: one workgroup per CU (a workgroup takes a CU's whole LDS), each walking
    // every n_cu-th tile with the next tile's first slab requested under the current tile's last
    int grid = d.nt_m * d.nt_n * d.k_slices;
    d.round = 0;
    if (MI == 3 && d.k_slices == 1) {
        int n_cu = 0;
        ATTS_TRY_RC(device_cu_count(&n_cu));
        n_cu &= ~7;                                   // the tile order deals workgroup ids to the 8 XCDs in turn
        if (n_cu >= 8 && grid > n_cu) grid = n_cu;
        d.round = grid;
    }
    hipLaunchKernelGGL((gemm_bf16_wide_kernel<EPI, kWavesM, MI, NI, kRaggedB>), dim3(grid), dim3(128 * kWavesM), lds, stream,
                       reinterpret_cast<const char*>(g.a), reinterpret_cast<const char*>(g.w), g.out, g.targets, g.partials,
                       g.target_logit, g.rope, g.vt, d);
    ATTS_LAUNCH_CHECK("gemm_bf16_wide_kernel");
    return ATTS_OK;
}

template <int EPI>
int32_t launch_tile_rows(int rows, const GemmArgs& g, hipStream_t stream) {
    if (rows == 128) return launch_wide_tile<EPI, 1>(g, stream);
    return rows == 256 ? launch_wide_tile<EPI, 2>(g, stream) : launch_wide_tile<EPI, 3>(g, stream);
}

template <int EPI>
int32_t launch_fast(const GemmRoute& r, const GemmArgs& g, hipStream_t stream) {
    if constexpr (EPI == EPI_PARTIAL_F32) {
        return r.tile_rows == 128 ? launch_wide_tile<EPI, 1, 2>(g, stream) : launch_tile_rows<EPI>(r.tile_rows, g, stream);
    } else {
        if (r.tail_rows == 0) return launch_tile_rows<EPI>(r.tile_rows, g, stream);
        GemmArgs head = g, tail = g;
        if (r.head_cols) {
            // the columns from head_cols on: weights (SwiGLU: gate and up rows, N apart as before) and output further on
            head.n_cols = r.head_cols;
            ATTS_TRY_RC(launch_tile_rows<EPI>(r.tile_rows, head, stream));
            tail.n_cols = g.N - r.head_cols;
            tail.w = static_cast<const char*>(g.w) + (int64_t)r.head_cols * g.ldw * 2;
            tail.out = static_cast<char*>(g.out) + (int64_t)r.head_cols * ((EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32) ? 4 : 2);
            return launch_tile_rows<EPI>(r.tail_rows, tail, stream);
        }
        head.M = r.head_rows;
        ATTS_TRY_RC((launch_wide_tile<EPI, 3>(head, stream)));
        const int64_t r0 = head.M;
        constexpr int64_t out_bytes = (EPI == EPI_STORE_F32 || EPI == EPI_RESID_F32) ? 4 : 2;
        tail.M = g.M - head.M;
        tail.a = static_cast<const char*>(g.a) + r0 * g.lda * 2;
        if (g.out) tail.out = static_cast<char*>(g.out) + r0 * g.ldc * out_bytes;
        if (EPI == EPI_LMHEAD) {
            tail.targets = g.targets + r0;
            tail.partials = g.partials + r0 * g.n_part;
            tail.target_logit = g.target_logit + r0;
        }
        return launch_tile_rows<EPI>(r.tail_rows, tail, stream);
    }
}

template <typename T, int BM, int BN, int EPI>
int32_t launch_cfg(const GemmArgs& g, hipStream_t stream) {
    constexpr int n_out = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
    GemmDims d{};
    d.M = g.M; d.N = g.N; d.Kd = g.Kd;
    d.lda = g.lda; d.ldw = g.ldw; d.ldc = g.ldc;
    d.n_part = g.n_part;
    d.ldv = g.ldv;
    d.n_rot_heads = g.n_rot_heads;
    d.k_slices = 1;
    d.slice_pitch = 0;
    d.nt_m = (int)ceil_div(g.M, BM);
    d.nt_n = (int)ceil_div(g.N, n_out);
    const size_t lds = 2 * (size_t)(BM + BN) * kRowBytes;
    ATTS_TRY_RC((allow_dynamic_lds<gemm_nt_kernel<T, BM, BN, EPI>>(lds)));
    hipLaunchKernelGGL((gemm_nt_kernel<T, BM, BN, EPI>), dim3(d.nt_m * d.nt_n), dim3(kThreads), lds, stream, reinterpret_cast<const char*>(g.a),
                       reinterpret_cast<const char*>(g.w), g.out, g.targets, g.partials, g.target_logit, g.rope, g.vt, d);
    ATTS_LAUNCH_CHECK("gemm_nt_kernel");
    return ATTS_OK;
}

// Tile choice of the general kernel: 256 x 256 when the problem fills the chip with such tiles, else 128 x 128.
bool use_big_tile(int32_t M, int32_t N) {
    return ceil_div(M, 256) * ceil_div(N, 256) >= 192;
}

// Products of few tiles go to the kernel with 32 x 32 tiles and K split over a workgroup's wavefronts (small.hip).  Its time
// grows with its tiles, the general kernel's with its rounds of 128 x 128 tiles, of which a compute unit takes two at a
// time in 1.64 times the time of one (fp32).  The most small tiles it is taken for, and times around them in us:
//   fp32, one round    2048 up to K = 256, else 1920:  1024 x 2048 x 128  14.2 (16.7 general); 1000 x 1900 x 2048  165 (168);
//                      2000 x 1000 (2016 tiles) x 2048  181 (169)
//   fp32, two rounds   twice that up to K = 256, 1.7 times up to 512, else 1.5:  260 x 11000 (3096 tiles)  71 (75) at K = 512,
//                      284 (273) at 2048; 129 x 16600 (2595 tiles) x 8192  964 (1090); 300 x 12000 (3750 tiles) x 2048  331 (279)
//   fp32, 32 x 64 tiles (SwiGLU, LM head), which read a third fewer operands a product: 2048 a round; above K = 4096 1.7 times that in
//                      two:  LM head 2000 x 1000 x 2048  147 (187); 300 x 12000 x 2048  273 (298), x 8192  1170 (1121);
//                      260 x 11000 x 8192  1010 (1104)
//   bf16               768 a round, as its matrix instructions take a sixteenth of the time so that the unshared operand reads
//                      count:  1000 x 768 x 2048  25 (33); 17 x 49000 (1532 tiles) x 2048  44 (75); 33 x 24000 (1500 tiles of
//                      one round): general.  Above K = 4096 the weights come from memory once either way and the general kernel's
//                      second round only counts as it fills: 17 x 33000 (1032 tiles) x 8192  201 (165), 17 x 49000  253 (280)
bool use_small_tile(int32_t dtype, int epi, int32_t M, int32_t N, int32_t Kd) {
    const int64_t general = ceil_div(M, 128) * ceil_div(N, 128), rounds = ceil_div(general, kPlanCus), tiles = ceil_div(M, 32) * ceil_div(N, 32);
    if (tiles >= (1 << 24)) return false;                        // 2^32 threads a launch
    if (dtype == ATTS_DTYPE_F32) {
        const bool wide = epi == EPI_SWIGLU || epi == EPI_LMHEAD;
        const double pair = wide ? (Kd <= 4096 ? 2.0 : 1.7) : (Kd <= 256 ? 2.0 : (Kd <= 512 ? 1.7 : 1.5));
        return (double)tiles <= (wide || Kd <= 256 ? 2048 : 1920) * ((double)(rounds / 2) * pair + (double)(rounds % 2));
    }
    return tiles <= (Kd <= 4096 || general <= 256 ? rounds * 768 : 768 + 7 * (general - 256));
}

template <typename T, int EPI>
int32_t launch_epi(const GemmRoute& r, const GemmArgs& g, hipStream_t stream) {
    switch (r.kernel) {
        case ATTS_KERNEL_ALIGNED:
            if constexpr (sizeof(T) == 2) return launch_fast<EPI>(r, g, stream);
            break;
        case ATTS_KERNEL_SMALL: return launch_gemm_small(sizeof(T) == 2 ? ATTS_DTYPE_BF16 : ATTS_DTYPE_F32, (GemmEpilogue)EPI, g, stream);
        case ATTS_KERNEL_GENERAL_256:
            if constexpr (EPI != EPI_PARTIAL_F32) return launch_cfg<T, 256, 256, EPI>(g, stream);
            break;
        case ATTS_KERNEL_GENERAL_128:
            if constexpr (EPI != EPI_PARTIAL_F32) return launch_cfg<T, 128, 128, EPI>(g, stream);
            break;
    }
    return fail(ATTS_ERR_SHAPE, "gemm: no kernel for epilogue %d of this shape", EPI);
}

template <typename T>
int32_t launch_t(const GemmRoute& r, GemmEpilogue epi, const GemmArgs& g, hipStream_t stream) {
    switch (epi) {
        case EPI_STORE_ACT: return launch_epi<T, EPI_STORE_ACT>(r, g, stream);
        case EPI_STORE_F32: return launch_epi<T, EPI_STORE_F32>(r, g, stream);
        case EPI_RESID_F32: return launch_epi<T, EPI_RESID_F32>(r, g, stream);
        case EPI_SWIGLU: return launch_epi<T, EPI_SWIGLU>(r, g, stream);
        case EPI_LMHEAD: return launch_epi<T, EPI_LMHEAD>(r, g, stream);
        case EPI_PARTIAL_F32: return launch_epi<T, EPI_PARTIAL_F32>(r, g, stream);
        case EPI_QKV_ROPE: break;   // fast path only, dispatched by launch_gemm
        case EPI_LMHEAD_T: break;   // taken by launch_gemm itself, never asked for
    }
    return fail(ATTS_ERR_INVALID_ARG, "unknown GEMM epilogue %d", (int)epi);
}

// log of the sum of exponentials of a row's logits from its n_part (maximum, sum) partials; one wavefront.
template <int kHeld>
__device__ __forceinline__ float row_logsumexp(const float2* __restrict__ p, int n_part, int lane) {
    // Two passes over the row's partials, the sum against the row's final maximum and in the order of the columns.  The first
    // 64 kHeld are requested at once and held in registers in between, the rest eight at a time (one load at a time was a
    // chain of fifty load latencies: 4096 rows of 1584 partials 31.4 -> 12.1 us, 385 rows 11.8 -> 5.2; one pass with a running
    // maximum per lane 11.3 and 5.3, for other roundings of the sum).
    const float2 none = make_float2(-INFINITY, 0.f);
    float2 held[kHeld];
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) held[u] = lane + 64 * u < n_part ? p[lane + 64 * u] : none;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) mx = fmaxf(mx, held[u].x);
    for (int i0 = lane + 64 * kHeld; i0 < n_part; i0 += 64 * 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = i0 + 64 * u < n_part ? p[i0 + 64 * u].x : -INFINITY;
#pragma unroll
        for (int u = 0; u < 8; ++u) mx = fmaxf(mx, x[u]);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const float with = sum + held[u].y * __expf(held[u].x - mx);
        sum = held[u].y > 0.f ? with : sum;                          // selected, not branched over
    }
    for (int i0 = lane + 64 * kHeld; i0 < n_part; i0 += 64 * 8) {
        float2 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = i0 + 64 * u < n_part ? p[i0 + 64 * u] : none;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (q[u].y > 0.f) sum += q[u].y * __expf(q[u].x - mx);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) sum += __shfl_xor(sum, o);
    return mx + __logf(sum);
}

template <int kHeld>
__global__ void lmhead_combine_kernel(const float2* __restrict__ partials, const float* __restrict__ target_logit, int B, int n_part,
                                      const uint8_t* __restrict__ valid, float* __restrict__ lp) {
    // one wavefront per row
    const int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= B) return;
    if (valid && !valid[row]) {
        if (lane == 0) lp[row] = 0.f;
        return;
    }
    const float z = row_logsumexp<kHeld>(partials + (int64_t)row * n_part, n_part, lane);
    if (lane == 0) lp[row] = target_logit[row] - z;
}

// Log-probabilities and score of one draft of at most kScoreTokens tokens by one workgroup, a wavefront a token and round: what the
// combine and the score reduction would do in a launch each, where a draft's partials are what one compute unit reads in less than a
// launch takes (16 drafts of 8 tokens and 594 partials: a pass 832 -> 826 us; 10 of 32 and 1584, 400 KB a draft: 8 us slower, so not).  The
// sums are the score reduction's.
constexpr int kScoreTokens = 32, kScorePartials = 10000;
template <int kHeld>
__global__ __launch_bounds__(1024) void lmhead_score_kernel(const float2* __restrict__ partials, const float* __restrict__ target_logit, int Tn, int n_part,
                                                            const int32_t* __restrict__ draft_lens, int mode, float* __restrict__ token_logprobs,
                                                            float* __restrict__ scores) {
    __shared__ float lp[kScoreTokens];
    const int k = blockIdx.x, lane = threadIdx.x & 63;
    const int len = draft_lens ? min(max(draft_lens[k], 0), Tn) : Tn;
    for (int t = threadIdx.x >> 6; t < Tn; t += 16) {
        const int64_t row = (int64_t)k * Tn + t;
        float v = 0.f;
        if (t < len) v = target_logit[row] - row_logsumexp<kHeld>(partials + row * n_part, n_part, lane);
        if (lane == 0) {
            lp[t] = v;
            if (token_logprobs) token_logprobs[row] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    float s = lane < Tn ? lp[lane] : 0.f;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) scores[k] = mode == ATTS_SCORE_MEAN_NLL ? -s / (float)max(len, 1) : -s;
}

}  // namespace

// The LM head with the operands exchanged: vocabulary entries are the rows of the tiles, scoring rows (any number, read in
// place without padding) their columns; the epilogue reduces inside the lanes.
//   more than 128 scoring rows: 384 x 256 tiles, vocabulary a multiple of 384.  No row of padding is computed in the
//       long direction (4096 scoring rows are 10.67 tiles of 384 in the other orientation) and the tile count drops (7B: 6336
//       instead of 6534, 25 rounds instead of 26).  Rows that the caller has not padded (385 of 152,064 x 3584): 447 us
//       against 825 with the general kernel.  Padded rows take the other orientation where the model's time for it is shorter by
//       more than it leaves out: the epilogue that reduces across lanes (the less the longer K is), and the vocabulary matrix that a
//       single row of tiles, or a second launch for the last rows, streams by alone (lmhead_exchanged_ok).  Of 504 heads of 16 models
//       (K 1024 to 16384, 129 to 3900 rows) timed both ways the rule takes none that is more than 0.3 % slower than the other way
//       round.  Short passes with the head, other orientation and exchanged (model's ratio): one row of tiles 7B 300 rows 474 and 434 us
//       (1.16), 32B 300 643 and 631 (1.15), 70B 300 698 and 815 (1.38), K 8192 with 152,064 entries 320 957 and 986 (1.15); second
//       launch 70B 600 1225 and 1173 (1.14), K 16384 520 2391 and 2298 (1.14); whole rows 7B 1090 1063 and 1027 (1.14), 32B
//       1425 and 1458 (1.14), 70B 1800 2980 and 3047 (1.10).
//       Small vocabularies leave most of the chip idle, and a tile of 384 x 256 is then the longer chain: exchanged only where its
//       1.43 (nearly no tile) to 1.69 us (256 tiles) a slab of 64 k elements and 3.5 us are less than the other kernel's time (first
//       orientation 0.95 to 1.47 and 17, general kernel 0.82 and 15 up to a tile a compute unit, 0.95 to 1.23 and 17.5 up to
//       two): 300 rows of 9216 entries d 1024 35.4 (general 37.7), 1536 47.3 (44.0), 4096 103.6 (76.6); 256 rows d 768 28.7
//       (first 36.8), 1536 45 (48), 4096 102 (88).
//   up to 128: 256 x 128 tiles, vocabulary a multiple of 256.  Bound by the vocabulary matrix streaming by once: three
//       stages of 48 KB keep 96 KB a CU in flight.  64 rows of 152,064 x 3584 217 us (5.0 TB/s; general kernel
//       484), 128 rows 226 (unpadded: 496; padded, 128 x 256 tiles the other way round: 248).  128 x 128 tiles, two
//       workgroups a CU, read the scoring rows twice as often: 229 and 256.
static bool lmhead_aligned_k(int32_t dtype, int32_t Kd, int64_t lda, int64_t ldw) {
    return dtype == ATTS_DTYPE_BF16 && Kd % kWideBK == 0 && Kd >= kMinSlabs * kWideBK && lda * 2 * 17 < (1ll << 31) && ldw * 2 * 17 < (1ll << 31);
}
// 384 x 256 tiles of g.N vocabulary entries and g.M scoring rows: whole rounds of them, and where the last round would leave
// many CUs idle, the vocabulary's last entries in a second launch of smaller tiles (one partial per row and tile there).  7B head,
// the call alone: 256 rows (396 tiles) 315 -> 293 us, 385 rows (792 tiles: three rounds and 24) 495 -> 447, 800 rows 855 ->
// 818; 70B head 200 rows 580 -> 491, 1000 rows 1650 -> 1620.
static TilePlan lmhead_exchanged_plan(const GemmArgs& g) {
    const int64_t nt_m = g.N / 384, nt_n = ceil_div(g.M, 256), slabs = g.Kd / kWideBK, full = nt_m * nt_n / kPlanCus;
    TilePlan best{384, 1, (double)ceil_div(nt_m * nt_n, kPlanCus) * fast_tile_us(384, false, slabs), 0, 0, 0};
    if (full == 0 || nt_m * nt_n % kPlanCus == 0) return best;
    const double base = best.us;
    for (int rows : {256, 128}) {
        int64_t head = full * kPlanCus / nt_n;
        if (rows == 256 && (nt_m - head) % 2) --head;               // whole tiles in the second launch
        if (head < 1) continue;
        const int64_t tail_tiles = (nt_m - head) * 384 / rows * nt_n;
        const double us = (double)ceil_div(head * nt_n, kPlanCus) * fast_tile_us(384, false, slabs) +
                          (double)ceil_div(tail_tiles, kPlanCus) * fast_tile_us(rows, false, slabs) + 4.0;
        if (us < best.us && us < 0.95 * base) best = TilePlan{384, 1, us, (int)(head * 384), rows, 0};
    }
    return best;
}
static bool lmhead_exchanged_ok(int32_t dtype, const GemmArgs& g) {
    if (g.N % 384 != 0 || g.M <= 128 || !lmhead_aligned_k(dtype, g.Kd, g.lda, g.ldw)) return false;
    const double slabs = (double)(g.Kd / kWideBK);
    const int64_t tiles = (int64_t)g.N / 384 * ceil_div(g.M, 256);
    const double light_us = (1.43 + 0.001 * (double)tiles) * slabs + 3.5;     // tiles of a partly filled round
    if (fast_path_ok(dtype, EPI_LMHEAD, g)) {
        const TilePlan first = direct_plan(EPI_LMHEAD, g);
        const double other = (double)(ceil_div(g.M, 256) * (g.N / 256));
        if (tiles <= 256 && first.rows == 256 && other <= 256) return light_us <= (0.95 + 8e-6 * other * other) * slabs + 17.0;
        const double alone = first.tail_rows != 0 ? 1.14 : (g.M <= first.rows ? 1.05 : 1.0);
        return lmhead_exchanged_plan(g).us <= (0.98 + 12.0 / slabs) * alone * first.us;
    }
    if (use_small_tile(dtype, EPI_LMHEAD, g.M, g.N, g.Kd)) return false;
    const int64_t general = ceil_div(g.M, 128) * ceil_div(g.N, 128);
    if (use_big_tile(g.M, g.N) || general > 512) return true;
    return light_us <= (general <= 256 ? 0.82 * slabs + 15.0 : (0.95 + 0.28 * (double)(general - 256) / 256) * slabs + 17.5);
}
static bool lmhead_few_ok(int32_t dtype, const GemmArgs& g) {
    return g.N % 256 == 0 && g.M <= 128 && lmhead_aligned_k(dtype, g.Kd, g.lda, g.ldw);
}

GemmRoute gemm_route(int32_t dtype, GemmEpilogue epi, const GemmArgs& g) {
    GemmRoute r{ATTS_KERNEL_GENERAL_128, 0, 1, 0, 0, 0, 0};
    if (epi == EPI_LMHEAD && lmhead_few_ok(dtype, g)) {
        r.kernel = ATTS_KERNEL_EXCHANGED; r.tile_rows = 256; r.n_part = g.N / 256;
        return r;
    }
    if (epi == EPI_LMHEAD && lmhead_exchanged_ok(dtype, g)) {
        const TilePlan plan = lmhead_exchanged_plan(g);
        r.kernel = ATTS_KERNEL_EXCHANGED; r.tile_rows = 384; r.n_part = g.N / 384 * 4;
        if (plan.tail_rows) {
            r.head_rows = plan.head_m; r.tail_rows = plan.tail_rows;
            r.n_part = r.head_rows / 384 * 4 + (g.N - r.head_rows) / r.tail_rows;
        }
        return r;
    }
    // A decoding step or a batch of short drafts streams the weights once: the kernel built for that takes the SwiGLU and the narrow
    // projections (partial-sum epilogue) of few rows whose tiles fill the chip.  At most 16 rows of other narrow outputs go to the kernel
    // that cuts K over single wavefronts; wide outputs (logits) give the aligned kernel enough tiles and it streams them as fast,
    // so they only go there when it cannot serve the shape.
    const bool fast = fast_path_ok(dtype, epi, g);
    if (gemm_streamed_ok(dtype, epi, g)) {
        r.kernel = ATTS_KERNEL_STREAMED;
        if (epi == EPI_PARTIAL_F32) r.slices = streamed_partial_slices(dtype, g);
        return r;
    }
    if (gemm_skinny_ok(dtype, epi, g) && (epi == EPI_PARTIAL_F32 || !fast)) {
        r.kernel = ATTS_KERNEL_FEW_ROWS;
        if (epi == EPI_PARTIAL_F32) r.slices = skinny_partial_slices(g);
        return r;
    }
    if (fast) {
        const TilePlan plan = epi == EPI_PARTIAL_F32 ? partial_plan(g) : direct_plan(epi, g);
        r.kernel = ATTS_KERNEL_ALIGNED; r.tile_rows = plan.rows; r.slices = plan.slices;
        r.head_rows = plan.head_m; r.tail_rows = plan.tail_rows; r.head_cols = plan.head_n;
        r.n_part = g.N / 256 * 2;
        return r;
    }
    const int32_t n_cols = epi == EPI_SWIGLU ? 2 * g.N : g.N;
    if (use_small_tile(dtype, epi, g.M, n_cols, g.Kd)) {
        r.kernel = ATTS_KERNEL_SMALL; r.n_part = small_lmhead_partials(g.N);
    } else {
        const bool big = use_big_tile(g.M, n_cols);
        r.kernel = big ? ATTS_KERNEL_GENERAL_256 : ATTS_KERNEL_GENERAL_128;
        r.n_part = (int32_t)ceil_div(g.N, big ? 256 : 128) * 2;
    }
    return r;
}

size_t partial_bytes_bound(int32_t dtype, int32_t M, int32_t N, int32_t Kd, bool a_rows_padded) {
    if (dtype != ATTS_DTYPE_BF16) return 0;
    const size_t few = skinny_partial_bound(M, N, Kd), streamed = streamed_partial_bound(M, N, Kd);
    size_t bytes = few > streamed ? few : streamed;
    GemmArgs g{};
    g.M = M; g.N = N; g.Kd = Kd; g.lda = Kd; g.ldw = Kd; g.a_rows_padded = a_rows_padded;
    const size_t max_slices = (size_t)Kd / kWideBK / 6;              // as partial_plan: and at most one round of tiles
    if (max_slices < 2 || !fast_path_ok(dtype, EPI_PARTIAL_F32, g)) return bytes;
    for (int rows : {128, 256, 384}) {
        if (rows > 128 && M <= rows - 128) continue;                 // 256-row tiles from 129 rows on, 384 from 257
        const size_t by_slices = max_slices * (size_t)M * N * sizeof(float), by_tiles = (size_t)kPlanCus * rows * (rows == 128 ? 128 : 256) * sizeof(float);
        const size_t b = by_slices < by_tiles ? by_slices : by_tiles;
        if (b > bytes) bytes = b;
    }
    return bytes;
}

int64_t lmhead_partials_bound(int32_t dtype, int32_t B, int32_t N, int32_t Kd, bool a_rows_padded) {
    const int64_t any = lmhead_max_partials(N);
    if (!lmhead_aligned_k(dtype, Kd, Kd, Kd) || N % 256 != 0) return B * any;
    if (B <= 128) return (int64_t)B * (N / 256);
    const int64_t first = a_rows_padded ? (int64_t)N / 256 * 2 : any, exchanged = N % 384 == 0 ? (int64_t)N / 384 * 4 : 0;
    return B * (first > exchanged ? first : exchanged);
}
int32_t lmhead_max_partials(int32_t N) { return (int32_t)ceil_div(N, 128) * 2; }

bool qkv_rope_fusable(int32_t dtype, int32_t M, int32_t N, int32_t Kd, int32_t head_dim, bool a_rows_padded) {
    GemmArgs g{};
    g.M = M; g.N = N; g.Kd = Kd; g.lda = Kd; g.ldw = Kd; g.a_rows_padded = a_rows_padded;
    return head_dim == 128 && fast_path_ok(dtype, EPI_QKV_ROPE, g);
}

int32_t launch_gemm(int32_t dtype, GemmEpilogue epi, const GemmArgs& g, hipStream_t stream) {
    const size_t es = dtype_size(dtype);
    if (g.M <= 0 || g.N <= 0 || g.Kd <= 0) return fail(ATTS_ERR_SHAPE, "gemm: empty shape %d x %d x %d", g.M, g.N, g.Kd);
    if ((g.Kd * es) % 16 || (g.lda * es) % 16 || (g.ldw * es) % 16)
        return fail(ATTS_ERR_SHAPE, "gemm: K (%d) and leading dimensions must be multiples of 16 bytes", g.Kd);
    if (((uintptr_t)g.a | (uintptr_t)g.w) & 15) return fail(ATTS_ERR_INVALID_ARG, "gemm: operands must be 16-byte aligned");
    const GemmRoute r = gemm_route(dtype, epi, g);
    if (epi == EPI_LMHEAD && g.n_part != r.n_part) return fail(ATTS_ERR_INVALID_ARG, "gemm: wrong partial count for the LM-head epilogue");
    if (epi == EPI_PARTIAL_F32 && (r.slices < 2 || g.n_slices != r.slices))
        return fail(ATTS_ERR_INVALID_ARG, "gemm: wrong slice count for the partial-sum epilogue");
    if (r.kernel == ATTS_KERNEL_EXCHANGED) {
        if (!g.targets || !g.partials || !g.target_logit) return fail(ATTS_ERR_INVALID_ARG, "gemm: LM-head epilogue without its buffers");
        GemmArgs x = g;
        x.a = g.w; x.lda = g.ldw; x.M = g.N;
        x.w = g.a; x.ldw = g.lda; x.N = g.M;
        x.a_rows_padded = false;
        if (r.tile_rows == 256) return launch_wide_tile<EPI_LMHEAD_T, 2, 2, true>(x, stream);
        GemmArgs tail = x;
        if (r.tail_rows) x.M = r.head_rows;
        ATTS_TRY_RC((x.N % 256 ? launch_wide_tile<EPI_LMHEAD_T, 3, 4, true>(x, stream) : launch_wide_tile<EPI_LMHEAD_T, 3>(x, stream)));
        if (!r.tail_rows) return ATTS_OK;
        tail.a = static_cast<const char*>(x.a) + (int64_t)r.head_rows * x.lda * 2;
        tail.M -= r.head_rows;
        tail.v0 = r.head_rows;
        tail.partials = g.partials + r.head_rows / 384 * 4;
        return r.tail_rows == 128 ? launch_wide_tile<EPI_LMHEAD_T, 1, 4, true>(tail, stream) : launch_wide_tile<EPI_LMHEAD_T, 2, 4, true>(tail, stream);
    }
    if (epi == EPI_QKV_ROPE) {
        if (!qkv_rope_fusable(dtype, g.M, g.N, g.Kd, 128, g.a_rows_padded) || !g.rope || !g.vt || g.ldv < g.M || g.ldv % 4 ||
            g.n_rot_heads < 1 || g.n_rot_heads * 128 >= g.N)
            return fail(ATTS_ERR_SHAPE, "gemm: the fused QKV epilogue does not apply to this call");
        return launch_fast<EPI_QKV_ROPE>(r, g, stream);
    }
    if (r.kernel == ATTS_KERNEL_FEW_ROWS) return launch_gemm_skinny(epi, g, stream);
    if (r.kernel == ATTS_KERNEL_STREAMED) return launch_gemm_streamed(epi, g, stream);
    return dtype == ATTS_DTYPE_F32 ? launch_t<float>(r, epi, g, stream) : launch_t<bf16>(r, epi, g, stream);
}

bool lmhead_score_ok(int32_t T, int32_t n_part) { return T <= kScoreTokens && (int64_t)T * n_part <= kScorePartials; }
int32_t launch_lmhead_score(const float2* partials, const float* target_logit, int32_t K, int32_t T, int32_t n_part, const int32_t* draft_lens,
                            int32_t mode, float* token_logprobs, float* scores, hipStream_t stream) {
    if (!lmhead_score_ok(T, n_part)) return fail(ATTS_ERR_SHAPE, "score: drafts of %d tokens and %d partials take two launches", T, n_part);
    const dim3 grid((unsigned)K), block(1024);
    if (n_part <= 64 * 8)
        hipLaunchKernelGGL(lmhead_score_kernel<8>, grid, block, 0, stream, partials, target_logit, T, n_part, draft_lens, mode, token_logprobs, scores);
    else
        hipLaunchKernelGGL(lmhead_score_kernel<16>, grid, block, 0, stream, partials, target_logit, T, n_part, draft_lens, mode, token_logprobs, scores);
    ATTS_LAUNCH_CHECK("lmhead_score_kernel");
    return ATTS_OK;
}

int32_t launch_lmhead_combine(const float2* partials, const float* target_logit, int32_t B, int32_t n_part,
                              const uint8_t* valid, float* lp, hipStream_t stream) {
    const int rows_per_block = 4;
    const dim3 grid((unsigned)ceil_div(B, rows_per_block)), block(64 * rows_per_block);
    if (n_part <= 64 * 8)
        hipLaunchKernelGGL(lmhead_combine_kernel<8>, grid, block, 0, stream, partials, target_logit, B, n_part, valid, lp);
    else if (n_part <= 64 * 16)
        hipLaunchKernelGGL(lmhead_combine_kernel<16>, grid, block, 0, stream, partials, target_logit, B, n_part, valid, lp);
    else
        hipLaunchKernelGGL(lmhead_combine_kernel<32>, grid, block, 0, stream, partials, target_logit, B, n_part, valid, lp);
    ATTS_LAUNCH_CHECK("lmhead_combine_kernel");
    return ATTS_OK;
}

}  // namespace atts
