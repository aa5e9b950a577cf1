// SwiGLU projection of at most 128 rows (bf16):  out[M, F] = silu(A Wg^T) * (A Wu^T),  W = [gate rows (F) ; up rows (F)], and the partial
// sums of a narrow projection of at most 64 rows (EPI_PARTIAL_F32).
//
// A decoding step and a batch of short drafts multiply a few rows with a matrix that is read from memory once, so what counts is
// that every compute unit streams its share of it: the output is cut into tiles of 16 NB features, NB the smallest for which at
// most 256 tiles are left, one workgroup a CU.  (The aligned kernel's tiles of 128 features are 148 at F = 18,944: 108 CUs without work.)
// Measured, aligned kernel and this one, us: F 18,944 K 3584 4 rows 62.8 -> 49.5 (5.5 TB/s of weights: the memory is the bound), 128 rows
// 67.7 -> 59.2 (A, read by every workgroup, is 44 % of what reaches the LDS); F 27,648 K 5120 110 -> 99.6 and 121.9 -> 119.2; F 9216
// K 2560 46.4 -> 22.8 and 47.6 -> 33.6.
//
//   * Block j of a tile's 32 NB weight rows holds 16 gate rows and the up rows of the same 16 features, so gate and up of a feature
//     sit in the same accumulator register 16 lanes apart, and one row swap between two registers brings them together.  (Partial
//     sums: 32 consecutive weight rows; the K range is cut over workgroups too, every slice storing its sums in its own copy of the output.)
//   * 128-byte slabs (64 k elements a row) of the 32 MB rows of A and the 32 NB weight rows are DMA-ed global -> LDS, S stages, S - 1
//     slabs in flight; one wait and one barrier a slab.  16-byte chunks are XOR-swizzled with (row >> 1) & 7 on the global side.
//   * The wavefronts that share a block of 32 rows (2 of 8 with 65 to 128 rows, 2 of 4 with up to 64, all 4 with up to 32) divide the four
//     k-steps of a slab and add their sums through LDS at the end, in wavefront order.  Four wavefronts issue the DMA.
#include "common.h"

#include <type_traits>

namespace atts {
namespace {

constexpr int kStreamBK = 64, kStreamBKB = 128;
constexpr int kStreamStages = 6;                 // (10 where the LDS holds them: no faster)
constexpr int kStreamTiles = 256;                // at most one tile a compute unit

struct StreamedDims {
    int32_t M, F, n_slabs;                       // F: features, or (partial sums) columns
    int32_t n_tiles, slices;
    int64_t slice_pitch;                         // floats
    int64_t ld;                                  // of both operands
    int64_t ldc;
};

template <int MB, int NB, bool kPartial>
__global__ __launch_bounds__(MB == 4 ? 512 : 256) void gemm_streamed_kernel(const char* __restrict__ gA, const char* __restrict__ gW,
                                                                            void* __restrict__ g_out, const StreamedDims d) {
    constexpr int KW = MB == 4 ? 2 : 4 / MB;                      // wavefronts that share a block of 32 rows
    constexpr int DMA = MB + NB;                                  // DMA instructions (8 rows each) a wavefront issues for a slab
    constexpr int STAGE = 32 * (MB + NB) * kStreamBKB;
    constexpr int S = 160 * 1024 / STAGE < kStreamStages ? 160 * 1024 / STAGE : kStreamStages;
    static_assert(S >= 3 && (S - 2) * DMA <= 63, "slabs in flight");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int mb = wave % MB, kw = wave / MB;
    const int l32 = lane & 31, half = lane >> 5;
    constexpr int kCols = kPartial ? 32 : 16;                     // output columns of a block
    const int slice = kPartial ? (int)blockIdx.x / d.n_tiles : 0;
    const int col0 = ((int)blockIdx.x - slice * d.n_tiles) * kCols * NB;
    const int k_first = kPartial ? (int)((int64_t)slice * d.n_slabs / d.slices) : 0;
    const int n_slabs = kPartial ? (int)((int64_t)(slice + 1) * d.n_slabs / d.slices) - k_first : d.n_slabs;
    const bool feeds = wave < 4;                                  // four wavefronts issue the DMA (and wait for it)

    // instruction j of this wavefront fills LDS rows 8 q .. 8 q + 7, q = wave DMA + j: lane i lands at row 8 q + i / 8, chunk i % 8,
    // and fetches chunk (i % 8) ^ swizzle(row), which depends on q's parity
    const char* base[DMA];
#pragma unroll
    for (int j = 0; j < DMA; ++j) {
        const int row = (wave * DMA + j) * 8;
        if (row < 32 * MB) {
            base[j] = gA + (int64_t)row * d.ld * 2;
        } else {
            const int w = row - 32 * MB, i = w & 31;
            const int col = min(col0 + kCols * (w >> 5), d.F - kCols);      // blocks past the last column repeat it; they are dropped
            base[j] = gW + (int64_t)(kPartial ? col + i : col + (i & 15) + (i >= 16 ? d.F : 0)) * d.ld * 2;
        }
    }
    uint32_t lane_off[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int dq = lane >> 3, sw = (4 * ((wave * DMA + p) & 1) + (dq >> 1)) & 7;
        lane_off[p] = (uint32_t)dq * (uint32_t)(d.ld * 2) + (uint32_t)(((lane & 7) ^ sw) * 16) + (uint32_t)k_first * kStreamBKB;
    }
    auto issue = [&](int stage) __attribute__((always_inline)) {
        if (!feeds) return;
        char* dst = smem + stage * STAGE + wave * DMA * 1024;
#pragma unroll
        for (int j = 0; j < DMA; ++j)
            __builtin_amdgcn_global_load_lds(ATTS_GPTR(base[j] + lane_off[j & 1]), ATTS_LPTR(dst + j * 1024), 16, 0, 0);
        lane_off[0] += kStreamBKB;
        lane_off[1] += kStreamBKB;
    };
    f32x16 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    const int frag_xor = (l32 >> 1) & 7;
    auto compute = [&](int stage) __attribute__((always_inline)) {
        const char* const pa = smem + stage * STAGE + (mb * 32 + l32) * kStreamBKB;
        const char* const pw = smem + stage * STAGE + (MB * 32 + l32) * kStreamBKB;
#pragma unroll
        for (int t = 0; t < 4 / KW; ++t) {
            const int chunk = ((2 * (kw * (4 / KW) + t) + half) ^ frag_xor) << 4;
            const bf16x8 fa = *reinterpret_cast<const bf16x8*>(pa + chunk);
            bf16x8 fb[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(pw + j * 32 * kStreamBKB + chunk);
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb[j], acc[j], 0, 0, 0);
        }
    };
#pragma unroll
    for (int k = 0; k < S - 1; ++k) issue(k);                     // n_slabs >= S - 1 (checked on the host)
    int stage = 0, k = 0;
    for (; k + S - 1 < n_slabs; ++k) {
        wait_vmcnt<(S - 2) * DMA>();                              // slab k has landed for every wavefront, and every one is
        block_barrier();                                          // through with slab k - 1, whose stage is filled next
        issue(stage == 0 ? S - 1 : stage - 1);
        compute(stage);
        stage = stage + 1 == S ? 0 : stage + 1;
    }
    auto tail = [&](auto left) __attribute__((always_inline)) {   // slabs still in flight behind this one
        wait_vmcnt<decltype(left)::value * DMA>();
        block_barrier();
        compute(stage);
        stage = stage + 1 == S ? 0 : stage + 1;
    };
    if constexpr (S > 5) tail(std::integral_constant<int, 4>{});
    if constexpr (S > 4) tail(std::integral_constant<int, 3>{});
    if constexpr (S > 3) tail(std::integral_constant<int, 2>{});
    tail(std::integral_constant<int, 1>{});
    tail(std::integral_constant<int, 0>{});

    if constexpr (KW > 1) {
        // Sums of the wavefronts that share rows, block j by wavefront j % KW, in wavefront order.  Two wavefronts a block of rows leave
        // only the other's blocks (slot j / 2), four leave all of theirs.
        constexpr int kSlots = KW == 2 ? (NB + 1) / 2 : NB;
        static_assert(KW * MB * kSlots * 16 * 64 * 4 <= 160 * 1024, "");
        float* const red = reinterpret_cast<float*>(smem);        // [KW][MB][kSlots][16][64]
        auto slot = [&](int w, int j) { return red + (((w * MB + mb) * kSlots + (KW == 2 ? j >> 1 : j)) * 16) * 64 + lane; };
        block_barrier();                                          // every wavefront is through with the last slab
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (j % KW != kw)
#pragma unroll
                for (int v = 0; v < 16; ++v) slot(kw, j)[v * 64] = acc[j][v];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (j % KW == kw)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float sum = 0.f;
#pragma unroll
                    for (int w = 0; w < KW; ++w) sum += w == kw ? acc[j][v] : slot(w, j)[v * 64];
                    acc[j][v] = sum;
                }
    }
    if constexpr (kPartial) {
        float* const sums = reinterpret_cast<float*>(g_out) + (int64_t)slice * d.slice_pitch;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (j % KW != kw || col0 + 32 * j >= d.F) continue;   // wave-uniform
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = mb * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                if (row < d.M) sums[(int64_t)row * d.ldc + col0 + 32 * j + l32] = acc[j][v];
            }
        }
        return;
    }
    bf16* const out = reinterpret_cast<bf16*>(g_out);
    // acc[j][v]: row 8 (v / 4) + 4 half + v % 4 of the wavefront's 32, weight row l32 of block j: gate below 16, up from 16 on.  Swapping
    // the odd 16-lane rows of register v with the even ones of v + 1 gathers the gates of both in one register and the ups in the other.
    const int first = mb * 32 + 4 * half + ((lane >> 4) & 1);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if (j % KW != kw || col0 + 16 * j >= d.F) continue;      // wave-uniform
        bf16* const o = out + col0 + 16 * j + (lane & 15);
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[j][v]), __float_as_uint(acc[j][v + 1]), false, false);
            const float gate = __uint_as_float(p[0]), up = __uint_as_float(p[1]);
            const int row = first + 8 * (v >> 2) + (v & 3);
            if (row < d.M) o[(int64_t)row * d.ldc] = from_f32<bf16>(gate * __builtin_amdgcn_rcpf(1.f + __expf(-gate)) * up);   // as in the tiled kernels
        }
    }
}

template <int MB, int NB, bool kPartial>
int32_t launch_streamed(const GemmArgs& g, hipStream_t stream) {
    StreamedDims d{};
    d.M = g.M; d.F = g.N; d.n_slabs = g.Kd / kStreamBK;
    d.ld = g.lda; d.ldc = g.ldc;
    d.n_tiles = (int)ceil_div(g.N, (kPartial ? 32 : 16) * NB);
    d.slices = kPartial ? g.n_slices : 1;
    d.slice_pitch = (int64_t)g.M * g.ldc;
    const size_t lds = 160 * 1024;
    int32_t rc = allow_dynamic_lds<gemm_streamed_kernel<MB, NB, kPartial>>(lds);
    if (rc != ATTS_OK) return rc;
    hipLaunchKernelGGL((gemm_streamed_kernel<MB, NB, kPartial>), dim3((unsigned)(d.n_tiles * d.slices)), dim3(MB == 4 ? 512 : 256), lds, stream,
                       reinterpret_cast<const char*>(g.a), reinterpret_cast<const char*>(g.w), g.out, d);
    ATTS_LAUNCH_CHECK("gemm_streamed_kernel");
    return ATTS_OK;
}

template <int MB>
int32_t launch_swiglu(const GemmArgs& g, int nb, hipStream_t stream) {
    switch (nb) {
        case 3: return launch_streamed<MB, 3, false>(g, stream);
        case 4: return launch_streamed<MB, 4, false>(g, stream);
        case 5: return launch_streamed<MB, 5, false>(g, stream);
        case 6: return launch_streamed<MB, 6, false>(g, stream);
        case 7: return launch_streamed<MB, 7, false>(g, stream);
    }
    return fail(ATTS_ERR_SHAPE, "gemm (streamed): no tile of %d blocks", nb);
}
template <int MB>
int32_t launch_partial(const GemmArgs& g, int nb, hipStream_t stream) {
    return nb == 2 ? launch_streamed<MB, 2, true>(g, stream) : launch_streamed<MB, 4, true>(g, stream);
}

// Blocks of 16 features a tile: 3 to 7.  Fewer would let A outweigh the weights, and from 224 of the aligned kernel's tiles on that one
// streams as fast (F 28,672, K 8192: 163.2 and 166.3 us with 4 rows, 175.6 and 179.2 with 128).
int stream_blocks(int32_t F) { return (int)ceil_div(ceil_div(F, 16), kStreamTiles); }

// Partial sums of up to 64 rows: blocks of 32 columns a tile (0: not served) and K slices, which every slice's sums make dearer for this
// kernel and for the pass that adds them.  Tiles of 64 columns while that leaves at least three slices, else of 128 with at least four;
// more than 32 rows and a long K want the wider ones, whose A weighs less.  us with their share of the residual pass, before and now:
// 7B O 11.3 -> 10.3 (20 rows) and 12.0 -> 11.7 (64), down 32.4 -> 28.8 and 36.4 -> 34.1, QKV 16.4 -> 15.0; 16 rows, where one wavefront a
// piece of K had them: down 31.3 -> 28.4, 32B 57.6 -> 52.3; 4 rows alike (a pass 547 -> 541).  70B QKV (80 tiles of 128): 41.7 and 43.2.
// From 65 rows on 128 x 128 tiles are faster (72 rows: down 36.6 and 37.7, O 12.4 and 13.9).
int partial_blocks(int32_t M, int32_t N, int64_t slabs) {
    const int64_t narrow = ceil_div(N, 64), wide = ceil_div(N, 128);
    if (narrow <= kStreamTiles / 3 && !(M > 32 && slabs >= 128)) return 2;
    return wide <= kStreamTiles / 4 ? 4 : 0;
}
int64_t partial_slices(int nb, int32_t N, int64_t slabs) {
    const int64_t s = kStreamTiles / ceil_div(N, 32 * nb), longest = slabs / 12;
    return s < longest ? s : longest;
}

}  // namespace

// K in whole slabs, one row pitch, rows of A readable up to the end of their blocks
static bool operands_ok(const GemmArgs& g) {
    const int rows = g.M <= 32 ? 32 : (g.M <= 64 ? 64 : 128);
    return g.Kd % kStreamBK == 0 && g.Kd >= 12 * kStreamBK && g.lda == g.ldw && g.lda * 2 * 9 < (1ll << 31) && (g.a_rows_padded || g.M == rows);
}

bool gemm_streamed_ok(int32_t dtype, GemmEpilogue epi, const GemmArgs& g) {
    if (dtype != ATTS_DTYPE_BF16 || g.M < 1) return false;
    if (epi == EPI_PARTIAL_F32) return streamed_partial_slices(dtype, g) >= 2;
    return epi == EPI_SWIGLU && g.M <= 128 && g.N >= 16 && g.N % 16 == 0 && stream_blocks(g.N) >= 3 &&
           ceil_div(g.N, 128) * 8 < kStreamTiles * 7 && operands_ok(g);
}

int32_t launch_gemm_streamed(GemmEpilogue epi, const GemmArgs& g, hipStream_t stream) {
    if (epi == EPI_PARTIAL_F32) {
        const int nb = partial_blocks(g.M, g.N, g.Kd / kStreamBK);
        return g.M <= 32 ? launch_partial<1>(g, nb, stream) : launch_partial<2>(g, nb, stream);
    }
    const int nb = stream_blocks(g.N);
    if (g.M <= 32) return launch_swiglu<1>(g, nb, stream);
    return g.M <= 64 ? launch_swiglu<2>(g, nb, stream) : launch_swiglu<4>(g, nb, stream);
}

int32_t streamed_partial_slices(int32_t dtype, const GemmArgs& g) {
    if (dtype != ATTS_DTYPE_BF16 || g.M < 1 || g.M > 64 || g.N < 32 || g.N % 32 != 0 || !operands_ok(g)) return 0;
    const int64_t slabs = g.Kd / kStreamBK, fitting = (int64_t)(g.room / ((size_t)g.M * g.N * sizeof(float)));
    const int nb = partial_blocks(g.M, g.N, slabs);
    if (nb == 0) return 0;
    const int64_t s = partial_slices(nb, g.N, slabs);
    // most of the chip at work, and every slice's sums stored
    return s >= 2 && s <= fitting && s * ceil_div(g.N, 32 * nb) * 4 >= kStreamTiles * 3 ? (int32_t)s : 0;
}

size_t streamed_partial_bound(int32_t M, int32_t N, int32_t Kd) {
    int64_t s = 0;
    for (int nb : {2, 4})
        if (partial_slices(nb, N, Kd / kStreamBK) > s) s = partial_slices(nb, N, Kd / kStreamBK);
    return (size_t)s * (size_t)(M < 64 ? M : 64) * N * sizeof(float);
}

}  // namespace atts
