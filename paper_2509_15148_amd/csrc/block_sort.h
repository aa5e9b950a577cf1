// Sorting keys inside one workgroup: a bitonic network over 8 keys per thread (device code; shared by calib.hip and sort.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace atts {

constexpr int kPer = 8;                      // keys per thread
constexpr int kWaveKeys = 64 * kPer;

// keep the smaller (c = 0) or the larger (c = ~0) of a and b: one three-operand median
__device__ __forceinline__ uint32_t keep(uint32_t a, uint32_t b, uint32_t c) { return max(min(a, b), min(max(a, b), c)); }

__device__ __forceinline__ void cswap(uint32_t& x, uint32_t& y) {
    const uint32_t lo = min(x, y), hi = max(x, y);
    x = lo;
    y = hi;
}

// Compare-exchange of every key with the same register of lane ^ X, the lower lane keeping the smaller key.
template <int X>
__device__ __forceinline__ void lane_step(uint32_t (&k)[kPer]) {
    if constexpr (X <= 8) {
        const uint32_t c = (threadIdx.x & X) ? ~0u : 0u;
        int o[kPer];
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            if constexpr (X == 1) o[e] = __builtin_amdgcn_mov_dpp((int)k[e], 0xB1, 0xF, 0xF, true);     // lanes (1, 0, 3, 2)
            if constexpr (X == 2) o[e] = __builtin_amdgcn_mov_dpp((int)k[e], 0x4E, 0xF, 0xF, true);     // lanes (2, 3, 0, 1)
            if constexpr (X == 4) o[e] = __builtin_amdgcn_mov_dpp((int)k[e], 0x141, 0xF, 0xF, true);    // ^ 7, then ^ 3
            if constexpr (X == 8) o[e] = __builtin_amdgcn_mov_dpp((int)k[e], 0x128, 0xF, 0xF, true);    // half a row of 16 round
        }
        __builtin_amdgcn_sched_barrier(0);                         // a DPP read right behind its register's write costs two idle slots
        if constexpr (X == 4) {
#pragma unroll
            for (int e = 0; e < kPer; ++e) o[e] = __builtin_amdgcn_mov_dpp(o[e], 0x1B, 0xF, 0xF, true);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < kPer; ++e) k[e] = keep(k[e], (uint32_t)o[e], c);
        __builtin_amdgcn_sched_barrier(0);
    } else {
        // two registers at a time: the swap puts the lower partners of both into one register and the upper ones into the
        // other, and a second swap takes them back
#pragma unroll
        for (int e = 0; e < kPer; e += 2) {
            auto swap = [](uint32_t x, uint32_t y) {
                if constexpr (X == 16) return __builtin_amdgcn_permlane16_swap(x, y, false, false);
                else return __builtin_amdgcn_permlane32_swap(x, y, false, false);
            };
            const auto p = swap(k[e], k[e + 1]);
            const auto q = swap(min(p[0], p[1]), max(p[0], p[1]));
            k[e] = q[0];
            k[e + 1] = q[1];
        }
    }
}

// The last steps of a stage: keys S lanes apart down to neighbouring registers.
template <int S>
__device__ __forceinline__ void merge_lanes(uint32_t (&k)[kPer]) {
    if constexpr (S >= 1) {
        lane_step<S>(k);
        merge_lanes<S / 2>(k);
    } else {
#pragma unroll
        for (int stride = kPer / 2; stride > 0; stride >>= 1)
#pragma unroll
            for (int e = 0; e < kPer; ++e)
                if ((e & stride) == 0) cswap(k[e], k[e + stride]);
    }
}

// Keys 8 t .. 8 t + 7 of thread t become the keys of those places in ascending order of the first `size` ones (a power of two
// from 512 on, at most 8 THREADS; block-uniform).  Everything up to 512 keys happens in the registers of a wavefront
// (neighbours by DPP, rows and halves by lane swaps); partners in other wavefronts exchange through LDS, one barrier each
// (two buffers in turn).  A stage's descending groups work on complemented keys, so that the lower place always keeps the smaller.
// What bounds it is the chain of steps: 512 keys about 620 vector instructions.  A launch that sorts 2048 keys takes 5.2 us and
// one of 8192 about 12 (16 wavefronts share four SIMDs), against 12.2 and 24 with pairwise merges in LDS, whose binary searches
// are chains of LDS reads.  buf: 2 x 8 THREADS words if THREADS > 64.
template <int THREADS>
__device__ __forceinline__ void sort_in_block(uint32_t (&k)[kPer], int size, uint32_t* buf) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t flip = 0;
    auto face = [&](bool descending) __attribute__((always_inline)) {
        const uint32_t now = descending ? ~0u : 0u, change = now ^ flip;
        flip = now;
#pragma unroll
        for (int e = 0; e < kPer; ++e) k[e] ^= change;
    };
    const bool active = THREADS == 64 || wave * kWaveKeys < size;  // wavefronts past the last place only keep the barriers
    if (active) {
        face(lane & 1);
#pragma unroll
        for (int round = 0; round < kPer; ++round) {               // eight keys by odd-even transposition
#pragma unroll
            for (int e = round & 1; e + 1 < kPer; e += 2) cswap(k[e], k[e + 1]);
        }
        face(lane & 2);
        merge_lanes<1>(k);
        face(lane & 4);
        merge_lanes<2>(k);
        face(lane & 8);
        merge_lanes<4>(k);
        face(lane & 16);
        merge_lanes<8>(k);
        face(lane & 32);
        merge_lanes<16>(k);
        face(size > kWaveKeys && (wave & 1));
        merge_lanes<32>(k);
    }
    if constexpr (THREADS > 64) {
        int cur = 0;
        for (int waves = 2; waves * kWaveKeys <= size; waves *= 2) {
            face(waves * kWaveKeys < size && (wave & waves));
            for (int s = waves / 2; s > 0; s >>= 1) {
                uint4* own = reinterpret_cast<uint4*>(buf + cur * (kPer * THREADS));       // two planes of 16 bytes per thread
                cur ^= 1;
                if (active) {
                    own[tid] = make_uint4(k[0], k[1], k[2], k[3]);
                    own[THREADS + tid] = make_uint4(k[4], k[5], k[6], k[7]);
                }
                __syncthreads();
                if (!active) continue;
                const uint4 x = own[tid ^ (64 * s)], y = own[THREADS + (tid ^ (64 * s))];
                const uint32_t c = (wave & s) ? ~0u : 0u;
                k[0] = keep(k[0], x.x, c);
                k[1] = keep(k[1], x.y, c);
                k[2] = keep(k[2], x.z, c);
                k[3] = keep(k[3], x.w, c);
                k[4] = keep(k[4], y.x, c);
                k[5] = keep(k[5], y.y, c);
                k[6] = keep(k[6], y.z, c);
                k[7] = keep(k[7], y.w, c);
            }
            if (active) merge_lanes<32>(k);
        }
    }
}

}  // namespace atts
