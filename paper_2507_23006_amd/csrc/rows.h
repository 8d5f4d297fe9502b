// Coefficient rows of packed Gaussians, between memory and LDS, for one wave.
#pragma once

#include "gs_internal.h"

namespace gs {

typedef float F4 __attribute__((ext_vector_type(4)));

// orders a wave's LDS accesses before and after it
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's 64 coefficient rows (192 bytes each) between memory and LDS.  A lane
// reading its own row touches two cache lines with each of its twelve 16-byte
// loads, 16 KB of lines per instruction and wave, which the compute unit's L1
// does not hold until the next piece is read; here twelve neighbouring lanes
// move a row's pieces.  Rows lie 13 pieces apart in LDS, so that a piece of all
// rows spreads over all banks.
constexpr int kRowF4 = 13;
constexpr int kWaveRows = 64 * kRowF4;     // float4s of LDS per wave

struct RowLanes {
    int rc[3], qc[3];      // row (of 16) and piece that the lane moves in step c of three
    __device__ explicit RowLanes(int lane) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            rc[c] = (64 * c + lane) / 12;
            qc[c] = 64 * c + lane - 12 * rc[c];
        }
    }
};

// rows of the Gaussians g (one per lane) into s
__device__ __forceinline__ void load_rows(const float* __restrict__ sh, uint32_t g, int nq,
                                          const RowLanes& rl, F4* s) {
    const F4* src = reinterpret_cast<const F4*>(sh);
    F4 piece[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const uint32_t r = __shfl(g, 16 * (i / 3) + rl.rc[i % 3]);
        piece[i] = rl.qc[i % 3] < nq ? src[(int64_t)12 * r + rl.qc[i % 3]] : F4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int i = 0; i < 12; ++i) s[(16 * (i / 3) + rl.rc[i % 3]) * kRowF4 + rl.qc[i % 3]] = piece[i];
    wave_sync();
}

// the first m rows of s to those of their Gaussians
__device__ __forceinline__ void store_rows(float* __restrict__ sh, uint32_t g, int m, const RowLanes& rl,
                                           const F4* s) {
    F4* dst = reinterpret_cast<F4*>(sh);
    wave_sync();
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const int r = 16 * (i / 3) + rl.rc[i % 3];
        const uint32_t to = __shfl(g, r);
        if (r < m) __builtin_nontemporal_store(s[r * kRowF4 + rl.qc[i % 3]], dst + (int64_t)12 * to + rl.qc[i % 3]);
    }
    wave_sync();
}

}  // namespace gs
