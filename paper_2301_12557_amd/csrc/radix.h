// radix.h -- one 8-bit digit of a stable LSD radix sort over a tile of pairs
// held in the registers of a workgroup.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fcfc {

constexpr int RS_T = 512, RS_I = 8, RS_WAVES = RS_T / 64;

struct RsShared {
    uint32_t wcnt[RS_WAVES][256];  // per wave: pairs of each digit, then those of the waves before
    uint32_t base[256];            // pairs of lower digits in the tile
    uint32_t wsum[4];
};

__device__ inline void rs_wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline uint32_t rs_wave_inclusive(uint32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t a = __shfl_up(v, o);
        v += lane >= o ? a : 0u;
    }
    return v;
}

// Position in the tile, ordered by digit, of the pairs of this thread: pair r
// of lane l of wave w is element 512 w + 64 r + l of a tile of m.  Each wave
// ranks its elements 64 at a time (the lanes of one digit find each other by
// eight ballots) against its own counters, so no barrier is needed until the
// waves' counts are summed.  s.base is left for the caller.
__device__ __attribute__((always_inline)) inline void rs_rank(RsShared& s, const uint32_t key[RS_I], int shift, int m,
                                                              uint32_t pos[RS_I]) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint32_t* cnt = s.wcnt[w];
#pragma unroll
    for (int q = 0; q < 4; q++) cnt[q * 64 + lane] = 0u;
    rs_wave_fence();
#pragma unroll
    for (int r = 0; r < RS_I; r++) {
        const bool valid = w * 64 * RS_I + r * 64 + lane < m;
        const uint32_t d = (key[r] >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const bool bit = (d >> b) & 1u;
            const uint64_t on = __ballot(bit);
            peers &= bit ? on : ~on;
        }
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
        const uint32_t have = cnt[d];
        rs_wave_fence();
        if (valid && before == 0) cnt[d] = have + (uint32_t)__popcll(peers);
        rs_wave_fence();
        pos[r] = have + before;
    }
    __syncthreads();
    uint32_t run = 0, incl = 0;
    if (t < 256) {
#pragma unroll
        for (int q = 0; q < RS_WAVES; q++) {
            const uint32_t c = s.wcnt[q][t];
            s.wcnt[q][t] = run;
            run += c;
        }
        incl = rs_wave_inclusive(run, lane);
        if (lane == 63) s.wsum[w] = incl;
    }
    __syncthreads();
    if (t < 256) {
        uint32_t b = incl - run;
        for (int q = 0; q < w; q++) b += s.wsum[q];
        s.base[t] = b;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_I; r++) {
        const uint32_t d = (key[r] >> shift) & 255u;
        pos[r] += s.base[d] + cnt[d];
    }
}

}  // namespace fcfc
