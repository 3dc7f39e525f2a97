// What the two packers (vgc_pack.hip, vgc_compact.hip) have in common on the device.
#ifndef VGC_SCAN_H
#define VGC_SCAN_H
#include "vgc_internal.h"

namespace vgc {

// Parameter sets of so few tiles and groups have packers of their own, whose workgroups each read all tile records.
constexpr uint32_t kSmallTiles = 2048, kSmallGroups = 512;

// Inclusive scan over a workgroup of kWaves waves; returns the inclusive value, total through `total`.
template <int kWaves>
__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t* sh /*[kWaves]*/, uint32_t& total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t incl = wave_inclusive_sum(x);
    __syncthreads();                       // protects sh against the previous use
    if (lane == 63) sh[wave] = incl;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = sh[w];
        if ((uint32_t)w < wave) base += c;
        tot += c;
    }
    total = tot;
    return incl + base;
}

// Words of a tile that are encoded in a group of exponent E: entries with rel <= 8 - shift.
__device__ __forceinline__ uint32_t kept_words(uint4 lo, uint32_t w4, uint32_t E, uint32_t& shift) {
    shift = E - (w4 >> 16);
    uint32_t kept = 0;
    if (E != 0 && shift <= 8) {
        const uint32_t h[9] = {lo.x & 0xFFFFu, lo.x >> 16, lo.y & 0xFFFFu, lo.y >> 16, lo.z & 0xFFFFu, lo.z >> 16, lo.w & 0xFFFFu,
                               lo.w >> 16, w4 & 0xFFFFu};
        const uint32_t lim = 8 - shift;
#pragma unroll
        for (int q = 0; q < 9; ++q) kept += ((uint32_t)q <= lim) ? h[q] : 0u;
    }
    return kept;
}

// An empty message: the plan belongs to another group list.
__device__ __forceinline__ void empty_message(uint32_t threads, uint32_t n_groups, vgc_group_hdr* __restrict__ hdrs_out, vgc_pack_status* __restrict__ status) {
    for (uint32_t k = threadIdx.x; k < n_groups; k += threads) {
        vgc_group_hdr h;
        h.exp_field = 0; h.count = 0; h.word_offset = 0;
        hdrs_out[k] = h;
    }
    if (threadIdx.x == 0) {
        vgc_pack_status st;
        st.total_words = 0; st.overflow = 0; st.plan_mismatch = 1;
        *status = st;
    }
}

}  // namespace vgc
#endif
