// Compressed index encoding of a message (Section 4.2 ends by noting that the index bits can be reduced further by
// compressing the indexes; the paper gives no algorithm, the format is this library's own).  Elements are in
// ascending index order, so each is stored as its distance from the previous element of its tile:
//     gap  = position in tile - position of the tile's previous element - 1   (the first element counts from -1)
//     code = sign << 3 | d                                                   (the 4-bit value of Section 4.2)
//     gap < 8: one byte gap << 4 | code;  else two bytes 0x80 | (gap & 7) << 4 | code, gap >> 3   (gap <= 2047)
// plus a directory: bytes per tile (uint16) and the byte offset of every run of 64 tiles (uint64).  The chain of
// distances restarts in every tile, so one wave encodes or decodes a tile without looking at any other.
//
//   k_compact_count   one wave per one or two tiles: bytes the tile's kept entries take -> tile_bytes
//   (k_run_sums and k_header_scan of vgc_pack.hip add them up: run offsets, group byte offsets, total)
//   k_compact_emit    one wave per one or two tiles: the bytes
// The encoder waits on memory, for a few entries per tile: what counts is how many loads depend on one another.  Entries asked
// for before it is known how many there are, a tile's place found from two tables instead of four, and the runs scanned where
// the segments are: 3 % of 138 M elements 80.5 -> 56 us, 30 % 180 -> 139.  Sums over a wave
// without LDS and two tiles a wave since then: a stream of 4.5 MB of 138 M elements 54 -> 45 us, of 42 MB 125 -> 111.
//   k_compact_count_small, k_compact_emit_small   all of it in two launches, for parameter sets of few tiles
//   k_unpack_compact  one wave per few tiles of a run, tile in LDS, messages in order (the batched decoder for this format)
#include <algorithm>

#include "vgc_scan.h"

namespace vgc {

__device__ __forceinline__ uint64_t lanes_below(uint32_t lane) { return (1ull << lane) - 1ull; }

// What is read of tile t (a wave) before it is known whether it has anything: its record and the first two rounds of 64 entries.  A
// tile owns kTile staging slots; what lies behind its count is ignored.
struct TileAhead { uint32_t record, entries[2]; };
__device__ __forceinline__ TileAhead tile_ahead(const TileHdr* __restrict__ hdrs, const uint16_t* __restrict__ staging, uint64_t t, uint32_t lane) {
    const uint16_t* st = staging + t * kTile;
    TileAhead a;
    a.entries[0] = st[lane];
    a.entries[1] = st[64 + lane];
    a.record = (lane < 8) ? hdrs[t].w[lane] : 0u;
    return a;
}

// The staged entries of tile t (a wave) that the group keeps, 64 at a time, as (first byte, second byte, two bytes?, byte
// offset inside the tile).  Calls `sink(keep, b0, b1, is_long, offset)` once per round in every lane; returns the
// tile's bytes.  `found(w)` is given the record and says whether the tile has some (it may complete w[7]).  Two rounds are
// requested while the two before are encoded.
template <class Found, class Sink>
__device__ __forceinline__ uint32_t encode_tile(const TileAhead& a, const uint16_t* __restrict__ staging,
                                                uint64_t t, uint32_t lane, Found found, Sink sink) {
    const uint16_t* st = staging + t * kTile;
    uint32_t ahead[2] = {a.entries[0], a.entries[1]};
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = (uint32_t)__builtin_amdgcn_readlane((int)a.record, i);
    if (!found(w)) return 0;
    const uint32_t cnt = min((w[0] & 0xFFFFu) + (w[0] >> 16) + (w[1] & 0xFFFFu) + (w[1] >> 16) + (w[2] & 0xFFFFu) +
                             (w[2] >> 16) + (w[3] & 0xFFFFu) + (w[3] >> 16) + (w[4] & 0xFFFFu), kTile);
    const uint32_t shift = w[7] >> 16, lim = 8 - shift;        // kept != 0 implies shift <= 8
    int32_t prev = -1;                                         // position of the last kept entry so far (uniform)
    uint32_t bytes = 0;
    for (uint32_t j0 = 0; j0 < cnt; j0 += 128) {
        const uint32_t now[2] = {ahead[0], ahead[1]};
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q)
            if (j0 + 128 + 64 * q < cnt) ahead[q] = st[j0 + 128 + 64 * q + lane];           // (uniform; below kTile, as cnt is)
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {
            if (j0 + 64 * q >= cnt) break;
            const uint32_t e = now[q];
            const uint32_t rel = e >> 12;
            const bool keep = (j0 + 64 * q + lane < cnt) && (rel <= lim);
            const uint32_t sr = shift + rel;
            const uint32_t d = sr ? sr - 1u : 0u;              // E_k minus min(rounded exponent, E_k)
            const uint32_t code = (((e >> 11) & 1u) << 3) | d;
            const int32_t pos = (int32_t)(e & 0x7FFu);
            const uint64_t b = __ballot(keep), lower = b & lanes_below(lane);
            const int src = lower ? 63 - __builtin_clzll(lower) : 0;
            const int32_t before = __shfl(pos, src);
            const uint32_t gap = (uint32_t)(pos - (lower ? before : prev) - 1);
            const bool is_long = keep && gap >= 8u;
            const uint64_t bl = __ballot(is_long);
            const uint32_t offset = bytes + (uint32_t)__popcll(lower) + (uint32_t)__popcll(bl & lanes_below(lane));
            const uint32_t b0 = (is_long ? 0x80u : 0u) | ((gap & 7u) << 4) | code, b1 = gap >> 3;
            sink(keep, b0, b1, is_long, offset);
            if (b) prev = __builtin_amdgcn_readlane(pos, 63 - __builtin_clzll(b));
            bytes += (uint32_t)__popcll(b) + (uint32_t)__popcll(bl);
        }
    }
    return bytes;
}

// kPer: consecutive tiles a wave does, whose first loads it asks for together.  The launches are rounds of waves that wait for memory
// (8192 are resident), and with two tiles there are half as many.  With few rounds the last ones, partly empty, cost more than that
// where tiles have many entries.  vgc_pack_compact at 3, 109, 293, 650 and 1230 bytes a tile, one tile -> two, us:
//   43984 tiles   36.4 -> 34.3, 40.8 -> 38.5, 53.0 -> 52.0,  84.5 ->  86.4, 127.7 -> 132.6
//   56000         44.5 -> 41.9, 50.7 -> 47.0, 64.4 -> 63.3, 103.5 -> 106.0, 158.0 -> 163.4
//   61000         47.4 -> 44.0, 56.2 -> 49.2, 69.0 -> 66.5, 111.1 -> 112.3, 171.5 -> 174.5
//   65536         44.6 -> 39.7, 51.3 -> 45.4, 66.7 -> 64.1, 111.9 -> 112.2, 176.2 -> 179.0
//   82000         52.8 -> 45.2, 59.1 -> 52.7, 77.6 -> 74.2, 133.7 -> 134.7, 219.2 -> 221.4
//   100000        60.0 -> 52.5, 67.3 -> 59.9, 89.6 -> 85.4, 158.0 -> 157.3, 272.6 -> 269.2
// So the line is where dense messages lose no more than 1.6 % and thin ones gain a tenth.  Three or four tiles lose up to 150 M elements
// (138 M at 620 bytes 112.6 -> 116.0, 121.7) and gain 3 % where few are sent.
template <uint32_t kPer>
__global__ __launch_bounds__(256) void k_compact_count(PlanCheck pc, uint64_t n_tiles, const TileHdr* __restrict__ hdrs,
                                                       const uint16_t* __restrict__ staging, uint16_t* __restrict__ tile_bytes) {
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t t0 = ((uint64_t)blockIdx.x * 4 + wave) * kPer;
    if (t0 >= n_tiles || !plan_ok(pc)) return;
    TileAhead a[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) a[q] = tile_ahead(hdrs, staging, min(t0 + q, n_tiles - 1), lane);
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        if (t0 + q >= n_tiles) break;
        const uint32_t bytes = encode_tile(a[q], staging, t0 + q, lane, [](const uint32_t* w) { return (w[7] & 0xFFFFu) != 0; },
                                           [](bool, uint32_t, uint32_t, bool, uint32_t) {});
        if (lane == 0) tile_bytes[t0 + q] = (uint16_t)bytes;
    }
}

template <uint32_t kPer>
__global__ __launch_bounds__(256) void k_compact_emit(PlanCheck pc, const PlanTile* __restrict__ tiles, uint64_t n_tiles,
                                                      const TileHdr* __restrict__ hdrs, const uint16_t* __restrict__ staging,
                                                      const uint16_t* __restrict__ tile_bytes, const uint64_t* __restrict__ run_offsets,
                                                      uint8_t* __restrict__ stream, uint64_t stream_cap) {
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t t0 = ((uint64_t)blockIdx.x * 4 + wave) * kPer;
    if (t0 >= n_tiles || !plan_ok(pc)) return;
    TileAhead a[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) a[q] = tile_ahead(hdrs, staging, min(t0 + q, n_tiles - 1), lane);
    // where the first tile's bytes go: the run's offset plus the bytes of the run's earlier tiles; the others' follow
    const PlanTile pt = tiles[t0];
    uint64_t out = 0;
    auto find_place = [&]() {
        const uint32_t in_run = (pt.start >> kTileShift) % kRunTiles;
        const uint32_t x = lane < in_run ? (uint32_t)tile_bytes[t0 - in_run + lane] : 0u;
        out = run_offsets[pt.run] + (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(x), 63);
    };
    uint32_t run[kPer] = {pt.run};
    uint64_t run_at[kPer] = {};
#pragma unroll
    for (uint32_t q = 1; q < kPer; ++q) run[q] = tiles[min(t0 + q, n_tiles - 1)].run;
#pragma unroll
    for (uint32_t q = 1; q < kPer; ++q) run_at[q] = run_offsets[run[q]];
    if (kPer > 1) find_place();                            // (one alone: only if it has some)
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
        if (t0 + q >= n_tiles) break;
        if (q > 0 && run[q] != run[q - 1]) out = run_at[q];
        out += encode_tile(a[q], staging, t0 + q, lane, [&](const uint32_t* w) {
            if ((w[7] & 0xFFFFu) == 0) return false;
            if (kPer == 1) find_place();
            return true;
        }, [&](bool keep, uint32_t b0, uint32_t b1, bool is_long, uint32_t offset) {
            const uint64_t o = out + offset;
            if (keep && o < stream_cap) stream[o] = (uint8_t)b0;
            if (is_long && o + 1 < stream_cap) stream[o + 1] = (uint8_t)b1;
        });
    }
}

// The same for parameter sets of at most kSmallTiles tiles, where the kernels are chains of a few us and the launches between
// them what counts: every workgroup reads all tile records and finds its groups' exponents by itself (k_compact_count_small), then
// all tiles' bytes and finds its own place (k_compact_emit_small, whose first workgroup also writes directory, headers and
// status).  us a call before -> now at few and at many sent: 20,000 elements 12.5 -> 7.2, 17.5 -> 11.3; 1.8 M 14.8 -> 9.9, 19.6 -> 14.0;
// 4.19 M (2046 tiles) 17.6 -> 15.7, 22.5 -> 19.7: what every workgroup reads grows with the set, and there its registers end it.
__global__ __launch_bounds__(256) void k_compact_count_small(PlanCheck pc, const uint32_t* __restrict__ flags, const PlanTile* __restrict__ tiles,
                                                             uint32_t n_tiles, uint32_t n_groups, TileHdr* __restrict__ hdrs,
                                                             const uint16_t* __restrict__ staging, uint16_t* __restrict__ tile_bytes) {
    constexpr uint32_t kPer = kSmallTiles / 256;
    __shared__ uint32_t max_e[kSmallGroups];
    if (!plan_ok(pc) || flags[0] != 0u) return;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6), t = blockIdx.x * 4 + wave;
    const uint32_t mine = min(t, n_tiles - 1);
    const TileAhead ahead = tile_ahead(hdrs, staging, mine, lane);
    const uint32_t own_group = tiles[mine].group;
    uint32_t w4[kPer], group[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = j * 256 + tid;
        w4[j] = i < n_tiles ? hdrs[i].w[4] : 0u;
        group[j] = i < n_tiles ? tiles[i].group : 0u;
    }
    for (uint32_t k = tid; k < n_groups; k += 256) max_e[k] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j)
        if (w4[j] >> 16) atomicMax(&max_e[group[j]], w4[j] >> 16);
    __syncthreads();
    if (t >= n_tiles) return;
    const uint32_t E = max_e[own_group];
    uint32_t w7 = 0;
    const uint32_t bytes = encode_tile(ahead, staging, t, lane, [&](uint32_t* w) {
        uint32_t shift;
        const uint32_t kept = kept_words(make_uint4(w[0], w[1], w[2], w[3]), w[4], E, shift);
        w[7] = w7 = kept | min(shift, 255u) << 16;
        return kept != 0;
    }, [](bool, uint32_t, uint32_t, bool, uint32_t) {});
    if (lane == 0) {
        tile_bytes[t] = (uint16_t)bytes;
        hdrs[t].w[7] = w7;
    }
}

__global__ __launch_bounds__(256) void k_compact_emit_small(PlanCheck pc, const uint32_t* __restrict__ flags, const PlanTile* __restrict__ tiles,
                                                            uint32_t n_tiles, uint32_t n_groups, const TileHdr* __restrict__ hdrs,
                                                            const uint16_t* __restrict__ staging, const uint16_t* __restrict__ tile_bytes,
                                                            uint64_t* __restrict__ run_offsets, uint8_t* __restrict__ stream, uint64_t stream_cap,
                                                            vgc_group_hdr* __restrict__ hdrs_out, vgc_pack_status* __restrict__ status) {
    constexpr uint32_t kPer = kSmallTiles / 256;
    __shared__ uint32_t max_e[kSmallGroups], count[kSmallGroups], place[kSmallGroups], sh[4], own[4];
    if (!plan_ok(pc) || flags[0] != 0u) {
        if (blockIdx.x == 0) empty_message(256, n_groups, hdrs_out, status);
        return;
    }
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6), t0 = blockIdx.x * 4, t = t0 + wave;
    const TileAhead ahead = tile_ahead(hdrs, staging, min(t, n_tiles - 1), lane);
    uint32_t bytes[kPer], sum = 0, before = 0;              // of a thread's consecutive tiles; those before the workgroup's
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = tid * kPer + j;
        bytes[j] = i < n_tiles ? (uint32_t)tile_bytes[i] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = tid * kPer + j;
        if (i < t0) before += bytes[j];
        if (i - t0 < 4u) own[i - t0] = bytes[j];
        sum += bytes[j];
    }
    before = wave_inclusive_sum(before);
    if (lane == 63) sh[wave] = before;
    __syncthreads();
    if (t < n_tiles) {
        uint32_t out = sh[0] + sh[1] + sh[2] + sh[3];       // (2048 tiles have at most 2^23 bytes)
        for (uint32_t q = 0; q < wave; ++q) out += own[q];
        encode_tile(ahead, staging, t, lane, [](const uint32_t* w) { return (w[7] & 0xFFFFu) != 0; },
                    [&](bool keep, uint32_t b0, uint32_t b1, bool is_long, uint32_t offset) {
            const uint64_t o = (uint64_t)out + offset;
            if (keep && o < stream_cap) stream[o] = (uint8_t)b0;
            if (is_long && o + 1 < stream_cap) stream[o + 1] = (uint8_t)b1;
        });
    }
    if (blockIdx.x != 0) return;
    uint32_t total;
    uint32_t at = block_scan<4>(sum, sh, total) - sum;
    for (uint32_t k = tid; k < n_groups; k += 256) max_e[k] = count[k] = place[k] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = tid * kPer + j;
        if (i < n_tiles) {
            const PlanTile pt = tiles[i];
            const uint32_t w4 = hdrs[i].w[4], kept = hdrs[i].w[7] & 0xFFFFu;
            if (w4 >> 16) atomicMax(&max_e[pt.group], w4 >> 16);
            if (kept) atomicAdd(&count[pt.group], kept);
            if (pt.start == 0) place[pt.group] = at;
            if ((pt.start >> kTileShift) % kRunTiles == 0) run_offsets[pt.run] = at;
        }
        at += bytes[j];
    }
    __syncthreads();
    for (uint32_t k = tid; k < n_groups; k += 256) {
        vgc_group_hdr h;
        h.exp_field = count[k] ? max_e[k] : 0u;
        h.count = count[k];
        h.word_offset = place[k];
        hdrs_out[k] = h;
    }
    if (tid == 0) {
        vgc_pack_status s;
        s.total_words = total;
        s.overflow = total > stream_cap ? 1u : 0u;
        s.plan_mismatch = 0;
        *status = s;
    }
}

constexpr uint64_t kTwoTiles = 65536;                       // tiles from which on a wave does two: eight rounds of waves (figures at the kernels)
int launch_pack_compact(PlanCheck pc, const uint32_t* flags, const PlanGroup* groups, const PlanTile* tiles, const PlanRun* runs,
                        const PlanSeg* segs, uint64_t n_tiles, uint64_t n_runs, uint32_t n_groups, uint32_t n_segs, uint32_t max_group_tiles,
                        TileHdr* hdrs, SegTmp* stmp, const uint16_t* staging, uint8_t* stream_out, uint64_t stream_cap,
                        uint16_t* tile_bytes_out, uint64_t* run_offsets_out, vgc_group_hdr* hdrs_out, vgc_pack_status* status_out,
                        hipStream_t stream) {
    const uint32_t tb = (uint32_t)((n_tiles + 3) / 4);
    if (n_tiles <= kSmallTiles && n_groups <= kSmallGroups) {
        hipLaunchKernelGGL(k_compact_count_small, dim3(tb), dim3(256), 0, stream, pc, flags, tiles, (uint32_t)n_tiles, n_groups, hdrs, staging,
                           tile_bytes_out);
        hipLaunchKernelGGL(k_compact_emit_small, dim3(tb), dim3(256), 0, stream, pc, flags, tiles, (uint32_t)n_tiles, n_groups, hdrs, staging,
                           tile_bytes_out, run_offsets_out, stream_out, stream_cap, hdrs_out, status_out);
        return hip_check(hipGetLastError(), "launch compact pack kernels (few tiles)");
    }
    const int rc = launch_part_scans(pc, groups, tiles, segs, n_tiles, n_segs, max_group_tiles, hdrs, stmp, stream);
    if (rc != VGC_OK) return rc;
    const bool two = n_tiles >= kTwoTiles;
    const uint32_t blocks = two ? (uint32_t)((n_tiles + 7) / 8) : tb;
    if (two) hipLaunchKernelGGL(k_compact_count<2>, dim3(blocks), dim3(256), 0, stream, pc, n_tiles, hdrs, staging, tile_bytes_out);
    else hipLaunchKernelGGL(k_compact_count<1>, dim3(blocks), dim3(256), 0, stream, pc, n_tiles, hdrs, staging, tile_bytes_out);
    const CompactDirectory dir = {tiles, runs, n_runs, tile_bytes_out, run_offsets_out, stream_cap};
    const int rc2 = launch_header_scan(pc, flags, groups, segs, n_groups, n_segs, max_group_tiles, hdrs, stmp, hdrs_out, status_out, ~0ull,
                                       &dir, stream);
    if (rc2 != VGC_OK) return rc2;
    if (two)
        hipLaunchKernelGGL(k_compact_emit<2>, dim3(blocks), dim3(256), 0, stream, pc, tiles, n_tiles, hdrs, staging, tile_bytes_out,
                           run_offsets_out, stream_out, stream_cap);
    else
        hipLaunchKernelGGL(k_compact_emit<1>, dim3(blocks), dim3(256), 0, stream, pc, tiles, n_tiles, hdrs, staging, tile_bytes_out,
                           run_offsets_out, stream_out, stream_cap);
    return hip_check(hipGetLastError(), "launch compact pack kernels");
}

// ------------------------------------------------------------------------------------------------
// decoder: several messages in one pass over the dense buffer, message order kept per element
// ------------------------------------------------------------------------------------------------
struct CompactArgs {
    const uint8_t* streams[kBatchMax];
    const uint16_t* tile_bytes[kBatchMax];
    const uint64_t* run_offsets[kBatchMax];
    const vgc_group_hdr* hdrs[kBatchMax];
    uint64_t n_bytes[kBatchMax];
    uint32_t p;
};

typedef float f4c __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) float* lds_float;
struct __attribute__((packed)) Unaligned64 { uint64_t x; };
typedef const __attribute__((address_space(1))) Unaligned64* global_u64;

constexpr uint32_t kLaneBytes = 8;                              // bytes of a message a lane decodes per round
constexpr uint32_t kRoundBytes = 64 * kLaneBytes;

// Bits 0..3 of x as bytes of 0x00 or 0xFF.
__device__ __forceinline__ uint32_t byte_mask(uint32_t x) {
    const uint32_t y = ((x & 15u) * 0x00204081u) & 0x01010101u;
    return __builtin_amdgcn_perm(0u, 0u, y | 0x0C0C0C0Cu);       // a selector of 12 gives 0x00, one of 13 0xFF
}

// One wave owns tiles_per_wave consecutive tiles of a run (tile in LDS, messages in order).
//
// What bounds it: fetched 64 bytes at a time, each fetch waiting for the end of the element before, by one wave per run
// of 64 tiles, 8 messages of 0.17 x 138 M elements took 2.57 ms, all of it latency (0.79 GB have to move: 0.13 ms).
// The directory says where every tile's bytes lie, so here a wave can start at any tile of a run, requests the first
// kRoundBytes of a message's tile while the message before it is decoded, and a lane decodes kLaneBytes consecutive
// bytes: 0.28 ms, and 0.19 ms (4.1 TB/s) since no byte takes a branch; bound by the vector instructions (188 a round of 512 bytes,
// which keep the units busy for 3/4 of the time) and the places in LDS that lanes share a bank for.
//
// Whether a lane's bytes begin inside an element follows from two ballots: a byte is the second of an element iff an
// odd number of bytes with bit 7 set precede it without a gap, so a lane whose bytes all have bit 7 set (an even number
// of them) passes the state of the lane before it on, and any other lane's outgoing state is the parity of its trailing
// bytes with bit 7 set.  An element is added at its last byte, up to which its position is the sum of all steps (gap + 1
// at a first byte, 8 times the value at a second byte); positions are kept in bytes of LDS.
// kMany: messages of at most 32, 16 or 8 lanes' bytes in a tile are decoded two, four or eight at once, each in its part of the
// wave, and then added one after the other.  A round takes its instructions whether a message fills it or not: 8 messages over
// 138 M elements took 182 to 188 us at any density up to 17 % and take now, at 0.2, 3 and 5 %, 109, 138 and 165 (writing alone: 95);
// over 4 M 12.5 -> 7.9, 11.2 (0.5, 4 %), over 20000 9.8 -> 6.1, 8.1; two messages of 0.5 to 4 % of 4 M 7.1 -> 6.7.
// kShort: some stream is shorter than a lane's access (1 to 7 bytes); its bytes are fetched one by one.
template <bool kShort, bool kMany>
__global__ __launch_bounds__(256, 5) void k_unpack_compact(PlanCheck pc, CompactArgs A, const PlanGroup* __restrict__ groups,
                                                           const PlanRun* __restrict__ runs, uint32_t n_runs, float scale,
                                                           float* __restrict__ dense, int overwrite, uint32_t tiles_per_wave) {
    static_assert(kBatchMax == 8, "a lane per (message, tile of a block of 8)");
    __shared__ __attribute__((aligned(4 * kTile))) float sh_tile[4][kTile];         // (a tile's address and a place in it are or-ed)
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t per_run = (uint32_t)kRunTiles / tiles_per_wave;
    const uint32_t gw = blockIdx.x * 4 + wave, run = gw / per_run;
    if (run >= n_runs || !plan_ok(pc)) return;
    float* T = sh_tile[wave];
    const uint32_t Tb = (uint32_t)(uintptr_t)(lds_float)T;
    uint32_t in_tile = 4u * (kTile - 1);                        // a mask in a register: and-or is one instruction then
    asm volatile("" : "+v"(in_tile));
    const uint32_t k = runs[run].group, first = runs[run].first_tile;
    const PlanGroup pg = groups[k];
    const uint32_t nt_group = (pg.size + kTile - 1) / kTile;
    const uint32_t run_end = min(first + (uint32_t)kRunTiles, nt_group);
    const uint32_t t0 = first + (gw % per_run) * tiles_per_wave;
    if (t0 >= run_end) return;
    const uint32_t t1 = min(t0 + tiles_per_wave, run_end);

    // Lanes 8 w .. 8 w + 7 keep message w: where the run's bytes begin, how many bytes the stream has from there (none
    // past them is read, whatever a damaged directory says; kShort, bit 31: the whole stream is shorter than a lane's access), the
    // group's exponent field, and for tile tb + lane % 8 of the block of 8 tiles being requested: offset inside the run << 13
    // | bytes (at most 2 kTile a tile).
    const uint32_t mw = lane >> 3, mj = lane & 7u;
    const bool mine = mw < A.p;
    uint64_t run_bytes = 0;
    uint32_t run_left = 0, expf = 0;
    const uint16_t* counts = nullptr;
    if (mine) {
        const uint64_t at = A.run_offsets[mw][run], n_bytes = A.n_bytes[mw];
        run_bytes = reinterpret_cast<uint64_t>(A.streams[mw]) + at;
        run_left = n_bytes > at ? (uint32_t)min(n_bytes - at, (uint64_t)1 << 20) : 0u;
        if (kShort && n_bytes < kLaneBytes) run_left |= 0x80000000u;
        expf = A.hdrs[mw][k].exp_field;
        counts = A.tile_bytes[mw] + pg.first_tile;
    }
    auto count_of = [&](uint32_t t) { return (mine && t < run_end) ? (uint32_t)counts[t] : 0u; };
    uint32_t cur = 0;                                           // bytes of the run's tiles before the block
    for (uint32_t t = first + mj; t < t0; t += 8) cur += min(count_of(t), 2u * kTile);
    cur += (uint32_t)__shfl_xor((int)cur, 1);
    cur += (uint32_t)__shfl_xor((int)cur, 2);
    cur += (uint32_t)__shfl_xor((int)cur, 4);
    uint32_t block = 0, most = 0, ahead = count_of(t0 + mj);      // most: the most bytes any message has of tile tb + lane % 8
    auto next_block = [&](uint32_t tb) {                        // ahead: the counts of the block that begins at tile tb
        const uint32_t here = min(ahead, 2u * kTile);
        uint32_t incl = here;
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)incl, off, 8);
            if (mj >= (uint32_t)off) incl += y;
        }
        block = ((cur + incl - here) << 13) | here;
        most = here;
#pragma unroll
        for (int off = 8; kMany && off < 64; off <<= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off));
        cur += (uint32_t)__shfl((int)incl, 7, 8);
        ahead = count_of(tb + 8 + mj);
    };
    // Bytes off .. off + 7 of the tile's message at S, `left` bytes of which may be read, once shifted down by `down` bits: the
    // shift is the reader's, who would otherwise wait for the bytes here.
    struct Bytes { uint64_t x; uint32_t down; };
    auto fetch = [&](const uint8_t* S, uint32_t off, int left, Bytes& y) {
        const int a = min((int)off, left - (int)kLaneBytes);    // the stream's last bytes: read from before them
        y.x = ((global_u64)((S - kLaneBytes) + (uint32_t)(a + (int)kLaneBytes)))->x;
        y.down = 8u * (off - (uint32_t)a);
    };
    // the same where the stream has fewer than 8 bytes in all (so the tile has, and off is 0): one by one
    auto fetch_few = [&](const uint8_t* S, int left, Bytes& y) {
        y.x = 0;
        for (int i = 0; i < left; ++i) y.x |= (uint64_t)S[i] << (8 * i);
        y.down = 0;
    };
    // the item (tile, first of its messages, how many: a power of two of lanes for each) requested next, and what has been requested
    uint32_t tn = t0, wn = 0, log_n = 6, many_n = 1, nb_n = 0, here_n = 0;
    int left_n = 0;
    const uint8_t* S_n = nullptr;
    Bytes x_n = {0, 0};
    auto request = [&]() {
        if (tn >= t1) return;
        const uint32_t tile = (tn - t0) & 7u;
        if (wn == 0 && tile == 0) next_block(tn);
        if (kMany && wn == 0) {
            const uint32_t top = (uint32_t)__builtin_amdgcn_readlane((int)most, (int)tile);
            log_n = top > 32 * kLaneBytes ? 6u : top > 16 * kLaneBytes ? 5u : top > 8 * kLaneBytes ? 4u : 3u;
        }
        if (kMany && log_n < 6) {
            many_n = min(64u >> log_n, A.p - wn);
            const uint32_t seg = lane >> log_n, off = (lane & ((1u << log_n) - 1u)) * kLaneBytes;
            const int src = (int)(8u * min(wn + seg, (uint32_t)kBatchMax - 1u));
            const uint32_t d = (uint32_t)__shfl((int)block, src + (int)tile);
            const uint64_t at = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(run_bytes >> 32), src) << 32) | (uint32_t)__shfl((int)(uint32_t)run_bytes, src);
            const int left = (int)(uint32_t)__shfl((int)run_left, src) - (int)(d >> 13);
            const uint32_t nb = seg < many_n ? (uint32_t)max(0, min((int)(d & 8191u), left)) : 0u;
            here_n = off < nb ? min(nb - off, kLaneBytes) : 0u;
            if (here_n) fetch(reinterpret_cast<const uint8_t*>(at) + (d >> 13), off, left, x_n);
        } else {
            many_n = 1;
            const int src = (int)(wn * 8u);
            const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)block, src + (int)tile);
            const uint64_t at = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(run_bytes >> 32), src) << 32) |
                                (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)run_bytes, src);
            const uint32_t left_of_run = (uint32_t)__builtin_amdgcn_readlane((int)run_left, src);
            const bool few = kShort && left_of_run >> 31;
            left_n = (int)(kShort ? left_of_run & 0x7FFFFFFFu : left_of_run) - (int)(d >> 13);
            nb_n = (uint32_t)max(0, min((int)(d & 8191u), left_n));
            S_n = reinterpret_cast<const uint8_t*>(at) + (d >> 13);
            if (lane * kLaneBytes < nb_n) {
                if (few) fetch_few(S_n, left_n, x_n);
                else fetch(S_n, lane * kLaneBytes, left_n, x_n);
            }
        }
        wn += many_n;
        if (wn == A.p) { wn = 0; ++tn; }
    };
    if (A.p) request();
    // what has been requested, waited for behind the message before: a wait in front of a tile's first message would be for the
    // stores of the tile before it as well (1 to 2 %)
    uint64_t bytes_n = x_n.x >> x_n.down;

    // A lane's `here` bytes in y of a message whose group has the exponent field ef: where in LDS each one's element lies and what
    // the codes amount to.  under: the lanes before it that hold bytes of the same message; inside, last: whether its first byte
    // there follows a first byte of two, and the byte before; from(sum over all lanes before): position in bytes of LDS.
    struct Elements { uint32_t at[kLaneBytes], hi[2], lo[2], c0, c1, ends, incl, back; bool by_byte; uint64_t stops, odd; };
    auto elements = [&](uint64_t y, uint32_t here, uint32_t ef, uint64_t under, uint32_t inside, uint32_t last, auto from) __attribute__((always_inline)) -> Elements {
        Elements E;
        uint32_t (&at)[kLaneBytes] = E.at, (&hi)[2] = E.hi, (&lo)[2] = E.lo;
        const uint32_t valid = (1u << here) - 1u;
        const uint64_t there = ~0ull >> ((8u * (kLaneBytes - here)) & 63u);         // (a lane with none: of no consequence)
        const uint64_t bytes = y & there;
        const uint2 x = make_uint2((uint32_t)bytes, (uint32_t)(bytes >> 32));
        // bit i: byte i has bit 7 set
        const uint32_t high = (__builtin_amdgcn_udot4((x.x >> 7) & 0x01010101u, 0x08040201u, 0u, false) |
                               __builtin_amdgcn_udot4((x.y >> 7) & 0x01010101u, 0x80402010u, 0u, false)) & valid;
        const uint64_t stops = __ballot(high != 0xFFu);
        const uint64_t odd = __ballot((__builtin_clz(~(high << 24)) & 1) != 0);
        const uint64_t before = stops & under;
        const uint32_t in = before ? (uint32_t)(odd >> (63 - __builtin_clzll(before))) & 1u : inside;
        // second bytes: those after an odd number of set bits, counted from where a run of them begins (the
        // carry of an addition runs through each run and comes out with its parity)
        const uint32_t opens = high & ~in;
        const uint32_t second = (((opens << 1) | 0xAAAAAAAAu) - opens) ^ 0xAAAAAAAAu ^ (high | in);
        const uint32_t ends = valid & (second | ~high);
        // the bytes that add their element: its last one, and the first of two in the same lane as well (see below)
        const uint32_t adds = ends | (second >> 1 & valid >> 1);
        const uint32_t m0 = byte_mask(second), m1 = byte_mask(second >> 4);
        // the 4-bit value of the element a byte ends: its own, or that of the byte before a second byte
        const uint32_t prev_lane = (uint32_t)__builtin_amdgcn_update_dpp((int)(last << 24), (int)x.y, 0x138, 0xF, 0xF, false);  // wave_shr:1
        const uint32_t c0 = (m0 & __builtin_amdgcn_alignbyte(x.x, prev_lane, 3)) | (~m0 & x.x);
        const uint32_t c1 = (m1 & __builtin_amdgcn_alignbyte(x.y, x.x, 3)) | (~m1 & x.y);
        // the first bytes' steps (gap + 1, low bits) and the second bytes' values; a sum over bytes is a dot product, with
        // the position in bytes of LDS 4 times the one and 32 times the other.  A second byte's value is counted at the
        // first byte before it (`lead`: that one is in the lane before), which so has its element's position already.
        const uint32_t f0 = ((((x.x >> 4) & 0x07070707u) + 0x01010101u) & (uint32_t)there) & ~m0, s0 = x.x & m0;
        const uint32_t f1 = ((((x.y >> 4) & 0x07070707u) + 0x01010101u) & (uint32_t)(there >> 32)) & ~m1, s1 = x.y & m1;
        const uint32_t q0 = __builtin_amdgcn_alignbyte(s1, s0, 1), q1 = s1 >> 8;
        const uint32_t lead = __builtin_amdgcn_udot4(s0, 0x00000020u, 0u, false);
        const uint32_t half = __builtin_amdgcn_udot4(q0, 0x20202020u, __builtin_amdgcn_udot4(f0, 0x04040404u, lead, false), false);
        const uint32_t sum = __builtin_amdgcn_udot4(q1, 0x20202020u, __builtin_amdgcn_udot4(f1, 0x04040404u, half, false), false);
        const uint32_t incl = wave_inclusive_sum(sum);
        const uint32_t p = from(incl - sum), p0 = p + lead, p1 = p + half;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t four = 0x04040404u >> (24 - 8 * i), eight = 0x20202020u >> (24 - 8 * i);     // of the bytes up to i
            at[i] = __builtin_amdgcn_udot4(q0, eight, __builtin_amdgcn_udot4(f0, four, p0, false), false);
            at[4 + i] = __builtin_amdgcn_udot4(q1, eight, __builtin_amdgcn_udot4(f1, four, p1, false), false);
        }
        at[3] = p1;
        at[7] = adds & 0x80u ? p + sum : at[6];
#pragma unroll
        for (int i = 0; i < (int)kLaneBytes; ++i) at[i] = (at[i] & in_tile) | Tb;
        // No byte needs a branch: each of a lane's eight writes its element's sum, or what the lane itself overwrites.  The
        // first byte of two writes the same as the second; one whose second is in the next lane writes where byte 6 does, and
        // the bytes behind the message's end where its last one does, both of which come later.  That leaves a message
        // that is cut inside an element, and exponents too small for some of the codes: there each byte is looked at.
        E.by_byte = ef < 8u || ((adds ^ valid) & 0x7Fu) != 0u;
        // the elements' values, sign and exponent (which reaches into the third byte), put together four at a time
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t c = h ? c1 : c0, exps = ef * 0x01010101u - (c & 0x07070707u);
            hi[h] = ((exps >> 1) & 0x7F7F7F7Fu) | ((c << 4) & 0x80808080u);
            lo[h] = (exps << 7) & 0x80808080u;
        }
        E.c0 = c0; E.c1 = c1; E.ends = ends; E.incl = incl; E.back = x.y; E.stops = stops; E.odd = odd;
        return E;
    };
    auto add_by_byte = [&](const Elements& E, uint32_t ef) {
#pragma unroll
        for (int i = 0; i < (int)kLaneBytes; ++i) {
            const uint32_t c = (i < 4 ? E.c0 : E.c1) >> (8 * (i & 3)), d = c & 7u;
            if ((E.ends >> i & 1u) && d < ef) {
                const float val = __uint_as_float((ef - d) << 23 | (c << 28 & 0x80000000u));
                const float contrib = scale * val;
                const lds_float e = (lds_float)(uintptr_t)E.at[i];
                *e = *e + contrib;
            }
        }
    };
    // the elements of one message are distinct: all are read before any is written
    auto contribution = [&](const Elements& E, int i) {
        const uint32_t sel = 0x04000C0Cu + 0x01010000u * (uint32_t)(i & 3);
        return scale * __uint_as_float(__builtin_amdgcn_perm(E.hi[i >> 2], E.lo[i >> 2], sel));
    };
    auto add = [&](const Elements& E, auto contrib) __attribute__((always_inline)) {
        float old[kLaneBytes];
#pragma unroll
        for (int i = 0; i < (int)kLaneBytes; ++i) old[i] = *(lds_float)(uintptr_t)E.at[i];
#pragma unroll
        for (int i = (int)kLaneBytes - 1; i >= 0; --i) *(lds_float)(uintptr_t)E.at[i] = old[i] + contrib(i);
    };

    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t start = t * kTile;
        const uint32_t m = min(kTile, pg.size - start);
        float* base = dense + pg.offset + start;
        const bool vec = m == kTile, whole = (reinterpret_cast<uintptr_t>(base) & 15u) == 0;
        if (overwrite) {
#pragma unroll
            for (int q = 0; q < 8; ++q) reinterpret_cast<f4c*>(T)[q * 64 + lane] = (f4c){0.f, 0.f, 0.f, 0.f};
        } else if (vec && whole) {
#pragma unroll
            for (int q = 0; q < 8; ++q) reinterpret_cast<f4c*>(T)[q * 64 + lane] = load_four<true>(base + 4 * (q * 64 + lane));
        } else if (vec) {
#pragma unroll
            for (int q = 0; q < 8; ++q) reinterpret_cast<f4c*>(T)[q * 64 + lane] = load_four<false>(base + 4 * (q * 64 + lane));
        } else {
            for (uint32_t i = lane; i < kTile; i += 64) T[i] = (i < m) ? base[i] : 0.f;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (uint32_t w = 0, many; w < A.p; w += many) {
            many = many_n;
            uint64_t y = bytes_n;
            if (kMany && log_n < 6) {
                const uint32_t log = log_n, here = here_n, seg = lane >> log;
                const uint32_t ef = (uint32_t)__shfl((int)expf, (int)(8u * min(w + seg, (uint32_t)kBatchMax - 1u)));
                request();
                const uint32_t begin = lane & ~((1u << log) - 1u);
                const Elements E = elements(y, here, ef, lanes_below(lane) & ~lanes_below(begin), 0u, 0u,
                                            [&](uint32_t sum) { return ~3u + sum - (uint32_t)__shfl((int)sum, (int)begin); });
                const bool on = here && ef - 1u < 254u;          // (else nothing of this message can be decoded)
                float contrib[kLaneBytes];
#pragma unroll
                for (int i = 0; i < (int)kLaneBytes; ++i) contrib[i] = contribution(E, i);
                const uint64_t slow = __ballot(on && E.by_byte);
#pragma unroll 1
                for (uint32_t s = 0; s < many; ++s) {
                    const bool turn = on && seg == s;
                    if (slow) { if (turn && E.by_byte) add_by_byte(E, ef); }
                    if (turn && !E.by_byte) add(E, [&](int i) { return contrib[i]; });
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
            } else {
                const uint32_t nb = nb_n;
                const int left = left_n;
                const uint8_t* S = S_n;
                const uint32_t ef = (uint32_t)__builtin_amdgcn_readlane((int)expf, (int)(w * 8u));
                request();
                const uint32_t ends_at = ef == 0 || ef > 254u ? 0u : nb;      // (0: nothing of this message can be decoded)
                uint32_t pos0 = ~3u;                            // position of the last element so far (-1: none), in bytes
                uint32_t inside = 0, last = 0;                  // whether the round begins inside an element, the byte before it
                for (uint32_t o = 0; o < ends_at; o += kRoundBytes) {
                    const uint32_t off = o + lane * kLaneBytes;
                    Bytes more = {0, 0};
                    if (off + kRoundBytes < nb) fetch(S, off + kRoundBytes, left, more);
                    const uint32_t here = off < nb ? min(nb - off, kLaneBytes) : 0u;
                    const Elements E = elements(y, here, ef, lanes_below(lane), inside, last, [&](uint32_t sum) { return pos0 + sum; });
                    if (E.by_byte) add_by_byte(E, ef);
                    if (off < nb && !E.by_byte) add(E, [&](int i) { return contribution(E, i); });
                    pos0 += (uint32_t)__builtin_amdgcn_readlane((int)E.incl, 63);
                    inside = E.stops ? (uint32_t)(E.odd >> (63 - __builtin_clzll(E.stops))) & 1u : inside;
                    last = (uint32_t)__builtin_amdgcn_readlane((int)E.back, 63) >> 24;
                    y = more.x >> more.down;
                }
            }
            bytes_n = x_n.x >> x_n.down;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (vec && whole) {
#pragma unroll
            for (int q = 0; q < 8; ++q) store_four<true>(reinterpret_cast<f4c*>(T)[q * 64 + lane], base + 4 * (q * 64 + lane));
        } else if (vec) {
#pragma unroll
            for (int q = 0; q < 8; ++q) store_four<false>(reinterpret_cast<f4c*>(T)[q * 64 + lane], base + 4 * (q * 64 + lane));
        } else {
            for (uint32_t i = lane; i < m; i += 64) base[i] = T[i];
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Whether some stream has bytes, but fewer than a lane reads at once.  From an empty one (a worker whose test fired nowhere)
// nothing is read, so it takes no part in the choice.  The variant with the test per message costs 1.4 % (7 messages of 17 % over
// 138 M elements and a short one: 181 against 179 us).
bool compact_short_streams(const uint64_t* n_bytes, uint32_t p) {
    for (uint32_t w = 0; w < p; ++w)
        if (n_bytes[w] != 0 && n_bytes[w] < kLaneBytes) return true;
    return false;
}

// Whether the messages are so thin that several fit a round in most tiles (at most 256 bytes each; the longest of them decides).
// The variant that looks for it costs 6 to 15 % where they do not: at 247 bytes a tile (8 % of 138 M elements, 8 messages) it takes
// 215 us against 187, at 170 165 against 185.  Lengths are what the caller knows: one given as a bound only keeps the other form.
// They say nothing of how the bytes are spread: with as few in all, but half of the tiles at 12 % and half empty, it takes 217 us
// against 186, an eighth of them at 24 % 331 against 301, two messages over 25.6 M 24.4 against 21.3.  A loop of either kind in one
// kernel, chosen by a wave's first tiles, took 199, 311 and 25.8, and where all tiles are thin 1 to 5 % more (8 messages of 0.5 % of
// 25.6 M: 28.5 -> 29.8): messages of one density are what is usual, so there is one loop.
bool compact_thin_streams(const uint64_t* n_bytes, uint32_t p, uint64_t n_tiles) {
    uint64_t most = 0;
    for (uint32_t w = 0; w < p; ++w) most = std::max(most, n_bytes[w]);
    return p > 1 && most <= 200 * n_tiles;
}

int launch_unpack_compact_batch(PlanCheck pc, const uint8_t* const* streams, const uint64_t* stream_bytes, const uint16_t* const* tile_bytes,
                                const uint64_t* const* run_offsets, const vgc_group_hdr* const* hdrs, uint32_t p,
                                const PlanGroup* groups, const PlanRun* runs, uint64_t n_tiles, uint64_t n_runs, float scale,
                                int overwrite, float* dense, uint32_t tiles_per_wave, hipStream_t stream) {
    const uint32_t tpw = decode_tiles_per_wave(n_runs, 16384, tiles_per_wave);
    const uint32_t blocks = (uint32_t)((n_runs * (kRunTiles / tpw) + 3) / 4);
    const uint32_t chunks = p ? (p + kBatchMax - 1) / kBatchMax : 1;
    for (uint32_t ch = 0; ch < chunks; ++ch) {
        CompactArgs A;
        const uint32_t first = ch * kBatchMax;
        A.p = p - first < (uint32_t)kBatchMax ? p - first : (uint32_t)kBatchMax;
        for (uint32_t w = 0; w < (uint32_t)kBatchMax; ++w) {
            const bool on = w < A.p;
            A.streams[w] = on ? streams[first + w] : nullptr;
            A.n_bytes[w] = on ? stream_bytes[first + w] : 0;
            A.tile_bytes[w] = on ? tile_bytes[first + w] : nullptr;
            A.run_offsets[w] = on ? run_offsets[first + w] : nullptr;
            A.hdrs[w] = on ? hdrs[first + w] : nullptr;
        }
#define VGC_COMPACT(SHORT, MANY)                                                                                              \
    hipLaunchKernelGGL((k_unpack_compact<SHORT, MANY>), dim3(blocks), dim3(256), 0, stream, pc, A, groups, runs, (uint32_t)n_runs, \
                       scale, dense, (overwrite && ch == 0) ? 1 : 0, tpw)
        if (compact_short_streams(A.n_bytes, A.p)) VGC_COMPACT(true, false);
        else if (compact_thin_streams(A.n_bytes, A.p, n_tiles)) VGC_COMPACT(false, true);
        else VGC_COMPACT(false, false);
#undef VGC_COMPACT
    }
    return hip_check(hipGetLastError(), "launch k_unpack_compact");
}

}  // namespace vgc
