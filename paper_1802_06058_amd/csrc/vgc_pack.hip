// Second half of Encode() (Sections 4.2 and 4.4): fix floor(log2 M_k) per group, turn the staged
// tile-relative exponent codes into the final 3-bit codes, drop what falls below 2^(E_k-7), and
// write the words of every group contiguously, in ascending index order.
//
// The scans are chains of dependent loads and barriers, not bandwidth, so their time is that of the largest unit one workgroup
// owns.  A group is cut into parts of up to kPartTiles tiles for them.  (One workgroup per segment of 8192 tiles took 16.5 us
// and its maximum 7.5 on 102.8 M elements in one group; with parts of 1024 tiles 6.0 and 5.0.  vgc_pack on ResNet-50: as before.)
//
//   k_part_max     (only when some group has more than two parts) largest tile exponent per part.
//   k_part_scan    one workgroup per part: E_k = max of the tile exponents, then per tile the
//                  number of words it keeps and its exclusive prefix inside the part.
//   k_header_scan  one workgroup: exclusive scan of the parts' counts -> headers, status and the
//                  position of every segment's and part's first word.
//   k_emit         one wave per tile: read the staged entries, filter, re-rank, write words.
//   k_pack_small   all of it in one launch, for parameter sets of few tiles.
#include "vgc_scan.h"

namespace vgc {

__device__ __forceinline__ uint32_t rank_below64(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Workgroup maximum.
template <int kWaves>
__device__ __forceinline__ uint32_t block_max(uint32_t e, uint32_t* sh /*[kWaves]*/) {
    e = wave_max(e);
    __syncthreads();
    if ((threadIdx.x & 63u) == 0) sh[threadIdx.x >> 6] = e;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) e = max(e, sh[w]);
    return e;
}

// The part of a workgroup: its tile records and how many there are (0: none).  Workgroup i < n_segs has the first part of segment
// i.  The other parts begin at least kPartTiles tiles apart, each behind a part of the same segment: workgroup n_segs + j has
// the one that begins among the tiles from j kPartTiles on, if any, and that is one of the segment of the first of these.  (A
// workgroup for as many parts as the largest group's segments have, of every segment: 100,000 groups of 700 elements and one of
// 20 M, vgc_pack 1760 us; so 787, and 707 without the large one.)
struct Part {
    uint32_t seg, index, cnt, group_tiles;
    uint64_t first, group_first;           // its first tile; its group's first tile
};
__device__ __forceinline__ Part part_of_block(const PlanGroup* __restrict__ groups, const PlanTile* __restrict__ tiles, const PlanSeg* __restrict__ segs,
                                              uint32_t n_segs) {
    Part q;
    uint32_t group, in_group;
    if (blockIdx.x < n_segs) {
        q.seg = blockIdx.x;
        q.index = 0;
        const PlanSeg ps = segs[q.seg];
        group = ps.group;
        in_group = ps.first_tile;
    } else {
        const PlanTile pt = tiles[(uint64_t)(blockIdx.x - n_segs) * kPartTiles];
        const uint32_t tile = pt.start >> kTileShift, in_seg = tile % kSegTiles;
        q.seg = pt.seg;
        q.index = (in_seg + kPartTiles - 1) / kPartTiles;
        group = pt.group;
        in_group = tile - in_seg + q.index * kPartTiles;
        if (q.index == 0 || q.index == kSegTiles / kPartTiles) in_group = ~0u;      // a segment's first part: not here
    }
    const PlanGroup pg = groups[group];
    q.group_tiles = (pg.size + kTile - 1) / kTile;
    q.group_first = pg.first_tile;
    q.first = (uint64_t)pg.first_tile + in_group;
    q.cnt = in_group < q.group_tiles ? min(kPartTiles, q.group_tiles - in_group) : 0u;
    return q;
}

constexpr uint32_t kScanThreads = 256;

// Groups of two parts have their exponent found by both parts' workgroups of the scan kernel, from all their records; a launch
// of its own would cost ResNet-50 (one group of 1152 tiles) 2.7 us.  From three parts on it is worth it.
constexpr uint32_t kOwnMaxTiles = 2 * kPartTiles;

// Only for groups of more than kOwnMaxTiles tiles: the largest tile exponent of every part into w[6] of its first record, so that the
// scan kernel's workgroups can each derive E_k of the whole group.
__global__ __launch_bounds__(kScanThreads) void k_part_max(PlanCheck pc, const PlanGroup* __restrict__ groups, const PlanTile* __restrict__ tiles,
                                                  const PlanSeg* __restrict__ segs, TileHdr* __restrict__ hdrs, uint32_t n_segs) {
    __shared__ uint32_t sh[kScanThreads / 64];
    if (!plan_ok(pc)) return;
    const Part q = part_of_block(groups, tiles, segs, n_segs);
    if (q.cnt == 0 || q.group_tiles <= kOwnMaxTiles) return;            // the scan kernel finds E_k itself
    const TileHdr* H = hdrs + q.first;
    uint32_t w[kPartTiles / kScanThreads], e = 0;
#pragma unroll
    for (uint32_t j = 0; j < kPartTiles / kScanThreads; ++j) {       // independent loads in flight
        const uint32_t i = j * kScanThreads + threadIdx.x;
        w[j] = (i < q.cnt) ? H[i].w[4] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < kPartTiles / kScanThreads; ++j) e = max(e, w[j] >> 16);
    e = block_max<kScanThreads / 64>(e, sh);
    if (threadIdx.x == 0) hdrs[q.first].w[6] = e;
}

// One workgroup per part: E_k, then per tile the number of words it keeps and its exclusive prefix inside the part (the first
// tile's, which is 0, gives its place to the part's count).  Each thread owns consecutive tile records: they are loaded
// together, scanned in registers, and only the per-thread totals go through the workgroup scan.
__global__ __launch_bounds__(kScanThreads) void k_part_scan(PlanCheck pc, const PlanGroup* __restrict__ groups, const PlanTile* __restrict__ tiles,
                                                   const PlanSeg* __restrict__ segs, TileHdr* __restrict__ hdrs, SegTmp* __restrict__ stmp, uint32_t n_segs) {
    constexpr uint32_t kPer = kPartTiles / kScanThreads;
    __shared__ uint32_t sh[kScanThreads / 64];
    if (!plan_ok(pc)) return;
    const Part q = part_of_block(groups, tiles, segs, n_segs);
    if (q.cnt == 0) return;
    TileHdr* H = hdrs + q.first;
    const uint32_t tid = threadIdx.x;

    // the loads of the records do not depend on E_k: issue them first
    uint4 lo[kPer];
    uint32_t w4[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = tid * kPer + j;
        lo[j] = make_uint4(0u, 0u, 0u, 0u);
        w4[j] = 0u;
        if (i < q.cnt) {
            lo[j] = reinterpret_cast<const uint4*>(H + i)[0];
            w4[j] = H[i].w[4];
        }
    }
    uint32_t E = 0;
    if (q.group_tiles <= kPartTiles) {
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) E = max(E, w4[j] >> 16);
    } else if (q.group_tiles <= kOwnMaxTiles) {
        const TileHdr* G = hdrs + q.group_first;
        uint32_t x[kOwnMaxTiles / kScanThreads];
#pragma unroll
        for (uint32_t j = 0; j < kOwnMaxTiles / kScanThreads; ++j) {
            const uint32_t i = j * kScanThreads + tid;
            x[j] = i < q.group_tiles ? G[i].w[4] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < kOwnMaxTiles / kScanThreads; ++j) E = max(E, x[j] >> 16);
    } else {
        const uint32_t n_parts = (q.group_tiles + kPartTiles - 1) / kPartTiles;         // at most 128
        if (tid < n_parts) E = hdrs[q.group_first + (uint64_t)tid * kPartTiles].w[6];
    }
    E = block_max<kScanThreads / 64>(E, sh);

    uint32_t kept[kPer], shift[kPer], mine = 0;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        kept[j] = kept_words(lo[j], w4[j], E, shift[j]);
        mine += kept[j];
    }
    uint32_t total;
    const uint32_t incl = block_scan<kScanThreads / 64>(mine, sh, total);
    uint32_t prefix = incl - mine;
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = tid * kPer + j;
        if (i < q.cnt) {
            H[i].w[5] = i == 0 ? total : prefix;
            H[i].w[7] = kept[j] | min(shift[j], 255u) << 16;
        }
        prefix += kept[j];
    }
    if (tid == 0 && q.index == 0) stmp[q.seg].exp_field = E;
}

// Bytes of a run of the compressed index format: the sum over its tiles (at most 64, of at most 2 kTile bytes each), by one thread.
struct __attribute__((packed, aligned(2))) EightCounts { uint32_t w[4]; };
__device__ __forceinline__ uint32_t run_bytes(const uint16_t* __restrict__ tile_bytes, uint32_t n) {
    static_assert(kRunTiles == 64, "eight loads of eight tiles");
    EightCounts x[8];
    uint16_t y[7];
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) x[q] = 8 * q + 8 <= n ? reinterpret_cast<const EightCounts*>(tile_bytes + 8 * q)[0] : EightCounts{{0, 0, 0, 0}};
#pragma unroll
    for (uint32_t i = 0; i < 7; ++i) y[i] = (n & ~7u) + i < n ? tile_bytes[(n & ~7u) + i] : (uint16_t)0;
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q)
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) sum += (x[q].w[i] & 0xFFFFu) + (x[q].w[i] >> 16);
#pragma unroll
    for (uint32_t i = 0; i < 7; ++i) sum += y[i];
    return sum;
}

// The bytes of every run, in the place of its offset: for more runs than kFoldedRuns, whose sums the header scan leaves alone.
// Its one workgroup takes 1024 runs at a time, each behind a chain of three loads: 10^9 elements (7630 runs) 100 us, so 15 and 5
// for the sums, vgc_pack_compact of 3 M elements of them 333 -> 267 us.  A launch is some 3 us: for one chunk it is not worth it.
constexpr uint64_t kFoldedRuns = 1024;
__global__ __launch_bounds__(256) void k_run_sums(PlanCheck pc, const PlanGroup* __restrict__ groups, const PlanRun* __restrict__ runs, uint64_t n_runs,
                                                  const uint16_t* __restrict__ tile_bytes, uint64_t* __restrict__ run_offsets) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t r = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= n_runs || !plan_ok(pc)) return;
    const PlanRun pr = runs[r];
    const PlanGroup pg = groups[pr.group];
    const uint32_t tiles = (pg.size + kTile - 1) / kTile - pr.first_tile;
    uint32_t x = lane < tiles ? (uint32_t)tile_bytes[(uint64_t)pg.first_tile + pr.first_tile + lane] : 0u;
    static_assert(kRunTiles == 64, "a lane a tile");
    x = wave_inclusive_sum(x);
    if (lane == 63) run_offsets[r] = x;
}

// One workgroup: the parts' counts become their places inside the segment, an exclusive scan over the segments gives their
// places in the message, and from these follow headers and status.  kCompact: the message is one with compressed indexes; the
// same scan over the runs' bytes gives run offsets, and the groups' offsets and the total are in bytes.
template <bool kCompact>
__global__ __launch_bounds__(1024) void k_header_scan(PlanCheck pc, const uint32_t* __restrict__ flags,
                                                      const PlanGroup* __restrict__ groups, const PlanSeg* __restrict__ segs,
                                                      TileHdr* __restrict__ hdrs, SegTmp* __restrict__ stmp,
                                                      uint32_t n_groups, uint32_t n_segs, uint32_t parts_per_seg,
                                                      vgc_group_hdr* __restrict__ hdrs_out,
                                                      vgc_pack_status* __restrict__ status, uint64_t words_cap, CompactDirectory dir) {
    constexpr uint32_t kParts = kSegTiles / kPartTiles;
    __shared__ uint32_t sh[16];
    if (!plan_ok(pc) || flags[0] != 0u) {
        empty_message(1024, n_groups, hdrs_out, status);
        return;
    }
    uint64_t running = 0;
    for (uint32_t base = 0; base < n_segs; base += 1024) {
        const uint32_t i = base + threadIdx.x;
        uint32_t count = 0;
        if (i < n_segs) {
            const PlanSeg ps = segs[i];
            const PlanGroup pg = groups[ps.group];
            const uint32_t tiles = (pg.size + kTile - 1) / kTile - ps.first_tile;           // of the segment and those behind it
            TileHdr* H = hdrs + pg.first_tile + ps.first_tile;
            uint32_t c[kParts];
#pragma unroll
            for (uint32_t q = 0; q < kParts; ++q) c[q] = q < parts_per_seg && q * kPartTiles < tiles ? H[q * kPartTiles].w[5] : 0u;
#pragma unroll
            for (uint32_t q = 0; q < kParts; ++q) {
                if (q < parts_per_seg && q * kPartTiles < tiles) H[q * kPartTiles].w[5] = count;
                count += c[q];
            }
        }
        // a chunk of 1024 segments holds at most 1024 * 2^24 words: scan the low and high parts separately
        const uint32_t lo = count & 0xFFFFu, hi = count >> 16;
        uint32_t tot_lo, tot_hi;
        const uint32_t incl_lo = block_scan<16>(lo, sh, tot_lo);
        const uint32_t incl_hi = block_scan<16>(hi, sh, tot_hi);
        if (i < n_segs) {
            stmp[i].count = count;
            stmp[i].base = running + (uint64_t)incl_lo + ((uint64_t)incl_hi << 16) - count;
        }
        running += (uint64_t)tot_lo + ((uint64_t)tot_hi << 16);
    }
    if (kCompact) {
        running = 0;
        for (uint64_t base = 0; base < dir.n_runs; base += 1024) {
            const uint64_t q = base + threadIdx.x;
            uint32_t bytes = 0;
            if (q >= dir.n_runs) {
            } else if (dir.n_runs > kFoldedRuns) {
                bytes = (uint32_t)dir.run_offsets[q];
            } else {
                const PlanRun pr = dir.runs[q];
                const PlanGroup pg = groups[pr.group];
                const uint32_t tiles = (pg.size + kTile - 1) / kTile - pr.first_tile;
                bytes = run_bytes(dir.tile_bytes + pg.first_tile + pr.first_tile, min(tiles, kRunTiles));
            }
            uint32_t total;                                  // (1024 runs hold at most 2^28 bytes)
            const uint32_t incl = block_scan<16>(bytes, sh, total);
            if (q < dir.n_runs) dir.run_offsets[q] = running + incl - bytes;
            running += total;
        }
    }
    __threadfence_block();
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_segs; i += 1024) {
        const PlanSeg ps = segs[i];
        if (ps.seg_in_group != 0) continue;
        const uint32_t nt = (groups[ps.group].size + kTile - 1) / kTile, last = i + (nt + kSegTiles - 1) / kSegTiles - 1;
        vgc_group_hdr h;
        h.word_offset = stmp[i].base;
        h.count = (uint32_t)(stmp[last].base + stmp[last].count - h.word_offset);
        h.exp_field = h.count ? stmp[i].exp_field : 0u;
        if (kCompact) h.word_offset = dir.run_offsets[dir.tiles[groups[ps.group].first_tile].run];
        hdrs_out[ps.group] = h;
    }
    if (threadIdx.x == 0) {
        vgc_pack_status st;
        st.total_words = running;
        st.overflow = running > (kCompact ? dir.stream_cap : words_cap) ? 1u : 0u;
        st.plan_mismatch = 0;
        *status = st;
    }
}

constexpr int kAhead = 8;                                   // rounds of 64 staged entries loaded before anything is known

// Every tile owns kTile staging slots, so the first rounds can be fetched before the tile's count is known (slots past the
// count hold stale data and are ignored): the loads overlap those of the records.
__device__ __forceinline__ void first_entries(const uint16_t* __restrict__ st, uint32_t lane, uint32_t* e) {
#pragma unroll
    for (int j = 0; j < kAhead; ++j) e[j] = __builtin_nontemporal_load(st + j * 64 + lane);
}

// The words of one tile (a wave): the entries e, then those behind them, `cnt` in all, kept where rel <= 8 - shift.
__device__ __forceinline__ void emit_tile(const uint16_t* __restrict__ st, uint32_t* e, uint32_t cnt, uint32_t shift, uint32_t start,
                                          uint64_t out, uint32_t lane, uint32_t* __restrict__ words, uint64_t words_cap) {
    const uint32_t lim = 8 - shift;
    for (uint32_t j0 = 0; j0 < cnt; j0 += 64 * kAhead) {
        if (j0) {
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const uint32_t jj = j0 + j * 64 + lane;
                e[j] = (jj < kTile) ? (uint32_t)__builtin_nontemporal_load(st + jj) : 0xFFFFu;
            }
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const uint32_t jj = j0 + j * 64 + lane;
            const uint32_t rel = e[j] >> 12;
            const bool keep = (jj < cnt) && (rel <= lim);
            const uint32_t sr = shift + rel;
            const uint32_t d = sr ? sr - 1u : 0u;           // E_k minus min(rounded exponent, E_k)
            const uint32_t word = (((e[j] >> 11) & 1u) << 31) | (d << 28) | (start + (e[j] & 0x7FFu));
            const uint64_t b = __ballot(keep);
            const uint64_t pos = out + rank_below64(b);
            if (keep && pos < words_cap) words[pos] = word;         // (in the cache: see k_emit)
            out += (uint32_t)__popcll(b);
        }
    }
}

// The words are left in the cache, where tiles meet in their lines: past it (non-temporal) the kernel is 1.05 to 1.3 times slower
// (75 M elements, 59 % sent, 67 against 86 us), and so is the decoder that reads them next.  Only 10^9 elements with few sent
// are 0.7 % faster past it, select and pack together (4595 against 4565 us).
__global__ __launch_bounds__(256) void k_emit(PlanCheck pc, const PlanTile* __restrict__ tiles, uint64_t n_tiles,
                                              const TileHdr* __restrict__ hdrs, const uint16_t* __restrict__ staging,
                                              const SegTmp* __restrict__ stmp,
                                              uint32_t* __restrict__ words, uint64_t words_cap) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t t = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= n_tiles || !plan_ok(pc)) return;
    const uint16_t* st = staging + t * kTile;
    uint32_t e[kAhead];
    first_entries(st, lane, e);
    const uint32_t hw = (lane < 8) ? hdrs[t].w[lane] : 0u;  // one 32-byte read per wave
    const PlanTile pt = tiles[t];
    uint32_t w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = (uint32_t)__builtin_amdgcn_readlane((int)hw, i);
    if ((w[7] & 0xFFFFu) == 0) return;                      // (else the shift is at most 8)
    const uint32_t cnt = (w[0] & 0xFFFFu) + (w[0] >> 16) + (w[1] & 0xFFFFu) + (w[1] >> 16) + (w[2] & 0xFFFFu) +
                         (w[2] >> 16) + (w[3] & 0xFFFFu) + (w[3] >> 16) + (w[4] & 0xFFFFu);
    // the segment's place in the message, the part's in the segment (a segment's first part: none), the tile's in the part
    const uint32_t in_seg = (pt.start >> kTileShift) % kSegTiles, in_part = in_seg % kPartTiles;
    uint64_t out = stmp[pt.seg].base + w[5];
    if (in_seg >= kPartTiles && in_part) out += hdrs[t - in_part].w[5];
    emit_tile(st, e, cnt, w[7] >> 16, pt.start, out, lane, words, words_cap);
}

// The whole of vgc_pack for parameter sets of at most kSmallTiles tiles: every workgroup reads all tile records (32 bytes each,
// from L2) and finds the groups' exponents and its own four tiles' place by itself, so that two launches and the waits between
// them fall away.  1.8 M elements (880 tiles): 4.7 + 4.0 + 5.2 us in three kernels, 14.2 us a call -> 9.0.  The records every
// workgroup reads grow with the set: at 4.1 M elements 11.6 against 15.0 us, and there the registers that hold them end it.
__global__ __launch_bounds__(256) void k_pack_small(PlanCheck pc, const uint32_t* __restrict__ flags, const PlanTile* __restrict__ tiles,
                                                    uint32_t n_tiles, uint32_t n_groups, const TileHdr* __restrict__ hdrs,
                                                    const uint16_t* __restrict__ staging, uint32_t* __restrict__ words,
                                                    uint64_t words_cap, vgc_group_hdr* __restrict__ hdrs_out,
                                                    vgc_pack_status* __restrict__ status) {
    constexpr uint32_t kPer = kSmallTiles / 256;
    __shared__ uint32_t max_e[kSmallGroups], count[kSmallGroups], sh[4], own_kept[4], own_shift[4], own_cnt[4];
    if (!plan_ok(pc) || flags[0] != 0u) {
        if (blockIdx.x == 0) empty_message(256, n_groups, hdrs_out, status);
        return;
    }
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6), t0 = blockIdx.x * 4, t = t0 + wave;
    const bool first_block = blockIdx.x == 0;               // it writes headers and status too
    const uint16_t* st = staging + (uint64_t)min(t, n_tiles - 1) * kTile;
    uint32_t e[kAhead];
    first_entries(st, lane, e);
    uint4 lo[kPer];
    uint32_t w4[kPer], group[kPer];
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = j * 256 + tid;
        lo[j] = make_uint4(0u, 0u, 0u, 0u);
        w4[j] = group[j] = 0;
        if (i < n_tiles) {
            lo[j] = reinterpret_cast<const uint4*>(hdrs + i)[0];
            w4[j] = hdrs[i].w[4];
            group[j] = tiles[i].group;
        }
    }
    const uint32_t start = tiles[min(t, n_tiles - 1)].start;
    for (uint32_t k = tid; k < n_groups; k += 256) max_e[k] = count[k] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j)
        if (w4[j] >> 16) atomicMax(&max_e[group[j]], w4[j] >> 16);
    __syncthreads();
    uint32_t before = 0;                                    // words of the tiles before the workgroup's
#pragma unroll
    for (uint32_t j = 0; j < kPer; ++j) {
        const uint32_t i = j * 256 + tid;
        if (i >= n_tiles) continue;
        uint32_t shift;
        const uint32_t kept = kept_words(lo[j], w4[j], max_e[group[j]], shift);
        if (i < t0) before += kept;
        if (i - t0 < 4u) {
            const uint32_t h = lo[j].x + lo[j].y + lo[j].z + lo[j].w + (w4[j] & 0xFFFFu);     // (no carry: at most 2048 in all)
            own_kept[i - t0] = kept; own_shift[i - t0] = shift; own_cnt[i - t0] = (h & 0xFFFFu) + (h >> 16);
        }
        if (first_block && kept) atomicAdd(&count[group[j]], kept);
    }
    before = wave_inclusive_sum(before);
    if (lane == 63) sh[wave] = before;
    __syncthreads();
    if (t < n_tiles && own_kept[wave] != 0) {
        uint32_t out = sh[0] + sh[1] + sh[2] + sh[3];
        for (uint32_t q = 0; q < wave; ++q) out += own_kept[q];
        emit_tile(st, e, own_cnt[wave], own_shift[wave], start, out, lane, words, words_cap);
    }
    if (!first_block) return;
    uint32_t running = 0;                                   // at most kSmallTiles * kTile words
    for (uint32_t base = 0; base < n_groups; base += 256) {
        const uint32_t k = base + tid;
        const uint32_t c = k < n_groups ? count[k] : 0u;
        uint32_t total;
        const uint32_t incl = block_scan<4>(c, sh, total);
        if (k < n_groups) {
            vgc_group_hdr h;
            h.exp_field = c ? max_e[k] : 0u;
            h.count = c;
            h.word_offset = running + incl - c;
            hdrs_out[k] = h;
        }
        running += total;
    }
    if (tid == 0) {
        vgc_pack_status s;
        s.total_words = running;
        s.overflow = running > words_cap ? 1u : 0u;
        s.plan_mismatch = 0;
        *status = s;
    }
}

static uint32_t parts_per_seg(uint32_t max_group_tiles) {
    const uint32_t parts = (max_group_tiles + kPartTiles - 1) / kPartTiles;
    return parts < kSegTiles / kPartTiles ? parts : kSegTiles / kPartTiles;
}

int launch_part_scans(PlanCheck pc, const PlanGroup* groups, const PlanTile* tiles, const PlanSeg* segs, uint64_t n_tiles, uint32_t n_segs,
                      uint32_t max_group_tiles, TileHdr* hdrs, SegTmp* stmp, hipStream_t stream) {
    const uint32_t blocks = n_segs + (max_group_tiles > kPartTiles ? (uint32_t)((n_tiles + kPartTiles - 1) / kPartTiles) : 0u);
    if (max_group_tiles > kOwnMaxTiles)
        hipLaunchKernelGGL(k_part_max, dim3(blocks), dim3(kScanThreads), 0, stream, pc, groups, tiles, segs, hdrs, n_segs);
    hipLaunchKernelGGL(k_part_scan, dim3(blocks), dim3(kScanThreads), 0, stream, pc, groups, tiles, segs, hdrs, stmp, n_segs);
    return hip_check(hipGetLastError(), "launch part scans");
}

int launch_header_scan(PlanCheck pc, const uint32_t* flags, const PlanGroup* groups, const PlanSeg* segs, uint32_t n_groups,
                       uint32_t n_segs, uint32_t max_group_tiles, TileHdr* hdrs, SegTmp* stmp, vgc_group_hdr* hdrs_out,
                       vgc_pack_status* status_out, uint64_t words_cap, const CompactDirectory* compact, hipStream_t stream) {
    const uint32_t pps = parts_per_seg(max_group_tiles);
    if (compact && compact->n_runs > kFoldedRuns)
        hipLaunchKernelGGL(k_run_sums, dim3((uint32_t)((compact->n_runs + 3) / 4)), dim3(256), 0, stream, pc, groups, compact->runs, compact->n_runs,
                           compact->tile_bytes, compact->run_offsets);
    if (compact)
        hipLaunchKernelGGL(k_header_scan<true>, dim3(1), dim3(1024), 0, stream, pc, flags, groups, segs, hdrs, stmp, n_groups, n_segs, pps,
                           hdrs_out, status_out, words_cap, *compact);
    else
        hipLaunchKernelGGL(k_header_scan<false>, dim3(1), dim3(1024), 0, stream, pc, flags, groups, segs, hdrs, stmp, n_groups, n_segs, pps,
                           hdrs_out, status_out, words_cap, CompactDirectory{});
    return hip_check(hipGetLastError(), "launch k_header_scan");
}

int launch_pack(PlanCheck pc, const uint32_t* flags, const PlanGroup* groups, const PlanTile* tiles, const PlanSeg* segs, uint64_t n_tiles,
                uint32_t n_groups, uint32_t n_segs, uint32_t max_group_tiles,
                TileHdr* hdrs, SegTmp* stmp, const uint16_t* staging,
                uint32_t* words_out, uint64_t words_cap, vgc_group_hdr* hdrs_out,
                vgc_pack_status* status_out, hipStream_t stream) {
    const uint32_t blocks = (uint32_t)((n_tiles + 3) / 4);
    if (n_tiles <= kSmallTiles && n_groups <= kSmallGroups) {
        hipLaunchKernelGGL(k_pack_small, dim3(blocks), dim3(256), 0, stream, pc, flags, tiles, (uint32_t)n_tiles, n_groups, hdrs, staging,
                           words_out, words_cap, hdrs_out, status_out);
        return hip_check(hipGetLastError(), "launch k_pack_small");
    }
    int rc = launch_part_scans(pc, groups, tiles, segs, n_tiles, n_segs, max_group_tiles, hdrs, stmp, stream);
    if (rc == VGC_OK)
        rc = launch_header_scan(pc, flags, groups, segs, n_groups, n_segs, max_group_tiles, hdrs, stmp, hdrs_out, status_out, words_cap, nullptr, stream);
    if (rc != VGC_OK) return rc;
    hipLaunchKernelGGL(k_emit, dim3(blocks), dim3(256), 0, stream, pc, tiles, n_tiles, hdrs, staging,
                       stmp, words_out, words_cap);
    return hip_check(hipGetLastError(), "launch pack kernels");
}

}  // namespace vgc
