// Decode-and-sum half of CommunicateAndUpdate() (Section 4.3): one launch adds one worker's
// message into the dense gradient buffer.  Indices inside a message are distinct, so plain
// read-modify-write is race free and the float32 result does not depend on scheduling; messages
// are ordered by the stream.
#include <type_traits>

#include "vgc_internal.h"

namespace vgc {

__global__ __launch_bounds__(256) void k_unpack_add(PlanCheck pc, const uint32_t* __restrict__ words, uint64_t n_words,
                                                    const vgc_group_hdr* __restrict__ hdrs,
                                                    const PlanGroup* __restrict__ groups, uint32_t n_groups,
                                                    float scale, float* __restrict__ dense) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (!plan_ok(pc)) return;
    const vgc_group_hdr last = hdrs[n_groups - 1];
    uint64_t total = last.word_offset + last.count;
    if (total > n_words) total = n_words;
    if (i >= total) return;
    // the group whose word range holds i: the last one whose first word is at or before i
    uint32_t lo = 0, hi = n_groups - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (hdrs[mid].word_offset <= i) lo = mid; else hi = mid - 1;
    }
    const vgc_group_hdr h = hdrs[lo];
    const PlanGroup pg = groups[lo];
    const uint32_t w = __builtin_nontemporal_load(words + i);
    const uint32_t idx = w & 0x0FFFFFFFu;
    const uint32_t d = (w >> 28) & 7u;
    // a well-formed message never trips these; a damaged one is skipped rather than written out of range
    if (idx >= pg.size || h.exp_field <= d || h.exp_field > 254u || i >= h.word_offset + h.count) return;
    const float val = __uint_as_float(((h.exp_field - d) << 23) | (w & 0x80000000u));
    const float contrib = scale * val;
    float* p = dense + pg.offset + idx;
    *p = *p + contrib;
}

int launch_unpack_add(PlanCheck pc, const uint32_t* words, uint64_t n_words, const vgc_group_hdr* hdrs,
                      const PlanGroup* groups, uint32_t n_groups, float scale, float* dense,
                      hipStream_t stream) {
    if (n_words == 0) return VGC_OK;
    const uint64_t blocks = (n_words + 255) / 256;
    if (blocks > 0x7FFFFFFFull) {
        set_error("vgc_unpack_add: %llu words exceed the launch limit", (unsigned long long)n_words);
        return VGC_ERR_SIZE;
    }
    hipLaunchKernelGGL(k_unpack_add, dim3((uint32_t)blocks), dim3(256), 0, stream, pc, words, n_words, hdrs, groups,
                       n_groups, scale, dense);
    return hip_check(hipGetLastError(), "launch k_unpack_add");
}

}  // namespace vgc

// ------------------------------------------------------------------------------------------------
// Several messages in one pass over the dense buffer.  When the messages together touch most cache
// lines of the dense buffer (the synthetic workloads send 20-35 % of all elements per worker), one
// launch per message re-reads and re-writes the whole buffer p times.  Here one wave owns a run of
// consecutive tiles of one group: it keeps the current tile (2048 floats) in LDS, and for every
// message, in message order, streams that message's words of the tile from a cursor and adds them.
// The float32 additions an element receives are the same, in the same order, as p single-message
// launches would perform, so the result is bit-identical.
//
// Bound by memory: the words once, the buffer (or the optimizer's arrays) once or twice.  What kept it from there was the
// search for the cursors, each message's words being asked for only when the one before was done, and words asked for
// past a tile's end that a non-temporal load did not leave in the cache.  Before and after: 10^9 elements, 8 messages of
// 17 % overwriting, 2388 -> 1888 us (5.0 TB/s); of 0.2 % over 3 x 10^8, 473 -> 225 us; 25.6 M elements with Adam,
// 220 -> 163 us; 138 M with momentum SGD and sparse messages, 433 -> 387 us (5.8 TB/s).  The words are read 1.33 (33 %
// sent) to 1.60 times (19 %): 1.17 to 1.37 times with an eighth of the waves, so the rest are the cursors' searches.
// ------------------------------------------------------------------------------------------------
namespace vgc {


template <int kMax>
struct BatchArgs {
    const uint32_t* words[kMax];
    const vgc_group_hdr* hdrs[kMax];
    uint64_t n_words[kMax];
    uint32_t p;
};

// What happens to a tile once every message has been added into it.
//   kToDense       it is the tile of the dense gradient buffer: written back.
//   kMomentumSgd   it is the decoded gradient ghat (elements nobody sent are zero, Section 4.1):
//                  m <- mu m - lr ghat;  w <- w + m.
//   kAdam          m <- b1 m + (1 - b1) ghat;  v <- b2 v + (1 - b2) ghat^2;
//                  w <- w - lr (m / bias1) / (sqrt(v / bias2) + eps),  bias_i = 1 - b_i^t.
// One float32 rounding per operation, in the order written (no contraction).
enum { kToDense = 0, kMomentumSgd = 1, kAdam = 2 };

struct UpdateArgs {
    float* w;
    float* s1;
    float* s2;
    float lr, mu, b1, b2, omb1, omb2, bias1, bias2, eps;
};

template <int kMode>
__device__ __forceinline__ void update_element(const UpdateArgs& O, float ghat, float& w, float& s1, float& s2) {
    if (kMode == kMomentumSgd) {
        const float t1 = O.mu * s1;
        const float t2 = O.lr * ghat;
        s1 = t1 - t2;
        w = w + s1;
    } else {
        const float a = O.b1 * s1, b = O.omb1 * ghat;
        s1 = a + b;
        const float g2 = ghat * ghat;
        const float c = O.b2 * s2, d = O.omb2 * g2;
        s2 = c + d;
        const float mhat = s1 / O.bias1;
        const float vhat = s2 / O.bias2;
        const float denom = sqrtf(vhat) + O.eps;
        const float step = (O.lr * mhat) / denom;
        w = w - step;
    }
}

typedef float f4u __attribute__((ext_vector_type(4)));

// Whether the group's elements begin at a multiple of 16 bytes in every array that is read or written.
template <int kMode>
__device__ __forceinline__ bool whole_group(const float* dense, const UpdateArgs& O, const PlanGroup& pg) {
    auto at = [&](const float* p) { return (reinterpret_cast<uintptr_t>(p + pg.offset) & 15u) == 0; };
    return kMode == kToDense ? at(dense) : at(O.w) && at(O.s1) && (kMode != kAdam || at(O.s2));
}

// The first words of one message's tile, on their way: `n` of them, 64 to a round.
template <int kFirst>
struct Request {
    uint32_t word[kFirst];
    uint32_t n;
};

// What a lane keeps of its message (lane w: message w): where the words not yet added begin, how many are left of the
// group's segment, the segment's exponent field, and how many rounds the first request of a tile has.
struct Cursor {
    uint64_t at;
    uint32_t left, exp_field, rounds;
};

__device__ __forceinline__ uint32_t lane_of(uint32_t x, uint32_t w) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)w);
}

// Requests min(left, rounds x 64) words of message w.  The range of the buffer resource ends with the last of them: the
// rounds behind it are answered without memory traffic, and there is no branch, so that the wait for one message's words
// can be counted past the next message's.  A round's place is part of the vector offset and there the instruction's own
// (at most 2816 bytes): the scalar offset is not held against the range.
template <int kFirst>
__device__ __forceinline__ void request_words(Request<kFirst>& Q, const Cursor& C, uint32_t w, uint32_t lane) {
    const uint64_t at = (uint64_t)lane_of((uint32_t)C.at, w) | (uint64_t)lane_of((uint32_t)(C.at >> 32), w) << 32;
    Q.n = min(lane_of(C.left, w), lane_of(C.rounds, w) * 64u);
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(at), 0, (int)(Q.n * 4u), 0x00020000);
    uint32_t at_lane = lane * 4u;
    asm volatile("" : "+v"(at_lane));                        // or each sum is kept in a register of its own through the loops
#pragma unroll
    for (int j = 0; j < kFirst; ++j)
        Q.word[j] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)at_lane + j * 256, 0, 0);
}

// Adds kRounds x 64 words (the first n of them exist) into the tile; returns how many belong to it.  A message's indices
// are distinct, so the tile's elements are read together and written together.
template <int kRounds>
__device__ __forceinline__ uint32_t add_rounds(const uint32_t* word, uint32_t n, uint32_t start, uint32_t m, uint32_t ef,
                                               float scale, float* T, uint32_t lane) {
    float old[kRounds];
    uint32_t used = 0;
#pragma unroll
    for (int j = 0; j < kRounds; ++j) old[j] = T[min((word[j] & 0x0FFFFFFFu) - start, kTile - 1u)];
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const uint32_t idx = word[j] & 0x0FFFFFFFu;
        const uint32_t d = (word[j] >> 28) & 7u;
        const bool in_tile = ((uint32_t)j * 64u + lane < n) && (idx < start + m);
        // a well-formed message has idx >= start here and exp_field > d; anything else is skipped
        if (in_tile && idx >= start && ef > d && ef <= 254u) {
            const float val = __uint_as_float(((ef - d) << 23) | (word[j] & 0x80000000u));
            const float contrib = scale * val;
            T[idx - start] = old[j] + contrib;
        }
        used += (uint32_t)__popcll(__ballot(in_tile));
    }
    return used;
}

// Adds message w's words of the tile: those of its first request, and while the tile holds more, further requests.
template <int kFirst>
__device__ __forceinline__ void add_message(const Request<kFirst>& Q, Cursor& C, uint32_t w, uint32_t start, uint32_t m,
                                            float scale, float* T, uint32_t lane) {
    constexpr int kGroup = kFirst < 4 ? kFirst : 4;
    if (Q.n == 0) return;
    const uint32_t ef = lane_of(C.exp_field, w);
    uint32_t used = 0;
#pragma unroll
    for (int j = 0; j < kFirst; j += kGroup)
        if ((uint32_t)j * 64u < Q.n) used += add_rounds<kGroup>(Q.word + j, Q.n - (uint32_t)j * 64u, start, m, ef, scale, T, lane);
    uint32_t left = lane_of(C.left, w) - used;
    uint64_t at = ((uint64_t)lane_of((uint32_t)C.at, w) | (uint64_t)lane_of((uint32_t)(C.at >> 32), w) << 32) + 4ull * used;
    bool more = used == Q.n && left != 0;
    while (more) {
        constexpr int kRounds = 4;
        const uint32_t n = min(left, (uint32_t)kRounds * 64u);
        uint32_t word[kRounds];
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const uint32_t i = (uint32_t)j * 64u + lane;
            word[j] = i < n ? reinterpret_cast<const uint32_t*>(at)[i] : 0u;
        }
        used = add_rounds<kRounds>(word, n, start, m, ef, scale, T, lane);
        left -= used;
        at += 4ull * used;
        more = used == n && left != 0;
    }
    if (lane == w) { C.at = at; C.left = left; }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The tiles [t0, t1) of one wave.  While a message is added, the next one's words (after the last message: the next
// tile's first) are on their way; an odd number of messages is made even with one that has no words.
// kWhole: the group's first element lies at a multiple of 16 bytes in every array, and so do its whole tiles.
template <int kFirst, int kMode, bool kWhole>
__device__ __forceinline__ void decode_tiles(Cursor C, uint32_t p, const PlanGroup& pg, uint32_t t0, uint32_t t1, float scale,
                                             float* __restrict__ dense, int overwrite, const UpdateArgs& O, float* T, uint32_t lane) {
    const uint32_t pe = p < 2 ? 2u : (p + 1u) & ~1u;
    C.rounds = min(C.rounds, (uint32_t)kFirst);
    Request<kFirst> QA, QB;
    request_words(QA, C, 0, lane);
    for (uint32_t t = t0; t < t1; ++t) {
        const uint32_t start = t * kTile;
        const uint32_t m = min(kTile, pg.size - start);
        const uint64_t e0 = pg.offset + start;
        float* base = (kMode == kToDense) ? dense + e0 : O.w + e0;
        const bool vec = m == kTile;
        // ---- tile -> LDS ----
        if (overwrite || kMode != kToDense) {
#pragma unroll
            for (int q = 0; q < 8; ++q) reinterpret_cast<f4u*>(T)[q * 64 + lane] = (f4u){0.f, 0.f, 0.f, 0.f};
        } else if (vec) {
            f4u x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = load_four<kWhole>(base + 4 * (q * 64 + lane));
#pragma unroll
            for (int q = 0; q < 8; ++q) reinterpret_cast<f4u*>(T)[q * 64 + lane] = x[q];
        } else {
            for (uint32_t i = lane; i < kTile; i += 64) T[i] = (i < m) ? base[i] : 0.f;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        request_words(QB, C, 1, lane);
        // the optimizer's arrays are requested now and arrive while the messages are decoded
        f4u W4[kMode == kToDense ? 1 : 8], S1[kMode == kToDense ? 1 : 8], S2[kMode == kAdam ? 8 : 1];
        if (kMode != kToDense && vec) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                W4[q] = load_four<kWhole>(O.w + e0 + 4 * (q * 64 + lane));
                S1[q] = load_four<kWhole>(O.s1 + e0 + 4 * (q * 64 + lane));
                if (kMode == kAdam) S2[q] = load_four<kWhole>(O.s2 + e0 + 4 * (q * 64 + lane));
            }
        }

        // ---- messages in order ----
        add_message(QA, C, 0, start, m, scale, T, lane);
        for (uint32_t w = 1; w + 1 < pe; w += 2) {
            request_words(QA, C, w + 1, lane);
            add_message(QB, C, w, start, m, scale, T, lane);
            request_words(QB, C, w + 2, lane);
            add_message(QA, C, w + 1, start, m, scale, T, lane);
        }
        request_words(QA, C, 0, lane);                       // the next tile's (behind the last one: not used)
        add_message(QB, C, pe - 1, start, m, scale, T, lane);

        // ---- LDS -> tile ----
        if (kMode == kToDense) {
            if (vec) {
#pragma unroll
                for (int q = 0; q < 8; ++q) store_four<kWhole>(reinterpret_cast<f4u*>(T)[q * 64 + lane], base + 4 * (q * 64 + lane));
            } else {
                for (uint32_t i = lane; i < m; i += 64) base[i] = T[i];
            }
        } else if (vec) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const f4u G = reinterpret_cast<f4u*>(T)[q * 64 + lane];
                f4u w4 = W4[q], a4 = S1[q], b4 = S2[kMode == kAdam ? q : 0];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float w = w4[c], a = a4[c], b = b4[c];
                    update_element<kMode>(O, G[c], w, a, b);
                    w4[c] = w; a4[c] = a; b4[c] = b;
                }
                store_four<kWhole>(w4, O.w + e0 + 4 * (q * 64 + lane));
                store_four<kWhole>(a4, O.s1 + e0 + 4 * (q * 64 + lane));
                if (kMode == kAdam) store_four<kWhole>(b4, O.s2 + e0 + 4 * (q * 64 + lane));
            }
        } else {
            for (uint32_t i = lane; i < m; i += 64) {
                float w = O.w[e0 + i], a = O.s1[e0 + i], b = (kMode == kAdam) ? O.s2[e0 + i] : 0.f;
                update_element<kMode>(O, T[i], w, a, b);
                O.w[e0 + i] = w;
                O.s1[e0 + i] = a;
                if (kMode == kAdam) O.s2[e0 + i] = b;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int kMax, int kMode>
__global__ __launch_bounds__(256) void k_unpack_add_batch(PlanCheck pc, BatchArgs<kMax> A, const PlanGroup* __restrict__ groups,
                                                          const PlanRun* __restrict__ runs, uint32_t n_runs,
                                                          float scale, float* __restrict__ dense, int overwrite,
                                                          UpdateArgs O, uint32_t tiles_per_wave) {
    __shared__ __attribute__((aligned(16))) float sh_tile[4][kTile];
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // a run of kRunTiles tiles is shared by kRunTiles / tiles_per_wave waves (small parameter sets have few runs)
    const uint32_t per_run = (uint32_t)kRunTiles / tiles_per_wave;
    // Workgroups are dealt round the eight L2 caches.  Of every 128 consecutive ones each cache gets 16 that lie next to
    // each other, so that the words a wave requests past its last tile are in the cache that wants them next (one tile a
    // wave, 25.6 M elements, 8 messages of 5 %: 51.3 -> 45.2 us; with eight tiles a wave it makes no difference).
    const uint32_t in_block = blockIdx.x & 127u, block0 = blockIdx.x - in_block;
    const uint32_t block = block0 + 128u <= gridDim.x ? block0 + (in_block & 7u) * 16u + (in_block >> 3) : blockIdx.x;
    const uint32_t gw = block * 4 + wave;
    const uint32_t run = gw / per_run;
    if (run >= n_runs || !plan_ok(pc)) return;
    float* T = sh_tile[wave];
    const uint32_t k = runs[run].group;
    const PlanGroup pg = groups[k];
    const uint32_t nt_group = (pg.size + kTile - 1) / kTile;
    const uint32_t run_end = min(runs[run].first_tile + (uint32_t)kRunTiles, nt_group);
    const uint32_t t0 = runs[run].first_tile + (gw % per_run) * tiles_per_wave;   // first tile of this wave, counted inside the group
    if (t0 >= run_end) return;
    const uint32_t t1 = min(t0 + tiles_per_wave, run_end);

    Cursor C = {0, 0, 0, 0};
    if (lane < A.p) {
        const vgc_group_hdr h = A.hdrs[lane][k];
        // first request of a tile: the mean of a tile's count plus 3 standard deviations if the sent elements were
        // spread evenly.  Words requested past the tile's end are requested again with the next tile.
        const float mu = (float)h.count * ((float)kTile / (float)pg.size);
        C.rounds = (uint32_t)fminf((mu + 3.0f * sqrtf(mu)) * (1.0f / 64.0f), 32.0f) + 1u;
        uint64_t lo = h.word_offset, hi = h.word_offset + h.count;
        if (hi > A.n_words[lane]) hi = A.n_words[lane];
        if (lo > hi) lo = hi;
        C.at = reinterpret_cast<uint64_t>(A.words[lane]) + 4ull * lo;
        C.left = (uint32_t)min(hi - lo, (uint64_t)0xFFFFFFFFu);
        C.exp_field = h.exp_field;
    }
    if (t0 != 0) {
        // every cursor to its message's first word with an index at or behind the wave's first element.  64 / p lanes (a
        // power of two) look for one cursor, each of them at another word: 8 messages of 2^19 words take 7 dependent loads
        // where one lane a message took 19, and with one tile a wave (small parameter sets) they are what the wave waits for.
        uint32_t lg = 6;
        while (lg > 0 && (64u >> lg) < A.p) --lg;
        const uint32_t w = lane >> lg, sub = lane & ((1u << lg) - 1u);
        const uint32_t first = t0 * kTile;
        const uint64_t at = (uint64_t)(uint32_t)__shfl((int)(uint32_t)C.at, (int)w) |
                            (uint64_t)(uint32_t)__shfl((int)(uint32_t)(C.at >> 32), (int)w) << 32;
        uint32_t lo = 0, hi = (uint32_t)__shfl((int)C.left, (int)w);
        const uint32_t* W = reinterpret_cast<const uint32_t*>(at);
        while (__ballot(lo < hi)) {
            const uint64_t n = lo < hi ? hi - lo : 0;
            const bool less = n != 0 && (W[lo + (uint32_t)((n * (2u * sub + 1u)) >> (lg + 1u))] & 0x0FFFFFFFu) < first;
            const uint64_t mine = (__ballot(less) >> (w << lg)) & (~0ull >> (64u - (1u << lg)));
            const uint32_t c = (uint32_t)__popcll(mine);     // so many of the lanes' words lie before the wave's elements
            if (n != 0) {
                const uint32_t below = lo + (uint32_t)((n * (2u * c - 1u)) >> (lg + 1u)) + 1u;
                const uint32_t above = lo + (uint32_t)((n * (2u * c + 1u)) >> (lg + 1u));
                if (c != (1u << lg)) hi = above;
                if (c != 0) lo = min(below, hi);             // (a damaged message may answer in no order)
            }
        }
        const uint32_t skip = (uint32_t)__shfl((int)lo, (int)((lane << lg) & 63u));
        if (lane < A.p) { C.at += 4ull * skip; C.left -= skip; }
    }

    // The rounds of a first request follow from the densest message: one that is not needed still costs an issue slot, one
    // that is missing is waited for.  The 12 are for densities from a fifth on (138 M elements, 3 messages of 30 % added:
    // 300 us, 326 with 8); next to the optimizer's arrays they cost a wave per SIMD.
    auto decode = [&](auto W) {
        constexpr bool kWhole = decltype(W)::value;
        if (__ballot(C.rounds > 2) == 0) decode_tiles<2, kMode, kWhole>(C, A.p, pg, t0, t1, scale, dense, overwrite, O, T, lane);
        else if (kMode == kToDense && __ballot(C.rounds > 8) != 0)
            decode_tiles<kMode == kToDense ? 12 : 8, kMode, kWhole>(C, A.p, pg, t0, t1, scale, dense, overwrite, O, T, lane);
        else decode_tiles<8, kMode, kWhole>(C, A.p, pg, t0, t1, scale, dense, overwrite, O, T, lane);
    };
    if (whole_group<kMode>(dense, O, pg)) decode(std::true_type{});
    else decode(std::false_type{});
}

// ------------------------------------------------------------------------------------------------
// The same for parameter sets too small to give every unit of the chip several waves of a tile each: a workgroup per tile.
// One wave a tile is then bound by a chain: cursors (six dependent loads), then every message's words asked for while the one
// before it is added.  Here the four waves look for a quarter of the messages' cursors each, with four times the lanes a
// message, the words of eight messages are requested at once, 256 a round, and a barrier keeps the messages' order.
// 1.8 M elements, 8 messages of 17 %, momentum SGD: 26.6 -> 18.2 us from a cold cache, Adam 37.8 -> 26.4; 16 messages of 30 %
// 54.6 -> 33.2; 20,000 elements 28.8 -> 14.3.
// ------------------------------------------------------------------------------------------------
template <int kRounds, int kMode, bool kWhole>
__device__ __forceinline__ void decode_tile(uint32_t p, const uint64_t* cur_at, const uint32_t* cur_left, const uint32_t* cur_exp, uint32_t* more,
                                            const PlanGroup& pg, uint32_t start, float scale, float* __restrict__ dense, int overwrite,
                                            const UpdateArgs& O, float* T, uint32_t tid) {
    const uint32_t m = min(kTile, pg.size - start);
    const uint64_t e0 = pg.offset + start;
    float* base = (kMode == kToDense) ? dense + e0 : O.w + e0;
    const bool vec = m == kTile;
    const bool fresh = overwrite || kMode != kToDense;
    // a thread's elements: two groups of four (vec), else eight, 256 apart
    f4u W4[2], S1[2], S2[2];
    uint32_t word[8][kRounds];
    auto request = [&](uint32_t w, uint32_t first, uint32_t* x) -> uint32_t {      // words first .. of message w; how many there are
        const uint32_t left = w < p ? cur_left[w] : 0u, n = left > first ? min(left - first, (uint32_t)kRounds * 256u) : 0u;
        const uint64_t at = w < p ? cur_at[w] + 4ull * first : 0ull;
        const uint32_t n_u = __builtin_amdgcn_readfirstlane(n);
        const uint32_t at_lo = __builtin_amdgcn_readfirstlane((uint32_t)at), at_hi = __builtin_amdgcn_readfirstlane((uint32_t)(at >> 32));   // (it returns an int)
        const uint64_t at_u = (uint64_t)at_lo | (uint64_t)at_hi << 32;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(at_u), 0, (int)(n_u * 4u), 0x00020000);
#pragma unroll
        for (int j = 0; j < kRounds; ++j) x[j] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)(tid * 4u) + j * 1024, 0, 0);
        return n_u;
    };
    auto add = [&](const uint32_t* x, uint32_t n, uint32_t w) {
        const uint32_t ef = __builtin_amdgcn_readfirstlane(cur_exp[w]);
        float old[kRounds];
#pragma unroll
        for (int j = 0; j < kRounds; ++j) old[j] = T[min((x[j] & 0x0FFFFFFFu) - start, kTile - 1u)];
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const uint32_t i = (uint32_t)j * 256u + tid, idx = x[j] & 0x0FFFFFFFu, d = (x[j] >> 28) & 7u;
            const bool in_tile = i < n && idx < start + m;
            // a well-formed message has idx >= start here and exp_field > d; anything else is skipped
            if (in_tile && idx >= start && ef > d && ef <= 254u) {
                const float val = __uint_as_float(((ef - d) << 23) | (x[j] & 0x80000000u));
                const float contrib = scale * val;
                T[idx - start] = old[j] + contrib;
            }
            if (in_tile && i == (uint32_t)kRounds * 256u - 1u) more[w] += 1u;      // the last of those requested: there may be others
        }
    };
    for (uint32_t w0 = 0; w0 == 0 || w0 < p; w0 += 8) {
        uint32_t n[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) n[u] = request(w0 + u, 0, word[u]);
        if (w0 == 0) {
            // the tile and the optimizer's arrays: behind the words, and used when those have been added
            if (vec) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (kMode != kToDense || !fresh) W4[q] = load_four<kWhole>(base + 4 * (q * 256 + tid));
                    if (kMode != kToDense) S1[q] = load_four<kWhole>(O.s1 + e0 + 4 * (q * 256 + tid));
                    if (kMode == kAdam) S2[q] = load_four<kWhole>(O.s2 + e0 + 4 * (q * 256 + tid));
                }
            }
            if (!fresh) {
                if (vec) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) reinterpret_cast<f4u*>(T)[q * 256 + tid] = W4[q];
                } else {
                    for (uint32_t i = tid; i < kTile; i += 256) T[i] = (i < m) ? base[i] : 0.f;
                }
                __syncthreads();
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            if (w0 + u >= p) break;
            if (n[u] == 0) continue;
            add(word[u], n[u], w0 + u);
            __syncthreads();
            if (n[u] == (uint32_t)kRounds * 256u) {
                uint32_t rounds = 1;
                while (more[w0 + u] == rounds) {
                    uint32_t x[kRounds];
                    const uint32_t k = request(w0 + u, rounds * (uint32_t)kRounds * 256u, x);
                    __syncthreads();                                 // (all have read the count)
                    if (k == 0) break;
                    add(x, k, w0 + u);
                    __syncthreads();
                    ++rounds;
                }
            }
        }
    }
    if (vec) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f4u G = reinterpret_cast<f4u*>(T)[q * 256 + tid];
            if (kMode == kToDense) {
                store_four<kWhole>(G, base + 4 * (q * 256 + tid));
                continue;
            }
            f4u w4 = W4[q], a4 = S1[q], b4 = S2[q];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float w = w4[c], a = a4[c], b = kMode == kAdam ? b4[c] : 0.f;
                update_element<kMode>(O, G[c], w, a, b);
                w4[c] = w; a4[c] = a; b4[c] = b;
            }
            store_four<kWhole>(w4, O.w + e0 + 4 * (q * 256 + tid));
            store_four<kWhole>(a4, O.s1 + e0 + 4 * (q * 256 + tid));
            if (kMode == kAdam) store_four<kWhole>(b4, O.s2 + e0 + 4 * (q * 256 + tid));
        }
        return;
    }
    for (uint32_t i = tid; i < m; i += 256) {
        if (kMode == kToDense) {
            base[i] = T[i];
            continue;
        }
        float w = O.w[e0 + i], a = O.s1[e0 + i], b = (kMode == kAdam) ? O.s2[e0 + i] : 0.f;
        update_element<kMode>(O, T[i], w, a, b);
        O.w[e0 + i] = w;
        O.s1[e0 + i] = a;
        if (kMode == kAdam) O.s2[e0 + i] = b;
    }
}

template <int kMax, int kMode>
__global__ __launch_bounds__(256) void k_unpack_tile(PlanCheck pc, BatchArgs<kMax> A, const PlanGroup* __restrict__ groups,
                                                     const PlanTile* __restrict__ tiles, uint32_t n_tiles, float scale,
                                                     float* __restrict__ dense, int overwrite, UpdateArgs O) {
    __shared__ __attribute__((aligned(16))) float T[kTile];
    __shared__ uint64_t cur_at[kMax];
    __shared__ uint32_t cur_left[kMax], cur_exp[kMax], more[kMax], rounds_of[4];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (neighbours share an L2, as above)
    const uint32_t in_block = blockIdx.x & 127u, block0 = blockIdx.x - in_block;
    const uint32_t t = block0 + 128u <= gridDim.x ? block0 + (in_block & 7u) * 16u + (in_block >> 3) : blockIdx.x;
    if (t >= n_tiles || !plan_ok(pc)) return;
    const PlanTile pt = tiles[t];
    const PlanGroup pg = groups[pt.group];
    const uint32_t first = pt.start;

    // The cursors: wave v finds those of messages v, v + 4, .., with 64 >> lg lanes for each (a power of two).
    const uint32_t mine_p = (A.p + 3u - wave) / 4u;                  // messages of the wave
    uint32_t lg = 6;
    while (lg > 0 && (64u >> lg) < mine_p) --lg;
    const uint32_t w = wave + 4u * (lane >> lg), sub = lane & ((1u << lg) - 1u);
    uint32_t rounds = 0;
    if (mine_p) {
        uint64_t at = 0;
        uint32_t left = 0, ef = 0;
        if (w < A.p) {
            const vgc_group_hdr h = A.hdrs[w][pt.group];
            const float mu = (float)h.count * ((float)kTile / (float)pg.size);
            rounds = (uint32_t)fminf((mu + 3.0f * sqrtf(mu)) * (1.0f / 256.0f), 8.0f) + 1u;
            uint64_t lo = h.word_offset, hi = h.word_offset + h.count;
            if (hi > A.n_words[w]) hi = A.n_words[w];
            if (lo > hi) lo = hi;
            at = reinterpret_cast<uint64_t>(A.words[w]) + 4ull * lo;
            left = (uint32_t)min(hi - lo, (uint64_t)0xFFFFFFFFu);
            ef = h.exp_field;
        }
        uint32_t lo = 0, hi = first != 0 ? left : 0u;
        const uint32_t* W = reinterpret_cast<const uint32_t*>(at);
        while (__ballot(lo < hi)) {
            const uint64_t n = lo < hi ? hi - lo : 0;
            const bool less = n != 0 && (W[lo + (uint32_t)((n * (2u * sub + 1u)) >> (lg + 1u))] & 0x0FFFFFFFu) < first;
            const uint64_t of_message = (__ballot(less) >> ((lane >> lg) << lg)) & (~0ull >> (64u - (1u << lg)));
            const uint32_t c = (uint32_t)__popcll(of_message);
            if (n != 0) {
                const uint32_t below = lo + (uint32_t)((n * (2u * c - 1u)) >> (lg + 1u)) + 1u;
                const uint32_t above = lo + (uint32_t)((n * (2u * c + 1u)) >> (lg + 1u));
                if (c != (1u << lg)) hi = above;
                if (c != 0) lo = min(below, hi);                     // (a damaged message may answer in no order)
            }
        }
        if (w < A.p && sub == 0) {
            cur_at[w] = at + 4ull * lo;
            cur_left[w] = left - lo;
            cur_exp[w] = ef;
            more[w] = 0;
        }
    }
    const uint32_t rounds_w = __ballot(rounds > 2) ? 4u : __ballot(rounds > 1) ? 2u : 1u;
    if (lane == 0) rounds_of[wave] = rounds_w;
    if (overwrite || kMode != kToDense) {
#pragma unroll
        for (int q = 0; q < 2; ++q) reinterpret_cast<f4u*>(T)[q * 256 + tid] = (f4u){0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    const uint32_t most = __builtin_amdgcn_readfirstlane(max(max(rounds_of[0], rounds_of[1]), max(rounds_of[2], rounds_of[3])));
    auto decode = [&](auto W) {
        constexpr bool kWhole = decltype(W)::value;
        if (most == 1) decode_tile<1, kMode, kWhole>(A.p, cur_at, cur_left, cur_exp, more, pg, first, scale, dense, overwrite, O, T, tid);
        else if (most == 2) decode_tile<2, kMode, kWhole>(A.p, cur_at, cur_left, cur_exp, more, pg, first, scale, dense, overwrite, O, T, tid);
        else decode_tile<4, kMode, kWhole>(A.p, cur_at, cur_left, cur_exp, more, pg, first, scale, dense, overwrite, O, T, tid);
    };
    if (whole_group<kMode>(dense, O, pg)) decode(std::true_type{});
    else decode(std::false_type{});
}

// Waves to aim for: 5120 are resident, and the last ones to be placed leave the others idle.  64 K of them against 16 K:
// 10^9 elements, 8 messages of 17 %, 1.87 against 2.05 ms; 138 M elements, sparse messages with momentum SGD, 384 against
// 423 us, although each wave's search reads 12 to 16 KB.  With 256 K that costs more: 2.36 ms and 386 us.
constexpr uint64_t kWaves = 65536;

// Up to so many tiles a workgroup takes each: as many workgroups as are resident at once (five per compute unit).  2.5 M elements
// (1221 tiles), 8 messages of 17 %: 22.7 -> 20.2 us overwriting, 38.0 -> 28.2 with Adam; 3 M (1465) 23.8 -> 28.2 and 45.0 -> 35.0;
// 4 M 24.9 -> 30.4 and 39.0 -> 38.9; beyond, the search for the cursors of every tile costs what it gives or more.
// Where every group is whole tiles (and the update is not Adam) waves have no last tile that they do element by element, the one
// all others wait for, and the line comes earlier unless there are many words to a tile.  By tile / by waves, us, buffers in the
// cache, 16 messages of 3 % added: 512 tiles 16.5 / 16.7, 768 19.5 / 17.3, 1024 21.9 / 18.1, but 1026 and a ragged one 22.1 / 27.1;
// 8 messages of 17 %, 1024 tiles, 12.8 / 14.5; momentum SGD, 16 of 3 %: 12.6 / 13.1, 14.2 / 13.7, 16.0 / 14.6, 15.9 / 18.2.
constexpr uint64_t kFewTiles = 1280, kFewWholeTiles = 512;
static bool few_tiles(uint64_t n_tiles, bool whole_tiles, const uint64_t* n_words, uint32_t p) {
    if (!whole_tiles || n_tiles <= kFewWholeTiles) return n_tiles <= kFewTiles;
    const uint64_t n = n_tiles * kTile;
    uint64_t total = 0;
    for (uint32_t w = 0; w < p; ++w) total += n_words[w] < n ? n_words[w] : n;
    return n_tiles <= kFewTiles && total >= n && total >= p * (n / 8);
}

template <int kMax>
static BatchArgs<kMax> batch_args(const uint32_t* const* words, const uint64_t* n_words, const vgc_group_hdr* const* hdrs,
                                  uint32_t first, uint32_t p) {
    BatchArgs<kMax> A;
    A.p = p - first < (uint32_t)kMax ? p - first : (uint32_t)kMax;
    for (uint32_t w = 0; w < (uint32_t)kMax; ++w) {
        const bool on = w < A.p;
        A.words[w] = on ? words[first + w] : nullptr;
        A.hdrs[w] = on ? hdrs[first + w] : nullptr;
        A.n_words[w] = on ? n_words[first + w] : 0;
    }
    return A;
}

int launch_unpack_add_batch(PlanCheck pc, const uint32_t* const* words, const uint64_t* n_words, const vgc_group_hdr* const* hdrs,
                            uint32_t p, const PlanGroup* groups, const PlanTile* tiles, const PlanRun* runs, uint64_t n_tiles, uint64_t n_runs,
                            bool whole_tiles, float scale, int overwrite, float* dense, uint32_t tiles_per_wave, hipStream_t stream) {
    const bool by_tile = tiles_per_wave == 0 && few_tiles(n_tiles, whole_tiles, n_words, p);
    const uint32_t tpw = decode_tiles_per_wave(n_runs, kWaves, tiles_per_wave);
    const uint32_t blocks = (uint32_t)((n_runs * (kRunTiles / tpw) + 3) / 4);
    const uint32_t chunks = p ? (p + kBatchMax - 1) / kBatchMax : 1;     // p == 0: only the optional clear
    for (uint32_t ch = 0; ch < chunks; ++ch) {
        const BatchArgs<kBatchMax> A = batch_args<kBatchMax>(words, n_words, hdrs, ch * kBatchMax, p);
        if (by_tile) {
            hipLaunchKernelGGL((k_unpack_tile<kBatchMax, kToDense>), dim3((uint32_t)n_tiles), dim3(256), 0, stream, pc, A, groups, tiles,
                               (uint32_t)n_tiles, scale, dense, (overwrite && ch == 0) ? 1 : 0, UpdateArgs{});
            continue;
        }
        hipLaunchKernelGGL((k_unpack_add_batch<kBatchMax, kToDense>), dim3(blocks), dim3(256), 0, stream, pc, A, groups, runs,
                           (uint32_t)n_runs, scale, dense, (overwrite && ch == 0) ? 1 : 0, UpdateArgs{}, tpw);
    }
    return hip_check(hipGetLastError(), "launch k_unpack_add_batch");
}

int launch_unpack_apply(PlanCheck pc, const uint32_t* const* words, const uint64_t* n_words, const vgc_group_hdr* const* hdrs,
                        uint32_t p, const PlanGroup* groups, const PlanTile* tiles, const PlanRun* runs, uint64_t n_tiles, uint64_t n_runs, bool whole_tiles,
                        float scale, int kind, float lr, float mu, float b1, float b2, float omb1, float omb2, float bias1, float bias2,
                        float eps, float* param, float* state1, float* state2, uint32_t tiles_per_wave, hipStream_t stream) {
    const uint32_t tpw = decode_tiles_per_wave(n_runs, kWaves, tiles_per_wave);
    const uint32_t blocks = (uint32_t)((n_runs * (kRunTiles / tpw) + 3) / 4);
    const BatchArgs<kApplyMax> A = batch_args<kApplyMax>(words, n_words, hdrs, 0, p);
    UpdateArgs O;
    O.w = param; O.s1 = state1; O.s2 = state2;
    O.lr = lr; O.mu = mu; O.b1 = b1; O.b2 = b2; O.omb1 = omb1; O.omb2 = omb2; O.bias1 = bias1; O.bias2 = bias2; O.eps = eps;
    if (tiles_per_wave == 0 && few_tiles(n_tiles, whole_tiles && kind != VGC_OPT_ADAM, n_words, p)) {
        if (kind == VGC_OPT_ADAM)
            hipLaunchKernelGGL((k_unpack_tile<kApplyMax, kAdam>), dim3((uint32_t)n_tiles), dim3(256), 0, stream, pc, A, groups, tiles,
                               (uint32_t)n_tiles, scale, static_cast<float*>(nullptr), 1, O);
        else
            hipLaunchKernelGGL((k_unpack_tile<kApplyMax, kMomentumSgd>), dim3((uint32_t)n_tiles), dim3(256), 0, stream, pc, A, groups, tiles,
                               (uint32_t)n_tiles, scale, static_cast<float*>(nullptr), 1, O);
        return hip_check(hipGetLastError(), "launch k_unpack_tile (update)");
    }
    if (kind == VGC_OPT_ADAM)
        hipLaunchKernelGGL((k_unpack_add_batch<kApplyMax, kAdam>), dim3(blocks), dim3(256), 0, stream, pc, A, groups, runs,
                           (uint32_t)n_runs, scale, static_cast<float*>(nullptr), 1, O, tpw);
    else
        hipLaunchKernelGGL((k_unpack_add_batch<kApplyMax, kMomentumSgd>), dim3(blocks), dim3(256), 0, stream, pc, A, groups, runs,
                           (uint32_t)n_runs, scale, static_cast<float*>(nullptr), 1, O, tpw);
    return hip_check(hipGetLastError(), "launch k_unpack_add_batch (update)");
}

}  // namespace vgc
