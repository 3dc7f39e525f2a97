// The statistic of a fully-connected layer fused into the accumulate / test / reset-or-decay pass of Alg. 1:
// g = c X^T D and s = c^2 (X.X)^T (D.D) (the first two lines of the loop body, Section 5's 2 N |B|
// multiply-adds each) are formed on the matrix cores and consumed in place by the rest of the loop body
// (r += g, v += s, the test of Eq. 2, reset or decay, and the first half of Encode()), so that neither g nor
// s of the layer ever reaches HBM: 16 bytes per parameter (r and v read and written) instead of 32.
//
// A workgroup (8 waves) owns 16 tiles of the select pass, i.e. 16 x 2048 consecutive-per-tile elements of the
// weight [J, C]: 16 rows x 2048 columns when C is a multiple of 2048 (a tile is a piece of a row), 16 R whole
// rows when C = 2048 / R (a tile is R rows).  The K = |B| contraction is short, so the operands are read
// from a pre-transposed copy (K contiguous per row / column: one 16-byte load per MFMA fragment, no LDS) that a
// small kernel prepares.  The columns are the M side of the MFMA and the rows its N side, so that a lane holds four
// consecutive columns of one row; 32 columns of 16 rows at a time are turned through a wave's own LDS so that each access
// to r and v covers whole 128-byte lines, and finished in registers down to 16 bits per element (sign and exponents of
// what is sent).  When all 16 tiles are through, these go to LDS in tile order and each wave encodes two tiles from there.
//
// What bounds it: r and v read and written, 16 bytes per parameter (25088 x 4096: 1.64 GB, 0.28 ms at the 5.9 TB/s of an
// in-place stream), and how far the contraction (0.20 ms alone) and that stream overlap.  Keeping all 16 tiles' g and s in
// accumulators and passing them through LDS into tile order took one workgroup of 131 KB of LDS per compute unit, whose
// waves contracted, streamed and encoded in step: 0.43 ms.  With 70 KB and at most 128 registers two workgroups share a
// compute unit: 0.38 ms.  Loads come back in the order of their request: with r and v requested before the fragments each
// MFMA waited for HBM (0.50 ms).  Kernel and transposes, before -> now, us: the same layer at batch 8, 32, 64, 128 in bf16
// 384 -> 353, 388 -> 350, 457 -> 383, 553 -> 511, in float32 428 -> 355, 508 -> 390, 638 -> 530, 901 -> 813.  The form before
// stays for long batches in bf16 (k_fused_fc_select_long).
#include <type_traits>

#include "vgc_tile_core.h"

namespace vgc {

typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

// [B, W] row-major -> [W, Kp] with the B values of a column contiguous and zeros up to Kp, for X (W = J) and, in the blocks
// from blocks_x on, for D (W = C).  One thread per (column, 16-byte piece of K); neighbouring threads take neighbouring
// columns, so the reads coalesce.
template <typename T>
__global__ __launch_bounds__(256) void k_fc_transpose(const T* __restrict__ X, const T* __restrict__ D, uint32_t B, uint32_t J, uint32_t C,
                                                      uint32_t Kp, uint32_t blocks_x, T* __restrict__ XT, T* __restrict__ DT) {
    constexpr uint32_t kPer = 16 / sizeof(T);
    const bool is_x = blockIdx.x < blocks_x;
    const T* src = is_x ? X : D;
    T* dst = is_x ? XT : DT;
    const uint32_t W = is_x ? J : C;
    const uint64_t idx = (uint64_t)(blockIdx.x - (is_x ? 0u : blocks_x)) * 256 + threadIdx.x;
    const uint32_t pieces = Kp / kPer;
    if (idx >= (uint64_t)W * pieces) return;
    const uint32_t w = (uint32_t)(idx % W), kc = (uint32_t)(idx / W);
    T out[kPer];
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
        const uint32_t k = kc * kPer + i;
        out[i] = k < B ? src[(size_t)k * W + w] : (T)0;
    }
    *reinterpret_cast<u4v*>(dst + (size_t)w * Kp + (size_t)kc * kPer) = *reinterpret_cast<const u4v*>(out);
}

// Squares of packed bf16 values: float32 products, rounded to nearest-even bf16 (2^-9 relative per factor) by the
// hardware's packed conversion.
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t sq_bf16x2(uint32_t w) {
    const float lo = __uint_as_float(w << 16), hi = __uint_as_float(w & 0xFFFF0000u);
    const f2v p = {lo * lo, hi * hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(p, bf2v));
}
__device__ __forceinline__ u4v sq_bf16x8(u4v x) {
    u4v y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = sq_bf16x2(x[e]);
    return y;
}

constexpr int kFusedTiles = 16;                     // tiles per workgroup
constexpr int kCodePitch = kTile + 64;              // codes per tile in LDS: two tiles start 32 banks apart
constexpr int kTurnPitch = 32 + 4;                  // floats per row of a wave's 16 x 32 turning buffer

struct FusedArgs {
    const void* XT;          // [J, Kp]
    const void* DT;          // [C, Kp]
    uint32_t J, C, Kp;
    float cg, cs;
    float* r;                // whole parameter space
    float* v;
    float* g_out;            // optional [J, C] of this layer
    float* s_out;
    uint32_t group;
    float alpha, zeta;
};

// What the encoder has to know of an element, in 16 bits: rounded exponent field (Section 4.4's recipe, 0 .. 256), whether
// rounding raised it, whether the element is sent, its sign.
__device__ __forceinline__ uint32_t element_code(uint32_t bits, bool send) {
    const uint32_t ab = bits & 0x7FFFFFFFu, ernd = (ab + 0x00400000u) >> 23;   // add one at the mantissa's top bit, drop the mantissa
    return (ernd | ((ernd - (ab >> 23)) << 9) | 0x4000u | ((bits >> 16) & 0x8000u)) & (send ? 0xFFFFu : 0u);
}

// The second half of the select pass on one tile, by one wave, from the tile's codes in LDS: send bitmap, largest exponent,
// histogram of the relative codes and the staged entries in index order (which replace the codes).  Chunk u of the tile is
// elements 256 u + 4 lane + c.
__device__ __forceinline__ void encode_codes(uint16_t* codes, TileHdr* __restrict__ hdr, uint32_t* __restrict__ bm,
                                             uint16_t* __restrict__ out, uint32_t lane) {
    uint2 code[8];
    uint32_t etr = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        code[u] = *reinterpret_cast<const uint2*>(codes + u * 256 + 4 * lane);
        uint32_t nib = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t w = ((c < 2 ? code[u].x : code[u].y) >> (16 * (c & 1))) & 0xFFFFu;
            const bool send = (w & 0x4000u) != 0;
            nib |= (send ? 1u : 0u) << c;
            etr = max(etr, send ? (w & 511u) - ((w >> 9) & 1u) : 0u);
        }
        // send bitmap: bit 256 u + 4 lane + c; eight lanes make one word
        const uint32_t x = eight_lanes_or(nib << (4 * (lane & 7u)));
        if ((lane & 7u) == 0) bm[u * 8 + (lane >> 3)] = x;
    }
    etr = wave_max(etr);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // every lane's codes are read before entries replace them
    __builtin_amdgcn_wave_barrier();

    HistPairs hist = {};                                     // of the lane's at most 32 entries
    uint32_t nibbles = 0;                                    // of those of up to three chunks
    uint32_t base = 0;                                       // entries of the chunks before u (uniform)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        uint32_t entry[4], below = 0, total = 0, st = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t w = ((c < 2 ? code[u].x : code[u].y) >> (16 * (c & 1))) & 0xFFFFu;
            const uint32_t ernd = w & 511u, rel = etr + 1u - ernd;              // >= 0 for sent elements
            const bool staged = (w & 0x4000u) && ernd >= 1u && rel <= 8u;
            entry[c] = ((rel & 15u) << 12) | ((w >> 15) << 11) | (uint32_t)(u * 256 + c) + 4u * lane;
            nibbles += staged && rel < 8u ? 1u << (4u * rel & 31u) : 0u;
            const uint64_t b = __ballot(staged);
            below += rank_below(b);
            total += (uint32_t)__popcll(b);
            st |= (staged ? 1u : 0u) << c;
        }
        uint32_t pos = base + below;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if ((st >> c) & 1u) codes[pos] = (uint16_t)entry[c];
            pos += (st >> c) & 1u;
        }
        base += total;
        if (u % 3 == 2 || u == 7) {
            const HistPairs s = spread_nibbles(nibbles);
#pragma unroll
            for (int q = 0; q < 4; ++q) hist.p[q] += s.p[q];
            nibbles = 0;
        }
    }
    hist = wave_hist(hist);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t piece = lane; piece * 8u < base; piece += 64u)
        __builtin_nontemporal_store(reinterpret_cast<const uint4v*>(codes)[piece], reinterpret_cast<uint4v*>(out) + piece);
    if (lane == 63) store_tile_record(hdr, hist, base, etr);
}

// Four consecutive floats, as 16 bytes where they are aligned (`vec`: the same for the whole launch).
__device__ __forceinline__ f4 load4(const float* p, bool vec) {
    if (vec) return __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
    return (f4){__builtin_nontemporal_load(p), __builtin_nontemporal_load(p + 1), __builtin_nontemporal_load(p + 2), __builtin_nontemporal_load(p + 3)};
}
__device__ __forceinline__ void store4(f4 x, float* p, bool vec) {
    if (vec) { __builtin_nontemporal_store(x, reinterpret_cast<f4*>(p)); return; }
#pragma unroll
    for (int c = 0; c < 4; ++c) __builtin_nontemporal_store(x[c], p + c);
}

// kR: rows of [J, C] per tile (1: C is a multiple of 2048 and a tile is a piece of a row; 2, 4, 8: C = 2048 / kR).
// kWaves: waves that share the block's 16 tiles.
// kSteps: fragments that Kp has (1 or 2), 0: any number.
template <int kR, bool kBf16, int kWaves, int kSteps>
__global__ __launch_bounds__(kWaves * 64, 4) void k_fused_fc_select(PlanCheck pc, uint32_t* __restrict__ flags, FusedArgs A,
                                                            const PlanGroup* __restrict__ groups,
                                                            TileHdr* __restrict__ hdrs, uint32_t* __restrict__ bitmap,
                                                            uint16_t* __restrict__ staging) {
    constexpr int kN = 64 / kWaves;                           // pieces of 32 columns a wave does
    constexpr int kParked = kN - 4;
    // first the waves' turning buffers for g and s and the codes of their first kParked pieces, then, when all are through, the
    // codes of the 16 tiles (those of a wave's last four pieces come from registers)
    union Lds {
        struct { float turn[2][16 * kTurnPitch]; uint2 park[kParked ? 2 * kParked : 1][64]; } w[kWaves];
        uint16_t codes[kFusedTiles][kCodePitch];
    };
    __shared__ __attribute__((aligned(16))) Lds sh;

    const bool ok = plan_ok(pc);
    if (blockIdx.x == 0 && threadIdx.x == 0) flags[0] = ok ? 0u : 1u;
    if (!ok) return;

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // uniform per wave: scalar registers, scalar branches
    const uint32_t lrow = lane & 15u, lgrp = lane >> 4;
    const PlanGroup pg = groups[A.group];
    constexpr uint32_t Cb = kTile / kR;                       // columns one block spans
    constexpr uint32_t CT = Cb / 16;                          // 16-column MFMA tiles per row tile
    const uint32_t ncb = kR == 1 ? A.C / kTile : 1u;          // column blocks
    const uint32_t cb = kR == 1 ? blockIdx.x % ncb : 0u, rb = kR == 1 ? blockIdx.x / ncb : blockIdx.x;
    const uint32_t j0 = rb * 16u * kR;                        // first row of the block
    const uint32_t colbase = cb * kTile;
    const uint32_t nt_group = (pg.size + kTile - 1) / kTile;

    // ---- this wave's part: one MFMA row tile (16 rows), 32 kN columns, 32 of them at a time.  Accumulator element i of a lane in
    // column tile t is row lane % 16, column 16 t + 4 (lane / 16) + i of them; turned through LDS, a lane has the four columns
    // 4 (lane % 8) .. + 3 of the rows 8 q + lane / 8, q = 0, 1 ----
    const uint32_t rt = (2u * kN * wave) / CT, ct0 = (2u * kN * wave) % CT;
    const uint32_t trow = lane >> 3, tcol = 4u * (lane & 7u);
    const bool frow_ok = j0 + 16u * rt + lrow < A.J;          // the fragment's row exists
    const uint32_t row = 16u * rt + trow, rows_left = j0 + row < A.J ? A.J - j0 - row : 0u;   // row of q = 0 in the block; rows from there on
    // addresses as a part that is the same for the wave and a lane's offset of 32 bits
    const uint64_t e0 = (uint64_t)(j0 + 16u * rt) * A.C + colbase + 16u * ct0;          // the wave's first element in the layer
    const uint32_t eoff = trow * A.C + tcol;
    float* r = A.r + pg.offset + e0;
    float* v = A.v + pg.offset + e0;
    const size_t row8 = (size_t)8u * A.C;                     // from q to q + 1
    const bool vec = ((reinterpret_cast<uintptr_t>(A.r + pg.offset) | reinterpret_cast<uintptr_t>(A.v + pg.offset)) & 15u) == 0;
    const bool vec_out = ((reinterpret_cast<uintptr_t>(A.g_out) | reinterpret_cast<uintptr_t>(A.s_out)) & 15u) == 0;
    float* turn_g = sh.w[wave].turn[0];
    float* turn_s = sh.w[wave].turn[1];
    constexpr uint32_t kPer = kBf16 ? 8u : 4u;                // K values a lane's 16 bytes hold
    constexpr uint32_t kStep = 4u * kPer;                     // K values of one fragment
    const uint32_t es = kBf16 ? 2u : 4u;
    const uint32_t doff = (lrow * A.Kp + kPer * lgrp) * es, xoff = frow_ok ? doff : 0u;
    const char* xp = static_cast<const char*>(A.XT) + (size_t)(j0 + 16u * rt < A.J ? j0 + 16u * rt : 0u) * A.Kp * es;
    const char* dp = static_cast<const char*>(A.DT) + (size_t)(colbase + 16u * ct0) * A.Kp * es;
    const size_t dstep = (size_t)16u * A.Kp * es;             // one column tile further
    struct Frags { u4v x, d[2]; };
    auto fetch = [&](int n, uint32_t k0) -> Frags {
        Frags F;
        F.x = *reinterpret_cast<const u4v*>(xp + (size_t)k0 * es + xoff);
        if (!frow_ok) F.x = (u4v){0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < 2; ++t) F.d[t] = *reinterpret_cast<const u4v*>(dp + (size_t)(2 * n + t) * dstep + (size_t)k0 * es + doff);
        return F;
    };
    f4v acc_g[2], acc_s[2];
    auto multiply = [&](const Frags& F) {
        if (kBf16) {
            const u4v x2 = sq_bf16x8(F.x);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const u4v d2 = sq_bf16x8(F.d[t]);
                acc_g[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, F.d[t]), __builtin_bit_cast(bf8v, F.x), acc_g[t], 0, 0, 0);
                acc_s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, d2), __builtin_bit_cast(bf8v, x2), acc_s[t], 0, 0, 0);
            }
        } else {
            // v_mfma_f32_16x16x4_f32 takes one k per lane group; a lane loads four consecutive k at once and k-step i of
            // a group of 16 uses element i, so lane group q supplies k = 16 step + 4 q + i (the same assignment for both
            // operands, every k exactly once)
            const f4v xf = __builtin_bit_cast(f4v, F.x), x2 = xf * xf;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const f4v df = __builtin_bit_cast(f4v, F.d[t]), d2 = df * df;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc_g[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(df[i], xf[i], acc_g[t], 0, 0, 0);
                    acc_s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(d2[i], x2[i], acc_s[t], 0, 0, 0);
                }
            }
        }
    };
    // Loads come back in the order of their request (and stores count among them): the first fragments of the next 32 columns are
    // requested before the r and v of these are waited for and written.  The wait for one of them is counted past those requested
    // after it where the number of these is known: with kWhole (all 16 rows exist, r and v lie at 16 bytes, g and s are not asked
    // for) and kSteps no branch is left around a load.  With them in branches each of these waits was for everything, the r and v
    // just requested among it.  In bf16, us: 25088 x 4096 at batch 32 363 -> 352, at batch 64 387 -> 385, 9216 x 1024 at 64
    // 72.3 -> 69.6, 4096 x 4096 80.5 -> 77.4, 5000 x 256 at 40 33.2 -> 30.2, 1001 x 512 at 20 29.1 -> 25.6; float32, 25088 x 4096
    // at 16, 367 -> 357.  With two fragments of float32 it is slower (25088 x 4096 at 32: 391 -> 398): they stay in branches.  With
    // one fragment there are registers left to request the r and v, too, 32 columns ahead (bf16, batch 32: 354 -> 351; with two:
    // 387 -> 401, spilled).
    constexpr bool kAhead = kSteps == 1;
    uint2 code[kN][2];                                        // of columns 32 n + tcol .. + 3, row q (n < kParked: in LDS meanwhile)
    auto pass = [&](auto whole_) __attribute__((always_inline)) {
        constexpr bool kWhole = decltype(whole_)::value;
        auto fetch_first = [&](int n, Frags& F0, Frags& F1) {
            F0 = fetch(n, 0);
            if (kSteps != 1) F1 = fetch(n, kSteps == 2 || A.Kp > kStep ? kStep : 0u);
        };
        f4 R4[2][2], V4[2][2];                                // of these columns and of the next
        auto request = [&](int n) {
            f4 (&R)[2] = R4[n & 1], (&V)[2] = V4[n & 1];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (!kWhole) R[q] = V[q] = (f4){0.f, 0.f, 0.f, 0.f};
                if (kWhole || 8u * q < rows_left) {
                    R[q] = load4(r + q * row8 + 32 * n + eoff, kWhole || vec);
                    V[q] = load4(v + q * row8 + 32 * n + eoff, kWhole || vec);
                }
            }
        };
        Frags F0, F1;
        fetch_first(0, F0, F1);
        if (kWhole && kAhead) request(0);
#pragma unroll
        for (int n = 0; n < kN; ++n) {
            if (!kWhole || !kAhead) request(n);
#pragma unroll
            for (int t = 0; t < 2; ++t) { acc_g[t] = (f4v){0.f, 0.f, 0.f, 0.f}; acc_s[t] = (f4v){0.f, 0.f, 0.f, 0.f}; }
            multiply(F0);
            if (kSteps == 2 || (kSteps == 0 && A.Kp > kStep)) multiply(F1);
            if (kSteps == 0) {
#pragma unroll 1
                for (uint32_t k0 = 2u * kStep; k0 < A.Kp; k0 += kStep) multiply(fetch(n, k0));
            }
            if (n + 1 < kN) {
                fetch_first(n + 1, F0, F1);
                if (kWhole && kAhead) request(n + 1);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                *reinterpret_cast<f4v*>(turn_g + lrow * kTurnPitch + 16 * t + 4 * lgrp) = acc_g[t] * A.cg;
                *reinterpret_cast<f4v*>(turn_s + lrow * kTurnPitch + 16 * t + 4 * lgrp) = acc_s[t] * A.cs;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const f4v g4 = *reinterpret_cast<const f4v*>(turn_g + (8 * q + trow) * kTurnPitch + tcol);
                const f4v s4 = *reinterpret_cast<const f4v*>(turn_s + (8 * q + trow) * kTurnPitch + tcol);
                const bool live = kWhole || 8u * q < rows_left;
                if (!kWhole && A.g_out && live) {
                    store4(__builtin_bit_cast(f4, g4), A.g_out + e0 + q * row8 + 32 * n + eoff, vec_out);
                    store4(__builtin_bit_cast(f4, s4), A.s_out + e0 + q * row8 + 32 * n + eoff, vec_out);
                }
                f4 ro, vo;
                uint32_t w[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float a, b;
                    uint32_t bits;
                    const bool send = alg1_step(g4[c], s4[c], R4[n & 1][q][c], V4[n & 1][q][c], A.alpha, A.zeta, a, b, bits) & live;
                    ro[c] = a;
                    vo[c] = b;
                    w[c] = element_code(bits, send);
                }
                if (live) {
                    store4(ro, r + q * row8 + 32 * n + eoff, kWhole || vec);
                    store4(vo, v + q * row8 + 32 * n + eoff, kWhole || vec);
                }
                const uint2 cw = make_uint2(w[0] | (w[1] << 16), w[2] | (w[3] << 16));
                if (n < kParked) sh.w[wave].park[2 * n + q][lane] = cw;
                else code[n][q] = cw;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            __builtin_amdgcn_wave_barrier();
        }
    };
    if (kSteps != 0 && vec && !A.g_out && j0 + 16u * rt + 16u <= A.J) pass(std::true_type{});    // (uniform per wave)
    else pass(std::false_type{});
#pragma unroll
    for (int n = 0; n < kParked; ++n)
#pragma unroll
        for (int q = 0; q < 2; ++q) code[n][q] = sh.w[wave].park[2 * n + q][lane];
    __syncthreads();                                          // the waves' own buffers have been read
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t rw = row + 8u * q;
#pragma unroll
        for (int n = 0; n < kN; ++n)
            *reinterpret_cast<uint2*>(sh.codes[rw / kR] + (rw % kR) * Cb + 16u * ct0 + 32u * n + tcol) = code[n][q];
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t q = 0; q < (uint32_t)(kFusedTiles / kWaves); ++q) {
        const uint32_t tl = (uint32_t)(kFusedTiles / kWaves) * wave + q;
        const uint32_t in_group = kR == 1 ? (j0 + tl) * ncb + cb : (uint32_t)blockIdx.x * kFusedTiles + tl;
        if (kR == 1 ? j0 + tl >= A.J : in_group >= nt_group) break;      // past the end of the layer
        const uint32_t t = pg.first_tile + in_group;
        encode_codes(sh.codes[tl], hdrs + t, bitmap + (size_t)t * (kTile / 32), staging + (size_t)t * kTile, lane);
    }
}

// The same for a long K in bf16: the contraction first, with all 16 tiles' g and s in the accumulators (2 x 64 registers per
// lane of eight waves, one workgroup per compute unit), which then pass through LDS in tile order, eight tiles at a time, and
// each wave runs the loop body on one tile while the r and v of its next chunks are on their way.  The fragments of X are
// fetched and squared once, where the kernel above does it once per 32 columns (one vector instruction in three).
constexpr int kSlotPitch = kTile + 8;               // floats per tile's slot: slots 2 q and 2 q + 2 start 16 banks apart

template <int kR>
__global__ __launch_bounds__(512) void k_fused_fc_select_long(PlanCheck pc, uint32_t* __restrict__ flags, FusedArgs A,
                                                              const PlanGroup* __restrict__ groups, TileHdr* __restrict__ hdrs,
                                                              uint32_t* __restrict__ bitmap, uint16_t* __restrict__ staging) {
    __shared__ __attribute__((aligned(16))) float lds_g[8][kSlotPitch];
    __shared__ __attribute__((aligned(16))) float lds_s[8][kSlotPitch];

    const bool ok = plan_ok(pc);
    if (blockIdx.x == 0 && threadIdx.x == 0) flags[0] = ok ? 0u : 1u;
    if (!ok) return;

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // uniform per wave: scalar registers, scalar branches
    const uint32_t lrow = lane & 15u, lgrp = lane >> 4;
    const PlanGroup pg = groups[A.group];
    constexpr uint32_t Cb = kTile / kR, CT = Cb / 16;         // columns of a block, its 16-column MFMA tiles per row tile
    const uint32_t ncb = kR == 1 ? A.C / kTile : 1u;          // column blocks
    const uint32_t cb = kR == 1 ? blockIdx.x % ncb : 0u, rb = kR == 1 ? blockIdx.x / ncb : blockIdx.x;
    const uint32_t j0 = rb * 16u * kR, colbase = cb * kTile;  // first row and column of the block
    const uint32_t nt_group = (pg.size + kTile - 1) / kTile;
    const bool vec = ((reinterpret_cast<uintptr_t>(A.r + pg.offset) | reinterpret_cast<uintptr_t>(A.v + pg.offset)) & 15u) == 0;
    const bool vec_out = ((reinterpret_cast<uintptr_t>(A.g_out) | reinterpret_cast<uintptr_t>(A.s_out)) & 15u) == 0;

    // Wave w runs the tile in slot w of each pass.  Accumulator element i of MFMA tile t of a lane is row 16 rt + 4 lgrp + i,
    // column 16 (ct0 + t) + lrow of the block; it belongs to tile row / kR.  For kR = 1 pass p takes elements 2 p, 2 p + 1 of
    // every lane (tiles 4 lgrp + i in slots 2 lgrp + i % 2: all lanes write), otherwise the tiles 8 p .. 8 p + 7.
    struct TileRef { uint32_t in_group, m; };                 // number inside the group, elements (0: past the end of the layer)
    auto ref_of = [&](uint32_t p) -> TileRef {
        const uint32_t tl = kR == 1 ? 4u * (wave >> 1) + 2u * p + (wave & 1u) : 8u * p + wave;
        const uint32_t in_group = kR == 1 ? (j0 + tl) * ncb + cb : (uint32_t)blockIdx.x * kFusedTiles + tl;
        const bool live = kR == 1 ? (j0 + tl) < A.J : in_group < nt_group;
        return TileRef{live ? in_group : 0u, live ? min(kTile, pg.size - in_group * kTile) : 0u};
    };
    // chunk u of a tile: elements 256 u + 4 lane + c; rows are whole multiples of 256, so a chunk exists as a whole or not at all
    f4 R4[4], V4[4];
    auto request = [&](const TileRef& q, int u, bool whole) {     // whole: all of it exists, 16 bytes at a time
        if (!whole) R4[u & 3] = V4[u & 3] = (f4){0.f, 0.f, 0.f, 0.f};
        if (!whole && 256u * u >= q.m) return;
        const size_t at = pg.offset + (size_t)q.in_group * kTile + 256u * u + 4u * lane;
        R4[u & 3] = load4(A.r + at, whole || vec);
        V4[u & 3] = load4(A.v + at, whole || vec);
    };
    TileRef q = ref_of(0);
    if (vec && q.m == kTile) {
#pragma unroll
        for (int u = 0; u < 4; ++u) request(q, u, true);      // they arrive while the matrix cores are busy
    }

    const uint32_t rt = (16u * wave) / CT, ct0 = (16u * wave) % CT;      // the wave's 16 MFMA tiles: one row tile, 16 column tiles
    f4v acc_g[16], acc_s[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) { acc_g[t] = (f4v){0.f, 0.f, 0.f, 0.f}; acc_s[t] = (f4v){0.f, 0.f, 0.f, 0.f}; }
    const uint32_t row = j0 + 16u * rt + lrow;
    const bool row_ok = row < A.J;
    const uint16_t* xp = static_cast<const uint16_t*>(A.XT) + (size_t)(row_ok ? row : 0u) * A.Kp + 8u * lgrp;
    const uint16_t* dp = static_cast<const uint16_t*>(A.DT) + (size_t)(colbase + 16u * ct0 + lrow) * A.Kp + 8u * lgrp;
    for (uint32_t k0 = 0; k0 < A.Kp; k0 += 32) {
        u4v x = *reinterpret_cast<const u4v*>(xp + k0);
        if (!row_ok) x = (u4v){0u, 0u, 0u, 0u};
        const u4v x2 = sq_bf16x8(x);
#pragma unroll
        for (int t0 = 0; t0 < 16; t0 += 8) {
            u4v d[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) d[t] = *reinterpret_cast<const u4v*>(dp + (size_t)(t0 + t) * 16u * A.Kp + k0);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const u4v d2 = sq_bf16x8(d[t]);
                acc_g[t0 + t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, x), __builtin_bit_cast(bf8v, d[t]), acc_g[t0 + t], 0, 0, 0);
                acc_s[t0 + t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, x2), __builtin_bit_cast(bf8v, d2), acc_s[t0 + t], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        if (p) __syncthreads();                               // every wave is done with the slots of the first pass
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (kR == 1 && i / 2 != p) continue;
            const uint32_t rw = 16u * rt + 4u * lgrp + i, tl = rw / kR;
            if (kR != 1 && (tl >> 3) != (uint32_t)p) continue;
            const uint32_t slot = kR == 1 ? 2u * lgrp + (uint32_t)(i & 1) : tl & 7u, at = (rw % kR) * Cb + 16u * ct0 + lrow;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                lds_g[slot][at + 16u * t] = acc_g[t][i] * A.cg;
                lds_s[slot][at + 16u * t] = acc_s[t][i] * A.cs;
            }
        }
        __syncthreads();
        if (p) q = ref_of(1);
        if (q.m == 0) continue;
        uint2 code[8];
        auto run = [&](auto is_whole) __attribute__((always_inline)) {
            constexpr bool whole = decltype(is_whole)::value;
            if (p || !whole) {
#pragma unroll
                for (int u = 0; u < 4; ++u) request(q, u, whole);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const f4 g4 = reinterpret_cast<const f4*>(lds_g[wave])[u * 64 + lane], s4 = reinterpret_cast<const f4*>(lds_s[wave])[u * 64 + lane];
                const f4 r4 = R4[u & 3], v4 = V4[u & 3];
                if (u + 4 < 8) request(q, u + 4, whole);      // into the registers that this chunk leaves
                const bool live = whole || 256u * u < q.m;
                const size_t in_layer = (size_t)q.in_group * kTile + 256u * u + 4u * lane;
                if (A.g_out && live) {
                    store4(g4, A.g_out + in_layer, vec_out);
                    store4(s4, A.s_out + in_layer, vec_out);
                }
                f4 ro, vo;
                uint32_t w[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float a, b;
                    uint32_t bits;
                    const bool send = alg1_step(g4[c], s4[c], r4[c], v4[c], A.alpha, A.zeta, a, b, bits) & live;
                    ro[c] = a;
                    vo[c] = b;
                    w[c] = element_code(bits, send);
                }
                if (live) {
                    store4(ro, A.r + pg.offset + in_layer, whole || vec);
                    store4(vo, A.v + pg.offset + in_layer, whole || vec);
                }
                code[u] = make_uint2(w[0] | (w[1] << 16), w[2] | (w[3] << 16));
            }
        };
        if (vec && q.m == kTile) run(std::true_type{});
        else run(std::false_type{});
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");      // the slot's g has been read: the codes take its place
        __builtin_amdgcn_wave_barrier();
        uint16_t* codes = reinterpret_cast<uint16_t*>(lds_g[wave]);
#pragma unroll
        for (int u = 0; u < 8; ++u) *reinterpret_cast<uint2*>(codes + u * 256 + 4 * lane) = code[u];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        const uint32_t t = pg.first_tile + q.in_group;
        encode_codes(codes, hdrs + t, bitmap + (size_t)t * (kTile / 32), staging + (size_t)t * kTile, lane);
    }
}

// Batches in bf16 above which the contraction comes first (kernel and transposes, interleaved / contraction first, us): 9216 x
// 1024 at 128 93 / 93, at 160 96 / 87, at 256 134 / 125, at 1024 387 / 309; 25088 x 4096 at 128 511 / 553, at 160 533 / 520, at
// 256 772 / 764, at 1024 2393 / 1938.  In float32 the squares are one instruction an element and it gains nothing.
constexpr uint32_t kLongK = 128;

// Shapes the fused kernel takes: C a multiple of 2048 (a tile is a piece of a row) or C = 1024, 512, 256 (a tile is
// 2, 4, 8 whole rows).  0 = not supported.
static int fused_rows_per_tile(uint32_t C) {
    if (C % kTile == 0) return 1;
    if (C == 1024) return 2;
    if (C == 512) return 4;
    if (C == 256) return 8;
    return 0;
}

static uint32_t fused_kp(int dtype, uint32_t B) { return dtype == VGC_BF16 ? (B + 31u) / 32u * 32u : (B + 15u) / 16u * 16u; }

size_t fused_fc_workspace_bytes(int dtype, uint32_t B, uint32_t J, uint32_t C) {
    if (fused_rows_per_tile(C) == 0 || B == 0 || J == 0) return 0;
    const size_t es = dtype == VGC_BF16 ? 2 : 4;
    return ((size_t)J + C) * fused_kp(dtype, B) * es;
}

int launch_fused_fc_select(PlanCheck pc, uint32_t* flags, int dtype, const void* X, const void* D, uint32_t B, uint32_t J, uint32_t C,
                           float c, float* r, float* v, const PlanGroup* groups, uint32_t group, TileHdr* hdrs, uint32_t* bitmap,
                           uint16_t* staging, float alpha, float zeta, void* workspace, float* g_out, float* s_out, hipStream_t stream) {
    const int kr = fused_rows_per_tile(C);
    if (kr == 0) { set_error("vgc_sqgrad_accumulate_select: C = %u is neither a multiple of 2048 nor 256, 512 or 1024", C); return VGC_ERR_SIZE; }
    const uint32_t Kp = fused_kp(dtype, B);
    const size_t es = dtype == VGC_BF16 ? 2 : 4;
    char* ws = static_cast<char*>(workspace);
    void* XT = ws;
    void* DT = ws + (size_t)J * Kp * es;
    const uint32_t per = 16 / (uint32_t)es;
    const uint64_t nx = (uint64_t)J * (Kp / per), nd = (uint64_t)C * (Kp / per);
    const uint32_t bx = (uint32_t)((nx + 255) / 256), bd = (uint32_t)((nd + 255) / 256);
    if (dtype == VGC_BF16)
        hipLaunchKernelGGL(k_fc_transpose<uint16_t>, dim3(bx + bd), dim3(256), 0, stream, (const uint16_t*)X, (const uint16_t*)D, B, J, C, Kp, bx,
                           (uint16_t*)XT, (uint16_t*)DT);
    else
        hipLaunchKernelGGL(k_fc_transpose<float>, dim3(bx + bd), dim3(256), 0, stream, (const float*)X, (const float*)D, B, J, C, Kp, bx,
                           (float*)XT, (float*)DT);
    FusedArgs A;
    A.XT = XT; A.DT = DT; A.J = J; A.C = C; A.Kp = Kp; A.cg = c; A.cs = c * c; A.r = r; A.v = v; A.g_out = g_out; A.s_out = s_out;
    A.group = group; A.alpha = alpha; A.zeta = zeta;
    const uint64_t rows_per_block = 16ull * kr;
    const uint64_t nblk = (J + rows_per_block - 1) / rows_per_block * (kr == 1 ? C / kTile : 1u);
    if (nblk > 0x7FFFFFFFull) { set_error("vgc_sqgrad_accumulate_select: shape exceeds the launch limit"); return VGC_ERR_SIZE; }
    // With no more blocks than compute units 16 waves share a block, each with half the columns and one tile to encode: what a
    // wave does in a row is then all the time there is (300 x 2048 in bf16 at batch 64: 31.4 us against 35.0 with eight waves;
    // 1000 x 256 in float32: 41.7 against 49.7).
#define VGC_FUSED(K_, NW) hipLaunchKernelGGL((K_), dim3((uint32_t)nblk), dim3(NW * 64), 0, stream, pc, flags, A, groups, hdrs, bitmap, staging)
#define VGC_FUSED_STEPS(KR, BF, NW)                                                                                           \
    do {                                                                                                                      \
        if (steps == 1) VGC_FUSED((k_fused_fc_select<KR, BF, NW, 1>), NW);                                                    \
        else if (BF && steps == 2) VGC_FUSED((k_fused_fc_select<KR, BF, NW, BF ? 2 : 0>), NW);                                \
        else VGC_FUSED((k_fused_fc_select<KR, BF, NW, 0>), NW);                                                               \
    } while (0)
#define VGC_FUSED_WAVES(KR)                                                                                                   \
    do {                                                                                                                      \
        if (bf && Kp > kLongK) VGC_FUSED(k_fused_fc_select_long<KR>, 8);                                                      \
        else if (bf && nblk <= 256) VGC_FUSED_STEPS(KR, true, 16);                                                            \
        else if (bf) VGC_FUSED_STEPS(KR, true, 8);                                                                            \
        else if (nblk <= 256) VGC_FUSED_STEPS(KR, false, 16);                                                                 \
        else VGC_FUSED_STEPS(KR, false, 8);                                                                                   \
    } while (0)
    const bool bf = dtype == VGC_BF16;
    const uint32_t steps = Kp / (bf ? 32u : 16u);
    if (kr == 1) VGC_FUSED_WAVES(1);
    else if (kr == 2) VGC_FUSED_WAVES(2);
    else if (kr == 4) VGC_FUSED_WAVES(4);
    else VGC_FUSED_WAVES(8);
#undef VGC_FUSED_WAVES
#undef VGC_FUSED_STEPS
#undef VGC_FUSED
    return hip_check(hipGetLastError(), "launch k_fused_fc_select");
}

}  // namespace vgc
