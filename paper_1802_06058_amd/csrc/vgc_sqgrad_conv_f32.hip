// float32 conv form of the per-parameter sums of Alg. 1 (per sample G_z = U_z^T D_z over the P positions, then
// g = c sum_z G_z, s = c^2 sum_z G_z . G_z) on the bf16 matrix cores, without giving up float32: every input element is
// cut into three bf16 pieces that add up to it exactly (hi: rounded to bf16; mid: the rest rounded to bf16; lo: what is
// left, at most 8 bits), and of the nine products of two elements' pieces the six largest are summed in the float32
// accumulators: hi hi, hi mid, mid hi, mid mid, hi lo, lo hi.  The products are exact.  What is left out, mid lo, lo mid and
// lo lo, is at most 2^-24 of the product (x x with x = 1.0038986), over random mantissas 2^-27.5 in the root mean square; for
// the same two mantissas it is the same each time.  (With hi cut off instead of rounded: 2^-22 and 2^-25.5.)
//
// Why: v_mfma_f32_32x32x2_f32 does 256 multiply-adds a cycle and compute unit, the bf16 instructions 4096, so six of the
// latter take 3/8 of the time.  3 x 3, 256 -> 256 at 56 x 56, batch 32, through k_conv_f32: 1.21 -> 0.66 ms (98 -> 180 TFLOP/s;
// k_conv_taps_f32 below, which takes such layers, 0.52 on a card where this kernel takes 0.70); the 53 layers of ResNet-50 at
// batch 32: 3.14 -> 2.30 ms in one batch call (1.19 ms at the rate of a large bf16 product), 2.17 with k_conv_taps_f32.  What bounds it now: the vector instructions that cut the elements (13 per pair, once per filter tap and
// column tile) and those that add up the chunks share the issue slots with the MFMAs (matrix pipes 28 to 41 % busy on ResNet's
// layers), and on the small layers a workgroup's 14 chunks take 19 us of its kernel's 31.
//
// The bf16 MFMA adds with truncation: chained over all positions, every instruction would cut off a little of the
// accumulator, always towards minus infinity.  So the six products of a chunk of 32 positions are summed from zero, where
// what is cut off is small, and the chunk's sum is added in float32, rounded to nearest; and odd chunks form the negative sum
// and subtract it, so that what is left of the one-sided error cancels instead of adding up over the samples into g.  Error
// of s against 64 bits over ResNet-50's layers: 0.51e-7 to 0.81e-7 (with the float32 instruction 0.66e-7 to 1.3e-7), of g
// 0.79e-7 to 1.5e-7 (1.1e-7 to 2.9e-7).  Below 16 positions the last truncation shows: at one position g errs by 0.95e-7
// (0.73e-7), s by 0.62e-7 (0.57e-7).
#include <cmath>

#include "vgc_internal.h"

namespace vgc {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef short s8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s4v* lds_s4v_ptr;
typedef __amdgpu_buffer_rsrc_t rsrc_t;

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

constexpr int kR32 = 32;                 // positions per LDS stage: one MFMA k-step
// Elements are cut at 2^24 times their size, so that no piece of any float32 number, subnormal ones included, falls below what
// bf16 holds in full (without it, lo lost bits of elements below 2^-110); samples' sums are scaled back before the square.
// The multiplications cost 1 % of ResNet-50's layers.
constexpr float kUp = 0x1p24f, kDown = 0x1p-48f;

// Two floats as three pairs of bf16 whose sum they are: hi and mid rounded to nearest, lo what is left of 24 bits.  (A magnitude
// within half a bf16 step of the largest float rounds up to infinity: its sums are formed again at the end.)
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){x0, x1}, bf2v));
    const float r0 = x0 - __uint_as_float(hi << 16), r1 = x1 - __uint_as_float(hi & 0xFFFF0000u);
    mid = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){r0, r1}, bf2v));
    const float l0 = r0 - __uint_as_float(mid << 16), l1 = r1 - __uint_as_float(mid & 0xFFFF0000u);
    lo = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);
}

// The first sample of group k of `groups`: k B / groups (in 32 bits where that is enough: a division of 64 takes a workgroup 0.2 us).
__device__ __forceinline__ uint32_t first_sample(uint32_t k, uint32_t B, uint32_t groups) {
    return B < 65536u ? k * B / groups : (uint32_t)((uint64_t)k * B / groups);
}

// One staged chunk in registers: kR32 rows of a BM-wide and of a BN-wide float matrix, PA resp. PB 16-byte
// pieces per thread of a workgroup of NT threads.  Piece idx of an operand W columns wide sits in row
// idx / (W / 4), columns 4 (idx % (W / 4)) .. + 3.
template <int PA, int PB> struct Chunk32 { f4v a[PA], b[PB]; };

// LDS image of one operand's chunk: three planes (hi, mid, lo) of kR32 rows of W bf16.  A transposing read takes one
// 32-byte unit of rows 0..3, 8..11, 16..19 and 24..27 at once, half of them per pass over the 64 banks: the units of a row are
// XOR-ed with bits of the row number so that the eight (row, unit) of a pass fall into different banks without padding.
template <int W> __device__ __forceinline__ constexpr uint32_t lds_swizzle(uint32_t row) {
    return W >= 128 ? (row & 3u) | ((row >> 1) & 4u) : ((row >> 1) & 1u) | ((row >> 2) & 2u);
}
template <int W> __device__ __forceinline__ uint32_t lds_piece(uint32_t row, uint32_t col) {      // byte offset inside a plane
    return row * (W * 2) + (((col >> 4) ^ lds_swizzle<W>(row)) << 5) + (col & 15u) * 2u;
}

// The pieces of an infinity add up to NaN, as do products beyond the range of float32 whose pieces differ in sign, and a pixel
// may reach taps that do not use it, by way of positions past P (in the linear mode of k_conv_f32, and between the rows and the
// samples of k_conv_taps_f32).  So an MFMA tile with a sum that is not finite is formed again with the float32 instruction,
// element by element of its own operands from memory, and gets what float32 arithmetic gives.  Where all of a tile's sums are NaN
// already, as they are throughout once a network has diverged, nothing more can change and the walk ends.  3 x 3, 256 -> 256 at
// 14 x 14, batch 32, through k_conv_f32: 78 us; with an infinity among the activations 181, among the gradients 328, with nothing but NaN 87.
// x_at(z, p), d_at(z, p): the operands of the lane's row and column (lane % 16) at a position, zero outside; valid(r): whether row
// r of the tile is an output in the lane's column.  What is formed, for the rows 4 (lane / 16) .. + 3: the last sample's product,
// the sum of the samples' squares, and of the products.
struct Formed { f4v sum, s, g; };
template <typename FX, typename FD, typename FV>
__device__ __forceinline__ Formed form_again(FX x_at, FD d_at, FV valid, uint32_t z_begin, uint32_t z_end, uint32_t p_begin, uint32_t p_end) {
    const uint32_t lane = threadIdx.x & 63u;
    // whether the sums at the lane's outputs are all NaN
    auto settled = [&](const f4v& v) {
        bool s = true;
#pragma unroll
        for (int i = 0; i < 4; ++i) s = s && (v[i] != v[i] || !valid(4u * (lane >> 4) + (uint32_t)i));
        return __ballot(!s) == 0;
    };
    Formed F = {};
#pragma unroll 1
    for (uint32_t z = z_begin; z < z_end && !settled(F.s); ++z) {
        F.sum = (f4v){0};
#pragma unroll 1
        for (uint32_t p0 = p_begin; p0 < p_end && !settled(F.sum); p0 += 16) {
            float x[4], d[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                x[k] = x_at(z, p0 + 4u * k + (lane >> 4));
                d[k] = d_at(z, p0 + 4u * k + (lane >> 4));
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) F.sum = __builtin_amdgcn_mfma_f32_16x16x4f32(x[k], d[k], F.sum, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) F.s[i] = __builtin_fmaf(F.sum[i], F.sum[i], F.s[i]);
        F.g = F.g + F.sum;
    }
    return F;
}
// at(r): where row r of the tile lies in the lane's column.
template <bool kWantG, typename FV, typename FO>
__device__ __forceinline__ void store_formed(const Formed& F, FV valid, FO at, bool parts, float fs, float fg, float* __restrict__ so, float* __restrict__ go) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t r = 4u * (lane >> 4) + (uint32_t)i;
        if (valid(r)) {
            const size_t o = at(r);
            __builtin_nontemporal_store(parts ? F.sum[i] : fs * F.s[i], so + o);
            if (kWantG) __builtin_nontemporal_store(fg * F.g[i], go + o);
        }
    }
}
// Whether one of the wave's sums is an infinity or NaN.
__device__ __forceinline__ bool not_finite(const f4v& v) {
    uint32_t most = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) most = max(most, __float_as_uint(v[i]) & 0x7FFFFFFFu);
    return __ballot(most >= 0x7F800000u) != 0;
}

// X is [B, P, J], D is [B, P, C], samples z_begin .. z_end-1 of this workgroup's split.
// Input modes other than kPatches: X is the layer's NHWC input [B, H, W, Cin] seen through the geometry G, J = kh kw Cin;
//         the thread's piece of 4 columns lies inside one filter tap (Cin is a multiple of 4).
//   kLinear   unit strides, an output as wide as the input: the input element of position p is a constant number of
//             elements after p's own, so offsets advance by a constant per chunk; whether the column lies inside the
//             image repeats every W / gcd(W, kR32) <= 32 chunks and is kept as one bit per chunk of that period.
//   kGeneral  offsets are formed per chunk from the output position of the row, which is kept incrementally.
// BM x BN: the block tile; WM x WN: the part of it a wave multiplies, in MFMA tiles of 16 x 16.
enum { kPatches = 0, kLinear = 1, kGeneral = 2 };

// kFew: samples of at most 16 positions.  A chunk is 16 positions then, and the 32 of an MFMA hold two of the six products:
// lo hi + hi lo, mid mid + mid hi, hi mid + hi hi, with the two halves of a wave reading different planes.  Half the MFMAs and
// half the elements to cut of a chunk padded to 32 positions: 3 x 3, 512 -> 512 at 4 x 4, batch 64: 89 -> 53 us (80 with the
// float32 instruction); one position, 512 -> 512, batch 32, without a workspace: 51 -> 32.5 (33).
template <bool kWantG, int kMode, int BM, int BN, int WM, int WN, bool kFew>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64, kFew && !kWantG ? 4 : 2)      // (one register above 128: 512 -> 512 at 4 x 4 53 -> 64 us)
void k_conv_f32(const float* __restrict__ X, const float* __restrict__ D, uint32_t B, uint32_t P, uint32_t J, uint32_t C,
                uint32_t splits, uint32_t split_p, float cg, float cs, float* __restrict__ g_out, float* __restrict__ s_out,
                float* __restrict__ ws, ConvGeom G) {
    static_assert(!kFew || kMode != kLinear, "one chunk per sample: nothing to advance");
    if (kFew) split_p = 1;
    constexpr int kRows = kFew ? kR32 / 2 : kR32;                    // positions of a chunk
    constexpr int NT = (BM / WM) * (BN / WN) * 64;                   // threads of the workgroup
    constexpr int MT = WM / 16, NTL = WN / 16;                       // MFMA tiles of a wave
    constexpr int PA = kRows * BM / 4 / NT, PB = kRows * BN / 4 / NT;   // 16-byte pieces per thread and chunk
    constexpr int kPlaneA = kRows * BM * 2, kPlaneB = kRows * BN * 2;   // bytes
    static_assert(NT % (BM / 4) == 0 && NT % (BN / 4) == 0, "all pieces of a thread lie in the same columns");
    __shared__ __attribute__((aligned(16))) uint8_t shA[2][3 * kPlaneA];
    __shared__ __attribute__((aligned(16))) uint8_t shB[2][3 * kPlaneB];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, wm = wave / (BN / WN), wn = wave % (BN / WN);
    const uint32_t tiles_c = (C + BN - 1) / BN, tiles_j = (J + BM - 1) / BM;
    const uint32_t nblk = gridDim.x, per = nblk / 8u, rem = nblk % 8u;
    const uint32_t xcd = blockIdx.x % 8u, slot = blockIdx.x / 8u;
    const uint32_t logical = xcd * per + min(xcd, rem) + slot;       // contiguous range of tiles per XCD
    const uint32_t tile_c = logical % tiles_c, tile_j = (logical / tiles_c) % tiles_j, split = logical / (tiles_c * tiles_j);
    const uint32_t j0 = tile_j * BM, c0 = tile_c * BN;
    // split_p > 1: the workgroup owns part `part` of the positions of the single sample split / split_p
    // and leaves the unsquared partial product in the workspace
    const uint32_t n_chunks = kFew ? 1u : (P + kR32 - 1) / kR32;
    const uint32_t part = split_p > 1 ? split % split_p : 0u;
    const uint32_t chunks_per_part = (n_chunks + split_p - 1) / split_p;
    const uint32_t c_begin = min(n_chunks, part * chunks_per_part);
    // sample ranges of the splits differ by at most one sample
    const uint32_t z_begin = split_p > 1 ? split / split_p : first_sample(split, B, splits);
    const uint32_t z_end = split_p > 1 ? z_begin + 1u : first_sample(split + 1u, B, splits);
    const uint32_t total = split_p > 1 ? min(n_chunks, c_begin + chunks_per_part) - c_begin : (z_end - z_begin) * n_chunks;

    f4v acc[MT][NTL], s_acc[MT][NTL], g_acc[MT][NTL];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NTL; ++b) { acc[a][b] = (f4v){0}; s_acc[a][b] = (f4v){0}; g_acc[a][b] = (f4v){0}; }

    // the thread's pieces lie in the same columns, kRowStep rows apart
    constexpr uint32_t kRowStepA = NT / (BM / 4), kRowStepB = NT / (BN / 4);
    const uint32_t rowA = tid / (BM / 4), rowB = tid / (BN / 4), colj = j0 + (tid % (BM / 4)) * 4u;
    const uint32_t offB0 = (rowB * C + c0 + (tid % (BN / 4)) * 4u) * 4u;
    uint32_t offA = 0, offA0 = (rowA * J + colj) * 4u, rowsA = kRowStepA * J * 4u, phase = 0;
    uint32_t y0A[PA], x0A[PA], yA[PA], xA[PA], outside[PA];
    int32_t tapX = 0, tapOff = 0;
    if (kMode != kPatches) {
        const uint32_t tap = colj / G.Cin, ky = tap / G.kw;
        const int32_t ty = (int32_t)ky - (int32_t)G.ph;
        tapX = (int32_t)(tap - ky * G.kw) - (int32_t)G.pw;
        tapOff = (ty * (int32_t)G.W + tapX) * (int32_t)G.Cin + (int32_t)(colj - tap * G.Cin);
        if (colj >= J) tapX = -0x400000;                     // a column past J: never inside the input
    }
    if (kMode == kLinear) {
        offA0 = (uint32_t)((int32_t)(rowA * G.Cin) + tapOff) * 4u;
        offA = offA0 + c_begin * (kR32 * G.Cin * 4u);
        rowsA = kRowStepA * G.Cin * 4u;
        phase = c_begin % G.period;
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            uint32_t x = (rowA + kRowStepA * (uint32_t)i) % G.W;
            outside[i] = 0;
            for (uint32_t k = 0; k < G.period; ++k) {
                outside[i] |= ((uint32_t)((int32_t)x + tapX) < G.W ? 0u : 1u) << k;
                x += G.step_x;                                       // kR32 modulo W
                x = min(x, x - G.W);
            }
        }
    }
    if (kMode == kGeneral) {
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const uint32_t pos0 = c_begin * kR32 + rowA + kRowStepA * (uint32_t)i;    // the row in the workgroup's first chunk
            y0A[i] = yA[i] = pos0 / G.Wo;
            x0A[i] = xA[i] = pos0 - y0A[i] * G.Wo;
        }
    }
    Chunk32<PA, PB> R;
    // The operands of the sample that is requested, kept as descriptors: formed per piece they were a quarter of the loop's
    // instructions.  `to_event` chunks from now the requests leave the sample, or the last chunk has been requested.
    const uint32_t bytesA = kMode == kPatches ? P * J * 4u : G.H * G.W * G.Cin * 4u, bytesB = P * C * 4u;
    const uint32_t stepA = (kMode == kPatches ? J : G.Cin) * (kR32 * 4u), stepB = C * (kR32 * 4u);
    uint32_t zl = z_begin, todo = total, to_event = min(n_chunks - c_begin, total);
    auto operand = [&](const float* base, uint32_t bytes, uint32_t z, bool live) {
        return make_rsrc(base + (size_t)z * (bytes / 4u), live ? bytes : 0u);
    };
    rsrc_t ra = operand(X, bytesA, z_begin, total > 0u), rb = operand(D, bytesB, z_begin, total > 0u);
    uint32_t offB = offB0 + c_begin * stepB;
    if (kMode == kPatches) offA = offA0 + c_begin * stepA;
    // request of piece i of the chunk (pieces of A, then those of B); past the last chunk the range is empty
    auto issue_into = [&](Chunk32<PA, PB>& Q, int i) {
        if (i >= PA) {
            const uint32_t voff = offB + (uint32_t)(i - PA) * (kRowStepB * C * 4u);
            Q.b[i < PA ? 0 : i - PA] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(rb, (int)voff, 0, 0));
            return;
        }
        const int ia = i < PA ? i : 0;
        uint32_t voff;
        if (kMode == kPatches) {
            voff = offA + (uint32_t)ia * rowsA;
        } else {
            // rows of the input outside the image give an offset that is negative or past the sample: the load answers with
            // zeros; columns outside are masked (as are positions past P in the general mode; in the linear one they alias
            // into pixels of the sample, where the rows of D read as zeros)
            if (kMode == kLinear) {
                voff = (offA + (uint32_t)ia * rowsA) | (uint32_t)__builtin_amdgcn_sbfe((int32_t)outside[ia], phase, 1u);
            } else {
                const int32_t ys = __mul24((int32_t)yA[ia], (int32_t)G.sh), xs = __mul24((int32_t)xA[ia], (int32_t)G.sw);
                const bool inside = ((uint32_t)(xs + tapX) < G.W) & (yA[ia] < G.Ho);
                const int32_t off = __mul24(__mul24(ys, (int32_t)G.W) + xs, (int32_t)G.Cin) + tapOff;
                voff = ((uint32_t)off << 2) | (inside ? 0u : 0xFFFFFFFFu);
            }
        }
        Q.a[ia] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)voff, 0, 0));
    };
    auto issue_done = [&]() {                                     // every piece of the chunk is requested: on to the next
        offB += stepB;
        if (kMode != kGeneral) offA += stepA;
        if (kMode == kLinear) phase = phase + 1u == G.period ? 0u : phase + 1u;
        const bool event = --to_event == 0u;
        if (kMode == kGeneral && !kFew) {
#pragma unroll
            for (int i = 0; i < PA; ++i) {                        // the row of the next chunk: kR32 positions further
                const uint32_t x = xA[i] + G.step_x, xw = x - G.Wo;
                yA[i] += G.step_y + (x >= G.Wo ? 1u : 0u);
                xA[i] = min(x, xw);
            }
        }
        if (event) {
            todo -= min(todo, n_chunks);                          // (a part of a sample is within one)
            offB = offB0;
            if (kMode != kGeneral) offA = offA0;
            phase = 0;
            if (kMode == kGeneral) {
#pragma unroll
                for (int i = 0; i < PA; ++i) { xA[i] = x0A[i]; yA[i] = y0A[i]; }
            }
            ++zl;
            const bool live = todo > 0u;
            to_event = live ? min(n_chunks, todo) : 0x7FFFFFFFu;
            ra = operand(X, bytesA, live ? zl : z_begin, live);
            rb = operand(D, bytesB, live ? zl : z_begin, live);
        }
    };
    // piece i of the requested chunk (those of A, then those of B); rows kRowStep apart differ in the swizzle by a constant
    static_assert(kRowStepA % 8 == 0 && kRowStepB % 8 == 0, "the low bits of the row are the thread's own");
    const uint32_t toA = lds_piece<BM>(rowA, (tid % (BM / 4)) * 4u), toB = lds_piece<BN>(rowB, (tid % (BN / 4)) * 4u);
    u2v sh_, sm_, sl_;                                               // the piece's three planes
    // half h of piece i: two of its four columns; the second half stores the piece and requests the next chunk's
    auto stage_half = [&](uint32_t buf, int i, int h, const Chunk32<PA, PB>& Q, bool next) {     // buf: the parity of the chunk
        const f4v x = i < PA ? Q.a[i < PA ? i : 0] : Q.b[i < PA ? 0 : i - PA];
        const float up = i < PA && buf ? -kUp : kUp;
        uint32_t a, b, c;
        split_pair(x[2 * h] * up, x[2 * h + 1] * up, a, b, c);
        sh_[h] = a; sm_[h] = b; sl_[h] = c;
        if (h == 0) return;
        // (rowA < kRowStepA: where that is 8, bit 3 of the row is that of i kRowStep alone)
        uint8_t* p = i < PA ? shA[buf] + (toA ^ (lds_swizzle<BM>((uint32_t)i * kRowStepA) << 5)) + (uint32_t)i * (kRowStepA * BM * 2)
                            : shB[buf] + (toB ^ (lds_swizzle<BN>((uint32_t)(i - PA) * kRowStepB) << 5)) + (uint32_t)(i - PA) * (kRowStepB * BN * 2);
        const int plane = i < PA ? kPlaneA : kPlaneB;
        *reinterpret_cast<u2v*>(p) = sh_;
        *reinterpret_cast<u2v*>(p + plane) = sm_;
        *reinterpret_cast<u2v*>(p + 2 * plane) = sl_;
        if (next) issue_into(R, i);
    };
    constexpr int kValu = 10;                                        // vector instructions after an MFMA; 4, 7 and 10: 2.265, 2.257, 2.260 ms
    constexpr int kHalves = 2 * (PA + PB), kSlots = 3 * MT;          // a chunk's staging is dealt out over so many places in the loop
    auto stage_slot = [&](uint32_t buf, int s) {
        // (from and to by arithmetic, so that the unrolled loop has one or two turns and every index is a constant)
        const int from = (s * kHalves + kSlots - 1) / kSlots, to = ((s + 1) * kHalves + kSlots - 1) / kSlots;
#pragma unroll
        for (int k = from; k < to; ++k) stage_half(buf, k >> 1, k & 1, R, true);
        if (s == kSlots - 1) issue_done();
    };

    // the lane's place in a transposed fragment (ds_read_b64_tr_b16): rows 8 (lane / 16) .. + 7 of the k-step in two reads
    // of four, of which it addresses row r / 4 (rows r and r + 4 share the swizzle), and the 32-byte unit of the MFMA tile's
    // 16 columns
    // (kFew: the upper half of the wave has the same rows again, of the other plane of a pair)
    const uint32_t r16 = lane & 15u, frow = ((lane >> 4) & (kFew ? 1u : 3u)) * 8u + (r16 >> 2);
    const uint32_t fA = lds_piece<BM>(frow, wm * (uint32_t)WM + 4u * (r16 & 3u)), fB = lds_piece<BN>(frow, wn * (uint32_t)WN + 4u * (r16 & 3u));
    auto frag = [&](const uint8_t* p, int pitch) -> bf8v {
        const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(p));
        const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(p + 4 * pitch));
        s8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf8v, v);
    };

    // the first two chunks are requested before the first is waited for
    {
        Chunk32<PA, PB> first;
#pragma unroll
        for (int i = 0; i < PA + PB; ++i) issue_into(first, i);
        issue_done();
#pragma unroll
        for (int i = 0; i < PA + PB; ++i) issue_into(R, i);
        issue_done();
#pragma unroll
        for (int k = 0; k < kHalves; ++k) stage_half(0, k >> 1, k & 1, first, false);
    }
#pragma unroll
    for (int s = 0; s < 3; ++s) stage_slot(1, s);
    __syncthreads();

    static_assert(MT % 2 == 0, "the fragments' sets go by the row's parity");
    // the products' operands, the smallest first: planes, or (kFew) pairs of planes of which the wave's halves read one each
    constexpr int kProducts = kFew ? 3 : 6, kFragsB = kFew ? 2 : 3;
    constexpr int kPa[6] = {kFew ? 0 : 2, kFew ? 1 : 0, kFew ? 2 : 1, 1, 0, 0}, kPb[6] = {0, kFew ? 1 : 2, 1, 0, 1, 0};
    const bool upper = lane >= 32u;
    const uint32_t planeA[3] = {kFew ? (upper ? 0u : 2u * kPlaneA) : 0u, (uint32_t)kPlaneA, kFew ? 0u : 2u * kPlaneA};
    const uint32_t planeB[3] = {kFew && upper ? 2u * kPlaneB : 0u, kFew && upper ? 0u : (uint32_t)kPlaneB, 2u * kPlaneB};
    bf8v a[2][3], b[2][NTL][kFragsB];                                // row m in set m % 2, chunk q's columns in set q % 2
    auto fetch_a = [&](uint32_t buf, int m, int f) { a[m & 1][f] = frag(shA[buf] + planeA[f] + (fA ^ ((uint32_t)m * 32u)), BM * 2); };
    auto fetch_b = [&](uint32_t buf, int f) {                        // the unit's XOR with the row is the lane's own: tiles XOR in
#pragma unroll
        for (int n = 0; n < NTL; ++n) b[buf][n][f] = frag(shB[buf] + planeB[f] + (fB ^ ((uint32_t)n * 32u)), BN * 2);
    };
    auto order = [](int e, int n) { return kFew ? e : n - 1 - e; };  // of the fragments' fetches: as the products use them
#pragma unroll
    for (int e = 0; e < 3; ++e) { fetch_a(0, 0, order(e, 3)); if (e < kFragsB) fetch_b(0, order(e, kFragsB)); }

    // Chunk q sits in LDS buffer q % 2.  The two waves of a SIMD pass the barrier together and would all multiply, then all
    // convert (measured: matrix and vector time added up), so the conversion of the chunks to come is cut into two-column
    // halves of a thread's pieces and spread between the MFMAs, each slice kept in its place, and a piece is requested
    // again, two chunks on, as soon as its registers are free.  The fragments of the next MFMA row are fetched during this one,
    // those of the next chunk during this one's last row.  The one barrier of a chunk stands before its last row: by then the
    // wave has fetched all of chunk q's fragments and stored its pieces of chunk q + 1; those of chunk q + 2 follow into
    // chunk q's buffer.
    uint32_t left = split_p > 1 ? 0u : n_chunks;                     // chunks until the sample's product is complete (0: never)
    for (uint32_t q0 = 0; q0 < total; q0 += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (u > 0 && q0 + (uint32_t)u >= total) break;
            const uint32_t buf = (uint32_t)u;
            const bool last = kFew || --left == 0;                           // sample finished with this chunk: G_z is complete in acc
            if (last) left = n_chunks;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const bool end = m + 1 == MT;
                const uint32_t fbuf = end ? buf ^ 1u : buf;
                const int fm = end ? 0 : m + 1;
                if (end) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                f4v T[NTL];                                          // the chunk's own sum (of -A B for odd chunks, see above)
#pragma unroll
                for (int n = 0; n < NTL; ++n) T[n] = (f4v){0};
#pragma unroll
                for (int e = 0; e < kProducts; ++e) {
#pragma unroll
                    for (int n = 0; n < NTL; ++n) T[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m & 1][kPa[e]], b[u][n][kPb[e]], T[n], 0, 0, 0);
                    if (e < 3) fetch_a(fbuf, fm, order(e, 3));
                    if (end && e < kFragsB) fetch_b(fbuf, order(e, kFragsB));
                    if (kFew || (e & 1)) {
                        const int slot_ = kFew ? e : e / 2;
                        stage_slot(end ? buf : buf ^ 1u, end ? slot_ : m * 3 + slot_ + 3);
#pragma unroll
                        for (int k = 0; k < (kFew ? 1 : 2) * NTL; ++k) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                            __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (u && !kFew) {
#pragma unroll
                    for (int n = 0; n < NTL; ++n) T[n] = -T[n];
                }
                if (last) {
#pragma unroll
                    for (int n = 0; n < NTL; ++n) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float x = kFew ? T[n][i] * (u ? -kDown : kDown) : (acc[m][n][i] + T[n][i]) * kDown;
                            s_acc[m][n][i] = __builtin_fmaf(x, x, s_acc[m][n][i]);
                            if (kWantG) g_acc[m][n][i] += x;
                        }
                        if (!kFew) acc[m][n] = (f4v){0};
                    }
                } else {
#pragma unroll
                    for (int n = 0; n < NTL; ++n) acc[m][n] = acc[m][n] + T[n];
                }
            }
        }
    }

    // split_p > 1: the partial product itself, for k_sqgrad_reduce_parts; else the scaled result or unscaled partial sums
    const bool direct = (splits == 1);
    const size_t JC = (size_t)J * C;
    float* so = split_p > 1 ? ws + (size_t)split * JC : direct ? s_out : ws + (size_t)split * 2 * JC;
    float* go = direct ? g_out : ws + (size_t)split * 2 * JC + JC;
    const float fs = direct && split_p == 1 ? cs : 1.0f, fg = direct ? cg : 1.0f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NTL; ++n) {
            const uint32_t col = c0 + wn * (uint32_t)WN + n * 16u + (lane & 15u);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t row = j0 + wm * (uint32_t)WM + m * 16u + 4u * (lane >> 4) + (uint32_t)i;
                if (row < J && col < C) {
                    const size_t o = (size_t)row * C + col;
                    __builtin_nontemporal_store(split_p > 1 ? kDown * acc[m][n][i] : fs * s_acc[m][n][i], so + o);
                    if (kWantG) __builtin_nontemporal_store(fg * g_acc[m][n][i], go + o);
                }
            }
        }

    // Tiles with a sum that is not finite are formed again (see form_again); the look at the sums costs 0.6 % of ResNet-50's layers.
    auto top = [](float x) { return __float_as_uint(x) & 0x7FFFFFFFu; };
    uint32_t most = 0;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NTL; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) most = max(most, top(split_p > 1 ? acc[m][n][i] : s_acc[m][n][i]));
    if (__ballot(most >= 0x7F800000u) == 0) return;
    uint32_t again = 0;                                              // one bit per tile
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NTL; ++n) {
            most = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) most = max(most, top(split_p > 1 ? acc[m][n][i] : s_acc[m][n][i]));
            again |= (__ballot(most >= 0x7F800000u) ? 1u : 0u) << (m * NTL + n);
        }
    const uint32_t p_begin = c_begin * kR32, p_end = split_p > 1 ? min(P, (c_begin + total) * kR32) : P;
#pragma unroll 1
    for (; again; again &= again - 1u) {
        const uint32_t tile = (uint32_t)__builtin_ctz(again), m = tile / NTL, n = tile % NTL;
        const uint32_t jt = j0 + wm * (uint32_t)WM + m * 16u, j = jt + (lane & 15u), col = c0 + wn * (uint32_t)WN + n * 16u + (lane & 15u);
        const uint32_t tap = kMode == kPatches ? 0u : j / G.Cin, ky = kMode == kPatches ? 0u : tap / G.kw, kx = tap - ky * G.kw;
        auto valid = [&](uint32_t r) { return jt + r < J && col < C; };
        const Formed F = form_again(
            [&](uint32_t z, uint32_t p) -> float {
                if (j >= J || p >= p_end) return 0.f;
                if (kMode == kPatches) return X[((size_t)z * P + p) * J + j];
                const uint32_t y = p / G.Wo, iy = y * G.sh + ky - G.ph, ix = (p - y * G.Wo) * G.sw + kx - G.pw;
                return iy < G.H && ix < G.W ? X[(((size_t)z * G.H + iy) * G.W + ix) * G.Cin + (j - tap * G.Cin)] : 0.f;
            },
            [&](uint32_t z, uint32_t p) -> float { return col < C && p < p_end ? D[((size_t)z * P + p) * C + col] : 0.f; },
            valid, z_begin, z_end, p_begin, p_end);
        store_formed<kWantG>(F, valid, [&](uint32_t r) -> size_t { return (size_t)(jt + r) * C + col; }, split_p > 1, fs, fg, so, go);
    }
}

// ------------------------------------------------------------------------------------------------
// 3 x 3 filters with unit stride and padding 1.  In the kernel above every element is fetched, cut and stored into LDS once per
// filter tap and column tile, and the instructions that do so take the issue slots that the matrix instructions leave: beyond
// two vector instructions per MFMA the two add up (measured: 7.4 ns a SIMD and MFMA with two, 10.4 with four, 13 with six).  Here
// a workgroup owns all nine taps of 64 input channels times 64 output channels (576 x 64 outputs), and cuts every input pixel
// once: pixels go through a ring in LDS, and the fragment of tap (ky, kx) is read from it at a shift.
//
// For the shift to be the same for all positions, rows are W + 1 pixels long here, the last one a zero: it is the padding to the
// right of its row and to the left of the next.  Position q = y (W + 1) + x of a sample reads ring pixel q + (ky - 1)(W + 1) +
// kx - 1; at x = W the output gradient is zero.  That costs 1 / W more positions (none in whole chunks of 32 at 14 x 14 and 7 x 7).
// A step multiplies 32 positions and takes in the 32 pixels behind those that it reads; samples follow each other in the ring with at
// least W + 2 zeros between their last and first pixels, which pad one's bottom and the other's top.
//
// Eight waves: wave w has channels 16 (w % 4) .. + 15 of the block and one half of the columns: nine MFMA tiles of rows times two
// of columns.  Pieces, products, signs and the sum of a chunk are those of the kernel above; the sign turns on the output
// gradient, since a pixel belongs to several chunks.  With g, whose sums would not fit the registers otherwise, 32 input channels
// and a quarter of the columns a wave.  So that there are as many workgroups then, each takes two of the groups of samples that
// the call without g is split into; the squares of a group are summed by themselves and groups by pairs, here or in the
// reduction: s is the same with g and without.
//
// s alone, batch 32, us before and now: 64 channels at 56 x 56 68 -> 57, 128 at 28 x 28 80 -> 53, 256 at 14 x 14 66 -> 57, 512 at
// 7 x 7 105 -> 67; 512 at 14 x 14, batch 64, 395 -> 275 (215 TFLOP/s); ResNet-50 in one call 2349 -> 2173.  A step takes 2.3 us, the
// MFMAs alone 1.7 at the 2.05 GHz that they leave the clock; layers with one or two samples a workgroup are bound by its
// beginning and end (17 us at 14 x 14) and by the planes of the split.
constexpr int kTapsRing = 248, kTapsMirror = 34;         // pixels; the first ones again at the end, so that a fragment's reads do not wrap
constexpr uint32_t kTapsMaxW = 78;                       // a step's window, the block taken in meanwhile and the pixels between samples fit the ring

// How a sample lies in the ring: n_chunks steps of 32, then `extra` (0 .. 4) pixels more, so that the gap to the next is wide enough.
// A step reads the block of 32 pixels it begins with and the `ahead` next ones.
constexpr uint32_t kTapsAhead = (2 * (kTapsMaxW + 2) + kR32 - 1) / kR32;
static_assert(kR32 * (kTapsAhead + 2) + 4 <= kTapsRing, "what is read and what is taken in are different pixels of the ring");
struct TapsGeom { uint32_t H, W, Cin, n_chunks, extra, ahead; };

template <bool kWantG>
__global__ __launch_bounds__(512, 2)
void k_conv_taps_f32(const float* __restrict__ X, const float* __restrict__ D, uint32_t B, uint32_t C, uint32_t splits, uint32_t split_p,
                     float cg, float cs, float* __restrict__ g_out, float* __restrict__ s_out, float* __restrict__ ws, TapsGeom G) {
    constexpr int kCh = kWantG ? 32 : 64, NTL = kWantG ? 1 : 2;      // input channels of the tile; MFMA tiles of columns of a wave
    // bytes of a pixel, of a position: three planes of bf16, consecutive ones 32 bytes apart in the banks (modulo 256)
    constexpr int kPlaneX = kCh * 2, kPitchX = 3 * kPlaneX + 32, kPlaneD = 128, kPitchD = 3 * kPlaneD + 32;
    static_assert(kPitchX % 64 == 32 && kPitchD % 64 == 32, "eight consecutive ones begin in different banks");
    __shared__ __attribute__((aligned(16))) uint8_t shX[(kTapsRing + kTapsMirror) * kPitchX];
    __shared__ __attribute__((aligned(16))) uint8_t shD[2][kR32 * kPitchD];
    __shared__ f4v shS[kWantG ? 9 * 512 : 1];                        // the first group's sums of s (each thread's own)
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), wc = kWantG ? wave & 1u : wave & 3u, wn = kWantG ? wave >> 1 : wave >> 2;
    const uint32_t tiles_c = (C + 63u) / 64u, tiles_i = (G.Cin + kCh - 1u) / kCh, J = 9u * G.Cin, Wp = G.W + 1u;
    const uint32_t nblk = gridDim.x, per = nblk / 8u, rem = nblk % 8u;
    const uint32_t xcd = blockIdx.x % 8u, slot_x = blockIdx.x / 8u;
    const uint32_t logical = xcd * per + min(xcd, rem) + slot_x;     // contiguous range of tiles per XCD
    const uint32_t tile_c = logical % tiles_c, tile_i = (logical / tiles_c) % tiles_i, split = logical / (tiles_c * tiles_i);
    const uint32_t i0 = tile_i * kCh, c0 = tile_c * 64u;
    const uint32_t n_chunks = G.n_chunks;
    const uint32_t part = split_p > 1 ? split % split_p : 0u;
    const uint32_t chunks_per_part = (n_chunks + split_p - 1) / split_p;
    const uint32_t c_begin = min(n_chunks, part * chunks_per_part);
    const auto z_of = [&](uint32_t g) { return first_sample(min(g, splits), B, splits); };
    const uint32_t z_begin = split_p > 1 ? split / split_p : z_of(kWantG ? 2u * split : split);
    const uint32_t z_end = split_p > 1 ? z_begin + 1u : z_of(kWantG ? 2u * split + 2u : split + 1u);
    const uint32_t total = split_p > 1 ? min(n_chunks, c_begin + chunks_per_part) - c_begin : (z_end - z_begin) * n_chunks;

    f4v acc[9][NTL], s_acc[9][NTL], g_acc[9][NTL];
#pragma unroll
    for (int a = 0; a < 9; ++a)
#pragma unroll
        for (int b = 0; b < NTL; ++b) { acc[a][b] = (f4v){0}; s_acc[a][b] = (f4v){0}; g_acc[a][b] = (f4v){0}; }

    // the sign of the first chunk's sum, by its number in the batch, so that it does not depend on where the workgroup begins
    const float sign = ((z_begin * n_chunks + c_begin) & 1u) ? -1.0f : 1.0f;

    // ---- what the thread takes in: pixel row_ of a block of 32, four channels; position row_ of a chunk, four columns ----
    const uint32_t prow = tid / (kCh / 4), quad = tid % (kCh / 4), drow = tid >> 4, dquad = tid & 15u;
    const bool has_x = kCh == 64 || wave < 4u;
    const uint32_t xch = i0 + quad * 4u, dcol = c0 + dquad * 4u;
    const uint32_t x_off = (uint32_t)(xch < G.Cin) - 1u, d_off = (uint32_t)(dcol < C) - 1u;      // all ones where there is nothing
    // (y, x) of the pixel (position) that the thread requests next; 32 pixels further is step_y rows and step_x columns
    const uint32_t step_y = (uint32_t)kR32 / Wp, step_x = (uint32_t)kR32 - step_y * Wp;
    const uint32_t back_y = n_chunks * kR32 / Wp, back_x = n_chunks * kR32 - back_y * Wp;
    const uint32_t lead = G.W + 2u;
    uint32_t py, px, dy, dx;
    {   // pixel c_begin 32 + prow - lead, from two rows above the image on (lead <= 2 Wp)
        const uint32_t at = c_begin * kR32 + prow + 2u * Wp - lead;
        py = at / Wp;
        px = at - py * Wp;
        py -= 2u;
        const uint32_t pos = c_begin * kR32 + drow;
        dy = pos / Wp;
        dx = pos - dy * Wp;
    }
    auto advance = [&](uint32_t& y, uint32_t& x) {
        x += step_x;
        const uint32_t xw = x - Wp;
        y += step_y + (x >= Wp ? 1u : 0u);
        x = min(x, xw);
    };
    auto rewind = [&](uint32_t& y, uint32_t& x) {                    // to the start of a sample
        y -= back_y + (x < back_x ? 1u : 0u);
        x = x < back_x ? x + Wp - back_x : x - back_x;
    };
    const uint32_t x_bytes = G.H * G.W * G.Cin * 4u, d_bytes = G.H * G.W * C * 4u;
    uint32_t zx = z_begin, bx = c_begin, zd = z_begin, bd = c_begin; // sample and block (chunk) requested next
    auto operand = [&](const float* base, uint32_t bytes, uint32_t z) {
        return make_rsrc(base + (size_t)(z < z_end ? z : z_begin) * (bytes / 4u), z < z_end ? bytes : 0u);
    };
    rsrc_t rx = operand(X, x_bytes, z_begin), rd = operand(D, d_bytes, z_begin);
    f4v RX = {0}, RD = {0}, RE = {0};
    auto load_at = [&](rsrc_t r, uint32_t y, uint32_t x, uint32_t ch, uint32_t width, uint32_t off) -> f4v {
        const uint32_t at = (uint32_t)__mul24(__mul24((int)y, (int)G.W) + (int)x, (int)width) + ch;
        const bool inside = (y < G.H) & (x < G.W);
        return __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, (int)((at << 2) | off | (inside ? 0u : 0xFFFFFFFFu)), 0, 0));
    };
    auto request_x = [&]() {
        if (has_x) RX = load_at(rx, py, px, xch, G.Cin, x_off);
        advance(py, px);
        if (++bx == n_chunks) {
            // the pixels beyond the sample's last block, by the first wave: thread row 0 .. 3 stands at exactly those
            if (G.extra && wave == 0u) RE = load_at(rx, py, px, xch, G.Cin, x_off | ((uint32_t)(prow < G.extra) - 1u));
            bx = 0;
            rx = operand(X, x_bytes, ++zx);
            rewind(py, px);
        }
    };
    auto request_d = [&]() {
        RD = load_at(rd, dy, dx, dcol, C, d_off);
        advance(dy, dx);
        if (++bd == n_chunks) { bd = 0; rd = operand(D, d_bytes, ++zd); rewind(dy, dx); }
    };
    // ---- into LDS ----
    uint32_t slot_w = 0, bw = c_begin;                               // ring slot of the block stored next, and its number in the sample
    auto store_pixel = [&](uint32_t slot, u2v h, u2v m, u2v l) {
        uint8_t* p = shX + slot * kPitchX + quad * 8u;
        *reinterpret_cast<u2v*>(p) = h;
        *reinterpret_cast<u2v*>(p + kPlaneX) = m;
        *reinterpret_cast<u2v*>(p + 2 * kPlaneX) = l;
    };
    auto cut = [&](const f4v& v, float up, u2v& h, u2v& m, u2v& l) {
        uint32_t a, b, c;
        split_pair(v[0] * up, v[1] * up, a, b, c);
        h[0] = a; m[0] = b; l[0] = c;
        split_pair(v[2] * up, v[3] * up, a, b, c);
        h[1] = a; m[1] = b; l[1] = c;
    };
    auto put_x = [&](uint32_t first, const f4v& v) {                 // pixel prow of those from ring slot `first` on
        if (!has_x) return;
        u2v h, m, l;
        cut(v, kUp, h, m, l);
        uint32_t slot = first + prow;
        slot = min(slot, slot - (uint32_t)kTapsRing);
        store_pixel(slot, h, m, l);
        if (first < (uint32_t)kTapsMirror || first + kR32 > (uint32_t)kTapsRing)
            if (slot < (uint32_t)kTapsMirror) store_pixel(slot + kTapsRing, h, m, l);
    };
    auto ring = [](uint32_t s) { return s >= (uint32_t)kTapsRing ? s - (uint32_t)kTapsRing : s; };
    auto stage_x = [&]() {
        put_x(slot_w, RX);
        slot_w = ring(slot_w + kR32);
        if (++bw == n_chunks) {
            bw = 0;
            if (G.extra) {
                if (wave == 0u && prow < G.extra) put_x(slot_w, RE);
                slot_w = ring(slot_w + G.extra);
            }
        }
        request_x();
    };
    auto put_d = [&](uint32_t buf, float up) {
        u2v h, m, l;
        cut(RD, up, h, m, l);
        uint8_t* p = shD[buf] + drow * kPitchD + dquad * 8u;
        *reinterpret_cast<u2v*>(p) = h;
        *reinterpret_cast<u2v*>(p + kPlaneD) = m;
        *reinterpret_cast<u2v*>(p + 2 * kPlaneD) = l;
    };

    // ---- fragments: lanes 16 g .. + 15 have k = 8 g .. + 7, which are positions 4 g .. + 3 and 16 + 4 g .. + 3 of the chunk: a
    // transposing read then takes eight consecutive rows per pass over the banks ----
    const uint32_t r16 = lane & 15u, frow = (lane >> 4) * 4u + (r16 >> 2);
    const uint32_t fX = frow * kPitchX + wc * 32u + 8u * (r16 & 3u);
    const uint32_t fD = frow * kPitchD + wn * (uint32_t)(NTL * 32) + 8u * (r16 & 3u);
    auto frag = [&](const uint8_t* p, int pitch) -> bf8v {
        const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(p));
        const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(p + 16 * pitch));
        s8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf8v, v);
    };
    uint32_t slot_r = 0, br = c_begin;                               // ring slot of the step's first pixel; the step's number in the sample
    uint32_t at[3];                                                  // the lane's byte offset in the ring for filter row ky
    auto place = [&]() {
#pragma unroll
        for (uint32_t ky = 0; ky < 3; ++ky) at[ky] = fX + __builtin_amdgcn_readfirstlane(ring(slot_r + ky * Wp)) * kPitchX;
    };
    // Taps are multiplied one at a time, or with one column of tiles two at a time, for two independent chains of MFMAs.
    constexpr int kGroup = 2 / NTL, kGroups = (9 + kGroup - 1) / kGroup;
    static_assert(kGroups % 2 == 1, "the fragments' sets change places from step to step");
    bf8v a[2][kGroup][3], b[NTL][3];
    auto fetch_a = [&](int set, int group, int f) {
#pragma unroll
        for (int k = 0; k < kGroup; ++k) {
            const int tap = group * kGroup + k;
            if (tap < 9) a[set][k][f] = frag(shX + at[tap / 3 % 3] + (tap % 3) * kPitchX + f * kPlaneX, kPitchX);
        }
    };
    auto fetch_b = [&](uint32_t buf, int f) {
#pragma unroll
        for (int n = 0; n < NTL; ++n) b[n][f] = frag(shD[buf] + fD + n * 32 + f * kPlaneD, kPitchD);
    };

    // ---- the blocks that the first step needs, all requested before the first is waited for ----
    {
        constexpr int kMost = (int)kTapsAhead;
        f4v first[kMost + 1], extra[kMost + 1];
#pragma unroll
        for (int i = 0; i <= kMost; ++i)
            if ((uint32_t)i <= G.ahead) { request_x(); first[i] = RX; extra[i] = RE; }
        request_d();
        const f4v d0 = RD;
        request_x();
        request_d();
        const f4v nextx = RX, nexte = RE, nextd = RD;
#pragma unroll
        for (int i = 0; i <= kMost; ++i)
            if ((uint32_t)i <= G.ahead) {
                put_x(slot_w, first[i]);
                slot_w = ring(slot_w + kR32);
                if (++bw == n_chunks) {
                    bw = 0;
                    if (G.extra) {
                        if (wave == 0u && prow < G.extra) put_x(slot_w, extra[i]);
                        slot_w = ring(slot_w + G.extra);
                    }
                }
            }
        RX = nextx; RE = nexte;
        RD = d0;
        put_d(0, sign * kUp);
        RD = nextd;
    }
    __syncthreads();
    place();
    constexpr int kPa[6] = {2, 0, 1, 1, 0, 0}, kPb[6] = {0, 2, 1, 0, 1, 0};   // the smallest products first
    constexpr int kOrder[3] = {2, 0, 1};                             // planes in the order in which the products use them
#pragma unroll
    for (int e = 0; e < 3; ++e) { fetch_a(0, 0, kOrder[e]); fetch_b(0, e); }

    // the sums, the products of a part, or the scaled result go here; the lane's output i of tile (t, n)
    const bool direct = (splits <= (kWantG ? 2u : 1u) && split_p == 1);
    const size_t JC = (size_t)J * C;
    float* so = direct ? s_out : ws + (size_t)split * (kWantG ? 2 : 1) * JC;
    float* go = direct ? g_out : ws + (size_t)split * 2 * JC + JC;
    const float fs = direct ? cs : 1.0f, fg = direct ? cg : 1.0f;
    const uint32_t out_ch = i0 + wc * 16u + 4u * (lane >> 4), out_col = c0 + wn * (uint32_t)(NTL * 16) + (lane & 15u);
    auto each_out = [&](auto f) __attribute__((always_inline)) {
        uint32_t ch = out_ch;
        asm("" : "+v"(ch));                                          // or the addresses are kept in registers through the loop
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int n = 0; n < NTL; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (ch + (uint32_t)i < G.Cin && out_col + (uint32_t)n * 16u < C)
                        f(t, n, i, (size_t)((uint32_t)t * G.Cin + ch + (uint32_t)i) * C + out_col + (uint32_t)n * 16u);
    };

    f4v T[2][kGroup][NTL];                                           // this group's sums and those of the one before it
    uint32_t left = split_p > 1 ? 0u : n_chunks;                     // steps until the sample's product is complete (0: never)
    int32_t to_second = kWantG ? (int32_t)(z_of(2u * split + 1u) - z_begin) : 1;   // samples until the second group; then at most 0
    // from four samples a group on, g is summed by groups too (16 samples in a row, 512 -> 512 at 7 x 7: error 9.3e-8, 8.2e-8 so; 6 us)
    const bool halve_g = to_second >= 4;
    // Step q multiplies chunk q from D buffer q % 2 and takes in the next step's pixels and positions.  The fragments of the next
    // tap are fetched during this one.  The one barrier of a step stands before its last tap: by then the wave has fetched all
    // of the step's fragments and stored its share of the next step's input; the fragments of the next step's first tap follow.
    for (uint32_t q0 = 0; q0 < total; q0 += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (u > 0 && q0 + (uint32_t)u >= total) break;
            const bool last = --left == 0;
            if (last) left = n_chunks;
            auto add = [&](int group) {
                const float turn = u ? -sign : sign;
#pragma unroll
                for (int k = 0; k < kGroup; ++k) {
                    const int t = group * kGroup + k;
                    if (t >= 9) break;
                    f4v (&V)[NTL] = T[group & 1][k];
#pragma unroll
                    for (int n = 0; n < NTL; ++n)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[t][n][i] = __builtin_fmaf(V[n][i], turn, acc[t][n][i]);
                    if (!last) continue;
#pragma unroll
                    for (int n = 0; n < NTL; ++n) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float x = acc[t][n][i] * kDown;
                            s_acc[t][n][i] = __builtin_fmaf(x, x, s_acc[t][n][i]);
                            if (kWantG) g_acc[t][n][i] += x;
                        }
                        acc[t][n] = (f4v){0};
                    }
                }
            };
#pragma unroll
            for (int h = 0; h < kGroups; ++h) {
                const int set = (h + u) & 1;
                if (h == kGroups / 3) stage_x();
                if (h == kGroups * 2 / 3) { put_d(u ^ 1u, (u ? sign : -sign) * kUp); request_d(); }
                if (h == kGroups - 1) {
                    slot_r += kR32;
                    if (++br == n_chunks) { br = 0; slot_r += G.extra; }
                    slot_r = ring(slot_r);
                    place();
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                __builtin_amdgcn_sched_barrier(0);
                f4v (&V)[kGroup][NTL] = T[h & 1];
#pragma unroll
                for (int k = 0; k < kGroup; ++k)
#pragma unroll
                    for (int n = 0; n < NTL; ++n) V[k][n] = (f4v){0};
#pragma unroll
                for (int e = 0; e < 6; ++e) {
#pragma unroll
                    for (int k = 0; k < kGroup; ++k)
#pragma unroll
                        for (int n = 0; n < NTL; ++n)
                            if (h * kGroup + k < 9) V[k][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[set][k][kPa[e]], b[n][kPb[e]], V[k][n], 0, 0, 0);
                    if (e < 3) fetch_a(set ^ 1, h == kGroups - 1 ? 0 : h + 1, kOrder[e]);
                    if (h == kGroups - 1) {                          // each plane of the positions after its last use
                        if (e == 1) fetch_b(u ^ 1u, 2);
                        if (e == 4) fetch_b(u ^ 1u, 1);
                        if (e == 5) fetch_b(u ^ 1u, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    // a group's sums are added while the next one's products run
                    if (e == 2 && h > 0) { add(h - 1); __builtin_amdgcn_sched_barrier(0); }
                }
            }
            add(kGroups - 1);
            if (kWantG && last && --to_second == 0) {                // the first group's sums of s wait in LDS, those of g in memory
#pragma unroll
                for (int t = 0; t < 9; ++t) { shS[t * 512 + tid] = s_acc[t][0]; s_acc[t][0] = (f4v){0}; }
                if (halve_g) {
                    each_out([&](int t, int n, int i, size_t o) { go[o] = g_acc[t][n][i]; });
#pragma unroll
                    for (int t = 0; t < 9; ++t) g_acc[t][0] = (f4v){0};
                }
            }
        }
    }

    // one bit per tile with a sum that is not finite: of a group's squares each by itself, so that with g as without only that group's
    // are formed again, and the other's stay (in shS from then on)
    uint32_t again = 0, again_first = 0;
    if (kWantG && to_second <= 0) {
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const f4v first = shS[t * 512 + tid], second = s_acc[t][0];
            s_acc[t][0] = first + second;
            again |= (not_finite(second) ? 1u : 0u) << t;
            if (not_finite(first)) {
                again_first |= 1u << t;
                shS[t * 512 + tid] = second;
            }
        }
        if (halve_g) each_out([&](int t, int n, int i, size_t o) { g_acc[t][n][i] = go[o] + g_acc[t][n][i]; });
    } else {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int n = 0; n < NTL; ++n) again |= (not_finite(split_p > 1 ? acc[t][n] : s_acc[t][n]) ? 1u : 0u) << (t * NTL + n);
    }
    each_out([&](int t, int n, int i, size_t o) {
        const float out = split_p > 1 ? kDown * acc[t][n][i] : fs * s_acc[t][n][i];
        if (direct) __builtin_nontemporal_store(out, so + o);
        else so[o] = out;                                            // read again at once by the reduction
        if (kWantG) {
            if (direct) __builtin_nontemporal_store(fg * g_acc[t][n][i], go + o);
            else go[o] = fg * g_acc[t][n][i];
        }
    });
    if ((again | again_first) == 0) return;
    const uint32_t q_begin = c_begin * kR32, q_end = min((uint32_t)(G.H * Wp), split_p > 1 ? (c_begin + total) * kR32 : G.H * Wp);
#pragma unroll 1
    for (uint32_t rest = again | again_first; rest; rest &= rest - 1u) {
        const uint32_t tile = (uint32_t)__builtin_ctz(rest), t = tile / NTL, n = tile % NTL, ky = t / 3u, kx = t - 3u * ky;
        const uint32_t chm = i0 + wc * 16u, colm = c0 + wn * (uint32_t)(NTL * 16) + n * 16u, ch = chm + (lane & 15u), col = colm + (lane & 15u);
        auto valid = [&](uint32_t r) { return chm + r < G.Cin && col < C; };
        auto form = [&](uint32_t z0, uint32_t z1) {
            return form_again(
                [&](uint32_t z, uint32_t q) -> float {
                    const uint32_t y = q / Wp, x = q - y * Wp, iy = y + ky - 1u, ix = x + kx - 1u;
                    return ch < G.Cin && q < q_end && x < G.W && iy < G.H && ix < G.W ? X[(((size_t)z * G.H + iy) * G.W + ix) * G.Cin + ch] : 0.f;
                },
                [&](uint32_t z, uint32_t q) -> float {
                    const uint32_t y = q / Wp, x = q - y * Wp;
                    return col < C && q < q_end && x < G.W ? D[(((size_t)z * G.H + y) * G.W + x) * C + col] : 0.f;
                },
                valid, z0, z1, q_begin, q_end);
        };
        Formed F;
        if (kWantG && to_second <= 0) {
            const uint32_t z_second = z_of(2u * split + 1u);
            F = form(z_begin, z_second);
            Formed second = form(z_second, z_end);
            if (!(again_first >> t & 1u)) F.s = shS[t * 512 + tid];
            else if (!(again >> t & 1u)) second.s = shS[t * 512 + tid];
            F.s = F.s + second.s;
            F.g = F.g + second.g;
        } else {
            F = form(z_begin, z_end);
        }
        store_formed<kWantG>(F, valid, [&](uint32_t r) -> size_t { return (size_t)(t * G.Cin + chm + r) * C + col; }, split_p > 1, fs, fg, so, go);
    }
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
bool conv_f32_tiled_supported(uint32_t P, uint32_t J, uint32_t C) {
    const uint64_t limit = 0x7FFFFFFFull;
    return J % 4 == 0 && C % 4 == 0 && (uint64_t)(P + 16) * J * 4 < limit && (uint64_t)(P + 16) * C * 4 < limit;
}

// Block tile of the float32 conv kernel for a shape: 64 instead of 128 rows (columns) where that wastes at
// least a fifth fewer of them (J or C at most 64, or just past a multiple of 128).  256 rows were tried: 10 to 15 % faster
// where every compute unit gets eight samples or more (14 x 14, 256 -> 256, 3 x 3 at batch 256: 315 us against 354), slower
// below (batch 32: 65 against 60), and s would depend on whether g is asked for, whose accumulators that tile has no room for.
struct F32Tile { uint32_t bm, bn; };
static uint32_t f32_tile_edge(uint32_t n) {
    const uint32_t pad128 = (n + 127) / 128 * 128, pad64 = (n + 63) / 64 * 64;
    return pad64 * 5 <= pad128 * 4 ? 64u : 128u;
}
static F32Tile conv_f32_tile(uint32_t J, uint32_t C) { return F32Tile{f32_tile_edge(J), f32_tile_edge(C)}; }
static uint64_t conv_f32_tiles(const F32Tile& t, uint32_t J, uint32_t C) {
    return (uint64_t)((J + t.bm - 1) / t.bm) * ((C + t.bn - 1) / t.bn);
}
// Workgroups resident at once: as many as 160 KB of LDS hold at two staged chunks each (one of 128 x 128, two of 128 x 64,
// three of 64 x 64).
static uint64_t conv_f32_slots(const F32Tile& t) {
    const uint64_t lds = 2ull * 3 * kR32 * (t.bm + t.bn) * sizeof(uint16_t);
    return 256 * ((160ull * 1024) / lds);
}

// How a shape's work is divided: the samples over `splits` workgroups per tile, or (split_p > 1) every sample's positions
// over split_p of them, for `slots` workgroups at once and chunks of `chunk` positions.  most: bytes of workspace; pairs: a
// split of the samples leaves one plane of [J, C] in it, or with g a pair of them two (see k_conv_taps_f32), else each two.
// least: of splits of the samples, where the workspace has room for as many; 1 split where it has not.
struct F32Split { uint32_t splits, split_p; };
static size_t f32_split_bytes(const F32Split& r, uint32_t J, uint32_t C, bool pairs) {
    const size_t JC = (size_t)J * C * sizeof(float);
    return r.split_p > 1 ? (size_t)r.splits * JC : r.splits > 1 ? (size_t)(pairs ? r.splits + r.splits % 2 : r.splits * 2) * JC : 0;
}
static F32Split f32_split(uint64_t tiles, uint64_t slots, uint32_t chunk, uint32_t B, uint32_t P, uint32_t J, uint32_t C, size_t most,
                          bool pairs = false, uint32_t least = 1) {
    const uint32_t n_chunks = (P + chunk - 1) / chunk;
    F32Split r{1, 1};
    if (tiles * B * 3 <= slots * 2 && n_chunks >= 256u / chunk) {
        // up to half a round: as many parts as fill one round; up to two thirds: just under two rounds
        const uint64_t sp = tiles * B * 2 <= slots ? slots / (tiles * B) : 2 * slots / (tiles * B);
        r.split_p = (uint32_t)(sp < n_chunks * chunk / 128u ? sp : n_chunks * chunk / 128u);
        while (r.split_p > 1 && f32_split_bytes(F32Split{B * r.split_p, r.split_p}, J, C, pairs) > most) --r.split_p;
        if (r.split_p > 1) { r.splits = B * r.split_p; return r; }
        r.split_p = 1;
    }
    // of the numbers of splits with the same largest number of samples the smallest; the next has fewer samples
    double best = 1e300;
    for (uint32_t s = 1, zper = B;; s = (B + zper - 2) / (zper - 1), zper = (B + s - 1) / s) {
        if (s >= least && f32_split_bytes(F32Split{s, 1}, J, C, pairs) <= most) {
            const uint64_t rounds = (tiles * s + slots - 1) / slots;
            const double cost = (double)rounds * zper + (s > 1 ? 0.5 * s * (double)tiles / slots + 0.5 : 0.0);
            if (cost < best - 1e-9) { best = cost; r.splits = s; }
        }
        if (zper == 1) return r;
    }
}
// The workspace a shape asks for, which is also what vgc_sqgrad_noalloc accepts or refuses it by, is a rule of its own: what
// two, four or six workgroups per compute unit of 128 x 128, 128 x 64 and 64 x 64 tiles would fill.  The kernel has fewer and
// larger workgroups in flight and needs less for nearly all shapes; where it would need more it splits less.
size_t conv_f32_workspace_bytes(uint32_t B, uint32_t P, uint32_t J, uint32_t C) {
    const F32Tile t = conv_f32_tile(J, C);
    const uint64_t slots = 256 * (t.bm + t.bn == 256 ? 2 : t.bm + t.bn == 192 ? 4 : 6);
    return f32_split_bytes(f32_split(conv_f32_tiles(t, J, C), slots, 16, B, P, J, C, ~(size_t)0), J, C, false);
}

// What k_conv_f32 would do with a shape: its tile and split; space: whether the caller's workspace is as large as asked for.
struct F32Way { F32Tile t; size_t asked; bool space; F32Split sp; };
static F32Way conv_f32_way(uint32_t B, uint32_t P, uint32_t J, uint32_t C, bool workspace, size_t workspace_bytes) {
    F32Way w{conv_f32_tile(J, C), conv_f32_workspace_bytes(B, P, J, C), false, {1, 1}};
    w.space = workspace && workspace_bytes >= w.asked;
    if (w.space) w.sp = f32_split(conv_f32_tiles(w.t, J, C), conv_f32_slots(w.t), kR32, B, P, J, C, w.asked);
    return w;
}

template <int kMode>
static int launch_conv_f32_any(const F32Way& way, const void* X, const void* D, uint32_t B, uint32_t P, uint32_t J, uint32_t C, float c,
                               float* g_out, float* s_out, void* workspace, const ConvGeom& G, hipStream_t stream) {
    const size_t JC = (size_t)J * C;
    const F32Tile t = way.t;
    const uint32_t splits = way.sp.splits, split_p = way.sp.split_p;
    // with the positions split the partial products are unsquared: the variant without g serves both
    const bool with_g = g_out && split_p == 1;
    const uint64_t nblk = conv_f32_tiles(t, J, C) * splits;
    if (nblk > 0x7FFFFFFFull) { set_error("vgc_sqgrad: shape exceeds the launch limit"); return VGC_ERR_SIZE; }
    const float cg = c, cs = c * c;
    float* ws = static_cast<float*>(workspace);
    const float* Xf = static_cast<const float*>(X);
    const float* Df = static_cast<const float*>(D);
#define VGC_LAUNCH_F32(G_, BM_, BN_, WM_, WN_, FEW_)                                                                       \
    hipLaunchKernelGGL((k_conv_f32<G_, kMode, BM_, BN_, WM_, WN_, FEW_>), dim3((uint32_t)nblk),                        \
                       dim3((BM_ / WM_) * (BN_ / WN_) * 64), 0, stream, Xf, Df, B, P, J, C, splits, split_p, cg, cs, g_out, s_out, ws, G)
#define VGC_LAUNCH_F32_TILES(G_, FEW_)                                                                                     \
    do {                                                                                                                   \
        if (t.bm == 128 && t.bn == 128) VGC_LAUNCH_F32(G_, 128, 128, 64, 32, FEW_);                                        \
        else if (t.bm == 128) VGC_LAUNCH_F32(G_, 128, 64, 64, 32, FEW_);                                                   \
        else if (t.bn == 128) VGC_LAUNCH_F32(G_, 64, 128, 64, 32, FEW_);                                                   \
        else VGC_LAUNCH_F32(G_, 64, 64, 32, 32, FEW_);                                                                     \
    } while (0)
    constexpr bool kHasFew = kMode != kLinear;
    if (kHasFew && P <= kR32 / 2) {
        if (with_g) VGC_LAUNCH_F32_TILES(true, kHasFew);
        else VGC_LAUNCH_F32_TILES(false, kHasFew);
    } else if (with_g) VGC_LAUNCH_F32_TILES(true, false);
    else VGC_LAUNCH_F32_TILES(false, false);
#undef VGC_LAUNCH_F32_TILES
#undef VGC_LAUNCH_F32
    if (split_p > 1) launch_sqgrad_reduce_parts(ws, B, split_p, JC, cg, cs, g_out, s_out, stream);
    else if (splits > 1) launch_sqgrad_reduce(ws, splits, JC, cg, cs, g_out, s_out, stream);
    return hip_check(hipGetLastError(), "launch k_conv_f32");
}

// ---- 3 x 3, unit stride, padding 1: k_conv_taps_f32 ----
static TapsGeom taps_geom(uint32_t H, uint32_t W, uint32_t Cin) {
    const uint32_t span = H * (W + 1) - 1, lead = W + 2;                 // from the first to the last pixel; zeros needed between samples
    TapsGeom G{H, W, Cin, (span + kR32 - 1) / kR32, 0, (2 * lead + kR32 - 1) / kR32};
    const uint32_t room = G.n_chunks * kR32;
    if (span + lead > room) {
        if (span + lead - room <= 4) G.extra = span + lead - room;       // (14 x 14: 225 and 224)
        else G.n_chunks = (span + lead + kR32 - 1) / kR32;
    }
    return G;
}
// About how long a shape takes, in us: 3.5 and rounds of workgroups, each of which begins and ends in `begin` and takes `step` for each of
// its chunks, and the planes that it leaves, written and read again at 5 TB/s with a launch of 4; parts of samples are added by 16
// threads for a sample's four outputs, most of them idle with few samples: 9 per million outputs.
static double f32_us(uint64_t workgroups, uint64_t slots, uint64_t chunks, double begin, double step, uint32_t planes, bool parts, uint32_t J, uint32_t C) {
    const double rounds = (double)((workgroups + slots - 1) / slots), JC = (double)J * C;
    return 3.5 + rounds * (begin + (double)chunks * step) + (planes ? 4.0 + planes * JC * 8.0 / 5e6 : 0.0) + (parts ? JC * 9e-6 : 0.0);
}
static uint64_t f32_chunks(const F32Split& s, uint32_t B, uint32_t n_chunks) {           // of a workgroup
    return s.split_p > 1 ? (n_chunks + s.split_p - 1) / s.split_p : (uint64_t)((B + s.splits - 1) / s.splits) * n_chunks;
}

// Which of the two kernels takes a shape follows from that estimate, whose steps were measured: 1.45 us a chunk with 128 x 128 tiles,
// 1.55 with two workgroups of half of that per compute unit, 2.35 for the 576 x 64 of k_conv_taps_f32, and 1.45 for its 288 x 64 with g.
// Both forms of a call have to take the same way, so that s is the same: k_conv_taps_f32 where it is 6 % faster without g and not
// slower with it.  Estimated and measured times, k_conv_f32 / k_conv_taps_f32, batch 32: 512 channels at 7 x 7 118 / 67 and 104 / 68; 256 at
// 14 x 14 71 / 62 and 67 / 58; 128 at 28 x 28 90 / 63 and 81 / 55; 64 at 56 x 56 71 / 66 and 69 / 58; what goes to
// k_conv_f32: 256 at 14 x 14, batch 33 71 / 74 and 63 / 67; 192 -> 160 at 14 x 14 51 / 54 and 50 / 51; 256 at 8 x 8, batch 64
// 50 / 57 and 47 / 57; 128 at 14 x 14, batch 7 26 / 32 and 21 / 28.  With g: 512 at 7 x 7 144 / 77 and 120 / 81; 256 at 14 x 14 78 / 71 and
// 66 / 63; 64 -> 640 at 30 x 15, batch 111 287 / 261 and 256 / 255.  Half the channels a workgroup often make two rounds of one there:
// 64 -> 832 at 50 x 7, batch 182 439 / 792 and 406 / 742, 408 -> 448 at 8 x 9, batch 19 75 / 117 and 62 / 117, for 10 to 36 %
// without g.  Of 190 shapes about the line the 96 that come here take 0.45 to 1.03 of
// k_conv_f32's time with g and 0.50 to 0.96 without; the others would have taken 0.88 to 1.90, 1.15 in the mean.
//
// The errors must not grow by that.  The part of them that depends on the split is the rounding of a group's sums, added in a row: for s
// with n samples in each of m groups about n / (3 m) times one addition's, squared.  The tiles here are larger, so that a layer of many
// channels fills the chip with fewer and longer groups: 1024 -> 1024 at 7 x 7, batch 64, in one group of 64 had errors of 1.22e-7 (s)
// and 1.54e-7 (g), k_conv_f32 0.53e-7 and 0.97e-7.  So n / m may be 2 more than there; beyond that the samples are split further:
// 0.51e-7 and 0.96e-7, 372 us instead of 325 (k_conv_f32 497); 512 -> 512 at 14 x 14, batch 128, 0.57e-7 -> 0.50e-7, 546 -> 558 us (752).
// Of 108 shapes, 72 of which are split further by this, s errs by 0.84 to 1.05 (mean 0.99) and g by 0.83 to 1.12 (mean 1.00) of what
// k_conv_f32 does, without the limit by up to 2.29 and 1.59.  Those 72 take 0.65 to 0.99 of its time without g and 0.67 to 1.07 with g
// (without the limit 0.61 to 0.89 and 0.54 to 2.1).  The layers of ResNet-50 and VGG-16 at batch 32 and 64 keep their splits.
static bool conv_taps_f32_way(const F32Way& way, uint32_t B, uint32_t H, uint32_t W, uint32_t Cin, uint32_t C, TapsGeom& G, F32Split& sp) {
    if (W > kTapsMaxW || H * W <= kR32 / 2) return false;
    G = taps_geom(H, W, Cin);
    const uint32_t J = 9 * Cin, P = H * W, tiles_c = (C + 63) / 64;
    const uint64_t tiles = (uint64_t)((Cin + 63) / 64) * tiles_c;
    const F32Tile t = way.t;
    const F32Split other = way.sp;
    // a group's samples for each group: see above
    const double samples = other.split_p > 1 ? 0.0 : (double)B / ((double)other.splits * other.splits);
    const uint32_t least = (uint32_t)std::ceil(std::sqrt(B / (samples + 2.0)) - 1e-9);
    sp = way.space ? f32_split(tiles, 256, kR32, B, G.n_chunks * kR32, J, C, way.asked, true, least) : F32Split{1, 1};
    if (sp.split_p == 1 && sp.splits < least) return false;
    const bool parts = sp.split_p > 1, other_parts = other.split_p > 1;
    const uint64_t chunks = f32_chunks(sp, B, G.n_chunks), other_chunks = f32_chunks(other, B, (P + kR32 - 1) / kR32);
    auto general = [&](bool g) {
        const uint32_t planes = other.splits > 1 ? other.splits * (g && !other_parts ? 2 : 1) : 0;
        return f32_us(conv_f32_tiles(t, J, C) * other.splits, conv_f32_slots(t), other_chunks, 6.5, t.bm + t.bn == 256 ? 1.45 : 1.55, planes, other_parts, J, C);
    };
    if (f32_us(tiles * sp.splits, 256, chunks, 6.5, 2.35, sp.splits > 1 ? sp.splits : 0, parts, J, C) > 0.94 * general(false)) return false;
    if (parts) return true;                                              // the variant without g serves both
    const uint32_t blocks = (sp.splits + 1) / 2;
    return f32_us((uint64_t)((Cin + 31) / 32) * tiles_c * blocks, 256, chunks * (sp.splits > 1 ? 2 : 1), 7.8, 1.45, blocks > 1 ? 2 * blocks : 0, false, J, C) <=
           general(true);
}
// How many splits k_conv_taps_f32 takes a layer in, 0 where k_conv_f32 takes it.
uint32_t conv_taps_f32_splits(uint32_t B, uint32_t H, uint32_t W, uint32_t Cin, uint32_t C, bool workspace) {
    TapsGeom G;
    F32Split sp;
    return conv_taps_f32_way(conv_f32_way(B, H * W, 9 * Cin, C, workspace, ~(size_t)0), B, H, W, Cin, C, G, sp) ? sp.splits : 0u;
}

// 0 or an error: launched; 1: k_conv_f32 takes the shape.
static int launch_conv_taps_f32(const F32Way& way, const void* X, const void* D, uint32_t B, uint32_t H, uint32_t W, uint32_t Cin,
                                uint32_t C, float c, float* g_out, float* s_out, void* workspace, hipStream_t stream) {
    TapsGeom G;
    F32Split sp;
    if (!conv_taps_f32_way(way, B, H, W, Cin, C, G, sp)) return 1;
    const size_t JC = (size_t)9 * Cin * C;
    const bool with_g = g_out && sp.split_p == 1;
    const uint32_t blocks = with_g ? (sp.splits + 1) / 2 : sp.splits;
    const uint64_t nblk = (uint64_t)(with_g ? (Cin + 31) / 32 : (Cin + 63) / 64) * ((C + 63) / 64) * blocks;
    if (nblk > 0x7FFFFFFFull) { set_error("vgc_sqgrad: shape exceeds the launch limit"); return VGC_ERR_SIZE; }
    const float cg = c, cs = c * c;
    float* ws = static_cast<float*>(workspace);
#define VGC_LAUNCH_TAPS(G_)                                                                                                \
    hipLaunchKernelGGL((k_conv_taps_f32<G_>), dim3((uint32_t)nblk), dim3(512), 0, stream, static_cast<const float*>(X), \
                       static_cast<const float*>(D), B, C, sp.splits, sp.split_p, cg, cs, g_out, s_out, ws, G)
    if (with_g) VGC_LAUNCH_TAPS(true);
    else VGC_LAUNCH_TAPS(false);
#undef VGC_LAUNCH_TAPS
    if (sp.split_p > 1) launch_sqgrad_reduce_parts(ws, B, sp.split_p, JC, cg, cs, g_out, s_out, stream);
    else if (blocks > 1) launch_sqgrad_reduce(ws, blocks, JC, cg, cs, g_out, s_out, stream, with_g ? ReducePlanes::kPairsDone : ReducePlanes::kPairs);
    return hip_check(hipGetLastError(), "launch k_conv_taps_f32");
}

int launch_conv_f32_tiled(const void* X, const void* D, uint32_t B, uint32_t P, uint32_t J, uint32_t C, float c,
                          float* g_out, float* s_out, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    const F32Way way = conv_f32_way(B, P, J, C, workspace != nullptr, workspace_bytes);
    return launch_conv_f32_any<kPatches>(way, X, D, B, P, J, C, c, g_out, s_out, workspace, ConvGeom{}, stream);
}

int launch_conv2d_f32(const void* act, const void* D, uint32_t B, uint32_t P, uint32_t J, uint32_t C, float c,
                      float* g_out, float* s_out, void* workspace, size_t workspace_bytes, ConvGeom G, hipStream_t stream) {
    const F32Way way = conv_f32_way(B, P, J, C, workspace != nullptr, workspace_bytes);
    if (G.kw == 3 && J == 9 * G.Cin && G.sh == 1 && G.sw == 1 && G.ph == 1 && G.pw == 1) {
        const int rc = launch_conv_taps_f32(way, act, D, B, G.H, G.W, G.Cin, C, c, g_out, s_out, workspace, stream);
        if (rc <= 0) return rc;
    }
    if (G.sh == 1 && G.sw == 1 && G.Wo == G.W && P > kR32 / 2) {
        uint32_t a = G.W, b = kR32 % G.W;
        while (b) { const uint32_t m = a % b; a = b; b = m; }
        G.period = G.W / a;
        G.step_x = kR32 % G.W;
        if (G.period <= 32) return launch_conv_f32_any<kLinear>(way, act, D, B, P, J, C, c, g_out, s_out, workspace, G, stream);
    }
    G.step_y = kR32 / G.Wo;
    G.step_x = kR32 % G.Wo;
    return launch_conv_f32_any<kGeneral>(way, act, D, B, P, J, C, c, g_out, s_out, workspace, G, stream);
}

}  // namespace vgc
