// FC form of the per-parameter sums of Alg. 1: the gradient of sample z is the outer product x_z d_z^T, so
// g = c X^T D and s = c^2 (X.X)^T (D.D) are two contractions over K = B (Section 5's 2 N |B| multiply-adds each).
//
//   k_fc_bf16   bf16 inputs.  The squares are taken in float32 and rounded to bf16 (2^-9 relative per factor, well
//               inside the 1e-2 budget for bf16 inputs); v_mfma_f32_32x32x16_bf16, float32 accumulate.
//               With K this small the kernel is bound by writing [J, C] floats, not by the matrix cores.
//   k_fc_f32    float32 inputs, and bf16 ones whose rows are not whole 16-byte pieces (widened); v_mfma_f32_32x32x2_f32
//               (float32 products and sums, which is what the 1e-5 tolerance on s needs).
//
// Block tile 128 x 128 of [J, C] (k_fc_f32 also 64 x 64, and for rows of any length only that), 4 waves (2 x 2), operands staged
// through LDS k-major (rows of the source matrices as they are in memory).  Rows past the end of the matrix are outside the
// bounded range of the buffer loads and read as zero; rows of any length are read by load_any, which checks the end itself.
#include "vgc_internal.h"

namespace vgc {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef short s8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4v* lds_s4v_ptr;
typedef __amdgpu_buffer_rsrc_t rsrc_t;

constexpr int kT = 128;                  // block tile edge
constexpr int kPitch16 = kT + 32;        // bf16 row pitch (elements): rows start 16 banks apart

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// ds_read_b64_tr_b16 operand fetch: see vgc_sqgrad_tiled.hip for the lane mapping.
__device__ __forceinline__ bf8v frag16(const uint16_t* tile, int ks, int mbase, uint32_t lane) {
    const uint32_t r = lane & 15u, grp = lane >> 4;
    const uint16_t* p = tile + (ks * 16 + (grp >> 1) * 8 + (r >> 2)) * kPitch16 + mbase + (grp & 1u) * 16 + 4 * (r & 3u);
    const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(p));
    const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(p + 4 * kPitch16));
    s8v v;
    v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3];
    v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
    return __builtin_bit_cast(bf8v, v);
}

// Square of two packed bf16 values: float32 product, rounded to nearest-even bf16.
__device__ __forceinline__ uint32_t square_bf16x2(uint32_t w) {
    const float lo = __uint_as_float(w << 16), hi = __uint_as_float(w & 0xFFFF0000u);
    const uint32_t a = __float_as_uint(lo * lo), b = __float_as_uint(hi * hi);
    const uint32_t ra = (a + 0x7FFFu + ((a >> 16) & 1u)) >> 16;
    const uint32_t rb = (b + 0x7FFFu + ((b >> 16) & 1u)) & 0xFFFF0000u;
    return ra | rb;
}

// A wave's MT x MT MFMA tiles, of the quarter (wm, wn) of the block.  kAnyRow: rows of the output begin anywhere in a cache line, so
// lines are written by two tiles, and have to meet in the cache (25087 x 4095 at batch 8: 285 us with non-temporal stores, 145 so).
template <int MT, bool kAnyRow>
__device__ __forceinline__ void store_tile(float fs, float fg, const f16v (&s_acc)[MT][MT], const f16v (&g_acc)[MT][MT],
                                           bool want_g, float* __restrict__ so, float* __restrict__ go,
                                           uint32_t j0, uint32_t c0, uint32_t J, uint32_t C, uint32_t wm, uint32_t wn,
                                           uint32_t lane) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < MT; ++nt) {
            const uint32_t col = c0 + wn * (MT * 32u) + nt * 32 + (lane & 31u);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t row = j0 + wm * (MT * 32u) + mt * 32 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
                if (row < J && col < C) {
                    const size_t o = (size_t)row * C + col;
                    if (kAnyRow) so[o] = fs * s_acc[mt][nt][i];
                    else __builtin_nontemporal_store(fs * s_acc[mt][nt][i], so + o);
                    if (want_g) {
                        if (kAnyRow) go[o] = fg * g_acc[mt][nt][i];
                        else __builtin_nontemporal_store(fg * g_acc[mt][nt][i], go + o);
                    }
                }
            }
        }
}

// ------------------------------------------------------------------------------------------------
// FC, bf16
// ------------------------------------------------------------------------------------------------
template <bool kWantG>
__global__ __launch_bounds__(256, 2) void k_fc_bf16(const uint16_t* __restrict__ X, const uint16_t* __restrict__ D,
                                                    uint32_t B, uint32_t J, uint32_t C, float cg, float cs,
                                                    float* __restrict__ g_out, float* __restrict__ s_out) {
    constexpr int kRows = 32;
    __shared__ __attribute__((aligned(16))) uint16_t shX[kRows * kPitch16], shD[kRows * kPitch16];
    __shared__ __attribute__((aligned(16))) uint16_t shX2[kRows * kPitch16], shD2[kRows * kPitch16];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, wm = wave >> 1, wn = wave & 1u;
    const uint32_t tiles_c = (C + kT - 1) / kT;
    const uint32_t j0 = (blockIdx.x / tiles_c) * kT, c0 = (blockIdx.x % tiles_c) * kT;
    const rsrc_t rx = make_rsrc(X, B * J * 2u), rd = make_rsrc(D, B * C * 2u);

    f16v s_acc[2][2], g_acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) { s_acc[a][b] = (f16v){0}; g_acc[a][b] = (f16v){0}; }

    for (uint32_t z0 = 0; z0 < B; z0 += kRows) {
        u4v vx[2], vd[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t idx = tid + 256u * i, row = idx >> 4, col = (idx & 15u) * 8u;
            vx[i] = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(((z0 + row) * J + j0 + col) * 2u), 0, 0));
            vd[i] = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(rd, (int)(((z0 + row) * C + c0 + col) * 2u), 0, 0));
        }
        if (z0) __syncthreads();                        // the previous chunk has been consumed
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t idx = tid + 256u * i, off = (idx >> 4) * kPitch16 + (idx & 15u) * 8u;
            // columns past the matrix edge wrapped into the next row: they feed outputs that are not stored
            if (kWantG) {
                *reinterpret_cast<u4v*>(shX + off) = vx[i];
                *reinterpret_cast<u4v*>(shD + off) = vd[i];
            }
            u4v x2, d2;
#pragma unroll
            for (int e = 0; e < 4; ++e) { x2[e] = square_bf16x2(vx[i][e]); d2[e] = square_bf16x2(vd[i][e]); }
            *reinterpret_cast<u4v*>(shX2 + off) = x2;
            *reinterpret_cast<u4v*>(shD2 + off) = d2;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < kRows / 16; ++ks) {
            bf8v a2[2], b2[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) { a2[t] = frag16(shX2, ks, wm * 64 + t * 32, lane); b2[t] = frag16(shD2, ks, wn * 64 + t * 32, lane); }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    s_acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2[mt], b2[nt], s_acc[mt][nt], 0, 0, 0);
            if (kWantG) {
                bf8v a[2], b[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) { a[t] = frag16(shX, ks, wm * 64 + t * 32, lane); b[t] = frag16(shD, ks, wn * 64 + t * 32, lane); }
#pragma unroll
                for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt)
                        g_acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mt], b[nt], g_acc[mt][nt], 0, 0, 0);
            }
        }
    }
    store_tile<2, false>(cs, cg, s_acc, g_acc, kWantG, s_out, g_out, j0, c0, J, C, wm, wn, lane);
}

// ------------------------------------------------------------------------------------------------
// FC, float32
// ------------------------------------------------------------------------------------------------
constexpr int kR32 = 16;                 // rows per LDS stage

// Two chains of v_mfma_f32_32x32x2_f32 (float32 products and sums), on the values and on their squares.  A chunk of kR32
// samples is in registers while the one before it is multiplied from LDS.  Four waves (2 x 2) share a block of kE x kE
// outputs.  kE = 128 where there are tiles enough (the kernel is then bound by writing [J, C] floats); kE = 64 where 128 x 128
// tiles would leave compute units idle, whose one tile's K = B steps are then all the time there is: 1000 x 1000 at batch 128,
// 64 tiles of 128 against 256 of 64: 15.8 -> 6.6 us; 4096 x 1000 at batch 64 with g (256 against 1024): 23.6 -> 17.7.
// kLong: how the chunks to come are held.  In two register sets without copies, the multiplication never waits for a load,
// but the unrolled loop of the large tile takes registers that are worth a wave per SIMD; with a copy from set to set each
// chunk waits for the loads of the one after the next, which costs nothing while the writes of [J, C] are the bound.
//
// T, kAnyRow: float rows whose length is a multiple of four are read by bounded buffer loads; rows of any other length, and
// bfloat16 ones that k_fc_bf16 does not take (widened exactly, the squares then float32's), by loads at the elements' own
// alignment, the last piece of the matrix element by element.  Before, such
// shapes went without LDS, a wave's loads a step or eight ahead: 25087 x 4095 at batch 64, float32, s alone 271 -> 186 us, with
// g 417 -> 312; bfloat16 477 -> 235 and 589 -> 329; 1000 x 10 at batch 128 10.4 -> 8.0 and (bfloat16) 20.0 -> 10.0.
template <typename T> struct Piece;                          // four elements as they are in memory
template <> struct Piece<float> {
    f4v x;
    __device__ __forceinline__ f4v value() const { return x; }
};
template <> struct Piece<uint16_t> {
    uint32_t x[2];
    __device__ __forceinline__ f4v value() const {
        return (f4v){__uint_as_float(x[0] << 16), __uint_as_float(x[0] & 0xFFFF0000u), __uint_as_float(x[1] << 16), __uint_as_float(x[1] & 0xFFFF0000u)};
    }
};
template <typename T> struct __attribute__((packed, aligned(sizeof(T)))) AtElement { Piece<T> p; };

// Elements at .. at + 3 of a matrix of `total`; those past its end, and all of them unless `live`, are zeros.
template <typename T>
__device__ __forceinline__ Piece<T> load_any(const T* __restrict__ M, uint32_t total, uint32_t at, bool live) {
    union { T e[4]; Piece<T> p; } u = {{0, 0, 0, 0}};
    if (live && at + 4u <= total) u.p = reinterpret_cast<const AtElement<T>*>(M + at)->p;
    else if (live)
        for (uint32_t i = 0; i < 4; ++i)
            if (at + i < total) u.e[i] = M[at + i];
    return u.p;
}

template <bool kWantG, int kE, bool kLong, typename T, bool kAnyRow>
__global__ __launch_bounds__(256, kLong ? 2 : 3) void k_fc_f32(const T* __restrict__ X, const T* __restrict__ D, uint32_t B, uint32_t J,
                                                   uint32_t C, float cg, float cs, float* __restrict__ g_out, float* __restrict__ s_out) {
    static_assert(kAnyRow || sizeof(T) == 4, "bounded loads are of floats");
    constexpr int kPitch = kE + 32, MT = kE / 64;            // floats per LDS row; 32 x 32 tiles of a wave per direction
    constexpr int kPieces = kR32 * kE / 4 / 256;             // 16-byte pieces per thread, operand and chunk
    __shared__ __attribute__((aligned(16))) float shA[2][kR32 * kPitch], shB[2][kR32 * kPitch];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6, wm = wave >> 1, wn = wave & 1u;
    const uint32_t tiles_c = (C + kE - 1) / kE;
    const uint32_t nblk = gridDim.x, per = nblk / 8u, rem = nblk % 8u;
    const uint32_t xcd = blockIdx.x % 8u, slot = blockIdx.x / 8u;
    const uint32_t logical = xcd * per + min(xcd, rem) + slot;       // contiguous range of tiles per XCD
    const uint32_t j0 = (logical / tiles_c) * kE, c0 = (logical % tiles_c) * kE;
    const rsrc_t rx = make_rsrc(X, B * J * 4u), rd = make_rsrc(D, B * C * 4u);

    f16v s_acc[MT][MT], g_acc[MT][MT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < MT; ++b) { s_acc[a][b] = (f16v){0}; g_acc[a][b] = (f16v){0}; }

    struct Chunk { Piece<T> a[kPieces], b[kPieces]; };
    auto load = [&](uint32_t z0) -> Chunk {                  // rows past B read as zeros
        Chunk R;
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const uint32_t idx = tid + 256u * i, row = idx / (kE / 4), col = (idx % (kE / 4)) * 4u;
            // (columns past the matrix edge are those of the next row: they feed outputs that are not stored)
            const uint32_t atx = (z0 + row) * J + j0 + col, atd = (z0 + row) * C + c0 + col;
            if constexpr (kAnyRow) {
                R.a[i] = load_any<T>(X, B * J, atx, z0 + row < B);
                R.b[i] = load_any<T>(D, B * C, atd, z0 + row < B);
            } else {
                R.a[i].x = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(atx * 4u), 0, 0));
                R.b[i].x = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(rd, (int)(atd * 4u), 0, 0));
            }
        }
        return R;
    };
    auto stage = [&](uint32_t buf, const Chunk& R) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const uint32_t idx = tid + 256u * i, off = (idx / (kE / 4)) * kPitch + (idx % (kE / 4)) * 4u;
            *reinterpret_cast<f4v*>(shA[buf] + off) = R.a[i].value();
            *reinterpret_cast<f4v*>(shB[buf] + off) = R.b[i].value();
        }
    };
    const uint32_t col = lane & 31u, kh = lane >> 5;
    auto multiply = [&](const float* A, const float* Bm) {
#pragma unroll
        for (int ks = 0; ks < kR32 / 2; ++ks) {
            float a[MT], b[MT];
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                a[t] = A[(ks * 2 + kh) * kPitch + wm * (kE / 2) + t * 32 + col];
                b[t] = Bm[(ks * 2 + kh) * kPitch + wn * (kE / 2) + t * 32 + col];
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < MT; ++nt) {
                    s_acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mt] * a[mt], b[nt] * b[nt], s_acc[mt][nt], 0, 0, 0);
                    if (kWantG) g_acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mt], b[nt], g_acc[mt][nt], 0, 0, 0);
                }
        }
    };
    // Chunk q is multiplied from LDS buffer q % 2, and two more are on their way: with few tiles their latency is what a chunk costs.
    stage(0, load(0));
    Chunk R[2];
    R[0] = load(kR32);
    if (kLong) {
        // through register set (q + 1) % 2, the loop unrolled over both (a set that is copied is waited for)
        R[1] = load(2 * kR32);
        __syncthreads();
        for (uint32_t z0 = 0; z0 < B; z0 += 2 * kR32) {
#pragma unroll
            for (uint32_t u = 0; u < 2; ++u) {
                if (u > 0 && z0 + kR32 >= B) break;
                multiply(shA[u], shB[u]);
                stage(u ^ 1u, R[u]);
                R[u] = load(z0 + (u + 3) * kR32);
                __syncthreads();
            }
        }
    } else {
        __syncthreads();
        uint32_t buf = 0;
        for (uint32_t z0 = 0; z0 < B; z0 += kR32, buf ^= 1u) {
            R[1] = load(z0 + 2 * kR32);
            multiply(shA[buf], shB[buf]);
            stage(buf ^ 1u, R[0]);
            R[0] = R[1];
            __syncthreads();
        }
    }
    store_tile<MT, kAnyRow>(cs, cg, s_acc, g_acc, kWantG, s_out, g_out, j0, c0, J, C, wm, wn, lane);
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
// Rows of whole 16-byte pieces, which bounded loads can take.
static bool fc_whole_pieces(int dtype, uint32_t J, uint32_t C) {
    const uint32_t per = dtype == VGC_BF16 ? 8 : 4;
    return J % per == 0 && C % per == 0;
}
bool fc_tiled_supported(int dtype, uint32_t B, uint32_t J, uint32_t C) {
    const uint64_t limit = 0x7FFFFFFFull;                            // buffer ranges and offsets are 32-bit
    const uint32_t size = dtype == VGC_BF16 ? 2 : 4, ahead = dtype == VGC_BF16 ? 32 : 16;
    if (fc_whole_pieces(dtype, J, C)) return (uint64_t)(B + ahead) * J * size < limit && (uint64_t)(B + ahead) * C * size < limit;
    return (uint64_t)(B + 64) * (J + 128ull) < limit && (uint64_t)(B + 64) * (C + 128ull) < limit;
}

// Shapes the tiled kernel takes, but a wave per 32 x 32 outputs without LDS (vgc_sqgrad.hip; the same bits) is faster with: few
// rows of 16-bit elements, whose way through LDS is not worth it (2049 x 1001 at batch 8: 7.7 us tiled, 6.4 by waves; with g 9.9
// and 8.2; at batch 16 they meet, and so they do once the outputs, which it stores element by element, outgrow the caches), and
// matrices so thin that half of a 64 x 64 tile is padding, once there are enough of them to fill the chip (100001 x 9: float32 at
// batch 16 8.3 and 6.9, with g 10.9 and 8.7, with g at batch 512 122 and 95; bfloat16 at batch 16 8.7 and 7.7).  From batch 64 on
// the tiled kernel catches up there without g (14.7 and 13.6), and in bfloat16 (16.8 and 23.2).
bool fc_by_waves(int dtype, uint32_t B, uint32_t J, uint32_t C, bool want_g) {
    if (fc_whole_pieces(dtype, J, C) || J > 65535u * 64u) return false;
    const uint64_t tiles = (uint64_t)((J + 63) / 64) * ((C + 63) / 64), out = (uint64_t)J * C * (want_g ? 8 : 4);
    if (dtype == VGC_BF16 && B <= 8 && out <= (64ull << 20)) return true;
    return (J < C ? J : C) <= 32 && tiles >= 2 * 256 && (B < 64 || (want_g && dtype == VGC_F32));
}

template <typename T, bool kAnyRow>
static void launch_fc_f32(const void* X, const void* D, uint32_t B, uint32_t J, uint32_t C, float c, float* g_out, float* s_out,
                          bool small, dim3 grid, hipStream_t stream) {
    const float cg = c, cs = c * c;
    const dim3 block(256);
#define VGC_FC_F32(G_, E_, L_) hipLaunchKernelGGL((k_fc_f32<G_, E_, L_, T, kAnyRow>), grid, block, 0, stream, (const T*)X, (const T*)D, B, J, C, cg, cs, g_out, s_out)
    if (small) { if (g_out) VGC_FC_F32(true, 64, true); else VGC_FC_F32(false, 64, true); }
    // the large tile's two forms cross between batches of 200 and 256: 4096 x 4096 with g, copied against in two sets: 117 against
    // 121 us at 200, 140 against 138 at 256, 1025 against 988 at 2048
    else if constexpr (!kAnyRow) {
        if (B >= 256) { if (g_out) VGC_FC_F32(true, 128, true); else VGC_FC_F32(false, 128, true); }
        else { if (g_out) VGC_FC_F32(true, 128, false); else VGC_FC_F32(false, 128, false); }
    }
#undef VGC_FC_F32
}

int launch_fc_tiled(int dtype, const void* X, const void* D, uint32_t B, uint32_t J, uint32_t C, float c,
                    float* g_out, float* s_out, hipStream_t stream) {
    const bool whole = fc_whole_pieces(dtype, J, C), bf16 = dtype == VGC_BF16 && whole;
    uint64_t nblk = (uint64_t)((J + kT - 1) / kT) * ((C + kT - 1) / kT);
    // Small tiles where there are fewer than two of 128 x 128 per compute unit, and for rows of any length: with g the large tile
    // spills there or is down to two waves per SIMD (25087 x 4095, float32 at batch 64: 425 us, 312 with the small one), and without
    // it is the slower one as well wherever its last wave of workgroups or its edges leave much of it idle (float32 at batch 64:
    // 25087 x 4095 184 -> 174 us, 129 x 100001 52 -> 35; at best, 4095 x 4095 in
    // bfloat16 at batch 128, the large one is 8 % ahead).
    const bool small = !bf16 && (nblk < 2 * 256 || !whole);
    if (small) nblk = (uint64_t)((J + 63) / 64) * ((C + 63) / 64);
    if (nblk > 0x7FFFFFFFull) { set_error("vgc_sqgrad: shape exceeds the launch limit"); return VGC_ERR_SIZE; }
    const dim3 grid((uint32_t)nblk), block(256);
    if (bf16) {
        const float cg = c, cs = c * c;
        if (g_out) hipLaunchKernelGGL(k_fc_bf16<true>, grid, block, 0, stream, (const uint16_t*)X, (const uint16_t*)D, B, J, C, cg, cs, g_out, s_out);
        else hipLaunchKernelGGL(k_fc_bf16<false>, grid, block, 0, stream, (const uint16_t*)X, (const uint16_t*)D, B, J, C, cg, cs, g_out, s_out);
    } else if (dtype == VGC_BF16) launch_fc_f32<uint16_t, true>(X, D, B, J, C, c, g_out, s_out, small, grid, stream);
    else if (whole) launch_fc_f32<float, false>(X, D, B, J, C, c, g_out, s_out, small, grid, stream);
    else launch_fc_f32<float, true>(X, D, B, J, C, c, g_out, s_out, small, grid, stream);
    return hip_check(hipGetLastError(), "launch fc tiled");
}

}  // namespace vgc
