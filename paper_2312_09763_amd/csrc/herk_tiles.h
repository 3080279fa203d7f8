// Tile geometry shared by the product kernels that form Z in LDS
// (kernels_herk_fused.hip, kernels_herk_x6.hip, kernels_tiles.hip).
#pragma once

#include "internal.h"

namespace mv {

namespace {

constexpr int kST = kAntBlock;  // antennas (or rows) per block
constexpr int kTI = 4;    // 16 x 16 tiles per side of a square wave tile

__device__ inline int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// Row of a forming thread (8 threads per row, two sources each): a wave's 8 rows
// in the order 0, 4, 1, 5, 2, 6, 3, 7, so the two rows that 16 consecutive
// lanes write are 4 rows (576 bytes) apart and fall in disjoint LDS banks.
__device__ inline int wrow(int t) {
    const int g = (t >> 3) & 7;
    return ((t >> 6) << 3) + (((g & 1) << 2) | (g >> 1));
}

// The same for 160-byte rows: rows 0, 2, 1, 3, 4, 6, 5, 7 (two rows 320 bytes, 16
// banks, apart)
__device__ inline int wrow160(int t) {
    const int g = (t >> 3) & 7;
    return ((t >> 6) << 3) + (g & 4) + ((g & 1) << 1) + ((g >> 1) & 1);
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

struct AntEntry {
    double ux, uy, uz;  // (nu / c) x_a
    int b;              // beam index, -1 for padding rows
    int pad;
};

// packed bf16 words of one complex64 value: z = hi + mid + lo, each round-to-nearest-even
__device__ inline void split3(float re, float im, uint32_t &hi, uint32_t &mid, uint32_t &lo) {
    const f32x2_t z = {re, im};
    const bf16x2_t h = __builtin_convertvector(z, bf16x2_t);
    const f32x2_t r = z - __builtin_convertvector(h, f32x2_t);
    const bf16x2_t m = __builtin_convertvector(r, bf16x2_t);
    const f32x2_t q = r - __builtin_convertvector(m, f32x2_t);
    const bf16x2_t l = __builtin_convertvector(q, bf16x2_t);
    hi = __builtin_bit_cast(uint32_t, h);
    mid = __builtin_bit_cast(uint32_t, m);
    lo = __builtin_bit_cast(uint32_t, l);
}

// packed (hi, lo) bf16 words of one complex64 value: hi = bf16(z), lo = bf16(z - hi),
// both round-to-nearest-even (v_cvt_pk_bf16_f32 on gfx950)
__device__ inline void split2(float re, float im, uint32_t &hi, uint32_t &lo) {
    const f32x2_t z = {re, im};
    const bf16x2_t h = __builtin_convertvector(z, bf16x2_t);
    const f32x2_t r = z - __builtin_convertvector(h, f32x2_t);
    const bf16x2_t l = __builtin_convertvector(r, bf16x2_t);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

// F = exp(-2 pi i p), p in cycles: FP64 reduction, hardware sine and cosine in revolutions
__device__ __forceinline__ void fringe(double p, float &fr, float &fi) {
    const float r = (float)__builtin_amdgcn_fract(p);
    fi = __builtin_amdgcn_sinf(-r);
    fr = __builtin_amdgcn_cosf(-r);
}

// the column fragment rotated for the imaginary part: (re, im) -> (-im, re) per bf16 pair
__device__ inline u32x4 bf16_rot_col(u32x4 v) {
    u32x4 r;
    for (int q = 0; q < 4; q++) r[q] = __builtin_amdgcn_alignbit(v[q], v[q], 16) ^ 0x00008000u;
    return r;
}

__device__ __forceinline__ void mfma_pair(const u32x4 &a, const u32x4 &b, const u32x4 &w, f32x4 &re, f32x4 &im) {
    re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), re, 0, 0,
                                                 0);
    im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, w), im, 0, 0,
                                                 0);
}

// Staged-row geometry: RS bytes per row, planes of PLANEB bytes, NKS k-steps of 16
// complex per stage.
template <int RS_, int PLANEB_, int NKS_>
struct RowGeom {
    static constexpr int RS = RS_, PLANEB = PLANEB_, NKS = NKS_;
};

// Row sets of the triangle waves and the first accumulator slot of each row
// (row r of a set holds columns 0..r in consecutive slots).  On a diagonal
// block the column operand of column c is the row operand of row c (same
// rows, same lane layout), so a wave loads only the columns that are not its
// own rows, and none right of its last row.  order[] interleaves loaded and
// reused columns so every load has at least one column of products to hide in.
template <int S>
struct TriSet {
    static constexpr int NR = 4;
    static constexpr int r[4] = {S == 0 ? 0 : 2, S == 0 ? 7 : 5, S == 0 ? 1 : 3, S == 0 ? 6 : 4};
    static constexpr int base[4] = {0, r[0] + 1, r[0] + r[1] + 2, r[0] + r[1] + r[2] + 3};
    static constexpr int ncol = S == 0 ? 8 : 6;
    static constexpr int order[8] = {S == 0 ? 0 : 2, S == 0 ? 2 : 0, S == 0 ? 1 : 3, S == 0 ? 3 : 1,
                                     S == 0 ? 6 : 4, S == 0 ? 4 : 5, S == 0 ? 7 : -1, S == 0 ? 5 : -1};
    // row slot holding column c, or -1 when the column is loaded
    static constexpr int slot(int c) { return r[0] == c ? 0 : r[1] == c ? 1 : r[2] == c ? 2 : r[3] == c ? 3 : -1; }
    // first position at or after p whose column is loaded, or -1
    static constexpr int next_loaded(int p) {
        return p >= ncol ? -1 : slot(order[p]) < 0 ? p : next_loaded(p + 1);
    }
};

// Two-row sets {S, 7 - S} of a 128-row triangle (nine tiles each), columns in
// natural order; rows S and 7 - S double as columns S and 7 - S.
template <int S>
struct TriPair {
    static constexpr int NR = 2;
    static constexpr int r[2] = {S, 7 - S};
    static constexpr int base[2] = {0, S + 1};
    static constexpr int ncol = 8 - S;
    static constexpr int order[8] = {0, 1, 2, 3, 4, 5, 6, 7};
    static constexpr int slot(int c) { return c == r[0] ? 0 : c == r[1] ? 1 : -1; }
    static constexpr int next_loaded(int p) {
        return p >= ncol ? -1 : slot(order[p]) < 0 ? p : next_loaded(p + 1);
    }
};

// A tile set passed as a value (to pick a set at run time among instantiations)
template <typename T>
struct SetTag {
    typedef T type;
};

// Row S alone of a two-row set, when row 7 - S lies wholly past the antennas of
// a short last block (its tiles are neither multiplied nor stored).
template <int S>
struct TriSingle {
    static constexpr int NR = 1;
    static constexpr int r[1] = {S};
    static constexpr int base[1] = {0};
    static constexpr int ncol = S + 1;
    static constexpr int order[8] = {0, 1, 2, 3, 4, 5, 6, 7};
    static constexpr int slot(int c) { return c == r[0] ? 0 : -1; }
    static constexpr int next_loaded(int p) {
        return p >= ncol ? -1 : slot(order[p]) < 0 ? p : next_loaded(p + 1);
    }
};

// Row sets of the triangle waves on a short diagonal block of at most 96
// antennas (six tile rows): {5, 0, 3} (eleven tiles) and {4, 1, 2} (ten).
template <int S>
struct TriSet6 {
    static constexpr int NR = 3;
    static constexpr int r[3] = {S == 0 ? 5 : 4, S == 0 ? 0 : 1, S == 0 ? 3 : 2};
    static constexpr int base[3] = {0, r[0] + 1, r[0] + r[1] + 2};
    static constexpr int ncol = S == 0 ? 6 : 5;
    static constexpr int order[6] = {S == 0 ? 0 : 1, S == 0 ? 1 : 0, S == 0 ? 3 : 2,
                                     S == 0 ? 2 : 3, S == 0 ? 5 : 4, S == 0 ? 4 : -1};
    static constexpr int slot(int c) { return r[0] == c ? 0 : r[1] == c ? 1 : r[2] == c ? 2 : -1; }
    static constexpr int next_loaded(int p) {
        return p >= ncol ? -1 : slot(order[p]) < 0 ? p : next_loaded(p + 1);
    }
};

// Calls f(slot, row, column) for every tile of a triangle row set.
template <typename T, typename F>
__device__ __forceinline__ void for_tri_tiles(F f) {
#pragma unroll
    for (int k = 0; k < T::NR; k++)
#pragma unroll
        for (int c = 0; c <= T::r[k]; c++) f(T::base[k] + c, T::r[k], c);
}

}  // namespace

}  // namespace mv
