// Loss and gradient of the learned beam (network and parameter order in
// mlp.h) in three launches:
//   k_train_rows    forward and backward of 16 rows per workgroup, activations
//                   in LDS and registers; writes what the weight gradients read;
//   k_train_weights every weight's gradient tiles over chunks of rows and the
//                   bias column sums, in one launch;
//   k_train_finish  the sums over the chunks, the loss, and in training the Adam
//                   update and the operand images of the next step.
// A step is bound by latency, not by work: 1024 rows are 0.6 GFLOP, under a
// microsecond of matrix time.  As one launch per layer, bias, activation
// and sum it was 40 launches of 5-25 us, 465 us a step of 1024 rows and 527 us
// a gradient of 4096; so what counts is how many dependent launches and memory
// round trips there are.  Now a step of 1024 rows is 13.3 + 8.5 + 4.5 us (29 us with
// the gaps, 15x) and a gradient of 4096 is 17.3 + 16.1 + 4.2 us after 3 us of packing
// (38 us, 14x), bitwise the same results.  Rows are cut in 16s (one MFMA tile) because a layer
// then costs one barrier and the 1024 rows reach 64 CUs; a wave owns 16 units of
// every layer and loads its operands of all layers before the first one starts,
// so their latency is paid once.
//
// Products and their order of summation are those of one MFMA chain per output
// (32 deep on bf16, ascending k): hidden layers and their gradients round both
// operands to bf16 and accumulate in FP32, the head and its gradients stay in
// FP32 (v_mfma_f32_16x16x4f32).
#include <algorithm>

#include "mlp_math.h"

namespace mv {

namespace {

using namespace mlp;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ inline int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// ---- operand images -------------------------------------------------------
// MFMA A operands as the waves of k_train_rows read them, 16 bytes per lane:
//   fwd (bf16): W1 blocks (h, kb < 8), then W2..W4 blocks (h, kb < 4): lane (l16, lk)
//               holds W[16 h + l16][32 kb + 8 lk + 0..7];
//   bwd (bf16): W2..W4 transposed, blocks (h, kb < 4): W[32 kb + 8 lk + 0..7][16 h + l16];
//   head (f32): W5 blocks (rt < 4, q < 8): W5[16 rt + l16][16 q + 4 e + lk], e = 0..3;
//   headT (f32): W5 transposed, blocks (h < 8, q < 4): W5[16 q + 4 e + lk][16 h + l16].
constexpr int kBlkB = 512;                                 // bf16 per operand block
constexpr int kFwdElems = kHid * kFeat + 3 * kHid * kHid;  // bf16
constexpr int kBwdElems = 3 * kHid * kHid;                 // bf16
constexpr int kHeadElems = kNet * kHid;                    // floats, each of head and headT

struct Images {
    __bf16 *fwd, *bwd;
    float *head, *headT;
};

__host__ __device__ inline Images images_of(float *base) {
    Images g;
    g.fwd = (__bf16 *)base;
    g.bwd = g.fwd + kFwdElems;
    g.head = base + (kFwdElems + kBwdElems) / 2;
    g.headT = g.head + kHeadElems;
    return g;
}

// position of element (row, col) in the bf16 blocks of a layer with nkb k blocks
__device__ inline int fwd_pos(int row, int col, int nkb) {
    const int lane = (row & 15) + 16 * ((col >> 3) & 3);
    return ((row >> 4) * nkb + (col >> 5)) * kBlkB + lane * 8 + (col & 7);
}

// Parameter i of the vector, value v, into every image that holds it.
__device__ inline void image_store(const Images &g, int64_t i, float v) {
    if (i >= kOffW5) {
        if (i < kOffB5) {
            const int j = (int)(i - kOffW5), o = j / kHid, k = j % kHid;
            g.head[(((o >> 4) * 8 + (k >> 4)) * 64 + (o & 15) + 16 * (k & 3)) * 4 + ((k >> 2) & 3)] = v;
            g.headT[(((k >> 4) * 4 + (o >> 4)) * 64 + (k & 15) + 16 * (o & 3)) * 4 + ((o >> 2) & 3)] = v;
        }
        return;
    }
    if (i < kOffB1) {
        if (i >= kOffW1) {
            const int j = (int)(i - kOffW1);
            g.fwd[fwd_pos(j / kFeat, j % kFeat, kFeat / 32)] = (__bf16)v;
        }
        return;
    }
    const int64_t j = i - kOffW2, per = kOffW3 - kOffW2;  // W2, b2, W3, b3, W4, b4
    if (j < 0) return;
    const int l = (int)(j / per), r = (int)(j % per);
    if (r >= kHid * kHid) return;
    const int row = r / kHid, col = r % kHid;
    g.fwd[kHid * kFeat + l * kHid * kHid + fwd_pos(row, col, kHid / 32)] = (__bf16)v;
    g.bwd[l * kHid * kHid + fwd_pos(col, row, kHid / 32)] = (__bf16)v;
}

__global__ void __launch_bounds__(256) k_train_pack(const float *__restrict__ P, float *images) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < kNParams) image_store(images_of(images), i, P[i]);
}

// ---- forward and backward of 16 rows --------------------------------------
struct RowsArgs {
    const float *P;
    float *images;
    const float *x, *y;
    const int32_t *perm;  // row m of the call is perm[m] of x and y, or m itself when null
    int64_t n;
    TrainBufs b;
};

constexpr int kRows = 16;               // rows per workgroup
constexpr int kPhiS = kFeat + 8;        // LDS row strides (elements), 16 bytes of padding
constexpr int kActS = kHid + 8;
constexpr int kH4S = kHid + 4, kNetS = kNet + 4;

__global__ void __launch_bounds__(512, 1) k_train_rows(RowsArgs a) {
    __shared__ __attribute__((aligned(16))) __bf16 phi[kRows * kPhiS];
    __shared__ __attribute__((aligned(16))) __bf16 act[2][kRows * kActS];
    __shared__ __attribute__((aligned(16))) float h4[kRows * kH4S];
    __shared__ __attribute__((aligned(16))) float net[kRows * kNetS];
    __shared__ float xs[kRows * 3], ys[kRows * kOut], red[kRows * kOut];
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane & 15, lk = lane >> 4;
    const int64_t m0 = (int64_t)blockIdx.x * kRows;
    const Images g = images_of(a.images);
    const float *__restrict__ P = a.P;

    // this block's inputs, and this wave's operands of every layer
    if (tid < kRows * 3) {
        const int64_t m = m0 + tid / 3;
        xs[tid] = m < a.n ? a.x[3 * (a.perm ? (int64_t)a.perm[m] : m) + tid % 3] : 0.f;
    } else if (tid >= 128 && tid < 128 + kRows * kOut) {
        const int t = tid - 128;
        const int64_t m = m0 + t / kOut;
        ys[t] = m < a.n ? a.y[kOut * (a.perm ? (int64_t)a.perm[m] : m) + t % kOut] : 0.f;
    }
    bf16x8 w1[8], wl[3][4], wt[3][4];
#pragma unroll
    for (int kb = 0; kb < 8; kb++) w1[kb] = *(const bf16x8 *)(g.fwd + (w * 8 + kb) * kBlkB + lane * 8);
#pragma unroll
    for (int l = 0; l < 3; l++)
#pragma unroll
        for (int kb = 0; kb < 4; kb++)
            wl[l][kb] = *(const bf16x8 *)(g.fwd + kHid * kFeat + l * kHid * kHid + (w * 4 + kb) * kBlkB + lane * 8);
    f32x4 bias[4], bias5;
    const int64_t offB[4] = {kOffB1, kOffB2, kOffB3, kOffB4};
#pragma unroll
    for (int e = 0; e < 4; e++) {  // (a caller's parameters may be aligned to one float only)
#pragma unroll
        for (int l = 0; l < 4; l++) bias[l][e] = P[offB[l] + 16 * w + 4 * lk + e];
        bias5[e] = P[kOffB5 + 16 * (w & 3) + 4 * lk + e];
    }
    __syncthreads();

    // Fourier features: sin in columns 0..127, cos in 128..255
#pragma unroll
    for (int q = 0; q < kRows * kFreq / 512; q++) {
        const int i = tid + 512 * q, m = i / kFreq, j = i % kFreq;
        const float *b = P + kOffBff + kBffCols * j;
        const float arg = b[0] * xs[3 * m] + b[1] * xs[3 * m + 1];
        float s, c;
        sincos_rev(arg, s, c);
        phi[m * kPhiS + j] = (__bf16)s;
        phi[m * kPhiS + kFreq + j] = (__bf16)c;
    }
    __syncthreads();
    {  // the weight gradient of layer 1 reads the features as bf16 rows: 16 x 512 bytes
        const int m = tid / 32, c = tid % 32;
        if (m0 + m < a.n) ((u32x4 *)(a.b.phi + (m0 + m) * kFeat))[c] = *(const u32x4 *)(phi + m * kPhiS + c * 8);
    }

    // Accumulator element e of lane (l16, lk): unit 16 w + 4 lk + e of row l16.
    f32x4 z[4];
    auto hidden_out = [&](int l, const f32x4 &acc, __bf16 *dst) {
#pragma unroll
        for (int e = 0; e < 4; e++) z[l][e] = acc[e] + bias[l][e];
        bf16x4 h;
#pragma unroll
        for (int e = 0; e < 4; e++) h[e] = (__bf16)silu(z[l][e]);
        *(bf16x4 *)(dst + l16 * kActS + 16 * w + 4 * lk) = h;
        if (m0 + l16 < a.n) *(bf16x4 *)(a.b.h[l] + (m0 + l16) * kHid + 16 * w + 4 * lk) = h;
    };
    {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 8; kb++) {
            const bf16x8 v = *(const bf16x8 *)(phi + l16 * kPhiS + 32 * kb + 8 * lk);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[kb], v, acc, 0, 0, 0);
        }
        hidden_out(0, acc, act[0]);
    }
    // the backward operands, in flight while the forward layers run
    f32x4 wh[8], wht[4];
    if (w < 4)
#pragma unroll
        for (int q = 0; q < 8; q++) wh[q] = *(const f32x4 *)(g.head + ((w * 8 + q) * 64 + lane) * 4);
#pragma unroll
    for (int q = 0; q < 4; q++) wht[q] = *(const f32x4 *)(g.headT + ((w * 4 + q) * 64 + lane) * 4);
#pragma unroll
    for (int l = 0; l < 3; l++)
#pragma unroll
        for (int kb = 0; kb < 4; kb++)
            wt[l][kb] = *(const bf16x8 *)(g.bwd + l * kHid * kHid + (w * 4 + kb) * kBlkB + lane * 8);
    __syncthreads();
    auto product = [&](const bf16x8 (&op)[4], const __bf16 *src) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 4; kb++) {
            const bf16x8 v = *(const bf16x8 *)(src + l16 * kActS + 32 * kb + 8 * lk);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[kb], v, acc, 0, 0, 0);
        }
        return acc;
    };
    hidden_out(1, product(wl[0], act[0]), act[1]);
    __syncthreads();
    hidden_out(2, product(wl[1], act[1]), act[0]);
    __syncthreads();
    {
        const f32x4 acc = product(wl[2], act[0]);
        f32x4 h;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            z[3][e] = acc[e] + bias[3][e];
            h[e] = silu(z[3][e]);
        }
        *(f32x4 *)(h4 + l16 * kH4S + 16 * w + 4 * lk) = h;
        if (m0 + l16 < a.n) *(f32x4 *)(a.b.h4 + (m0 + l16) * kHid + 16 * w + 4 * lk) = h;
    }
    __syncthreads();
    if (w < 4) {  // the head in FP32: coefficient rows 16 w + 4 lk + e of row l16
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 8; q++)
#pragma unroll
            for (int e = 0; e < 4; e++)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wh[q][e], h4[l16 * kH4S + 16 * q + 4 * e + lk], acc, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; e++) acc[e] += bias5[e];
        *(f32x4 *)(net + l16 * kNetS + 16 * w + 4 * lk) = acc;
    }
    __syncthreads();
    if (tid < kRows * kOut) {  // the series, the squared error and its gradient
        const int m = tid / kOut, o = tid % kOut;
        float T[kBasis];
        chebyshev(2.0f * xs[3 * m + 2] - 1.0f, T);
        float *gp = net + m * kNetS + o * kBasis;
        float out = 0.f;
#pragma unroll
        for (int k = 0; k < kBasis; k++) out += T[k] * gp[k];
        const bool live = m0 + m < a.n;
        const float d = live ? out - ys[tid] : 0.f;
        const float dout = 2.0f * d / (float)(kOut * a.n);
        f32x4 d0, d1;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            d0[k] = T[k] * dout;
            d1[k] = T[4 + k] * dout;
        }
        *(f32x4 *)gp = d0;
        *(f32x4 *)(gp + 4) = d1;
        if (live) {
            f32x4 *dst = (f32x4 *)(a.b.dnet + (m0 + m) * kNet + o * kBasis);
            dst[0] = d0;
            dst[1] = d1;
        }
        red[tid] = d * d;
    }
    __syncthreads();
    if (tid < kWave) {
        double s = (double)red[tid] + (double)red[tid + 64];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
        if (tid == 0) a.b.sq[blockIdx.x] = s;
    }
    auto grad_out = [&](int l, const f32x4 &dh, __bf16 *dst) {  // dZ of layer l + 1
        f32x4 dz;
#pragma unroll
        for (int e = 0; e < 4; e++) dz[e] = silu_grad(dh[e], z[l][e]);
        if (m0 + l16 < a.n) *(f32x4 *)(a.b.dz[l] + (m0 + l16) * kHid + 16 * w + 4 * lk) = dz;
        if (dst) {
            bf16x4 h;
#pragma unroll
            for (int e = 0; e < 4; e++) h[e] = (__bf16)dz[e];
            *(bf16x4 *)(dst + l16 * kActS + 16 * w + 4 * lk) = h;
        }
    };
    {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int e = 0; e < 4; e++)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wht[q][e], net[l16 * kNetS + 16 * q + 4 * e + lk], acc, 0, 0, 0);
        grad_out(3, acc, act[1]);
    }
    __syncthreads();
    grad_out(2, product(wt[2], act[1]), act[0]);
    __syncthreads();
    grad_out(1, product(wt[1], act[0]), act[1]);
    __syncthreads();
    grad_out(0, product(wt[0], act[1]), nullptr);
}

// ---- weight gradients and bias column sums --------------------------------
// dW(m, k) = sum over rows of dZ[row][m] H[row][k]: 64 x 64 tiles of every weight
// over chunks of rows, raw sums to part[z][M][N] (summed in chunk order by
// k_train_finish).  A chunk's operands (at most 128 rows at a time) are loaded
// at once and transposed into LDS, rows in pairs so a lane writes whole
// words.  Bias gradients: column sums over 256 rows, four row lanes each.
struct WeightSeg {
    int64_t part;        // first float of the segment's partials in TrainBufs::part
    int m, n;            // weight shape
    int chunk, nz;       // rows per chunk and chunks
    int first;           // first workgroup
};
struct WeightsArgs {
    TrainBufs b;
    int64_t n;
    WeightSeg seg[5];    // W1, W2, W3, W4, W5
    int first_col;       // first workgroup of the column sums
    int64_t col_part;    // their partials [layer chunk][width], layers b1..b4 then b5
    int n_col;           // chunks of kColRows rows
};
constexpr int kSub = 128;      // rows staged at once
constexpr int kColRows = 256;  // rows of a bias partial

template <bool BF16>
__device__ __forceinline__ void weight_tile(const WeightSeg &g, int local, const float *__restrict__ dz, int dzw,
                                            const void *__restrict__ hv, int64_t n, float *__restrict__ part,
                                            unsigned char *smem) {
    constexpr int T = 64;
    constexpr int RB = kSub + 8;  // bf16 row stride: 16-byte aligned operand reads
    constexpr int RF = kSub + 1;  // float row stride
    __bf16 *Ab = (__bf16 *)smem, *Bb = Ab + T * RB;
    float *Af = (float *)smem, *Bf = Af + T * RF;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave, l16 = lane & 15, lk = lane >> 4;
    const int nt = g.n / T, tiles = (g.m / T) * nt;
    const int zc = local / tiles, t = local % tiles;
    const int u0 = (t / nt) * T, v0 = (t % nt) * T;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    const int64_t kbeg = (int64_t)zc * g.chunk, kend = kbeg + g.chunk < n ? kbeg + g.chunk : n;
    f32x4 acc[2][2];
    for (int i = 0; i < 2; i++)
        for (int j = 0; j < 2; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t k0 = kbeg; k0 < kend; k0 += kSub) {
        const int nk = kend - k0 < kSub ? (int)(kend - k0) : kSub;
        if constexpr (BF16) {
            const __bf16 *h = (const __bf16 *)hv;
            // dZ: row pair tid / 16 + 16 i, units u0 + 4 (tid % 16) ..; H: row pair tid / 8 + 32 i, columns 8 (tid % 8) ..
            f32x4 av[4][2];
            u32x4 bv[2][2];
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    const int r = 2 * (tid / 16 + 16 * i) + q;
                    av[i][q] = r < nk ? *(const f32x4 *)(dz + (k0 + r) * dzw + u0 + 4 * (tid % 16)) : f32x4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    const int r = 2 * (tid / 8 + 32 * i) + q;
                    bv[i][q] = r < nk ? *(const u32x4 *)(h + (k0 + r) * g.n + v0 + 8 * (tid % 8)) : u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int e = 0; e < 4; e++)
                    *(bf16x2 *)(Ab + (4 * (tid % 16) + e) * RB + 2 * (tid / 16 + 16 * i)) =
                        bf16x2{(__bf16)av[i][0][e], (__bf16)av[i][1][e]};
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t lo = bv[i][0][e], hi = bv[i][1][e];  // columns 2 e, 2 e + 1 of the two rows
                    __bf16 *d = Bb + (8 * (tid % 8) + 2 * e) * RB + 2 * (tid / 8 + 32 * i);
                    *(uint32_t *)d = (lo & 0xffffu) | (hi << 16);
                    *(uint32_t *)(d + RB) = (lo >> 16) | (hi & 0xffff0000u);
                }
        } else {
            const float *h = (const float *)hv;
            f32x4 av[8], bv[8];
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const int r = tid / 16 + 16 * i;
                const bool on = r < nk;
                av[i] = on ? *(const f32x4 *)(dz + (k0 + r) * dzw + u0 + 4 * (tid % 16)) : f32x4{0.f, 0.f, 0.f, 0.f};
                bv[i] = on ? *(const f32x4 *)(h + (k0 + r) * g.n + v0 + 4 * (tid % 16)) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < 8; i++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    Af[(4 * (tid % 16) + e) * RF + tid / 16 + 16 * i] = av[i][e];
                    Bf[(4 * (tid % 16) + e) * RF + tid / 16 + 16 * i] = bv[i][e];
                }
        }
        __syncthreads();
        if constexpr (BF16) {
#pragma unroll
            for (int ks = 0; ks < kSub; ks += 32) {
                bf16x8 av[2], bv[2];
#pragma unroll
                for (int i = 0; i < 2; i++) av[i] = *(const bf16x8 *)(Ab + (wr + 16 * i + l16) * RB + ks + lk * 8);
#pragma unroll
                for (int j = 0; j < 2; j++) bv[j] = *(const bf16x8 *)(Bb + (wc + 16 * j + l16) * RB + ks + lk * 8);
                if (ks < nk)
#pragma unroll
                    for (int i = 0; i < 2; i++)
#pragma unroll
                        for (int j = 0; j < 2; j++)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
            }
        } else {
            for (int kk = 0; kk < nk; kk += 4) {
                float av[2], bv[2];
#pragma unroll
                for (int i = 0; i < 2; i++) av[i] = Af[(wr + 16 * i + l16) * RF + kk + lk];
#pragma unroll
                for (int j = 0; j < 2; j++) bv[j] = Bf[(wc + 16 * j + l16) * RF + kk + lk];
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int j = 0; j < 2; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    float *out = part + g.part + (int64_t)zc * g.m * g.n;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 4; e++)
                out[(int64_t)(u0 + wr + 16 * i + 4 * lk + e) * g.n + v0 + wc + 16 * j + l16] = acc[i][j][e];
}

__global__ void __launch_bounds__(256) k_train_weights(WeightsArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * 64 * (kSub + 1) * 4];
    const int blk = blockIdx.x;
    if (blk >= a.first_col) {
        // 64 columns of one layer over kColRows rows, four row lanes
        float *red = (float *)smem;
        const int per = 2 * 4 + 1;  // 64-column groups of b1..b4 and b5
        const int ch = (blk - a.first_col) / per, cg = (blk - a.first_col) % per;
        const int l = cg < 8 ? cg / 2 : 4, width = l < 4 ? kHid : kNet, c0 = l < 4 ? 64 * (cg & 1) : 0;
        const float *src = l < 4 ? a.b.dz[l] : a.b.dnet;
        const int cl = threadIdx.x % 64, rl = threadIdx.x / 64;
        const int64_t r0 = (int64_t)ch * kColRows, r1 = r0 + kColRows < a.n ? r0 + kColRows : a.n;
        float s = 0.f;
        if (r1 - r0 == kColRows) {
#pragma unroll 16
            for (int q = 0; q < kColRows / 4; q++) s += src[(r0 + rl + 4 * q) * width + c0 + cl];
        } else {
            for (int64_t m = r0 + rl; m < r1; m += 4) s += src[m * width + c0 + cl];
        }
        red[rl * 64 + cl] = s;
        __syncthreads();
        if (rl == 0)
            a.b.part[a.col_part + ((int64_t)l * a.n_col + ch) * kHid + c0 + cl] =
                (red[cl] + red[64 + cl]) + (red[128 + cl] + red[192 + cl]);
        return;
    }
    int l = 0;
    while (l < 4 && blk >= a.seg[l + 1].first) l++;
    const WeightSeg &g = a.seg[l];
    const int local = blk - g.first;
    if (l == 0)
        weight_tile<true>(g, local, a.b.dz[0], kHid, a.b.phi, a.n, a.b.part, smem);
    else if (l < 4)
        weight_tile<true>(g, local, a.b.dz[l], kHid, a.b.h[l - 1], a.n, a.b.part, smem);
    else
        weight_tile<false>(g, local, a.b.dnet, kNet, a.b.h4, a.n, a.b.part, smem);
}

// ---- sums over the chunks, loss, Adam --------------------------------------
struct FinishArgs {
    WeightsArgs w;
    int64_t n_sq;       // partial sums of squares
    float *loss;
    float *grad;        // or null
    // training: parameters and moments updated in place, operand images renewed
    float *P, *m1, *m2, *images;
    int64_t step;
    float lr;
};

__global__ void __launch_bounds__(256) k_train_finish(FinishArgs a) {
    if (blockIdx.x == gridDim.x - 1) {  // the loss: lanes in a fixed order
        if (threadIdx.x < kWave) {
            double s = 0.0;
            for (int64_t i = threadIdx.x; i < a.n_sq; i += kWave) s += a.w.b.sq[i];
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
            if (threadIdx.x == 0) a.loss[0] = (float)(s / (double)(kOut * a.w.n));
        }
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= kNParams) return;
    float g = 0.f;
    if (i >= kOffW1) {
        const int64_t offW[5] = {kOffW1, kOffW2, kOffW3, kOffW4, kOffW5}, offB[5] = {kOffB1, kOffB2, kOffB3, kOffB4, kOffB5};
        int l = 0;
        while (l < 4 && i >= offW[l + 1]) l++;
        const bool is_bias = i >= offB[l];
        const WeightSeg &sg = a.w.seg[l];
        const float *p = a.w.b.part + (is_bias ? a.w.col_part + (int64_t)l * a.w.n_col * kHid + (i - offB[l])
                                               : sg.part + (i - offW[l]));
        const int64_t stride = is_bias ? kHid : (int64_t)sg.m * sg.n;
        const int nz = is_bias ? a.w.n_col : sg.nz;
#pragma unroll 8
        for (int q = 0; q < nz; q++) g += p[q * stride];
    }
    if (a.grad) a.grad[i] = g;
    if (a.P && i >= kOffW1) {  // the Fourier matrix is fixed
        float m1 = a.m1[i], m2 = a.m2[i];
        const float p = adam_step(a.P[i], g, m1, m2, a.step, a.lr, 0.9f, 0.999f, 1e-8f);
        a.m1[i] = m1;
        a.m2[i] = m2;
        a.P[i] = p;
        image_store(images_of(a.images), i, p);
    }
}

// chunks of a weight's rows: enough that its tiles reach the CUs, at least 128
// rows each, and one chunk for fewer than 512 rows
void cut(WeightSeg &g, int64_t n) {
    const int tiles = (g.m / 64) * (g.n / 64);
    int64_t nz = 1;
    if (n >= 512) nz = std::min<int64_t>((n + 127) / 128, (256 + tiles - 1) / tiles);
    const int64_t chunk = ((n + nz - 1) / nz + 31) / 32 * 32;
    g.chunk = (int)chunk;
    g.nz = (int)((n + chunk - 1) / chunk);
}

WeightsArgs plan(const TrainBufs &b, int64_t n) {
    WeightsArgs a{};
    a.b = b;
    a.n = n;
    int64_t part = 0;
    int first = 0;
    for (int l = 0; l < 5; l++) {
        WeightSeg &g = a.seg[l];
        g.m = l < 4 ? kHid : kNet;
        g.n = l == 0 ? kFeat : kHid;
        cut(g, n);
        g.part = part;
        g.first = first;
        part += (int64_t)g.nz * g.m * g.n;
        first += (g.m / 64) * (g.n / 64) * g.nz;
    }
    a.first_col = first;
    a.col_part = part;
    a.n_col = (int)((n + kColRows - 1) / kColRows);
    return a;
}

}  // namespace

namespace mlp {

int64_t train_part_floats(int64_t n) {
    const WeightsArgs a = plan(TrainBufs{}, n);
    return a.col_part + (int64_t)5 * a.n_col * kHid;
}

int64_t train_image_floats() { return (kFwdElems + kBwdElems) / 2 + 2 * kHeadElems; }

int64_t train_sq_count(int64_t n) { return (n + kRows - 1) / kRows; }

hipError_t train_pack(const float *P, float *images, hipStream_t s) {
    k_train_pack<<<(unsigned)((kNParams + 255) / 256), 256, 0, s>>>(P, images);
    return hipGetLastError();
}

hipError_t train_step(const TrainBufs &b, const float *P, const float *x, const float *y, const int32_t *perm,
                      int64_t n, float *grad, float *loss, float *update, float *m1, float *m2, int64_t step, float lr,
                      hipStream_t s) {
    RowsArgs r{P, b.images, x, y, perm, n, b};
    k_train_rows<<<(unsigned)train_sq_count(n), 512, 0, s>>>(r);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const WeightsArgs w = plan(b, n);
    k_train_weights<<<(unsigned)(w.first_col + w.n_col * 9), 256, 0, s>>>(w);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    FinishArgs f{w, train_sq_count(n), loss, grad, update, m1, m2, b.images, step, lr};
    k_train_finish<<<(unsigned)((kNParams + 255) / 256 + 1), 256, 0, s>>>(f);
    return hipGetLastError();
}

}  // namespace mlp

}  // namespace mv
