// FP64 products with Z formed in LDS.
//
// Product over sources (2 feeds x 2 axes, one shared beam).  The axis sum is taken per source first,
//   V[(a,p),(b,q)] = sum_m F_a(m) conj(F_b(m)) C_pq(m),  C_pq = sum_k B_pk conj(B_qk),
// which halves the multiply-adds of Z Z^H, and the fringe rows F are formed in
// LDS, so Z never goes through device memory.
//
// v_mfma_f64_16x16x4f64 runs 32 flops a cycle and SIMD, so a stage is bound by its
// MFMAs (64 cycles each) and everything else has room beside them: only the
// plain rows F of two blocks of 64 antennas are staged (16 sources, 35 KB), and a
// wave weights its row operand with C in registers (two to four multiplies per
// 4 to 16 MFMAs).  Blocks of 64 because the accumulators set the limit: a 16 x 16
// tile takes 16 registers, so a wave holds nine.  Items of a (instance,
// k-split), all nearly equal and in one launch:
//   block pair I > J: four products (C_00, C_11, C_10, conj C_10) of 64 x 64, a
//     row tile and two column tiles per wave, eight tiles;
//   two diagonal blocks: waves 0-3 the first, 4-7 the second, nine tiles each:
//     row r of V^10, row r of V^00 and row 3 - r of V^11;
//   a last odd diagonal block alone: both halves of the workgroup take it, each
//     half of the item's sources, added through LDS at the end.
// Waves 0-3 multiply before they form the next stage's rows and waves 4-7 after,
// so the two waves of a SIMD overlap matrix and vector work.
//
// 128 antennas, 50 000 sources, 4 x 4 instances: 2.2 ms (43 useful TFLOP/s, 48 executed;
// MFMAs busy 70 % at 2.18 GHz) where writing Z took 2.1 ms and Z Z^H 4.3 ms; 4 antennas
// 351 against 656 us for the whole call, 33 antennas 649 against 1929 us, 200 antennas
// and 3000 sources 320 against 488 us, so every such context takes it.
#include <type_traits>

#include "internal.h"
#include "launch_rules.h"

namespace mv {

namespace {

__device__ inline int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

constexpr int kB64 = 64;                // antennas per block
constexpr int kS64 = 16;                // sources per stage
constexpr int kRS64 = kS64 * 16 + 16;   // bytes of a staged row
constexpr int kBuf64 = 2 * kB64 * kRS64;

struct Src64 {
    double c00, c11, c10x, c10y;  // coherency (0 past the split)
    double x, y, z, pad;          // s_hat
};

__device__ __forceinline__ void mfma64(double wr, double wi, const double2 &b, f64x4 &re, f64x4 &im) {
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(wr, b.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(wi, b.x, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(wi, b.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(-wr, b.y, im, 0, 0, 0);
}

// (cos, -sin) of 2 pi p: p less whole turns and its nearest 256th of a turn, exactly
// (|t| <= 1/512); the Taylor series of both functions there (first omitted terms
// below 2^-56), turned by the table's 256th.  FP64 vector instructions and FP64
// MFMAs do not run side by side, so the short form counts: 20 of them instead of
// the 35 of a reduction to an eighth of a turn.
constexpr int kTurn = 256;
__device__ __forceinline__ double2 fringe64(double p, const double2 *turn) {
    constexpr double S0 = 6.283185307179586, S1 = -41.34170224039976, S2 = 81.60524927607506;
    constexpr double C1 = -19.739208802178716, C2 = 64.9393940226683, C3 = -85.45681720669373;
    const double r = p - rint(p);
    const double q = rint(kTurn * r);
    const double t = fma(-1.0 / kTurn, q, r), u = t * t;
    const double sn = t * fma(u, fma(u, S2, S1), S0);
    const double cs = fma(u, fma(u, fma(u, C3, C2), C1), 1.0);
    const double2 w = turn[(int)q & (kTurn - 1)];
    return make_double2(fma(w.x, cs, w.y * sn), fma(w.y, cs, -(w.x * sn)));
}

__device__ __forceinline__ double2 row64(const unsigned char *buf, int row, int k) {
    return *(const double2 *)(buf + row * kRS64 + k * 16);
}

__global__ void __launch_bounds__(512, 1) k_herk_coh64(FusedArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * kBuf64];
    __shared__ __attribute__((aligned(16))) Src64 src[3][2][kS64];  // stage % 3, half of the rows
    __shared__ double tab[2 * kB64][3];                              // (nu / c) x_a
    __shared__ double2 turn[kTurn];                                  // (cos, -sin) of i / 256 turns
    const int tid = threadIdx.x;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane & 15, lk = lane >> 4;
    const int Np = a.n_rows_pad;
    const int nb = (a.n_ant + kB64 - 1) / kB64;
    const int n_pair = nb * (nb - 1) / 2, n_diag = nb / 2, n_kind = n_pair + (nb + 1) / 2;
    const int units = a.work[a.n_inst];
    const int total = units * n_kind;
    const int fs = tid % kS64, fr = tid / kS64;  // forming: source, rows fr + 32 k
    const bool mult_first = wave < 4;
    if (tid < kTurn) {
        double sn, cs;
        sincospi(tid * (2.0 / kTurn), &sn, &cs);
        turn[tid] = make_double2(cs, -sn);
    }

    // Kind by kind, the heavier first (two diagonal blocks, the pairs with a short
    // last block as their rows at the end, a diagonal block alone), so that the
    // last wave of the grid holds the light ones; with the kinds of a split side by side
    // and 256 a multiple of their count every workgroup would keep one kind.
    for (int item = blockIdx.x; item < total; item += a.grid) {
        const int kind = item / units, unit = item % units;
        int lo = 0, hi = a.n_inst - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.work[mid] <= unit)
                lo = mid;
            else
                hi = mid - 1;
        }
        const int inst = lo;
        const int s = unit - a.work[inst];
        const bool pair = kind >= n_diag && kind < n_diag + n_pair;
        int I, J;
        if (pair) {  // (1, 0), (2, 0), (2, 1), (3, 0), ...
            int q = kind - n_diag;
            I = 1;
            while (q >= I) {
                q -= I;
                I++;
            }
            J = q;
        } else {
            I = kind < n_diag ? 2 * kind : nb - 1;
            J = kind < n_diag ? I + 1 : I;
        }
        // (one body per kind of item, so that each has its own accumulators)
        auto run = [&](auto is_pair) __attribute__((always_inline)) {
            constexpr bool off = decltype(is_pair)::value;
            const bool halves = !off && I == J;  // one block, the rows of the second half at the split's later sources
            const int tslot = inst / a.nfb;
            const int f = a.f0 + inst % a.nfb;
            const int64_t M = a.count[tslot];
            const int64_t per = a.kcols[inst] / 2;
            const int64_t m_begin = (int64_t)s * per;
            const int64_t m_end = m_begin + per < M ? m_begin + per : M;
            const int n_all = (int)((m_end - m_begin + kS64 - 1) / kS64);
            const int n_stage = halves ? (n_all + 1) / 2 : n_all;
            const double *sh = a.s_hat + (int64_t)tslot * 3 * a.ld_src;
            const double2 *Bm = (const double2 *)a.B + (int64_t)inst * 4 * a.ld_src;

            __syncthreads();  // the previous item's last reads of the tables
            if (tid < 2 * kB64) {
                const int ant = (tid < kB64 ? I : J) * kB64 + tid % kB64;
                const double nu_c = a.freqs[f] / kSpeedOfLight;
                const bool on = ant < a.n_ant;  // rows past the antennas only reach outputs that are never stored
                tab[tid][0] = on ? nu_c * a.antc[3 * ant] : 0.0;
                tab[tid][1] = on ? nu_c * a.antc[3 * ant + 1] : 0.0;
                tab[tid][2] = on ? nu_c * a.antc[3 * ant + 2] : 0.0;
            }
            // source data, one stage ahead, by the first lanes of wave 0 (lane 16 h + i:
            // source i of the half h)
            const bool fetcher = tid < 2 * kS64;
            const int half = tid / kS64;
            double fx = 0.0, fy = 0.0, fz = 0.0;
            double2 fb[4];
            auto fetch = [&](int stage) {
                const int64_t m = m_begin + (int64_t)(stage + (halves && half ? n_stage : 0)) * kS64 + fs;
                fx = fy = fz = 0.0;
                for (int c = 0; c < 4; c++) fb[c] = make_double2(0.0, 0.0);
                if (stage < n_stage && m < m_end) {
                    fx = sh[m];
                    fy = sh[a.ld_src + m];
                    fz = sh[2 * a.ld_src + m];
                    for (int c = 0; c < 4; c++) fb[c] = Bm[(int64_t)c * a.ld_src + m];
                }
            };
            auto stash = [&](int stage) {
                Src64 &e = src[stage % 3][half][fs];
                e.x = fx;
                e.y = fy;
                e.z = fz;
                // B components c = 2 p + k; C_10 = B_10 conj(B_00) + B_11 conj(B_01)
                e.c00 = fb[0].x * fb[0].x + fb[0].y * fb[0].y + fb[1].x * fb[1].x + fb[1].y * fb[1].y;
                e.c11 = fb[2].x * fb[2].x + fb[2].y * fb[2].y + fb[3].x * fb[3].x + fb[3].y * fb[3].y;
                e.c10x = fb[2].x * fb[0].x + fb[2].y * fb[0].y + fb[3].x * fb[1].x + fb[3].y * fb[1].y;
                e.c10y = fb[2].y * fb[0].x - fb[2].x * fb[0].y + fb[3].y * fb[1].x - fb[3].x * fb[1].y;
            };
            // Fringe rows of one stage: F = exp(-2 pi i p), p in cycles.  A source past the
            // split has zero weights, so its rows need no mask.
            auto produce = [&](unsigned char *buf, int stage) {
#pragma unroll 1
                for (int k = 0; k < 4; k++) {
                    const int r = fr + 32 * k;
                    const Src64 &e = src[stage % 3][k >> 1][fs];
                    const double p = tab[r][0] * e.x + tab[r][1] * e.y + tab[r][2] * e.z;
                    *(double2 *)(buf + r * kRS64 + fs * 16) = fringe64(p, turn);
                }
            };

            f64x4 re[9], im[9];
#pragma unroll
            for (int t = 0; t < 9; t++) re[t] = im[t] = f64x4{0.0, 0.0, 0.0, 0.0};
            // roles
            const int n_i = a.n_ant - I * kB64, nt_i = n_i < kB64 ? (n_i + 15) / 16 : 4;  // tile rows of block I
            const int n_j = a.n_ant - J * kB64, nt_j = n_j < kB64 ? (n_j + 15) / 16 : 4;
            const int bh = wave >> 2;                      // diagonal items: block of this wave
            const int nt = off ? nt_i : (bh ? nt_j : nt_i);
            // row tile, and for pairs the first of two column tiles (one row tile of a
            // short block: a column tile to each of four waves, on four SIMDs)
            const int rt = off ? (nt == 1 ? wave >> 2 : wave >> 1) : wave & 3;
            const int ct = nt == 1 ? wave & 3 : 2 * (wave & 1), nj = nt == 1 ? 1 : 2;

            auto consume = [&](const unsigned char *buf, int stage) __attribute__((always_inline)) {
                const Src64 *sp = src[stage % 3][off ? 0 : bh];
                if constexpr (off) {
                    if (rt >= nt) return;
#pragma unroll 1
                    for (int kk = 0; kk < kS64; kk += 4) {
                        const double2 v = row64(buf, 16 * rt + l16, kk + lk);
                        const double c00 = sp[kk + lk].c00, c11 = sp[kk + lk].c11;
                        const double cx = sp[kk + lk].c10x, cy = sp[kk + lk].c10y;
                        double2 b[2];
#pragma unroll
                        for (int j = 0; j < 2; j++) b[j] = row64(buf, kB64 + 16 * ((ct + j) & 3) + l16, kk + lk);
                        const double w[4][2] = {{c00 * v.x, c00 * v.y},
                                                {c11 * v.x, c11 * v.y},
                                                {cx * v.x - cy * v.y, cx * v.y + cy * v.x},
                                                {cx * v.x + cy * v.y, cx * v.y - cy * v.x}};
#pragma unroll
                        for (int q = 0; q < 4; q++)
#pragma unroll
                            for (int j = 0; j < 2; j++)
                                if (j < nj) mfma64(w[q][0], w[q][1], b[j], re[2 * q + j], im[2 * q + j]);
                    }
                } else {
                    const int o = bh * kB64;
#pragma unroll 1
                    for (int kk = 0; kk < kS64; kk += 4) {
                        const double2 v = row64(buf, o + 16 * rt + l16, kk + lk);
                        const double2 u = row64(buf, o + 16 * (3 - rt) + l16, kk + lk);
                        const double c00 = sp[kk + lk].c00, c11 = sp[kk + lk].c11;
                        const double cx = sp[kk + lk].c10x, cy = sp[kk + lk].c10y;
                        const double w00x = c00 * v.x, w00y = c00 * v.y, w11x = c11 * u.x, w11y = c11 * u.y;
                        const double w10x = cx * v.x - cy * v.y, w10y = cx * v.y + cy * v.x;
                        // slots 4..4 + r: V^00 tiles (r, slot - 4); the rest: V^11 tiles (3 - r, slot - 5 - r)
#pragma unroll
                        for (int c = 0; c < 4; c++)
                            if (rt < nt && c < nt)
                                mfma64(w10x, w10y, row64(buf, o + 16 * c + l16, kk + lk), re[c], im[c]);
#pragma unroll
                        for (int t = 0; t < 5; t++) {
                            const bool v00 = t <= rt;
                            if ((v00 ? rt : 3 - rt) < nt)
                                mfma64(v00 ? w00x : w11x, v00 ? w00y : w11y,
                                       row64(buf, o + 16 * (v00 ? t : t - rt - 1) + l16, kk + lk), re[4 + t], im[4 + t]);
                        }
                    }
                }
            };

            if (fetcher) {
                fetch(0);
                stash(0);
                fetch(1);
                stash(1);
            }
            __syncthreads();  // tables and the first two stages' sources ready
            produce(lds, 0);
            __syncthreads();
            for (int stg = 0; stg < n_stage; stg++) {
                unsigned char *cur = lds + (stg & 1) * kBuf64;
                unsigned char *nxt = lds + ((stg + 1) & 1) * kBuf64;
                const bool more = stg + 1 < n_stage;
                if (fetcher && stg + 2 < n_stage) fetch(stg + 2);
                if (!mult_first && more) produce(nxt, stg + 1);
                consume(cur, stg);
                if (mult_first && more) produce(nxt, stg + 1);
                // these sources take the place of stage stg - 1's, which nothing reads any more
                if (fetcher && stg + 2 < n_stage) stash(stg + 2);
                __syncthreads();
            }
            if (halves) {  // add the second half of the sources: its accumulators through LDS, four tiles at a time
                double2 *xch = (double2 *)lds;
#pragma unroll
                for (int t0 = 0; t0 < 9; t0 += 4) {
                    __syncthreads();
#pragma unroll
                    for (int t = t0; t < 9 && t < t0 + 4; t++)
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            if (bh)
                                xch[(((t - t0) * 4 + e) * 4 + (wave & 3)) * 64 + lane] =
                                    make_double2(re[t][e], im[t][e]);
                    __syncthreads();
#pragma unroll
                    for (int t = t0; t < 9 && t < t0 + 4; t++)
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            if (!bh) {
                                const double2 v = xch[(((t - t0) * 4 + e) * 4 + (wave & 3)) * 64 + lane];
                                re[t][e] += v.x;
                                im[t][e] += v.y;
                            }
                }
            }

            // Tile element e of a lane: row 4 e + lk, column l16.
            double2 *P = (double2 *)a.part + ((int64_t)inst * a.max_splits + s) * (int64_t)Np * Np;
            if constexpr (off) {
                if (rt < nt)
#pragma unroll
                    for (int q = 0; q < 4; q++)
#pragma unroll
                        for (int j = 0; j < 2; j++)
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                const int A = I * kB64 + 16 * rt + 4 * e + lk, Bc = J * kB64 + 16 * (ct + j) + l16;
                                const int p0 = q == 1 || q == 2 ? 1 : 0, q0 = q == 1 || q == 3 ? 1 : 0;
                                if (j < nj && A < a.n_ant && Bc < a.n_ant)
                                    P[(int64_t)(2 * A + p0) * Np + 2 * Bc + q0] =
                                        make_double2(re[2 * q + j][e], im[2 * q + j][e]);
                            }
            } else if (!(halves && bh)) {
                const int base = (bh ? J : I) * kB64;
#pragma unroll
                for (int t = 0; t < 9; t++) {
                    const bool v10 = t < 4, v00 = !v10 && t - 4 <= rt;
                    const int R = v10 || v00 ? rt : 3 - rt, C = v10 ? t : v00 ? t - 4 : t - 5 - rt;
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const int A = base + 16 * R + 4 * e + lk, Bc = base + 16 * C + l16;
                        if (A >= a.n_ant || Bc >= a.n_ant) continue;
                        const double vr = re[t][e], vi = im[t][e];
                        if (!v10) {
                            const int p0 = v00 ? 0 : 1;
                            P[(int64_t)(2 * A + p0) * Np + 2 * Bc + p0] = make_double2(vr, vi);
                        } else if (A >= Bc) {
                            P[(int64_t)(2 * A + 1) * Np + 2 * Bc] = make_double2(vr, vi);
                        } else {  // above the diagonal: conjugated at the transposed lower position
                            P[(int64_t)(2 * Bc) * Np + 2 * A + 1] = make_double2(vr, -vi);
                        }
                    }
                }
            }
        };
        if (pair)
            run(std::true_type{});
        else
            run(std::false_type{});
    }
}

// ---------------------------------------------------------------------------
// FP64 product over lists of 16 x 16 tiles with Z formed in LDS: scalar arrays, several
// beams, and requested pairs.  Lists and bundles are those of kernels_tiles.hip:
// a workgroup forms all rows of its bundle once per stage of 16 columns and multiplies up
// to eight tiles a wave.  MFMA-bound (1024 cycles a tile and stage), forming beside it by the
// other wave of the SIMD: 8 waves with a CU's LDS, or 4 with half of it.
// Against Z written to memory and multiplied from there in blocks of 64 (with k-splits
// that fill the chip), whole calls: 37 antennas, 2000 sources, 8 instances 83 -> 52 us; 30 / 100
// antennas, 30 000 sources, 32 instances 434 / 1158 -> 171 / 600 us.
// ---------------------------------------------------------------------------
struct Col64 {
    double x, y, z, pad;  // s_hat
    double2 b[2];         // values of both feeds (one beam)
};

struct Row64 {
    double x, y, z;     // x_a
    int32_t bp, pad;    // beam n_feed + feed
};

template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES, 2) k_tiles64(TileArgs a) {
    constexpr int ROWS = 16 * tile64_blocks(WAVES), BUF = ROWS * kRS64, NT = kWaveTiles64;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * BUF];
    __shared__ __attribute__((aligned(16))) Col64 col[2][kS64];
    __shared__ Row64 row[ROWS];
    __shared__ double2 turn[kTurn];  // (cos, -sin) of i / 256 turns
    static_assert((2 * BUF + sizeof(col) + sizeof(row) + sizeof(turn)) * (8 / WAVES) <= 160 * 1024, "LDS");
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane & 15, lk = lane >> 4;
    const int64_t item = blockIdx.x;
    const int s = (int)(item % a.n_split);
    const int bundle = (int)((item / a.n_split) % a.n_bundle);
    const int inst = (int)(item / ((int64_t)a.n_split * a.n_bundle));
    const int tslot = inst / a.nfb;
    const int nx = a.n_ax, nf = a.n_feed;
    const int64_t K = (int64_t)nx * a.count[tslot];
    const int64_t kc = split_cols(K, a.n_split);
    const int64_t kb = (int64_t)s * kc, ke = kb + kc < K ? kb + kc : K;
    if (kb >= K) return;  // an empty k-split: the reduction leaves it out too
    const TileBundle bd = a.bundles[bundle];
    const int n_rows = bd.n_rows;
    const double nu_c = a.freqs[a.f0 + inst % a.nfb] / kSpeedOfLight;
    const double *sh = a.s_hat + (int64_t)tslot * 3 * a.ld_src;
    const double2 *Bi = (const double2 *)a.B + (int64_t)inst * a.n_beam * nf * nx * a.ld_src;  // [beam][feed][axis][m]
    const bool shared_beam = a.n_beam == 1;
    for (int q = tid; q < n_rows; q += 64 * WAVES) {
        const int z = a.rows[bd.row0 + q], ant = z < 0 ? 0 : z / nf;  // padding rows reach no stored output
        row[q] = Row64{a.antc[3 * ant], a.antc[3 * ant + 1], a.antc[3 * ant + 2],
                       a.bidx[ant] * nf + (z < 0 ? 0 : z % nf), 0};
    }
    for (int q = tid; q < kTurn; q += 64 * WAVES) {
        double sn, cs;
        sincospi(q * (2.0 / kTurn), &sn, &cs);
        turn[q] = make_double2(cs, -sn);
    }
    const int n_stage = (int)((ke - kb + kS64 - 1) / kS64);

    // the columns of a stage, one per lane of the first 16
    const bool fetcher = tid < kS64;
    Col64 fc;
    auto fetch = [&](int stage) {
        const int64_t c = kb + (int64_t)stage * kS64 + tid;
        fc.x = fc.y = fc.z = fc.pad = 0.0;
        fc.b[0] = fc.b[1] = make_double2(0.0, 0.0);
        if (c < ke) {
            const int64_t m = c / nx;
            fc.x = sh[m];
            fc.y = sh[a.ld_src + m];
            fc.z = sh[2 * a.ld_src + m];
            if (shared_beam) {
                fc.b[0] = Bi[(c % nx) * a.ld_src + m];
                if (nf == 2) fc.b[1] = Bi[(nx + c % nx) * a.ld_src + m];
            }
        }
    };
    // one column (fs) of rows fr + 4 WAVES k
    const int fs = tid % kS64, fr = tid / kS64;
    auto produce = [&](unsigned char *buf, int stage) __attribute__((always_inline)) {
        const Col64 &c = col[stage & 1][fs];
        const double x = c.x, y = c.y, z = c.z;
        const int64_t cg = kb + (int64_t)stage * kS64 + fs;
#pragma unroll 1
        for (int r = fr; r < n_rows; r += 4 * WAVES) {
            const Row64 e = row[r];
            double2 b;
            if (shared_beam)
                b = c.b[e.bp];
            else
                b = cg < ke ? Bi[(e.bp * nx + cg % nx) * a.ld_src + cg / nx] : make_double2(0.0, 0.0);
            const double2 f = fringe64(nu_c * (e.x * x + e.y * y + e.z * z), turn);
            *(double2 *)(buf + r * kRS64 + fs * 16) =
                make_double2(b.x * f.x - b.y * f.y, b.x * f.y + b.y * f.x);
        }
    };

    if (fetcher) {
        fetch(0);
        col[0][tid] = fc;
        fetch(1);
        col[1][tid] = fc;
    }
    // this wave's tiles, sorted by column block: LDS offsets of their row and column blocks
    // (`fresh`: bit t set where the column block is not that of tile t - 1)
    const int t0 = bd.n_tiles * wave / WAVES, nt = bd.n_tiles * (wave + 1) / WAVES - t0;
    uint32_t ro[NT], co[NT], fresh = 0;
#pragma unroll
    for (int t = 0; t < NT; t++) {
        const int32_t e = a.tiles[bd.tile0 + (t < nt ? t0 + t : 0)];
        ro[t] = __builtin_amdgcn_readfirstlane((e & 255) * 16 * kRS64);
        co[t] = __builtin_amdgcn_readfirstlane((e >> 8) * 16 * kRS64);
        if (t == 0 || co[t] != co[t - 1]) fresh |= 1u << t;
    }
    __syncthreads();
    produce(lds, 0);
    __syncthreads();

    auto stages = [&](auto first) __attribute__((always_inline)) {
        f64x4 re[NT], im[NT];
#pragma unroll
        for (int t = 0; t < NT; t++) re[t] = im[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        auto consume = [&](const unsigned char *buf) __attribute__((always_inline)) {
            const unsigned char *p = buf + l16 * kRS64 + lk * 16;
            double2 b[4];
            int n = nt;
            uint32_t fr_ = fresh;
            asm volatile("" : "+s"(n), "+s"(fr_));  // tested here: no condition is kept across the stages
#pragma unroll
            for (int t = 0; t < NT; t++) {
                if (t < n) {
                    if (fr_ >> t & 1)
#pragma unroll
                        for (int q = 0; q < 4; q++) b[q] = *(const double2 *)(p + co[t] + q * 64);
                    double2 r[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) r[q] = *(const double2 *)(p + ro[t] + q * 64);
#pragma unroll
                    for (int q = 0; q < 4; q++) mfma64(r[q].x, r[q].y, b[q], re[t], im[t]);
                }
            }
        };
        for (int stg = 0; stg < n_stage; stg++) {
            unsigned char *cur = lds + (stg & 1) * BUF;
            unsigned char *nxt = lds + ((stg + 1) & 1) * BUF;
            const bool more = stg + 1 < n_stage;
            if constexpr (decltype(first)::value) {
                consume(cur);
                // the columns of stage stg + 2 replace those of stage stg, last read a stage ago
                if (fetcher && stg + 2 < n_stage) fetch(stg + 2);
                if (more) produce(nxt, stg + 1);
                if (fetcher && stg + 2 < n_stage) col[stg & 1][tid] = fc;
            } else {
                if (more) produce(nxt, stg + 1);
                consume(cur);
            }
            __syncthreads();
        }
        // the write-out's addresses are formed here rather than kept live across the stages
        int r4 = lk, c = l16, ld = a.ld;
        asm volatile("" : "+v"(r4), "+v"(c), "+v"(ld));
        double2 *P = (double2 *)a.part + ((int64_t)inst * a.n_split + s) * a.part_stride;
        const int32_t *dst = a.dst + bd.tile0 + t0;
#pragma unroll
        for (int t = 0; t < NT; t++)
            if (t < nt)
#pragma unroll
                for (int e = 0; e < 4; e++)
                    P[(int64_t)dst[t] + (4 * e + r4) * ld + c] = make_double2(re[t][e], im[t][e]);
    };
    if (wave < WAVES / 2)
        stages(std::true_type{});
    else
        stages(std::false_type{});
}

}  // namespace

bool f64_over_sources(int n_feed, int n_ax, int n_beam) { return n_feed == 2 && n_ax == 2 && n_beam == 1; }

int f64_items(int n_ant) {
    const int nb = (n_ant + kB64 - 1) / kB64;
    return nb * (nb - 1) / 2 + (nb + 1) / 2;
}

hipError_t launch_herk_f64(const FusedArgs &a, hipStream_t s) {
    if (a.n_inst <= 0) return hipSuccess;
    k_herk_coh64<<<a.grid, 512, 0, s>>>(a);
    return hipGetLastError();
}

int tile64_waves(int n_rows, int n_tiles) {
    return n_rows <= 16 * tile64_blocks(4) && n_tiles <= 4 * kWaveTiles64 ? 4 : 8;
}

hipError_t launch_tiles64(const TileArgs &a, hipStream_t s) {
    const int64_t items = (int64_t)a.n_inst * a.n_bundle * a.n_split;
    if (items <= 0) return hipSuccess;
    if (items * 64 * a.waves >= kMaxThreadsX || a.n_feed > 2 || a.n_ax > 2 || a.coherent) return hipErrorInvalidValue;
    if (a.waves == 4)
        k_tiles64<4><<<(unsigned)items, 256, 0, s>>>(a);
    else if (a.waves == 8)
        k_tiles64<8><<<(unsigned)items, 512, 0, s>>>(a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace mv
