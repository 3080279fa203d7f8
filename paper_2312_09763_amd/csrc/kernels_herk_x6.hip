// FP32 products on the bf16 matrix cores: every FP32 operand is split exactly into
// three bf16 terms (hi, mid, lo: 8 bits each, 24 in all), and
//   a b = al bh + ah bl + am bm + am bh + ah bm + ah bh,
// the omitted terms am bl, al bm and al bl below 2^-26 of |a b|, i.e. below the
// rounding of one FP32 product.  Six v_mfma_f32_16x16x32_bf16 take 96 cycles for
// the multiply-adds that eight v_mfma_f32_16x16x4f32 do in 256.
//
// The bf16 MFMA aligns its products to the accumulator and drops what falls some
// 2^-26 below it, so products are not added to a grown sum: the six products of a
// stage (16 complex) start from zero and are added to the accumulator by one FP32
// addition.  That costs 8 vector additions per 12 MFMAs and makes the result more
// exact than the FP32 MFMAs it replaced: error against 64 bits 1.2e-6 -> 2.3e-7 on 128
// antennas and 200 000 sources (16 x 16 instances; accumulating on the MFMA itself was
// 2.1e-6), 5.2e-7 -> 1.5e-7 on 350 antennas and 786 432 pixels.
//
// Bound by MFMAs and vector instructions together (2.4 per MFMA: splitting, column
// rotations, the additions); MFMAs are busy 61 % at 2.05 GHz (59 % in the block pairs).
// Product of the first case above 53.3 -> 31.7 ms; 350 polarised antennas, 1 x 4
// instances, whole call 28.3 -> 14.9 ms; 350 scalar antennas, 1 x 8, 14.4 -> 9.0 ms.
//
// The kernels are the FP32 forms of the product over sources (k_coh_x6 for the
// diagonal blocks, k_pairs_x6 for the block pairs) and of the three-block scalar
// product (k_blk3_x6); their items, wave roles and overlap of forming and
// multiplying are those of the BF16X3 kernels in kernels_herk_fused.hip.  A staged
// row is 16 complex in three planes of 64 bytes, 208 bytes with 16 of padding, so
// two stages of 384 rows fill the 160 KB of LDS; the antenna table and the
// sources of a stage live in the padding.
#include <type_traits>

#include "herk_tiles.h"
#include "matvis.h"

namespace mv {

namespace {

typedef RowGeom<208, 64, 1> GeomX6;
constexpr int kSPS = 16;                  // sources per stage
constexpr int kPad = 3 * GeomX6::PLANEB;  // the padding's offset in a row

// two sources (2 mp, 2 mp + 1) of a row
__device__ __forceinline__ void store_row(unsigned char *buf, int row, int mp, const float (&vr)[2],
                                          const float (&vi)[2]) {
    uint32_t h[2], m[2], l[2];
#pragma unroll
    for (int q = 0; q < 2; q++) split3(vr[q], vi[q], h[q], m[q], l[q]);
    unsigned char *p = buf + row * GeomX6::RS + mp * 8;
    *(uint2 *)p = make_uint2(h[0], h[1]);
    *(uint2 *)(p + GeomX6::PLANEB) = make_uint2(m[0], m[1]);
    *(uint2 *)(p + 2 * GeomX6::PLANEB) = make_uint2(l[0], l[1]);
}

struct Terms {
    u32x4 h, m, l;
};

__device__ __forceinline__ Terms load_terms(const unsigned char *p) {
    Terms t;
    t.h = *(const u32x4 *)p;
    t.m = *(const u32x4 *)(p + GeomX6::PLANEB);
    t.l = *(const u32x4 *)(p + 2 * GeomX6::PLANEB);
    return t;
}

// Accumulator of a tile, one part: four scalars (a vector is copied whole around the
// stage loop).
struct Acc {
    float v[4];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int e = 0; e < 4; e++) v[e] = 0.f;
    }
};

// One part (real, or imaginary with the column rotated) of one column against n <= G
// row tiles: t = the six products of a stage from zero, the smallest first.  The
// column's terms are taken one at a time (lo, mid, hi) and the parts one after the
// other, which keeps the operands beside the accumulators within the registers.
template <int G>
struct Part {
    const Terms *a[G];
    int n;
    f32x4 t[G];
    template <u32x4 Terms::*T>
    __device__ __forceinline__ void round(const u32x4 &b) {
#pragma unroll
        for (int i = 0; i < G; i++)
            if (i < n)
                t[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[i]->*T),
                                                               __builtin_bit_cast(bf16x8, b), t[i], 0, 0, 0);
    }
    __device__ __forceinline__ void lo(const u32x4 &b) {
#pragma unroll
        for (int i = 0; i < G; i++) t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        round<&Terms::h>(b);
    }
    __device__ __forceinline__ void mid(const u32x4 &b) {
        round<&Terms::m>(b);
        round<&Terms::h>(b);
    }
    __device__ __forceinline__ void hi(const u32x4 &b) {
        round<&Terms::l>(b);
        round<&Terms::m>(b);
        round<&Terms::h>(b);
    }
    __device__ __forceinline__ void add(Acc *const (&acc)[G]) const {
#pragma unroll
        for (int i = 0; i < G; i++)
            if (i < n)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    acc[i]->v[e] += t[i][e];
                    asm volatile("" : "+v"(acc[i]->v[e]));  // added here, not after the stage's forming
                }
    }
};

// Both parts of the column at p (LDS) against the row tiles of `part`; next holds its
// lo term, and after the last term the word at `after` (the next column's lo term).
template <int G>
__device__ __forceinline__ void column(Part<G> &part, const unsigned char *p, const unsigned char *after, u32x4 &next,
                                       Acc *const (&re)[G], Acc *const (&im)[G]) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
        u32x4 b = h ? bf16_rot_col(next) : next;
        next = *(const u32x4 *)(p + GeomX6::PLANEB);
        __builtin_amdgcn_sched_barrier(0);  // keep each prefetch ahead of the products
        part.lo(b);
        __builtin_amdgcn_sched_barrier(0);
        b = h ? bf16_rot_col(next) : next;
        next = *(const u32x4 *)p;
        __builtin_amdgcn_sched_barrier(0);
        part.mid(b);
        __builtin_amdgcn_sched_barrier(0);
        b = h ? bf16_rot_col(next) : next;
        next = *(const u32x4 *)(h ? after : p + 2 * GeomX6::PLANEB);
        __builtin_amdgcn_sched_barrier(0);
        part.hi(b);
        __builtin_amdgcn_sched_barrier(0);
        part.add(h ? im : re);
    }
}

// Rows 16 (rb + i), i < NR, against columns 16 (cb + j), j < NC; slot i * kTI + j.
template <int NACC, int NR, int NC>
__device__ __forceinline__ void consume_sq(const unsigned char *buf, int rb, int cb, int l16, int lk, Acc (&re)[NACC],
                                           Acc (&im)[NACC]) {
    Terms a[NR];
    Part<NR> part;
    part.n = NR;
#pragma unroll
    for (int i = 0; i < NR; i++) {
        a[i] = load_terms(buf + (16 * (rb + i) + l16) * GeomX6::RS + lk * 16);
        part.a[i] = &a[i];
    }
    const unsigned char *pc = buf + (16 * cb + l16) * GeomX6::RS + lk * 16;
    u32x4 next = *(const u32x4 *)(pc + 2 * GeomX6::PLANEB);
#pragma unroll
    for (int j = 0; j < NC; j++) {
        Acc *r[NR], *m[NR];
#pragma unroll
        for (int i = 0; i < NR; i++) r[i] = &re[i * kTI + j], m[i] = &im[i * kTI + j];
        const unsigned char *p = pc + 16 * j * GeomX6::RS;
        column<NR>(part, p, p + (j + 1 < NC ? 16 * GeomX6::RS : 0) + 2 * GeomX6::PLANEB, next, r, m);
    }
}

// One diagonal triangle starting at LDS row o: tiles (r, c), c <= r, r in the set T.
template <typename T, int NACC>
__device__ __forceinline__ void consume_tri(const unsigned char *buf, int o, int l16, int lk, Acc (&re)[NACC],
                                            Acc (&im)[NACC]) {
    constexpr int NR = T::NR;
    const unsigned char *p0 = buf + (o + l16) * GeomX6::RS + lk * 16;
    Terms a[NR];
#pragma unroll
    for (int k = 0; k < NR; k++) a[k] = load_terms(p0 + 16 * T::r[k] * GeomX6::RS);
    u32x4 next = *(const u32x4 *)(p0 + 16 * T::order[0] * GeomX6::RS + 2 * GeomX6::PLANEB);
#pragma unroll
    for (int q = 0; q < T::ncol; q++) {
        const int c = T::order[q], cn = q + 1 < T::ncol ? T::order[q + 1] : c;
        Part<NR> part;  // the rows at or below this column
        Acc *r[NR], *m[NR];
        part.n = 0;
#pragma unroll
        for (int k = 0; k < NR; k++) part.a[k] = &a[0], r[k] = &re[0], m[k] = &im[0];
#pragma unroll
        for (int k = 0; k < NR; k++)
            if (T::r[k] >= c) {
                part.a[part.n] = &a[k];
                r[part.n] = &re[T::base[k] + c];
                m[part.n] = &im[T::base[k] + c];
                part.n++;
            }
        column<NR>(part, p0 + 16 * c * GeomX6::RS, p0 + 16 * cn * GeomX6::RS + 2 * GeomX6::PLANEB, next, r, m);
    }
}

// Work item of a persistent launch with n_kind items per k-split.
struct Item {
    int inst, s, kind;
};
__device__ __forceinline__ Item locate(const FusedArgs &a, int item, int n_kind) {
    int lo = 0, hi = a.n_inst - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.work[mid] * n_kind <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    const int local = item - a.work[lo] * n_kind;
    return Item{lo, local / n_kind, local % n_kind};
}

// Table and sources in the row padding of two stage buffers of BUF bytes: antenna
// entry as at rows as of both buffers, source m of stage parity st in three pieces
// from row SRC0 of buffer 0 on.
struct Src {
    double x, y, z;         // s_hat
    float f0, f1, f2, f3;   // per-source factors (0 past the split)
};
template <int BUF, int SRC0>
struct Pads {
    unsigned char *lds;
    __device__ void put_ant(int as, double x, double y, double z) const {
        unsigned char *p = lds + as * GeomX6::RS + kPad;
        *(double2 *)p = make_double2(x, y);
        *(double *)(p + BUF) = z;
    }
    __device__ void ant(int as, double &x, double &y, double &z) const {
        const unsigned char *p = lds + as * GeomX6::RS + kPad;
        const double2 v = *(const double2 *)p;
        x = v.x;
        y = v.y;
        z = *(const double *)(p + BUF);
    }
    __device__ unsigned char *at(int st, int m, int piece) const {
        return lds + (SRC0 + (kSPS * st + m) * 3 + piece) * GeomX6::RS + kPad;
    }
    __device__ void put_src(int st, int m, const Src &e) const {
        *(double2 *)at(st, m, 0) = make_double2(e.x, e.y);
        *(double *)at(st, m, 1) = e.z;
        *(float4 *)at(st, m, 2) = make_float4(e.f0, e.f1, e.f2, e.f3);
    }
    __device__ Src src(int st, int m) const {
        const double2 xy = *(const double2 *)at(st, m, 0);
        const float4 f = *(const float4 *)at(st, m, 2);
        return Src{xy.x, xy.y, *(const double *)at(st, m, 1), f.x, f.y, f.z, f.w};
    }
    // a factor more, of the other block's rows
    __device__ void put_factor(int st, int m, float g) const { *(float *)(at(st, m, 1) + 8) = g; }
    __device__ float factor(int st, int m) const { return *(const float *)(at(st, m, 1) + 8); }
};

// ---------------------------------------------------------------------------
// Diagonal blocks of the product over sources: planes P0 = s0 F, P1 = s1 F,
// L = l F of 128 antennas; waves 0-3 V^10 = L P0^H as 64 x 64 wave tiles, waves 4-7
// the triangles of V^00 and V^11.  SHORT: the last block, at most 96 antennas.
// SQ_ANT antennas are formed by the square waves, the rest by the triangle waves.
// ---------------------------------------------------------------------------
template <int SQ_ANT, bool SHORT>
__global__ void __launch_bounds__(512, 1) k_coh_x6(FusedArgs a) {
    constexpr int BUF = 3 * kST * GeomX6::RS;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * BUF];
    static_assert(2 * BUF <= 160 * 1024, "two stages exceed the LDS");
    const Pads<BUF, kST> pads{lds};
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const bool sq = wave < 4;
    const int l16 = lane & 15, lk = lane >> 4;
    const int Np = a.n_rows_pad;
    const int nb = Np / (2 * kST);
    const bool has_short = short_last_block(a.n_ant, nb);
    const int n_kind = SHORT ? 1 : has_short ? nb - 1 : nb;
    const int total = a.work[a.n_inst] * n_kind;
    const int per_xcd = a.grid / 8;
    const int slot_x = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const int mp = tid % (kSPS / 2);  // source pair
    const int a0 = SHORT ? (sq ? wrow(tid) : 64 + wrow(tid - 256)) : (sq ? wrow(tid) : SQ_ANT + wrow(tid - 256));
    const int sq_r0 = (SHORT ? 3 : 4) * (wave >> 1), sq_c0 = (SHORT ? 3 : 4) * (wave & 1);
    const int tri_t = (wave - 4) >> 1, tri_s = (wave - 4) & 1;
    const int tri_o = tri_t * kST;

    for (int item = slot_x; item < total; item += a.grid) {
        const Item it = locate(a, item, n_kind);
        const int I = SHORT ? nb - 1 : it.kind;
        const int tslot = it.inst / a.nfb;
        const int f = a.f0 + it.inst % a.nfb;
        const int64_t M = a.count[tslot];
        const int64_t per = a.kcols[it.inst] / 2;
        const int64_t m_begin = (int64_t)it.s * per, m_end = m_begin + per < M ? m_begin + per : M;
        const double *sh = a.s_hat + (int64_t)tslot * 3 * a.ld_src;
        const float2 *Bm = (const float2 *)a.B + (int64_t)it.inst * 4 * a.ld_src;
        const double nu_c = a.freqs[f] / kSpeedOfLight;
        if (tid < kST) {  // (padding antennas only reach outputs that are never stored)
            const int ant = I * kST + tid;
            const bool on = ant < a.n_ant;
            pads.put_ant(tid, on ? nu_c * a.antc[3 * ant] : 0.0, on ? nu_c * a.antc[3 * ant + 1] : 0.0,
                         on ? nu_c * a.antc[3 * ant + 2] : 0.0);
        }
        const int n_stage = (int)((m_end - m_begin + kSPS - 1) / kSPS);
        // direction and coherency factors, one stage ahead by the first lanes of wave 0
        const bool fetcher = tid < kSPS;
        double fx = 0.0, fy = 0.0, fz = 0.0;
        float2 fb[4];
        auto fetch = [&](int stage) {
            const int64_t m = m_begin + (int64_t)stage * kSPS + tid;
            fx = fy = fz = 0.0;
            for (int c = 0; c < 4; c++) fb[c] = make_float2(0.f, 0.f);
            if (stage < n_stage && m < m_end) {
                fx = sh[m];
                fy = sh[a.ld_src + m];
                fz = sh[2 * a.ld_src + m];
                for (int c = 0; c < 4; c++) fb[c] = Bm[(int64_t)c * a.ld_src + m];
            }
        };
        auto stash = [&](int stage) {
            // B components c = 2 p + k; C10 = B10 conj(B00) + B11 conj(B01)
            const float c00 = fb[0].x * fb[0].x + fb[0].y * fb[0].y + fb[1].x * fb[1].x + fb[1].y * fb[1].y;
            const float c11 = fb[2].x * fb[2].x + fb[2].y * fb[2].y + fb[3].x * fb[3].x + fb[3].y * fb[3].y;
            const float c10x = fb[2].x * fb[0].x + fb[2].y * fb[0].y + fb[3].x * fb[1].x + fb[3].y * fb[1].y;
            const float c10y = fb[2].y * fb[0].x - fb[2].x * fb[0].y + fb[3].y * fb[1].x - fb[3].x * fb[1].y;
            const float s0 = sqrtf(c00);
            pads.put_src(stage & 1, tid, Src{fx, fy, fz, s0, sqrtf(c11), s0 > 0.f ? c10x / s0 : 0.f,
                                             s0 > 0.f ? c10y / s0 : 0.f});
        };
        auto produce_n = [&](unsigned char *buf, int stage, auto na) __attribute__((always_inline)) {
            Src w[2];
            w[0] = pads.src(stage & 1, 2 * mp);
            w[1] = pads.src(stage & 1, 2 * mp + 1);
#pragma unroll
            for (int k = 0; k < decltype(na)::value; k++) {
                const int as = a0 + 32 * k;
                double ux, uy, uz;
                pads.ant(as, ux, uy, uz);
                float fr[2], fi[2], vr[2], vi[2];
#pragma unroll
                for (int q = 0; q < 2; q++) fringe(ux * w[q].x + uy * w[q].y + uz * w[q].z, fr[q], fi[q]);
#pragma unroll
                for (int q = 0; q < 2; q++) vr[q] = w[q].f0 * fr[q], vi[q] = w[q].f0 * fi[q];
                store_row(buf, as, mp, vr, vi);
#pragma unroll
                for (int q = 0; q < 2; q++) vr[q] = w[q].f1 * fr[q], vi[q] = w[q].f1 * fi[q];
                store_row(buf, kST + as, mp, vr, vi);
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    vr[q] = w[q].f2 * fr[q] - w[q].f3 * fi[q];
                    vi[q] = w[q].f2 * fi[q] + w[q].f3 * fr[q];
                }
                store_row(buf, 2 * kST + as, mp, vr, vi);
            }
        };
        auto produce = [&](unsigned char *buf, int stage) __attribute__((always_inline)) {
            if (sq)
                produce_n(buf, stage, std::integral_constant<int, SHORT ? 2 : SQ_ANT / 32>{});
            else
                produce_n(buf, stage, std::integral_constant<int, SHORT ? 1 : (kST - SQ_ANT) / 32>{});
        };

        if (fetcher) {
            fetch(0);
            stash(0);
            fetch(1);
            stash(1);
        }
        __syncthreads();  // antenna table and the first two stages' sources ready
        produce(lds, 0);
        __syncthreads();
        float2 *P = (float2 *)a.part + ((int64_t)it.inst * a.max_splits + it.s) * (int64_t)Np * Np;
        // The stages of one wave role (every wave meets the same barriers): a body for
        // each role, so that each has its own accumulators.  The square waves multiply
        // before they form, the triangle waves after.
        auto stages = [&](auto consume, auto write, auto first) __attribute__((always_inline)) {
            for (int stg = 0; stg < n_stage; stg++) {
                unsigned char *cur = lds + (stg & 1) * BUF;
                unsigned char *nxt = lds + ((stg + 1) & 1) * BUF;
                const bool more = stg + 1 < n_stage;
                if constexpr (decltype(first)::value) {
                    consume(cur);
                    // the sources of stage stg + 2 (those of its parity were last read a stage
                    // ago) are loaded while wave 0 forms: they hold no registers while it multiplies
                    if (fetcher && stg + 2 < n_stage) fetch(stg + 2);
                    if (more) produce_n(nxt, stg + 1, std::integral_constant<int, SHORT ? 2 : SQ_ANT / 32>{});
                    if (fetcher && stg + 2 < n_stage) stash(stg + 2);
                } else {
                    if (more)
                        produce_n(nxt, stg + 1, std::integral_constant<int, SHORT ? 1 : (kST - SQ_ANT) / 32>{});
                    consume(cur);
                }
                __syncthreads();
            }
            // the write-out's addresses are formed here rather than kept live across the stages
            int ld = Np, row = 4 * lk, col = l16;
            asm volatile("" : "+v"(ld), "+v"(row), "+v"(col));
            write(ld, row, col);
        };
        auto square = [&]() __attribute__((always_inline)) {
            constexpr int NT = SHORT ? 3 : kTI;
            Acc re[16], im[16];
#pragma unroll
            for (int t = 0; t < 16; t++) re[t].clear(), im[t].clear();
            stages([&](const unsigned char *buf) __attribute__((always_inline)) {
                consume_sq<16, NT, NT>(buf, 16 + sq_r0, sq_c0, l16, lk, re, im);
            }, [&](int ld, int row, int col) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < NT; i++)
#pragma unroll
                    for (int j = 0; j < NT; j++) {
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int ra = I * kST + 16 * (sq_r0 + i) + row + e;
                            const int cb = I * kST + 16 * (sq_c0 + j) + col;
                            const float vr = re[i * kTI + j].v[e], vi = im[i * kTI + j].v[e];
                            if (ra >= a.n_ant || cb >= a.n_ant) continue;
                            if (ra >= cb)
                                P[(int64_t)(2 * ra + 1) * ld + 2 * cb] = make_float2(vr, vi);
                            else  // above the diagonal: conjugated at the transposed lower position
                                P[(int64_t)(2 * cb) * ld + 2 * ra + 1] = make_float2(vr, -vi);
                        }
                    }
            }, std::true_type{});
        };
        auto triangle = [&](auto set) __attribute__((always_inline)) {
            typedef typename decltype(set)::type T;
            constexpr int NACC = T::base[T::NR - 1] + T::r[T::NR - 1] + 1;
            Acc re[NACC], im[NACC];
#pragma unroll
            for (int t = 0; t < NACC; t++) re[t].clear(), im[t].clear();
            stages([&](const unsigned char *buf) __attribute__((always_inline)) {
                consume_tri<T>(buf, tri_o, l16, lk, re, im);
            }, [&](int ld, int row, int col) __attribute__((always_inline)) {
                for_tri_tiles<T>([&](int t, int R, int C) __attribute__((always_inline)) {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const int ra = I * kST + 16 * R + row + e, cb = I * kST + 16 * C + col;
                        if (ra >= a.n_ant || cb >= a.n_ant) continue;
                        P[(int64_t)(2 * ra + tri_t) * ld + 2 * cb + tri_t] = make_float2(re[t].v[e], im[t].v[e]);
                    }
                });
            }, std::false_type{});
        };
        typedef typename std::conditional<SHORT, TriSet6<0>, TriSet<0>>::type T0;
        typedef typename std::conditional<SHORT, TriSet6<1>, TriSet<1>>::type T1;
        if (sq)
            square();
        else if (tri_s == 0)
            triangle(SetTag<T0>{});
        else
            triangle(SetTag<T1>{});
    }
}

// ---------------------------------------------------------------------------
// Block pairs I > J of the product over sources, two kinds of item per pair as in
// k_herk_pairs: rows w0 F_I, w1 F_I against the columns g F_J with (w0, w1) = (C_00, C_11)
// or (C_10, conj C_10), over g (see stash).  Waves s and s + 4 (one SIMD) take the two
// products with opposite row halves and the same column half; row tiles past a
// short block I are neither formed nor multiplied.  (The columns are rotated in
// registers: a fourth plane does not fit the LDS.)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(512, 1) k_pairs_x6(FusedArgs a) {
    constexpr int BUF = 3 * kST * GeomX6::RS;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * BUF];
    const Pads<BUF, 2 * kST> pads{lds};
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane & 15, lk = lane >> 4;
    const int Np = a.n_rows_pad;
    const int nb = Np / (2 * kST);
    const int n_kind = nb * (nb - 1);
    const int total = a.work[a.n_inst] * n_kind;
    const int per_xcd = a.grid / 8;
    const int slot_x = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const int mp = tid % (kSPS / 2);
    const int simd = wave & 3, pr = wave >> 2;
    const int rh = (simd >> 1) ^ pr, ch = simd & 1;
    const int a0 = wrow(tid);  // antennas a0 + 64 k of the 256 of blocks I (k < 2) and J
    const bool mult_first = wave < 4;

    for (int item = slot_x; item < total; item += a.grid) {
        const Item it = locate(a, item, n_kind);
        const bool kind_y = it.kind & 1;
        int q = it.kind >> 1, I = 1;  // pairs (1, 0), (2, 0), (2, 1), (3, 0), ...
        while (q >= I) {
            q -= I;
            I++;
        }
        const int J = q;
        const int n_i = a.n_ant - I * kST < kST ? a.n_ant - I * kST : kST;
        const int nt = (n_i + 15) / 16, nt0 = (nt + 1) / 2;
        const int r0 = rh ? nt0 : 0, nrt = rh ? nt - nt0 : nt0;  // this wave's first row tile and count
        const int tslot = it.inst / a.nfb;
        const int f = a.f0 + it.inst % a.nfb;
        const int64_t M = a.count[tslot];
        const int64_t per = a.kcols[it.inst] / 2;
        const int64_t m_begin = (int64_t)it.s * per, m_end = m_begin + per < M ? m_begin + per : M;
        const double *sh = a.s_hat + (int64_t)tslot * 3 * a.ld_src;
        const float2 *Bm = (const float2 *)a.B + (int64_t)it.inst * 4 * a.ld_src;
        const double nu_c = a.freqs[f] / kSpeedOfLight;
        if (tid < 2 * kST) {
            const int ant = tid < kST ? I * kST + tid : J * kST + (tid - kST);
            const bool on = ant < a.n_ant;
            pads.put_ant(tid, on ? nu_c * a.antc[3 * ant] : 0.0, on ? nu_c * a.antc[3 * ant + 1] : 0.0,
                         on ? nu_c * a.antc[3 * ant + 2] : 0.0);
        }
        const int n_stage = (int)((m_end - m_begin + kSPS - 1) / kSPS);
        const bool fetcher = tid < kSPS;
        double fx = 0.0, fy = 0.0, fz = 0.0;
        float2 fb[4];
        auto fetch = [&](int stage) {
            const int64_t m = m_begin + (int64_t)stage * kSPS + tid;
            fx = fy = fz = 0.0;
            for (int c = 0; c < 4; c++) fb[c] = make_float2(0.f, 0.f);
            if (stage < n_stage && m < m_end) {
                fx = sh[m];
                fy = sh[a.ld_src + m];
                fz = sh[2 * a.ld_src + m];
                for (int c = 0; c < 4; c++) fb[c] = Bm[(int64_t)c * a.ld_src + m];
            }
        };
        // the two complex weights (f0, f1), (f2, f3): C_00 and C_11, or C_10 and its conjugate, over
        // g = sqrt(max(C_00, C_11)), which the rows of block J take: both operands then stay of the
        // size of B and their low terms within FP32's range wherever B's square is
        auto stash = [&](int stage) {
            const float c00 = fb[0].x * fb[0].x + fb[0].y * fb[0].y + fb[1].x * fb[1].x + fb[1].y * fb[1].y;
            const float c11 = fb[2].x * fb[2].x + fb[2].y * fb[2].y + fb[3].x * fb[3].x + fb[3].y * fb[3].y;
            const float g = sqrtf(fmaxf(c00, c11)), r = g > 0.f ? 1.f / g : 0.f;
            float w0 = c00, w1 = c11;
            if (kind_y) {
                w0 = fb[2].x * fb[0].x + fb[2].y * fb[0].y + fb[3].x * fb[1].x + fb[3].y * fb[1].y;
                w1 = fb[2].y * fb[0].x - fb[2].x * fb[0].y + fb[3].y * fb[1].x - fb[3].x * fb[1].y;
            }
            w0 *= r;
            w1 *= r;
            pads.put_src(stage & 1, tid,
                         Src{fx, fy, fz, w0, kind_y ? w1 : 0.f, kind_y ? w0 : w1, kind_y ? -w1 : 0.f});
            pads.put_factor(stage & 1, tid, g);
        };
        // Weighted rows of block I or the rows of block J for this thread's two
        // sources; a source past the split has zero weights.
        auto produce = [&](unsigned char *buf, int stage) __attribute__((always_inline)) {
            Src w[2];
            w[0] = pads.src(stage & 1, 2 * mp);
            w[1] = pads.src(stage & 1, 2 * mp + 1);
            const float g[2] = {pads.factor(stage & 1, 2 * mp), pads.factor(stage & 1, 2 * mp + 1)};
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int as = a0 + 64 * k;
                if (k < 2 && as >= n_i) continue;
                double ux, uy, uz;
                pads.ant(as, ux, uy, uz);
                float fr[2], fi[2], vr[2], vi[2];
#pragma unroll
                for (int s = 0; s < 2; s++) fringe(ux * w[s].x + uy * w[s].y + uz * w[s].z, fr[s], fi[s]);
                if (k >= 2) {
#pragma unroll
                    for (int s = 0; s < 2; s++) vr[s] = g[s] * fr[s], vi[s] = g[s] * fi[s];
                    store_row(buf, kST + as, mp, vr, vi);  // plane 2: row as - kST of block J
                    continue;
                }
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    vr[s] = w[s].f0 * fr[s] - w[s].f1 * fi[s];
                    vi[s] = w[s].f0 * fi[s] + w[s].f1 * fr[s];
                }
                store_row(buf, as, mp, vr, vi);
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    vr[s] = w[s].f2 * fr[s] - w[s].f3 * fi[s];
                    vi[s] = w[s].f2 * fi[s] + w[s].f3 * fr[s];
                }
                store_row(buf, kST + as, mp, vr, vi);
            }
        };
        if (fetcher) {
            fetch(0);
            stash(0);
            fetch(1);
            stash(1);
        }
        __syncthreads();
        produce(lds, 0);
        __syncthreads();
        float2 *P = (float2 *)a.part + ((int64_t)it.inst * a.max_splits + it.s) * (int64_t)Np * Np;
        // a body per number of row tiles (every wave meets the same barriers)
        auto run = [&](auto rows) __attribute__((always_inline)) {
            constexpr int NR = decltype(rows)::value;
            Acc re[16], im[16];
#pragma unroll
            for (int t = 0; t < 16; t++) re[t].clear(), im[t].clear();
            for (int stg = 0; stg < n_stage; stg++) {
                unsigned char *cur = lds + (stg & 1) * BUF;
                unsigned char *nxt = lds + ((stg + 1) & 1) * BUF;
                const bool more = stg + 1 < n_stage;
                if (!mult_first && more) produce(nxt, stg + 1);
                if constexpr (NR > 0) consume_sq<16, NR, kTI>(cur, pr * 8 + r0, 2 * 8 + 4 * ch, l16, lk, re, im);
                if (mult_first && more) {
                    if (fetcher && stg + 2 < n_stage) fetch(stg + 2);
                    produce(nxt, stg + 1);
                    if (fetcher && stg + 2 < n_stage) stash(stg + 2);
                }
                __syncthreads();
            }
            if constexpr (NR > 0) {
                int ld = Np, row = 4 * lk, col = l16;
                asm volatile("" : "+v"(ld), "+v"(row), "+v"(col));
                // product pr at antennas A of I (rows), B of J (columns): X V^pp at (2 A + pr,
                // 2 B + pr); Y V^10 at (2 A + 1, 2 B) and V^01 at (2 A, 2 B + 1)
                const int row_off = kind_y ? 1 - pr : pr;
#pragma unroll
                for (int i = 0; i < NR; i++)
#pragma unroll
                    for (int j = 0; j < kTI; j++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int A = I * kST + 16 * (r0 + i) + row + e, Bc = J * kST + 16 * (4 * ch + j) + col;
                            if (A < a.n_ant && Bc < a.n_ant)
                                P[(int64_t)(2 * A + row_off) * ld + 2 * Bc + pr] =
                                    make_float2(re[i * kTI + j].v[e], im[i * kTI + j].v[e]);
                        }
            }
        };
        switch (nrt) {
            case 4: run(std::integral_constant<int, 4>{}); break;
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 2: run(std::integral_constant<int, 2>{}); break;
            case 1: run(std::integral_constant<int, 1>{}); break;
            default: run(std::integral_constant<int, 0>{}); break;
        }
    }
}

// ---------------------------------------------------------------------------
// Scalar rows (one feed, one axis, one shared beam) in three blocks of 128: the items
// of k_herk_blk3 (kind 0: V_10 and the triangle of block 0; 1: V_21 and block 1;
// 2: V_20 and block 2), plane 0 the column block, plane 1 the row block, rows |B| F.
// ---------------------------------------------------------------------------
template <int SQ_ROWS>
__global__ void __launch_bounds__(512, 1) k_blk3_x6(FusedArgs a) {
    constexpr int BUF = 2 * kST * GeomX6::RS;
    static_assert(SQ_ROWS % 32 == 0, "32 rows per pass of a wave group");
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * BUF];
    __shared__ double tab[2 * kST][3];
    __shared__ Src src[2][kSPS];
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const bool sq = wave < 4;
    const int l16 = lane & 15, lk = lane >> 4;
    const int Np = a.n_rows_pad;
    constexpr int n_kind = 3;
    const int total = a.work[a.n_inst] * n_kind;
    const int per_xcd = a.grid / 8;
    const int slot_x = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const int mp = tid % (kSPS / 2);
    const int a0 = sq ? wrow(tid) : SQ_ROWS + wrow(tid - 256);
    const int sq_c0 = 4 * (wave & 1), tri_s = (wave - 4) & 3;

    for (int item = slot_x; item < total; item += a.grid) {
        const Item it = locate(a, item, n_kind);
        const int kind = it.kind;
        const int R = kind == 0 ? 1 : 2, C = kind == 1 ? 1 : 0, T = kind;
        const int tri_o = (T == C ? 0 : 1) * kST;
        // only the last block (2) can be short: its rows past the antennas are not formed, the
        // square waves split its row tiles evenly and a triangle wave drops its rows past them
        const int n_r = a.n_ant - R * kST < kST ? a.n_ant - R * kST : kST;
        const int n_t = a.n_ant - T * kST < kST ? a.n_ant - T * kST : kST;
        const int nt_r = (n_r + 15) / 16, nt0 = (nt_r + 1) / 2, nt_t = (n_t + 15) / 16;
        const int sq_r0 = (wave >> 1) ? nt0 : 0, sq_nr = (wave >> 1) ? nt_r - nt0 : nt0;
        const int tri_nr = 7 - tri_s < nt_t ? 2 : tri_s < nt_t ? 1 : 0;
        const int tslot = it.inst / a.nfb;
        const int f = a.f0 + it.inst % a.nfb;
        const int64_t M = a.count[tslot];
        const int64_t per = a.kcols[it.inst];
        const int64_t m_begin = (int64_t)it.s * per, m_end = m_begin + per < M ? m_begin + per : M;
        const double *sh = a.s_hat + (int64_t)tslot * 3 * a.ld_src;
        const float2 *Bm = (const float2 *)a.B + (int64_t)it.inst * a.ld_src;
        const double nu_c = a.freqs[f] / kSpeedOfLight;
        if (tid < 2 * kST) {
            const int ant = (tid < kST ? C : R) * kST + (tid & (kST - 1));
            const bool on = ant < a.n_ant;
            for (int c = 0; c < 3; c++) tab[tid][c] = on ? nu_c * a.antc[3 * ant + c] : 0.0;
        }
        const int n_stage = (int)((m_end - m_begin + kSPS - 1) / kSPS);
        const bool fetcher = tid < kSPS;
        double fx = 0.0, fy = 0.0, fz = 0.0;
        float2 fb = make_float2(0.f, 0.f);
        auto fetch = [&](int stage) {
            const int64_t m = m_begin + (int64_t)stage * kSPS + tid;
            fx = fy = fz = 0.0;
            fb = make_float2(0.f, 0.f);
            if (stage < n_stage && m < m_end) {
                fx = sh[m];
                fy = sh[a.ld_src + m];
                fz = sh[2 * a.ld_src + m];
                fb = Bm[m];
            }
        };
        auto stash = [&](int stage) {
            src[stage & 1][tid] = Src{fx, fy, fz, sqrtf(fb.x * fb.x + fb.y * fb.y), 0.f, 0.f, 0.f};
        };
        auto produce_n = [&](unsigned char *buf, int stage, auto na) __attribute__((always_inline)) {
            const Src &s0 = src[stage & 1][2 * mp], &s1 = src[stage & 1][2 * mp + 1];
            const double x[2] = {s0.x, s1.x}, y[2] = {s0.y, s1.y}, z[2] = {s0.z, s1.z};
            const float g[2] = {s0.f0, s1.f0};
#pragma unroll
            for (int k = 0; k < decltype(na)::value; k++) {
                const int as = a0 + 32 * k;
                if (as >= kST + n_r) continue;
                float vr[2], vi[2];
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    float fr, fi;
                    fringe(tab[as][0] * x[s] + tab[as][1] * y[s] + tab[as][2] * z[s], fr, fi);
                    vr[s] = g[s] * fr;
                    vi[s] = g[s] * fi;
                }
                store_row(buf, as, mp, vr, vi);
            }
        };
        typedef std::integral_constant<int, SQ_ROWS / 32> SqN;
        typedef std::integral_constant<int, (2 * kST - SQ_ROWS) / 32> TriN;
        if (fetcher) {
            fetch(0);
            stash(0);
            fetch(1);
            stash(1);
        }
        __syncthreads();
        if (sq)
            produce_n(lds, 0, SqN{});
        else
            produce_n(lds, 0, TriN{});
        __syncthreads();
        float2 *P = (float2 *)a.part + ((int64_t)it.inst * a.max_splits + it.s) * (int64_t)Np * Np;
        auto square = [&](auto rows) __attribute__((always_inline)) {
            constexpr int NR = decltype(rows)::value;
            Acc re[16], im[16];
#pragma unroll
            for (int t = 0; t < 16; t++) re[t].clear(), im[t].clear();
            for (int stg = 0; stg < n_stage; stg++) {
                unsigned char *cur = lds + (stg & 1) * BUF;
                unsigned char *nxt = lds + ((stg + 1) & 1) * BUF;
                const bool more = stg + 1 < n_stage;
                if constexpr (NR > 0) consume_sq<16, NR, kTI>(cur, 8 + sq_r0, sq_c0, l16, lk, re, im);
                if (fetcher && stg + 2 < n_stage) fetch(stg + 2);
                if (more) produce_n(nxt, stg + 1, SqN{});
                if (fetcher && stg + 2 < n_stage) stash(stg + 2);
                __syncthreads();
            }
            if constexpr (NR > 0) {
                int ld = Np, row = 4 * lk, col = l16;
                asm volatile("" : "+v"(ld), "+v"(row), "+v"(col));
#pragma unroll
                for (int i = 0; i < NR; i++)
#pragma unroll
                    for (int j = 0; j < kTI; j++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int A = R * kST + 16 * (sq_r0 + i) + row + e;
                            const int Bc = C * kST + 16 * (sq_c0 + j) + col;
                            if (A < a.n_ant && Bc < a.n_ant)
                                P[(int64_t)A * ld + Bc] = make_float2(re[i * kTI + j].v[e], im[i * kTI + j].v[e]);
                        }
            }
        };
        auto triangle = [&](auto set) __attribute__((always_inline)) {
            typedef typename decltype(set)::type TS;
            constexpr int NACC = TS::base[TS::NR - 1] + TS::r[TS::NR - 1] + 1;
            Acc re[NACC], im[NACC];
#pragma unroll
            for (int t = 0; t < NACC; t++) re[t].clear(), im[t].clear();
            for (int stg = 0; stg < n_stage; stg++) {
                if (stg + 1 < n_stage) produce_n(lds + ((stg + 1) & 1) * BUF, stg + 1, TriN{});
                if (tri_nr > 0) consume_tri<TS>(lds + (stg & 1) * BUF, tri_o, l16, lk, re, im);
                __syncthreads();
            }
            if (tri_nr == 0) return;
            int ld = Np, row = 4 * lk, col = l16;
            asm volatile("" : "+v"(ld), "+v"(row), "+v"(col));
            for_tri_tiles<TS>([&](int t, int Rr, int Cc) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int A = T * kST + 16 * Rr + row + e, Bc = T * kST + 16 * Cc + col;
                    if (A < a.n_ant && Bc < a.n_ant) P[(int64_t)A * ld + Bc] = make_float2(re[t].v[e], im[t].v[e]);
                }
            });
        };
        if (sq) {
            switch (sq_nr) {
                case 4: square(std::integral_constant<int, 4>{}); break;
                case 3: square(std::integral_constant<int, 3>{}); break;
                case 2: square(std::integral_constant<int, 2>{}); break;
                case 1: square(std::integral_constant<int, 1>{}); break;
                default: square(std::integral_constant<int, 0>{}); break;
            }
        } else if (tri_nr == 2) {
            switch (tri_s) {
                case 0: triangle(SetTag<TriPair<0>>{}); break;
                case 1: triangle(SetTag<TriPair<1>>{}); break;
                case 2: triangle(SetTag<TriPair<2>>{}); break;
                default: triangle(SetTag<TriPair<3>>{}); break;
            }
        } else {  // one row of the set, or none
            switch (tri_s) {
                case 0: triangle(SetTag<TriSingle<0>>{}); break;
                case 1: triangle(SetTag<TriSingle<1>>{}); break;
                case 2: triangle(SetTag<TriSingle<2>>{}); break;
                default: triangle(SetTag<TriSingle<3>>{}); break;
            }
        }
    }
}

}  // namespace

hipError_t launch_coh_x6(const FusedArgs &a, hipStream_t s) {
    const int nb = a.n_rows_pad / (2 * kST);
    const bool has_short = short_last_block(a.n_ant, nb);
    if (nb > 1 || !has_short) {
        if ((a.tile & 15) == 2)
            k_coh_x6<64, false><<<a.grid, 512, 0, s>>>(a);
        else
            k_coh_x6<96, false><<<a.grid, 512, 0, s>>>(a);
    }
    if (has_short) k_coh_x6<96, true><<<a.grid, 512, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_pairs_x6(const FusedArgs &a, hipStream_t s) {
    k_pairs_x6<<<a.grid, 512, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_blk3_x6(const FusedArgs &a, hipStream_t s) {
    const int split = a.tile & 15;
    if (split == 2)
        k_blk3_x6<64><<<a.grid, 512, 0, s>>>(a);
    else if (split == 4)
        k_blk3_x6<128><<<a.grid, 512, 0, s>>>(a);
    else
        k_blk3_x6<96><<<a.grid, 512, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace mv
