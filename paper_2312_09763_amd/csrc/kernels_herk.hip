// Alg. 2 step (v): V = Z Z^H (Eq. zz) for a batch of instances with uneven
// column counts, on MFMA.
//
// Real embedding.  With Z = Zr + i Zi,
//   Re V = Zr Zr^T + Zi Zi^T,   Im V = Zi Zr^T - Zr Zi^T,
// so each 16x16 output tile takes four real products per k-chunk (FP32 and
// FP64: v_mfma_{f32,f64}_16x16x4, one complex element per lane), or six bf16
// products on BF16X3 (v_mfma_f32_16x16x32_bf16: eight bf16 = four complex per
// lane, re/im interleaved; the imaginary operand W = (im, -re) is formed in
// registers by swapping the bf16 halves and flipping one sign bit, and
// Z Z^H ~ hi hi^H + hi lo^H + lo hi^H).
//
// Work decomposition.  Output rows are padded to Np, a multiple of the
// super-tile ST (128 on FP32/BF16X3, 64 on FP64).  A work item is
// (instance, k-split, lower super-tile (I >= J)).  A 256-thread workgroup
// stages the rows of I and J (only I on the diagonal) for KC = 16 complex
// columns at a time in LDS, with the next chunk prefetched into registers;
// its four waves own the 2 x 2 wave tiles of the super-tile (the wave above
// the diagonal of a diagonal super-tile idles).  Each item writes its
// partial tile to its own slot, so the later sum over k-splits runs in a
// fixed order and the result is bitwise reproducible.
//
// Scheduling.  The grid is persistent (a multiple of 8 workgroups); the
// per-instance item counts come from the device-side visible counts through
// a prefix array built by k_worklist, so no host synchronisation is needed.
// Workgroup b runs on XCD b % 8; consecutive items (the super-tiles of one
// k-split, which share Z rows) are mapped to workgroups of the same XCD so
// the shared rows hit the same L2.
#include "internal.h"

namespace mv {

namespace {

template <int PREC>
struct HT;
template <>
struct HT<P32> {
    static constexpr int ST = 128, KC = 16, EB = 8, PLANES = 1;
};
template <>
struct HT<P64> {
    static constexpr int ST = 64, KC = 16, EB = 16, PLANES = 1;
};
template <>
struct HT<PB3> {
    static constexpr int ST = 128, KC = 16, EB = 4, PLANES = 2;
};

// Stage geometry of a square ST_ tile computed by four waves (2 x 2 wave tiles).
template <int PREC, int ST_>
struct HG {
    typedef HT<PREC> T;
    static constexpr int ST = ST_, WT = ST_ / 2, KC = T::KC, EB = T::EB, PLANES = T::PLANES;
    static constexpr int ROWB = KC * EB * PLANES;  // bytes of one staged row
    static constexpr int RS = ROWB + 16;           // LDS row stride (16 B pad against bank conflicts)
    static constexpr int CPR = ROWB / 16;          // 16-byte chunks per row
    static constexpr int NLD = 2 * ST * CPR / 256; // chunks per thread per stage
    static constexpr int LDS = 2 * ST * RS;
    static constexpr int TI = WT / 16;             // 16x16 tiles per wave side
};
template <int PREC>
struct HD : HG<PREC, HT<PREC>::ST> {};

__device__ inline int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Items of instance i: nsplit_i * n_st, with K_i = n_ax * visible count.
__device__ inline int64_t inst_k(const int32_t *count, int64_t fixed_k, int n_ax, int nfb, int i) {
    return count ? (int64_t)n_ax * count[i / nfb] : fixed_k;
}

// A wave as plan_splits wants it.  Reductions by DPP, within rows of 16 and then from row to
// row, into lane 63: a sixth of the time of shuffles through LDS, which count in a kernel of
// a few microseconds.
struct WaveGroup {
    int id;
    static constexpr int size = kWave;
    template <int CTRL, int ROWS, typename F>
    static __device__ int64_t step(int64_t v, int64_t none, F f) {
        const int lo = __builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp((int)(none >> 32), (int)(v >> 32), CTRL, ROWS, 0xf, false);
        return f(v, (int64_t)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo));
    }
    template <typename F>
    static __device__ int64_t reduce(int64_t v, int64_t none, F f) {
        v = step<0x111, 0xf>(v, none, f);  // row_shr:1, 2, 4, 8
        v = step<0x112, 0xf>(v, none, f);
        v = step<0x114, 0xf>(v, none, f);
        v = step<0x118, 0xf>(v, none, f);
        v = step<0x142, 0xa>(v, none, f);  // row_bcast:15 into rows 1 and 3
        v = step<0x143, 0xc>(v, none, f);  // row_bcast:31 into rows 2 and 3
        const uint32_t lo = __builtin_amdgcn_readlane((int)v, kWave - 1);
        const uint32_t hi = __builtin_amdgcn_readlane((int)(v >> 32), kWave - 1);
        return (int64_t)((uint64_t)hi << 32 | lo);
    }
    __device__ int64_t sum(int64_t v) {
        return reduce(v, 0, [](int64_t a, int64_t b) { return a + b; });
    }
    __device__ int64_t max(int64_t v) {
        return reduce(v, 0, [](int64_t a, int64_t b) { return a > b ? a : b; });
    }
    __device__ int64_t min(int64_t v) {
        return reduce(v, INT64_MAX, [](int64_t a, int64_t b) { return a < b ? a : b; });
    }
};

// k-splits per instance (the rule is plan_splits) and the item prefix.  Every workgroup
// then takes the same number of items of nearly the same size, and a call of few or
// small instances still reaches every CU: 15 instances of 20 000 columns at 91 antennas
// made 75 items for 256 CUs and took 711 us on FP32, 255 items take 241 us; 16 instances of
// 50 000 columns and 256 rows on FP64 with Z in memory filled 2.2 of 3 waves of the grid,
// 6.26 ms, and fill 3 of 3 in 4.34 ms.
__global__ void __launch_bounds__(1024) k_worklist(const int32_t *count, int64_t fixed_k, int n_ax, int nfb, int n_inst,
                                                   SplitRule rule, int32_t *work, int32_t *nsplit, int32_t *kcols) {
    __shared__ int wtot[1024 / kWave];
    __shared__ int carry_s;
    constexpr int kSlots = 256;
    __shared__ int32_t seen[kSlots];  // visible counts, where the slots fit
    __shared__ SplitPlan plan_s;
    const int n_slot = n_inst / nfb;
    const bool local = count && n_slot <= kSlots;
    if (threadIdx.x == 0) carry_s = 0;
    if (local && (int)threadIdx.x < n_slot) seen[threadIdx.x] = count[threadIdx.x];
    __syncthreads();
    const int lane = lane_id(), w = threadIdx.x / kWave;
    auto cols = [&](int slot) {
        return local ? (int64_t)n_ax * seen[slot] : inst_k(count, fixed_k, n_ax, 1, slot);
    };
    if (w == 0) {
        WaveGroup group{lane};
        const SplitPlan p = plan_splits(rule, n_slot, nfb, cols, group);
        if (lane == 0) plan_s = p;
    }
    __syncthreads();
    const SplitPlan plan = plan_s;
    for (int base = 0; base < n_inst; base += 1024) {
        int i = base + threadIdx.x;
        int v = 0;
        if (i < n_inst) {
            const Split sp = split_of(rule, plan, cols(i / nfb), i);
            nsplit[i] = sp.n;
            kcols[i] = (int32_t)sp.kc;
            v = sp.n * rule.n_st;
        }
        int x = v;
        for (int d = 1; d < kWave; d <<= 1) {
            int y = __shfl_up(x, d, kWave);
            if (lane >= d) x += y;
        }
        if (lane == kWave - 1) wtot[w] = x;
        __syncthreads();
        if (w == 0) {
            int t = lane < 1024 / kWave ? wtot[lane] : 0;
            for (int d = 1; d < kWave; d <<= 1) {
                int y = __shfl_up(t, d, kWave);
                if (lane >= d) t += y;
            }
            if (lane < 1024 / kWave) wtot[lane] = t;
        }
        __syncthreads();
        int carry = carry_s;
        if (i < n_inst) work[i] = carry + (w > 0 ? wtot[w - 1] : 0) + x - v;
        __syncthreads();
        if (threadIdx.x == 0) carry_s = carry + wtot[1024 / kWave - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0) work[n_inst] = carry_s;
}

// W = (im, -re) for four packed bf16 complex values.
__device__ inline u32x4 bf16_rot(u32x4 v) {
    u32x4 r;
    for (int q = 0; q < 4; q++) r[q] = __builtin_amdgcn_alignbit(v[q], v[q], 16) ^ 0x80000000u;
    return r;
}

// One KC-deep stage of a WT x WT wave tile: rows arow.. of the staged A block
// against rows brow.. of the staged B block (both in LDS, row stride RS).
template <int PREC, typename D, typename Acc>
__device__ __forceinline__ void mma_stage(const unsigned char *lds, int arow, int brow, int l16, int lk, bool on_diag,
                                          Acc (&acc_re)[D::TI][D::TI], Acc (&acc_im)[D::TI][D::TI]) {
    constexpr int KC = D::KC, RS = D::RS, TI = D::TI;
    if constexpr (PREC == PB3) {
        u32x4 ah[TI], al[TI], bh[TI], bl[TI];
#pragma unroll
        for (int i = 0; i < TI; i++) {
            const unsigned char *p = lds + (arow + 16 * i + l16) * RS + lk * 16;
            ah[i] = *(const u32x4 *)p;
            al[i] = *(const u32x4 *)(p + KC * 4);
        }
#pragma unroll
        for (int j = 0; j < TI; j++) {
            const unsigned char *p = lds + (brow + 16 * j + l16) * RS + lk * 16;
            bh[j] = *(const u32x4 *)p;
            bl[j] = *(const u32x4 *)(p + KC * 4);
        }
#pragma unroll
        for (int i = 0; i < TI; i++) {
            const u32x4 wh = bf16_rot(ah[i]), wl = bf16_rot(al[i]);
            const bf16x8 Ah = __builtin_bit_cast(bf16x8, ah[i]);
            const bf16x8 Al = __builtin_bit_cast(bf16x8, al[i]);
            const bf16x8 Wh = __builtin_bit_cast(bf16x8, wh);
            const bf16x8 Wl = __builtin_bit_cast(bf16x8, wl);
#pragma unroll
            for (int j = 0; j < TI; j++) {
                const bf16x8 Bh = __builtin_bit_cast(bf16x8, bh[j]);
                const bf16x8 Bl = __builtin_bit_cast(bf16x8, bl[j]);
                acc_re[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, Bh, acc_re[i][j], 0, 0, 0);
                acc_re[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, Bl, acc_re[i][j], 0, 0, 0);
                acc_re[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Al, Bh, acc_re[i][j], 0, 0, 0);
                acc_im[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wh, Bh, acc_im[i][j], 0, 0, 0);
                acc_im[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wh, Bl, acc_im[i][j], 0, 0, 0);
                acc_im[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wl, Bh, acc_im[i][j], 0, 0, 0);
                // On the output diagonal the dropped lo lo^H term is a sum of
                // |lo|^2, a one-signed bias of relative size ~2^-16; add it
                // there (elsewhere it averages out and is left out).
                if (on_diag && i == j) {
                    acc_re[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Al, Bl, acc_re[i][j], 0, 0, 0);
                    acc_im[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Wl, Bl, acc_im[i][j], 0, 0, 0);
                }
            }
        }
    } else {
        typedef typename std::conditional<PREC == P64, double2, float2>::type C;
        typedef typename std::conditional<PREC == P64, double, float>::type R;
#pragma unroll
        for (int kk = 0; kk < KC; kk += 4) {
            C av[TI], bv[TI];
#pragma unroll
            for (int i = 0; i < TI; i++)
                av[i] = *(const C *)(lds + (arow + 16 * i + l16) * RS + (kk + lk) * D::EB);
#pragma unroll
            for (int j = 0; j < TI; j++)
                bv[j] = *(const C *)(lds + (brow + 16 * j + l16) * RS + (kk + lk) * D::EB);
#pragma unroll
            for (int i = 0; i < TI; i++) {
                const R nre = -av[i].x;
#pragma unroll
                for (int j = 0; j < TI; j++) {
                    if constexpr (PREC == P64) {
                        acc_re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i].x, bv[j].x, acc_re[i][j], 0, 0, 0);
                        acc_re[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i].y, bv[j].y, acc_re[i][j], 0, 0, 0);
                        acc_im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i].y, bv[j].x, acc_im[i][j], 0, 0, 0);
                        acc_im[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(nre, bv[j].y, acc_im[i][j], 0, 0, 0);
                    } else {
                        acc_re[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i].x, bv[j].x, acc_re[i][j], 0, 0, 0);
                        acc_re[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i].y, bv[j].y, acc_re[i][j], 0, 0, 0);
                        acc_im[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i].y, bv[j].x, acc_im[i][j], 0, 0, 0);
                        acc_im[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(nre, bv[j].y, acc_im[i][j], 0, 0, 0);
                    }
                }
            }
        }
    }
}

template <int PREC>
__global__ void __launch_bounds__(256, 2) k_herk(HerkArgs a) {
    typedef HD<PREC> D;
    constexpr int ST = D::ST, WT = D::WT, KC = D::KC, RS = D::RS, CPR = D::CPR, NLD = D::NLD, TI = D::TI;
    typedef typename std::conditional<PREC == P64, f64x4, f32x4>::type Acc;
    typedef typename std::conditional<PREC == P64, double2, float2>::type PartT;
    __shared__ __attribute__((aligned(16))) unsigned char lds[D::LDS];

    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int wave = tid / kWave;
    const int wr = wave >> 1, wc = wave & 1;
    const int Np = a.n_rows_pad;
    const int nb = Np / ST;
    const int n_st = nb * (nb + 1) / 2;
    const int total = a.work[a.n_inst];
    const int per_xcd = a.grid / 8;
    const int slot = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    const char *zbase = (const char *)a.Z;
    const char *zlo = (const char *)a.Z_lo;
    const int64_t ldzb = a.ldz * D::EB;  // row stride in bytes of one plane

    for (int item = slot; item < total; item += a.grid) {
        // locate the instance: largest i with work[i] <= item
        int lo = 0, hi = a.n_inst - 1;
        while (lo < hi) {
            int mid = (lo + hi + 1) >> 1;
            if (a.work[mid] <= item)
                lo = mid;
            else
                hi = mid - 1;
        }
        const int inst = lo;
        const int local = item - a.work[inst];
        const int s = local / n_st;
        int st = local % n_st;
        int I = 0;
        while (st > I) {
            st -= I + 1;
            I++;
        }
        const int J = st;
        const bool diag = (I == J);
        const int64_t K = inst_k(a.count, a.fixed_k, a.n_ax, a.nfb, inst);
        const int64_t Kr = ((K + KC - 1) / KC) * KC;
        const int64_t kc = a.kcols[inst];
        const int64_t kb = (int64_t)s * kc;
        const int64_t ke = kb + kc < Kr ? kb + kc : Kr;
        const int64_t ioff = (int64_t)inst * a.inst_stride * D::EB;

        Acc acc_re[TI][TI], acc_im[TI][TI];
        for (int i = 0; i < TI; i++)
            for (int j = 0; j < TI; j++)
                for (int e = 0; e < 4; e++) {
                    acc_re[i][j][e] = 0;
                    acc_im[i][j][e] = 0;
                }

        u32x4 pre[NLD];
        auto load = [&](int64_t k0) {
#pragma unroll
            for (int j = 0; j < NLD; j++) {
                if (diag && j >= NLD / 2) break;
                const int q = tid + 256 * j;
                const int lr = q / CPR, c = q % CPR;
                const int grow = lr < ST ? I * ST + lr : J * ST + (lr - ST);
                const char *src;
                if constexpr (D::PLANES == 2) {
                    const int half = CPR / 2;
                    src = (c < half ? zbase : zlo) + ioff + grow * ldzb + k0 * D::EB + (c % half) * 16;
                } else {
                    src = zbase + ioff + grow * ldzb + k0 * D::EB + c * 16;
                }
                pre[j] = *(const u32x4 *)src;
            }
        };
        auto store = [&]() {
#pragma unroll
            for (int j = 0; j < NLD; j++) {
                if (diag && j >= NLD / 2) break;
                const int q = tid + 256 * j;
                const int lr = q / CPR, c = q % CPR;
                *(u32x4 *)(lds + lr * RS + c * 16) = pre[j];
            }
        };

        const bool active = !(diag && wc > wr);
        const bool on_diag = diag && wc == wr;  // this wave's tiles (i, i) hold output diagonal entries
        const int arow = wr * WT;
        const int brow = (diag ? 0 : ST) + wc * WT;
        const int l16 = lane & 15, lk = lane >> 4;

        if (kb < ke) load(kb);
        for (int64_t k0 = kb; k0 < ke; k0 += KC) {
            __syncthreads();
            store();
            __syncthreads();
            if (k0 + KC < ke) load(k0 + KC);
            if (active) mma_stage<PREC, D>(lds, arow, brow, l16, lk, on_diag, acc_re, acc_im);
        }

        if (active) {
            // Accumulator layout of a 16x16 tile: lane l, register e holds column l % 16 of
            // row 4 (l / 16) + e for the f32 products, and of row 4 e + l / 16 for
            // v_mfma_f64_16x16x4f64.
            PartT *P = (PartT *)a.part + ((int64_t)inst * a.max_splits + s) * (int64_t)Np * Np;
            const int rb = I * ST + wr * WT;
            const int c0 = J * ST + wc * WT + l16;
#pragma unroll
            for (int i = 0; i < TI; i++)
#pragma unroll
                for (int j = 0; j < TI; j++)
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        PartT v;
                        v.x = acc_re[i][j][e];
                        v.y = acc_im[i][j][e];
                        const int row = rb + 16 * i + (PREC == P64 ? 4 * e + lk : 4 * lk + e);
                        P[(int64_t)row * Np + c0 + 16 * j] = v;
                    }
        }
        __syncthreads();  // LDS is reused by the next item
    }
}

// Redundancy-aware product (App. A, Eq. Vpx): V'_x = A_x B_x^H with A_x, B_x
// gathered rows of Z.  One workgroup per (instance, ST x ST tile of a
// sub-matrix, k-split); the tile's rows are read through its two row lists
// straight from Z (a gather fused into the stage loads: no copy of A_x or
// B_x is formed), and the raw tile goes to its own partial slot.
template <int PREC, int STS>
__global__ void __launch_bounds__(256, 2) k_submat(SubmatArgs a) {
    typedef HG<PREC, STS> D;
    constexpr int ST = D::ST, WT = D::WT, KC = D::KC, RS = D::RS, CPR = D::CPR, NLD = D::NLD, TI = D::TI;
    typedef typename std::conditional<PREC == P64, f64x4, f32x4>::type Acc;
    typedef typename std::conditional<PREC == P64, double2, float2>::type PartT;
    __shared__ __attribute__((aligned(16))) unsigned char lds[D::LDS];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
    const int wr = wave >> 1, wc = wave & 1, l16 = lane & 15, lk = lane >> 4;
    const int64_t item = blockIdx.x;
    const int s = (int)(item % a.max_splits);
    const int tile = (int)((item / a.max_splits) % a.n_tiles);
    const int inst = (int)(item / ((int64_t)a.max_splits * a.n_tiles));
    const int64_t K = inst_k(a.count, a.fixed_k, a.n_ax, a.nfb, inst);
    const int64_t Kr = ((K + KC - 1) / KC) * KC;
    const int64_t kb = (int64_t)s * a.ksplit;
    if (kb >= Kr) return;  // an empty k-split: the reduction sums only ceil(K / ksplit) of them
    const int64_t ke = kb + a.ksplit < Kr ? kb + a.ksplit : Kr;
    const int32_t *rows = a.rows + (int64_t)tile * 2 * ST;
    const char *zbase = (const char *)a.Z + (int64_t)inst * a.inst_stride * D::EB;
    const char *zlo = PREC == PB3 ? (const char *)a.Z_lo + (int64_t)inst * a.inst_stride * D::EB : nullptr;
    const int64_t ldzb = a.ldz * D::EB;

    Acc acc_re[TI][TI], acc_im[TI][TI];
    for (int i = 0; i < TI; i++)
        for (int j = 0; j < TI; j++)
            for (int e = 0; e < 4; e++) {
                acc_re[i][j][e] = 0;
                acc_im[i][j][e] = 0;
            }
    int grow[NLD];
#pragma unroll
    for (int j = 0; j < NLD; j++) {
        const int lr = (tid + 256 * j) / CPR;
        grow[j] = rows[lr];  // A rows for lr < ST, then B rows
    }
    u32x4 pre[NLD];
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int j = 0; j < NLD; j++) {
            const int c = (tid + 256 * j) % CPR;
            pre[j] = u32x4{0u, 0u, 0u, 0u};
            if (grow[j] < 0) continue;
            if constexpr (D::PLANES == 2) {  // BF16X3: hi then lo plane of the staged row
                const int half = CPR / 2;
                pre[j] = *(const u32x4 *)((c < half ? zbase : zlo) + grow[j] * ldzb + k0 * D::EB + (c % half) * 16);
            } else {
                pre[j] = *(const u32x4 *)(zbase + grow[j] * ldzb + k0 * D::EB + c * 16);
            }
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int j = 0; j < NLD; j++) {
            const int q = tid + 256 * j;
            *(u32x4 *)(lds + (q / CPR) * RS + (q % CPR) * 16) = pre[j];
        }
    };
    const int arow = wr * WT, brow = ST + wc * WT;
    if (kb < ke) load(kb);
    for (int64_t k0 = kb; k0 < ke; k0 += KC) {
        __syncthreads();
        store();
        __syncthreads();
        if (k0 + KC < ke) load(k0 + KC);
        // BF16X3: any tile may hold an autocorrelation (a = b, p = q), where the
        // dropped lo lo^H term is a one-signed bias, so every tile takes it
        mma_stage<PREC, D>(lds, arow, brow, l16, lk, PREC == PB3, acc_re, acc_im);
    }
    PartT *P = (PartT *)a.part + (((int64_t)inst * a.max_splits + s) * a.n_tiles + tile) * ST * ST;
#pragma unroll
    for (int i = 0; i < TI; i++)
#pragma unroll
        for (int j = 0; j < TI; j++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                PartT v;
                v.x = acc_re[i][j][e];
                v.y = acc_im[i][j][e];
                const int r = arow + 16 * i + (PREC == P64 ? 4 * e + lk : 4 * lk + e);
                P[(int64_t)r * ST + wc * WT + 16 * j + l16] = v;
            }
}

// V of every requested pair: the k-split partials of its tile element summed in
// FP64 in split order, earlier source chunks carried in vacc.
template <int PREC>
__global__ void __launch_bounds__(256) k_submat_reduce(SubmatReduceArgs a) {
    typedef typename std::conditional<PREC == P64, double2, float2>::type C;
    const int nf = a.n_feed;
    const int64_t per_inst = (int64_t)a.n_pair * nf * nf;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= per_inst * a.n_inst) return;
    const int inst = (int)(gid / per_inst);
    const int64_t e = gid % per_inst;
    const int64_t K = inst_k(a.count, a.fixed_k, a.n_ax, a.nfb, inst);
    const int64_t kc = a.ksplit > 0 ? a.ksplit : split_cols(K, a.max_splits);
    const int ns = K > 0 ? (int)((K + kc - 1) / kc) : 0;
    const int32_t tile = a.loc[2 * e], off = a.loc[2 * e + 1];
    const int ST2 = a.st * a.st;
    double re = 0.0, im = 0.0;
    for (int s = 0; s < ns; s++) {
        const C v = ((const C *)a.part)[(((int64_t)inst * a.max_splits + s) * a.n_tiles + tile) * ST2 + off];
        re += (double)v.x;
        im += (double)v.y;
    }
    double2 *acc = (double2 *)a.vacc + (int64_t)inst * per_inst + e;
    if (!a.first) {
        const double2 o = *acc;
        re += o.x;
        im += o.y;
    }
    if (!a.last) {
        *acc = make_double2(re, im);
        return;
    }
    const int t = a.bt.t0 + inst / a.bt.nfb, f = a.bt.f0 + inst % a.bt.nfb;
    C out;
    out.x = re;
    out.y = im;
    ((C *)a.out)[((int64_t)t * a.n_freq_total + f) * per_inst + e] = out;
}

// Fixed-order sum of the k-split partials, Hermitian fill and the write of the
// output layout, over 32 x 32 tiles of the lower triangle: partial rows are
// read coalesced, each lower element is summed once (in FP64, splits in
// order), and both it and its conjugate mirror above the diagonal are written,
// the mirror through an LDS transpose.  Earlier source chunks are carried in vacc at the
// lower positions only.
template <int PREC, int NR>
__global__ void __launch_bounds__(1024 / NR) k_reduce_tiles(ReduceArgs a) {
    constexpr int DY = 32 / NR;              // between the rows of a thread
    constexpr int UNROLL = NR == 1 ? 16 : 4;  // splits in flight
    typedef typename std::conditional<PREC == P64, double2, float2>::type PartT;
    typedef typename std::conditional<PREC == P64, double2, float2>::type OutT;
    __shared__ double2 sm[32][33];
    const int inst = blockIdx.y;
    const int N = a.n_rows, Np = a.n_rows_pad, nf = a.n_feed, na = a.n_ant;
    // tile (R, C), R >= C, from the linear lower-triangle index
    int R = 0, t = blockIdx.x;
    while (t > R) {
        t -= R + 1;
        R++;
    }
    const int C = t;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int64_t K = a.count ? (int64_t)a.n_ax * a.count[inst / a.nfb] : a.fixed_k;
    const int64_t kc = a.ksplit > 0 ? a.ksplit : split_cols(K, a.max_splits);
    const int ns = a.nsplit ? a.nsplit[inst] : K > 0 ? (int)((K + kc - 1) / kc) : 0;
    const PartT *P = (const PartT *)a.part + (int64_t)inst * a.max_splits * Np * Np;
    double2 *acc = a.vacc ? (double2 *)a.vacc + (int64_t)inst * N * N : nullptr;
    OutT *out = (OutT *)a.out;
    if (a.out_kind == 0) {
        const int tt = a.bt.t0 + inst / a.bt.nfb, f = a.bt.f0 + inst % a.bt.nfb;
        out += ((int64_t)tt * a.n_freq_total + f) * (int64_t)N * N;
    }
    auto out_index = [&](int r, int c) -> int64_t {
        if (a.out_kind != 0) return (int64_t)r * N + c;
        const int aa = r / nf, p = r % nf, b = c / nf, q = c % nf;
        return (((int64_t)aa * na + b) * nf + p) * nf + q;
    };
    // The splits of this thread's rows are summed together, so that the loads of 4
    // splits x 4 rows, or 16 splits of one row, are in flight at once (the sums' order is
    // the splits' either way): summed a row at a time, 128 splits cost more than the
    // product of a small call.  (8 splits x 4 rows took 0.41 instead of 0.33 ms on 16
    // instances of 700 rows.)
    const int c = 32 * C + tx;
    double sr[NR], si[NR];
    const PartT *pp[NR];
    bool on[NR];
    for (int i = 0; i < NR; i++) {
        const int r = 32 * R + ty + DY * i;
        on[i] = r < N && c < N && r >= c;
        pp[i] = P + (on[i] ? (int64_t)r * Np + c : 0);  // element 0 is readable for every split
        sr[i] = si[i] = 0.0;
    }
#pragma unroll UNROLL
    for (int s = 0; s < ns; s++) {
#pragma unroll
        for (int i = 0; i < NR; i++) {
            const PartT v = pp[i][(int64_t)s * Np * Np];
            sr[i] += (double)v.x;
            si[i] += (double)v.y;
        }
    }
    for (int i = 0; i < NR; i++) {
        const int rl = ty + DY * i, r = 32 * R + rl;
        if (!on[i]) continue;
        if (r == c) si[i] = 0.0;
        if (!a.first) {
            const double2 prev = acc[(int64_t)r * N + c];
            sr[i] += prev.x;
            si[i] += prev.y;
        }
        if (!a.last) {
            acc[(int64_t)r * N + c] = make_double2(sr[i], si[i]);
            continue;
        }
        sm[rl][tx] = make_double2(sr[i], si[i]);
        OutT v;
        v.x = sr[i];
        v.y = si[i];
        out[out_index(r, c)] = v;
    }
    if (!a.last) return;
    __syncthreads();
    // mirror: element (32 C + ty + DY i, 32 R + tx) = conj(lower (32 R + tx, 32 C + ty + DY i))
    for (int i = 0; i < NR; i++) {
        const int cl = ty + DY * i, r = 32 * C + cl, c = 32 * R + tx;
        if (r >= N || c >= N || r >= c) continue;
        const double2 w = sm[tx][cl];
        OutT v;
        v.x = w.x;
        v.y = -w.y;
        out[out_index(r, c)] = v;
    }
}

}  // namespace

int herk_super_tile(int prec) { return prec == P64 ? HT<P64>::ST : HT<P32>::ST; }

hipError_t launch_submat(int prec, const SubmatArgs &a, hipStream_t s) {
    const int64_t items = (int64_t)a.n_inst * a.n_tiles * a.max_splits;
    if (items <= 0) return hipSuccess;
    if (prec == P64)
        k_submat<P64, kSubmatTile><<<(unsigned)items, 256, 0, s>>>(a);
    else if (prec == P32)
        k_submat<P32, kSubmatTile><<<(unsigned)items, 256, 0, s>>>(a);
    else if (prec == PB3)
        k_submat<PB3, kSubmatTile><<<(unsigned)items, 256, 0, s>>>(a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_submat_reduce(int prec, const SubmatReduceArgs &a, hipStream_t s) {
    const int64_t n = (int64_t)a.n_inst * a.n_pair * a.n_feed * a.n_feed;
    if (n <= 0) return hipSuccess;
    const unsigned g = (unsigned)((n + 255) / 256);
    if (prec == P64)
        k_submat_reduce<P64><<<g, 256, 0, s>>>(a);
    else if (prec == P32 || prec == PB3)
        k_submat_reduce<P32><<<g, 256, 0, s>>>(a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

int herk_occupancy(int prec) {
    int nb = 1;
    hipError_t e;
    if (prec == P64)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_herk<P64>, 256, 0);
    else if (prec == P32)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_herk<P32>, 256, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_herk<PB3>, 256, 0);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return nb < 1 ? 1 : nb;
}

hipError_t launch_worklist(int prec, const HerkArgs &a, int unit, hipStream_t s) {
    if (a.n_inst <= 0) return hipSuccess;
    const int st = herk_super_tile(prec);
    const int nb = a.n_rows_pad / st;
    SplitRule r = a.rule;
    r.ksplit = a.ksplit;
    r.max_splits = a.max_splits;
    r.n_st = unit ? 1 : nb * (nb + 1) / 2;
    if (r.n_bal < 1) r.n_bal = 1;
    k_worklist<<<1, 1024, 0, s>>>(a.count, a.fixed_k, a.n_ax, a.nfb, a.n_inst, r, a.work, a.nsplit, a.kcols);
    return hipGetLastError();
}

hipError_t launch_herk(int prec, const HerkArgs &a, hipStream_t s) {
    if (a.n_inst <= 0) return hipSuccess;
    if (prec == P64)
        k_herk<P64><<<a.grid, 256, 0, s>>>(a);
    else if (prec == P32)
        k_herk<P32><<<a.grid, 256, 0, s>>>(a);
    else
        k_herk<PB3><<<a.grid, 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_reduce(int prec, const ReduceArgs &a, hipStream_t s) {
    if (a.n_inst <= 0 || a.n_rows <= 0) return hipSuccess;
    const int nt = (a.n_rows + 31) / 32;
    dim3 g((unsigned)(nt * (nt + 1) / 2), a.n_inst);
    // One row a thread while the tiles are too few to fill the chip with four rows a
    // thread: 8 instances of 37 rows in 16 splits 18.5 -> 7.0 us, 15 of 182 rows in 17
    // splits 20.1 -> 10.2 us.
    const bool few = (int64_t)g.x * g.y <= 512;
    if (prec == P64 && few)
        k_reduce_tiles<P64, 1><<<g, 1024, 0, s>>>(a);
    else if (prec == P64)
        k_reduce_tiles<P64, 4><<<g, 256, 0, s>>>(a);
    else if (few)
        k_reduce_tiles<P32, 1><<<g, 1024, 0, s>>>(a);
    else
        k_reduce_tiles<P32, 4><<<g, 256, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace mv
