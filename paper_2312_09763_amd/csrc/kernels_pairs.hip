// Redundancy-aware product (App. A, Eq. Vpx) with Z formed in LDS, FP32 and BF16X3.
//
// Of V only the requested pairs are needed.  The host lists the rows of Z (antenna,
// feed) that some pair uses, in order, cuts them into blocks of 16, and lists the
// 16 x 16 tiles (I, J) in which a pair lies: 81 tiles for the 1344 unique baselines
// of a 350-antenna hexagon, a sixth of V and a third less than the planned
// sub-matrices hold.  Tiles are grouped into bundles of at most kPairTiles tiles on
// at most kPairBlocks blocks; a workgroup takes one (instance, k-split, bundle),
// forms every row of the bundle once per stage of 16 columns and multiplies the
// bundle's tiles from it, up to 6 a wave.  So Z is neither written nor gathered: in
// HBM it was 2.2 GB for 32 instances of 24 576 sources that are up (written at 2.0 TB/s,
// then read once per 32 x 32 tile).
//
// FP32 operands are three exact bf16 terms and six products, as in
// kernels_herk_x6.hip; BF16X3 operands hi + lo and all four products, because any
// tile may hold an autocorrelation, where lo lo^H is a one-signed bias.  The products
// of a stage start from zero and are added in FP32.
//
// Bound by vector instructions (63 % of the cycles: forming, rotation of columns, the
// additions), LDS (54 %) and MFMAs (45 %) together; half of the waves multiply before
// they form the next stage and half after.  350 antennas, 49 152 sources, 4 times of 8
// channels, FP32: forming Z and multiplying went from 1.08 + 2.29 to 0.80 ms, the error
// against 64 bits from 1.3e-6 to 2.2e-7.  16 waves of 6 tiles rather than 8 of 12 (with
// operands loaded a tile ahead) took 0.82 against 0.92 ms, rows and columns laid out for
// the banks 0.80.
#include <type_traits>

#include "herk_tiles.h"
#include "matvis.h"

namespace mv {

namespace {

constexpr int kSPS = 16;                       // columns per stage
constexpr int kRows = 16 * kPairBlocks;        // staged rows
constexpr int kWaves = 16;
constexpr int kWaveTiles = kPairTiles / kWaves;  // tiles of a wave
constexpr int kPlane = 4 * kSPS;               // bytes of a row's plane

template <int PREC>
struct PairGeom {
    static constexpr int NT = PREC == P32 ? 3 : 2;     // bf16 terms per value
    static constexpr int RS = NT * kPlane + 16;        // 16 bytes of padding spread the banks
    static constexpr int BUF = kRows * RS;
};

// Two staged columns: the sources' directions and their values of both feeds.  80 bytes,
// so that the eight pairs of a stage start in different banks.
struct __attribute__((aligned(16))) Columns {
    double x0, y0, z0, x1, y1, z1;
    float4 b0, b1;
};

struct Row {
    double ux, uy, uz;  // (nu / c) x_a
    int32_t bp;         // beam n_feed + feed
    int32_t pad;
};

template <int NT>
struct Ops {
    u32x4 t[NT];  // hi, [mid,] lo
    __device__ __forceinline__ void load(const unsigned char *p) {
#pragma unroll
        for (int q = 0; q < NT; q++) t[q] = *(const u32x4 *)(p + q * kPlane);
    }
};

__device__ __forceinline__ f32x4 mma(const u32x4 &a, const u32x4 &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                   0);
}

// The products of row terms a with column terms b (re) and w (im), smallest first.
template <int NT>
__device__ __forceinline__ void products(const Ops<NT> &a, const Ops<NT> &b, const Ops<NT> &w, f32x4 &re, f32x4 &im) {
    re = f32x4{0.f, 0.f, 0.f, 0.f};
    im = re;
#pragma unroll
    for (int order = 2 * (NT - 1); order >= 0; order--)
#pragma unroll
        for (int q = NT - 1; q >= 0; q--) {
            const int p = order - q;
            // three terms: those above 2^-26 only (p + q <= 2)
            if (p < 0 || p >= NT || (NT == 3 && order > 2)) continue;
            re = mma(a.t[p], b.t[q], re);
            im = mma(a.t[p], w.t[q], im);
        }
}

template <int PREC>
__global__ void __launch_bounds__(1024, 1) k_pair_tiles(PairArgs a) {
    typedef PairGeom<PREC> G;
    constexpr int NT = G::NT, RS = G::RS;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * G::BUF];
    __shared__ Row row[kRows];
    __shared__ Columns col[2][kSPS / 2];
    static_assert(2 * G::BUF + sizeof(Row) * kRows + sizeof(Columns) * kSPS <= 160 * 1024, "LDS");
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
    const PairBundle bd = a.bundles[bundle];
    const int n_rows = bd.n_rows;
    const double nu_c = a.freqs[a.f0 + inst % a.nfb] / kSpeedOfLight;
    const double *sh = a.s_hat + (int64_t)tslot * 3 * a.ld_src;
    const float2 *Bi = (const float2 *)a.B + (int64_t)inst * a.n_beam * nf * nx * a.ld_src;  // [beam][feed][axis][m]
    const bool shared_beam = a.n_beam == 1;
    if (tid < n_rows) {
        const int z = a.rows[bd.row0 + tid], ant = z < 0 ? 0 : z / nf;  // padding rows reach no stored output
        row[tid] = Row{nu_c * a.antc[3 * ant], nu_c * a.antc[3 * ant + 1], nu_c * a.antc[3 * ant + 2],
                       a.bidx[ant] * nf + (z < 0 ? 0 : z % nf), 0};
    }
    const int n_stage = (int)((ke - kb + kSPS - 1) / kSPS);

    // the columns of a stage, one per lane of the first 16
    const bool fetcher = tid < kSPS;
    double fx, fy, fz;
    float4 fb;
    auto fetch = [&](int stage) {
        const int64_t c = kb + (int64_t)stage * kSPS + tid;
        fx = fy = fz = 0.0;
        fb = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c < ke) {
            const int64_t m = c / nx;
            fx = sh[m];
            fy = sh[a.ld_src + m];
            fz = sh[2 * a.ld_src + m];
            if (shared_beam) {
                const float2 v = Bi[(c % nx) * a.ld_src + m];
                const float2 u = nf == 2 ? Bi[(nx + c % nx) * a.ld_src + m] : v;
                fb = make_float4(v.x, v.y, u.x, u.y);
            }
        }
    };
    auto stash = [&](int stage) {
        Columns &e = col[stage & 1][tid / 2];
        double *d = tid & 1 ? &e.x1 : &e.x0;
        d[0] = fx;
        d[1] = fy;
        d[2] = fz;
        *(tid & 1 ? &e.b1 : &e.b0) = fb;
    };
    // two columns (2 mp, 2 mp + 1) of rows r0 + 128 k; the rows that 32 lanes write are 4
    // (832 bytes, a quarter of the banks) apart
    const int mp = tid % 8, g = tid / 8 % 8;
    const int r0 = wave / 2 * 16 + wave % 2 * 2 + g % 4 * 4 + g / 4;
    auto produce = [&](unsigned char *buf, int stage) __attribute__((always_inline)) {
        const Columns c = col[stage & 1][mp];
        const int64_t cg = kb + (int64_t)stage * kSPS + 2 * mp;
        for (int r = r0; r < n_rows; r += 8 * kWaves) {
            const Row e = row[r];
            float vr[2], vi[2];
            if (shared_beam) {
                const bool second = e.bp != 0;
                vr[0] = second ? c.b0.z : c.b0.x;
                vi[0] = second ? c.b0.w : c.b0.y;
                vr[1] = second ? c.b1.z : c.b1.x;
                vi[1] = second ? c.b1.w : c.b1.y;
            } else {
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    const int64_t cq = cg + q;
                    const float2 v = cq < ke ? Bi[(e.bp * nx + cq % nx) * a.ld_src + cq / nx] : make_float2(0.f, 0.f);
                    vr[q] = v.x;
                    vi[q] = v.y;
                }
            }
            float fr[2], fi[2];
            fringe(e.ux * c.x0 + e.uy * c.y0 + e.uz * c.z0, fr[0], fi[0]);
            fringe(e.ux * c.x1 + e.uy * c.y1 + e.uz * c.z1, fr[1], fi[1]);
            uint32_t w[NT][2];
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const float zr = vr[q] * fr[q] - vi[q] * fi[q], zi = vr[q] * fi[q] + vi[q] * fr[q];
                if constexpr (NT == 3)
                    split3(zr, zi, w[0][q], w[1][q], w[2][q]);
                else
                    split2(zr, zi, w[0][q], w[1][q]);
            }
            unsigned char *p = buf + r * RS + mp * 8;
#pragma unroll
            for (int t = 0; t < NT; t++) *(uint2 *)(p + t * kPlane) = make_uint2(w[t][0], w[t][1]);
        }
    };

    if (fetcher) {
        fetch(0);
        stash(0);
        fetch(1);
        stash(1);
    }
    // this wave's tiles, sorted by column block: LDS offsets of their row and column blocks
    const int t0 = bd.n_tiles * wave / kWaves, nt = bd.n_tiles * (wave + 1) / kWaves - t0;
    // (`fresh`: bit t set where the column block is not that of tile t - 1)
    uint32_t ro[kWaveTiles], co[kWaveTiles], fresh = 0;
#pragma unroll
    for (int t = 0; t < kWaveTiles; t++) {
        const int32_t e = a.tiles[bd.tile0 + (t < nt ? t0 + t : 0)];
        ro[t] = __builtin_amdgcn_readfirstlane((e & 255) * 16 * RS);
        co[t] = __builtin_amdgcn_readfirstlane((e >> 8) * 16 * RS);
        if (t == 0 || co[t] != co[t - 1]) fresh |= 1u << t;
    }
    __syncthreads();
    produce(lds, 0);
    __syncthreads();

    auto stages = [&](auto first) __attribute__((always_inline)) {
        float re[kWaveTiles][4], im[kWaveTiles][4];
#pragma unroll
        for (int t = 0; t < kWaveTiles; t++)
#pragma unroll
            for (int e = 0; e < 4; e++) re[t][e] = im[t][e] = 0.f;
        auto consume = [&](const unsigned char *buf) __attribute__((always_inline)) {
            const unsigned char *p = buf + l16 * RS + lk * 16;
            Ops<NT> b, w;
            int n = nt;
            uint32_t fr = fresh;
            asm volatile("" : "+s"(n), "+s"(fr));  // tested here: no condition is kept across the stages
#pragma unroll
            for (int t = 0; t < kWaveTiles; t++) {
                if (t < n) {
                    if (fr >> t & 1) {
                        b.load(p + co[t]);
#pragma unroll
                        for (int q = 0; q < NT; q++) w.t[q] = bf16_rot_col(b.t[q]);
                    }
                    Ops<NT> r;
                    r.load(p + ro[t]);
                    __builtin_amdgcn_sched_barrier(0);
                    f32x4 pr, pi;
                    products<NT>(r, b, w, pr, pi);
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        re[t][e] += pr[e];
                        im[t][e] += pi[e];
                        asm volatile("" : "+v"(re[t][e]), "+v"(im[t][e]));  // added here, not after the forming
                    }
                }
            }
        };
        for (int stg = 0; stg < n_stage; stg++) {
            unsigned char *cur = lds + (stg & 1) * G::BUF;
            unsigned char *nxt = lds + ((stg + 1) & 1) * G::BUF;
            const bool more = stg + 1 < n_stage;
            if constexpr (decltype(first)::value) {
                consume(cur);
                // the columns of stage stg + 2 replace those of stage stg, last read a stage ago
                if (fetcher && stg + 2 < n_stage) fetch(stg + 2);
                if (more) produce(nxt, stg + 1);
                if (fetcher && stg + 2 < n_stage) stash(stg);
            } else {
                if (more) produce(nxt, stg + 1);
                consume(cur);
            }
            __syncthreads();
        }
        // the write-out's addresses are formed here rather than kept live across the stages
        int r4 = 4 * lk, c = l16;
        asm volatile("" : "+v"(r4), "+v"(c));
        float2 *P = (float2 *)a.part +
                    (((int64_t)inst * a.n_split + s) * a.n_tiles + bd.tile0 + t0) * (int64_t)(kPairTile * kPairTile);
#pragma unroll
        for (int t = 0; t < kWaveTiles; t++)
            if (t < nt)
#pragma unroll
                for (int e = 0; e < 4; e++)
                    P[t * kPairTile * kPairTile + (r4 + e) * kPairTile + c] = make_float2(re[t][e], im[t][e]);
    };
    if (wave < kWaves / 2)
        stages(std::true_type{});
    else
        stages(std::false_type{});
}

}  // namespace

hipError_t launch_pair_tiles(int prec, const PairArgs &a, hipStream_t s) {
    const int64_t items = (int64_t)a.n_inst * a.n_bundle * a.n_split;
    if (items <= 0) return hipSuccess;
    if (items > 0x7fffffff || a.n_feed > 2 || a.n_ax > 2) return hipErrorInvalidValue;
    if (prec == P32)
        k_pair_tiles<P32><<<(unsigned)items, 64 * kWaves, 0, s>>>(a);
    else if (prec == PB3)
        k_pair_tiles<PB3><<<(unsigned)items, 64 * kWaves, 0, s>>>(a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace mv
