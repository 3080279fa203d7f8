// Products over lists of 16 x 16 output tiles with Z formed in LDS, FP32 and BF16X3:
// the redundancy-aware product (App. A, Eq. Vpx) and the full product of small arrays
// and of several beams (MATVIS_PATH_FUSED).
//
// The host lists rows of Z (antenna, feed) in blocks of 16 and the tiles (I, J) to
// compute: those that hold a requested pair (81 tiles for the 1344 unique baselines of a
// 350-antenna hexagon, a sixth of V and a third less than the planned sub-matrices
// hold), or the lower triangle of V.  Tiles are grouped into bundles; a workgroup takes
// one (instance, k-split, bundle), forms every row of the bundle once per stage of 16
// columns and multiplies the bundle's tiles from it, up to 6 a wave.  So Z is neither
// written nor gathered, and nothing is done for padding beyond 16 rows: as blocks of 128
// rows, 12, 37 and 61 polarised antennas all took the time of 64.
//
// A polarised array with one beam (COHERENT; up to 64 antennas, on FP32 up to 80) stages, as the
// product over sources of larger ones does, the planes P0 = s0 F, P1 = s1 F and L = l F, with
// s_p = sqrt(C_pp) and l = C10 / s0 of the source's 2 x 2 coherency C = B B^H:
// V^00 = P0 P0^H, V^11 = P1 P1^H (lower triangles), V^10 = L P0^H: half the columns of Z.
//
// FP32 operands are three exact bf16 terms and six products, as in
// kernels_herk_x6.hip; BF16X3 operands hi + lo and all four products, because any
// tile may hold an autocorrelation, where lo lo^H is a one-signed bias.  The products
// of a stage start from zero and are added in FP32.
//
// A workgroup has 16 waves and a CU's LDS, or 8 and a half of it, or 4 and a quarter,
// whichever is the least that holds its bundle: a CU always has 16 waves, and small
// bundles have other workgroups to fill the waits at their barriers.
//
// Bound by vector instructions (66 % of the cycles, 4.4 per MFMA: forming, rotation of
// columns, the additions) and MFMAs (47 %) together, with LDS bank conflicts in 23 %; half of
// the waves multiply before they form the next stage and half after.  Requested pairs of 350 antennas, 49 152
// sources, 4 times of 8 channels, FP32: forming Z and multiplying went from 1.08 + 2.29
// to 0.80 ms, the error against 64 bits from 1.3e-6 to 2.2e-7.  16 waves of 6 tiles
// rather than 8 of 12 (with operands loaded a tile ahead) took 0.82 against 0.92 ms, rows
// and columns laid out for the banks 0.80.
// Whole calls of 100 000 sources, 4 times of 8 channels against blocks of 128 rows: FP32, 12
// / 37 / 61 polarised antennas 2.19 / 2.22 / 2.23 -> 0.31 / 0.60 / 0.98 ms, 30 / 100 / 200
// scalar ones 1.37 / 1.38 / 4.62 -> 0.23 / 0.60 / 1.41 ms; BF16X3, 12 / 37 / 61 polarised 0.83 /
// 0.85 / 0.86 -> 0.30 / 0.56 / 0.79 ms, 30 / 100 scalar 0.61 / 0.61 -> 0.22 / 0.50 ms.  The gain is
// least where the blocks had least padding: 113 / 128 scalar antennas on BF16X3 594 / 595 ->
// 544 / 557 us, 64 polarised ones 860 -> 784 us.  Errors against 64 bits: FP32 a quarter of what
// they were; BF16X3, set by its two-term split, 2.2e-6 -> 1.2e-6 at 100 to 128 scalar antennas
// and 100 000 sources, 1.9e-6 -> 5.1e-7 at 64 polarised ones.
#include <type_traits>

#include "herk_tiles.h"
#include "launch_rules.h"
#include "matvis.h"

namespace mv {

namespace {

constexpr int kSPS = 16;                       // columns per stage
constexpr int kPlane = 4 * kSPS;               // bytes of a row's plane

template <int PREC, int WAVES>
struct TileGeom {
    static constexpr int NT = PREC == P32 ? 3 : 2;     // bf16 terms per value
    static constexpr int RS = NT * kPlane + 16;        // 16 bytes of padding spread the banks
    static constexpr int ROWS = 16 * tile_blocks(WAVES);
    static constexpr int BUF = ROWS * RS;
};

// Two staged columns: the sources' directions and their values of both feeds (COHERENT:
// s0, s1 and l).  80 bytes,
// so that the eight pairs of a stage start in different banks.
struct __attribute__((aligned(16))) Columns {
    double x0, y0, z0, x1, y1, z1;
    float4 b0, b1;
};

struct Row {
    double ux, uy, uz;  // (nu / c) x_a
    int32_t bp;         // beam n_feed + feed; COHERENT: the plane
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

template <int PREC, int WAVES, bool COHERENT>
__global__ void __launch_bounds__(64 * WAVES, 4) k_tiles(TileArgs a) {
    typedef TileGeom<PREC, WAVES> G;
    constexpr int NT = G::NT, RS = G::RS;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * G::BUF];
    __shared__ Row row[G::ROWS];
    __shared__ Columns col[2][kSPS / 2];
    static_assert((2 * G::BUF + sizeof(Row) * G::ROWS + sizeof(Columns) * kSPS) * (16 / WAVES) <= 160 * 1024, "LDS");
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane & 15, lk = lane >> 4;
    const int64_t item = blockIdx.x;
    const int s = (int)(item % a.n_split);
    const int bundle = (int)((item / a.n_split) % a.n_bundle);
    const int inst = (int)(item / ((int64_t)a.n_split * a.n_bundle));
    const int tslot = inst / a.nfb;
    const int nx = COHERENT ? 1 : a.n_ax, nf = a.n_feed;
    const int64_t K = (int64_t)nx * a.count[tslot];
    const int64_t kc = split_cols(K, a.n_split);
    const int64_t kb = (int64_t)s * kc, ke = kb + kc < K ? kb + kc : K;
    if (kb >= K) return;  // an empty k-split: the reduction leaves it out too
    const TileBundle bd = a.bundles[bundle];
    const int n_rows = bd.n_rows;
    const int nr = COHERENT ? 3 : nf;  // rows of an antenna
    const double nu_c = a.freqs[a.f0 + inst % a.nfb] / kSpeedOfLight;
    const double *sh = a.s_hat + (int64_t)tslot * 3 * a.ld_src;
    const float2 *Bi = (const float2 *)a.B + (int64_t)inst * a.n_beam * nf * a.n_ax * a.ld_src;  // [beam][feed][axis][m]
    const bool shared_beam = a.n_beam == 1;
    for (int q = tid; q < n_rows; q += 64 * WAVES) {
        const int z = a.rows[bd.row0 + q], ant = z < 0 ? 0 : z / nr;  // padding rows reach no stored output
        const int p = z < 0 ? 0 : z % nr;
        row[q] = Row{nu_c * a.antc[3 * ant], nu_c * a.antc[3 * ant + 1], nu_c * a.antc[3 * ant + 2],
                       COHERENT ? p : a.bidx[ant] * nf + p, 0};
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
            if (COHERENT) {
                // B components c = 2 p + k; C10 = B10 conj(B00) + B11 conj(B01)
                const float2 b0 = Bi[m], b1 = Bi[a.ld_src + m], b2 = Bi[2 * a.ld_src + m], b3 = Bi[3 * a.ld_src + m];
                const float c00 = b0.x * b0.x + b0.y * b0.y + b1.x * b1.x + b1.y * b1.y;
                const float c11 = b2.x * b2.x + b2.y * b2.y + b3.x * b3.x + b3.y * b3.y;
                const float c10x = b2.x * b0.x + b2.y * b0.y + b3.x * b1.x + b3.y * b1.y;
                const float c10y = b2.y * b0.x - b2.x * b0.y + b3.y * b1.x - b3.x * b1.y;
                const float s0 = sqrtf(c00);
                fb = make_float4(s0, sqrtf(c11), s0 > 0.f ? c10x / s0 : 0.f, s0 > 0.f ? c10y / s0 : 0.f);
            } else if (shared_beam) {
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
    // two columns (2 mp, 2 mp + 1) of rows r0 + 8 WAVES k; the rows that 32 lanes write are 4
    // (832 bytes, a quarter of the banks) apart
    const int mp = tid % 8, g = tid / 8 % 8;
    const int r0 = wave / 2 * 16 + wave % 2 * 2 + g % 4 * 4 + g / 4;
    auto produce = [&](unsigned char *buf, int stage) __attribute__((always_inline)) {
        const Columns c = col[stage & 1][mp];
        const int64_t cg = kb + (int64_t)stage * kSPS + 2 * mp;
        for (int r = r0; r < n_rows; r += 8 * WAVES) {
            const Row e = row[r];
            float vr[2], vi[2];
            if (COHERENT) {
                const bool real = e.bp < 2, second = e.bp == 1;
                vr[0] = real ? (second ? c.b0.y : c.b0.x) : c.b0.z;
                vi[0] = real ? 0.f : c.b0.w;
                vr[1] = real ? (second ? c.b1.y : c.b1.x) : c.b1.z;
                vi[1] = real ? 0.f : c.b1.w;
            } else if (shared_beam) {
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
    const int t0 = bd.n_tiles * wave / WAVES, nt = bd.n_tiles * (wave + 1) / WAVES - t0;
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
        int r4 = 4 * lk, c = l16, ld = a.ld;
        asm volatile("" : "+v"(r4), "+v"(c), "+v"(ld));
        float2 *P = (float2 *)a.part + ((int64_t)inst * a.n_split + s) * a.part_stride;
        const int32_t *dst = a.dst + bd.tile0 + t0;
#pragma unroll
        for (int t = 0; t < kWaveTiles; t++)
            if (t < nt) {
                const int d = dst[t];
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    float2 v = make_float2(re[t][e], im[t][e]);
                    if constexpr (COHERENT) {
                        // rows and columns 2 a + p; V^10 above the antenna diagonal is V^01 below it
                        const int A = 16 * (d & 255) + r4 + e, B = 16 * (d >> 8 & 255) + c;
                        int r = 2 * A + (d >> 16 & 1), q = 2 * B + (d >> 17);
                        if (A < B && d >> 16 == 1) {
                            const int x = r;
                            r = q;
                            q = x;
                            v.y = -v.y;
                        }
                        P[(int64_t)r * ld + q] = v;
                    } else {
                        P[(int64_t)d + (r4 + e) * ld + c] = v;
                    }
                }
            }
    };
    if (wave < WAVES / 2)
        stages(std::true_type{});
    else
        stages(std::false_type{});
}

}  // namespace

int tile_waves(int n_rows, int n_tiles) {
    for (int w : {4, 8})
        if (n_rows <= 16 * tile_blocks(w) && n_tiles <= kWaveTiles * w) return w;
    return 16;
}

hipError_t launch_tiles(int prec, const TileArgs &a, hipStream_t s) {
    const int64_t items = (int64_t)a.n_inst * a.n_bundle * a.n_split;
    if (items <= 0) return hipSuccess;
    if (items * 64 * a.waves >= kMaxThreadsX || a.n_feed > 2 || a.n_ax > 2) return hipErrorInvalidValue;
    if (a.coherent && (a.n_feed != 2 || a.n_ax != 2 || a.n_beam != 1)) return hipErrorInvalidValue;
    auto launch = [&](auto waves) {
        constexpr int W = decltype(waves)::value;
        const unsigned g = (unsigned)items;
        if (prec == P32 && a.coherent)
            k_tiles<P32, W, true><<<g, 64 * W, 0, s>>>(a);
        else if (prec == P32)
            k_tiles<P32, W, false><<<g, 64 * W, 0, s>>>(a);
        else if (a.coherent)
            k_tiles<PB3, W, true><<<g, 64 * W, 0, s>>>(a);
        else
            k_tiles<PB3, W, false><<<g, 64 * W, 0, s>>>(a);
        return hipGetLastError();
    };
    if (prec != P32 && prec != PB3) return hipErrorInvalidValue;
    if (a.waves == 4) return launch(std::integral_constant<int, 4>{});
    if (a.waves == 8) return launch(std::integral_constant<int, 8>{});
    if (a.waves == 16) return launch(std::integral_constant<int, 16>{});
    return hipErrorInvalidValue;
}

}  // namespace mv
