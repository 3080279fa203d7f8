// Host side of the learned beam (include/matvis.h, "Learned beam").
// The loss and its gradient are the three launches of kernels_mlp_train.hip, or
// in the FP32 check mode a chain of the kernels in kernels_mlp.hip; the training
// loop is native, synchronises once per epoch, and draws the next epoch's order
// while the GPU runs the current one.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <mutex>
#include <new>
#include <numeric>
#include <random>
#include <vector>

#include "matvis.h"
#include "internal.h"
#include "mlp.h"

using namespace mv;

namespace {

#define CK(expr)                                       \
    do {                                               \
        hipError_t _e = (expr);                        \
        if (_e != hipSuccess) {                        \
            (void)hipGetLastError();                   \
            fprintf(stderr, "%s: %s\n", #expr, hipGetErrorString(_e)); \
            return MATVIS_EHIP;                        \
        }                                              \
    } while (0)

// Activation workspace of the FP32 check mode for n rows: buffer sizes in floats, in the order the
// workspace holds them.  alloc() gives each its own device allocation; bind()
// carves them, 256-byte aligned, out of one caller-provided block of
// Work::floats_for(rows) floats.
struct Work {
    int64_t n = 0;
    float *phi = nullptr, *Z[4] = {}, *H[4] = {}, *out = nullptr, *dout = nullptr, *dH = nullptr, *dZ = nullptr,
          *part = nullptr, *ws = nullptr;
    int64_t ws_elems = 0;  // split-k partial products and column-sum partials
    std::vector<void *> allocs;
    static int64_t ws_for(int64_t rows) { return std::max<int64_t>(384 * 4096, (rows + 255) / 256 * kHid); }
    // the (pointer, size) list in workspace order
    template <typename F>
    static hipError_t each(int64_t rows, float **phi, float **Z, float **H, float **out, float **dout, float **dH,
                           float **dZ, float **part, float **ws, F &&one) {
        hipError_t e = one(phi, rows * kFeat);
        for (int l = 0; l < 4 && e == hipSuccess; l++) e = one(&Z[l], rows * kHid);
        for (int l = 0; l < 4 && e == hipSuccess; l++) e = one(&H[l], rows * kHid);
        if (e == hipSuccess) e = one(out, rows * kNet);   // network outputs (basis coefficients)
        if (e == hipSuccess) e = one(dout, rows * kNet);
        if (e == hipSuccess) e = one(dH, rows * kHid);
        if (e == hipSuccess) e = one(dZ, rows * kHid);
        if (e == hipSuccess) e = one(part, (rows * kOut + 255) / 256 + 1);
        if (e == hipSuccess) e = one(ws, ws_for(rows));
        return e;
    }
    static constexpr int64_t kAlign = 64;  // floats (256 bytes)
    static int64_t round_a(int64_t c) { return (std::max<int64_t>(c, 1) + kAlign - 1) / kAlign * kAlign; }
    static int64_t floats_for(int64_t rows) {
        int64_t total = 0;
        float *dummy[16] = {};
        (void)each(rows, &dummy[0], &dummy[1], &dummy[5], &dummy[9], &dummy[10], &dummy[11], &dummy[12], &dummy[13],
                   &dummy[14], [&](float **, int64_t count) {
                 total += round_a(count);
                 return hipSuccess;
             });
        return total;
    }
    hipError_t alloc(int64_t rows) {
        n = rows;
        ws_elems = ws_for(rows);
        return each(rows, &phi, Z, H, &out, &dout, &dH, &dZ, &part, &ws, [&](float **p, int64_t count) {
            void *q = nullptr;
            hipError_t e = hipMalloc(&q, sizeof(float) * std::max<int64_t>(count, 1));
            if (e == hipSuccess) {
                allocs.push_back(q);
                *p = (float *)q;
            }
            return e;
        });
    }
    // no allocation: the buffers are consecutive pieces of base[0 .. floats_for(rows))
    void bind(float *base, int64_t rows) {
        n = rows;
        ws_elems = ws_for(rows);
        int64_t off = 0;
        (void)each(rows, &phi, Z, H, &out, &dout, &dH, &dZ, &part, &ws, [&](float **p, int64_t count) {
            *p = base + off;
            off += round_a(count);
            return hipSuccess;
        });
    }
    ~Work() {
        for (void *p : allocs) (void)hipFree(p);
    }
};

// Workspace of the bf16 mode for n rows: train_bind() carves the buffers, 256-byte
// aligned, out of one block of train_floats(n) floats.
mlp::TrainBufs train_bind(float *base, int64_t n, int64_t *total = nullptr) {
    int64_t off = 0;
    auto piece = [&](int64_t floats) {
        float *p = base ? base + off : nullptr;
        off += Work::round_a(floats);
        return p;
    };
    mlp::TrainBufs b{};
    b.phi = (__bf16 *)piece(n * kFeat / 2);
    for (int l = 0; l < 3; l++) b.h[l] = (__bf16 *)piece(n * kHid / 2);
    b.h4 = piece(n * kHid);
    for (int l = 0; l < 4; l++) b.dz[l] = piece(n * kHid);
    b.dnet = piece(n * kNet);
    b.part = piece(mlp::train_part_floats(n));
    b.sq = (double *)piece(2 * mlp::train_sq_count(n));
    b.images = piece(mlp::train_image_floats());
    if (total) *total = off;
    return b;
}
int64_t train_floats(int64_t n) {
    int64_t total = 0;
    (void)train_bind(nullptr, n, &total);
    return total;
}

// Loss and gradient of n rows on bf16 products in a block of train_floats(n) floats.
hipError_t loss_grad_bf16(const float *P, const float *x, const float *y, int64_t n, float *grad, float *loss,
                          float *base, hipStream_t s) {
    const mlp::TrainBufs b = train_bind(base, n);
    hipError_t e = mlp::train_pack(P, b.images, s);
    if (e == hipSuccess)
        e = mlp::train_step(b, P, x, y, nullptr, n, grad, loss, nullptr, nullptr, nullptr, 0, 0.f, s);
    return e;
}

// FP32 forward + backward of the squared error for w.n rows of (x, y).
hipError_t loss_grad_impl(const float *P, const float *x, const float *y, float *grad, float *loss, Work &w,
                          hipStream_t s) {
    const int64_t n = w.n;
    const int ni = (int)n;
    hipError_t e;
#define RET(expr)                      \
    if ((e = (expr)) != hipSuccess) return e
    RET(mlp::features(x, n, P, w.phi, s));
    RET(mlp::gemm(w.phi, kFeat, 1, P + kOffW1, kFeat, 1, ni, kHid, kFeat, P + kOffB1, w.Z[0], w.H[0], 1,
                  w.ws, w.ws_elems, s));
    const int64_t offW[3] = {kOffW2, kOffW3, kOffW4}, offB[3] = {kOffB2, kOffB3, kOffB4};
    for (int l = 1; l < 4; l++)
        RET(mlp::gemm(w.H[l - 1], kHid, 1, P + offW[l - 1], kHid, 1, ni, kHid, kHid, P + offB[l - 1], w.Z[l],
                      w.H[l], 1, w.ws, w.ws_elems, s));
    // the linear head, then the Chebyshev
    // sums of the frequency head and the squared error
    RET(mlp::gemm(w.H[3], kHid, 1, P + kOffW5, kHid, 1, ni, kNet, kHid, P + kOffB5, w.out, nullptr, 0,
                  w.ws, w.ws_elems, s));
    RET(mlp::loss_grad(w.out, x, y, n, w.dout, w.part, loss, s));
    RET(mlp::fill(grad, kOffW1, 0.f, s));  // the Fourier matrix is not trained
    // output layer
    RET(mlp::gemm(w.dout, 1, kNet, w.H[3], 1, kHid, kNet, kHid, ni, nullptr, grad + kOffW5, nullptr, 0,
                  w.ws, w.ws_elems, s));
    RET(mlp::colsum(w.dout, n, kNet, grad + kOffB5, w.ws, w.ws_elems, s));
    RET(mlp::gemm(w.dout, kNet, 1, P + kOffW5, 1, kHid, ni, kHid, kNet, nullptr, w.dH, nullptr, 0,
                  w.ws, w.ws_elems, s));
    // hidden layers 4..2
    const int64_t gW[4] = {kOffW1, kOffW2, kOffW3, kOffW4}, gB[4] = {kOffB1, kOffB2, kOffB3, kOffB4};
    for (int l = 3; l >= 1; l--) {
        RET(mlp::silu_bwd(w.dH, w.Z[l], w.dZ, n * kHid, s));
        RET(mlp::gemm(w.dZ, 1, kHid, w.H[l - 1], 1, kHid, kHid, kHid, ni, nullptr, grad + gW[l], nullptr, 0,
                      w.ws, w.ws_elems, s));
        RET(mlp::colsum(w.dZ, n, kHid, grad + gB[l], w.ws, w.ws_elems, s));
        RET(mlp::gemm(w.dZ, kHid, 1, P + gW[l], 1, kHid, ni, kHid, kHid, nullptr, w.dH, nullptr, 0,
                      w.ws, w.ws_elems, s));
    }
    RET(mlp::silu_bwd(w.dH, w.Z[0], w.dZ, n * kHid, s));
    RET(mlp::gemm(w.dZ, 1, kHid, w.phi, 1, kFeat, kHid, kFeat, ni, nullptr, grad + kOffW1, nullptr, 0,
                  w.ws, w.ws_elems, s));
    RET(mlp::colsum(w.dZ, n, kHid, grad + kOffB1, w.ws, w.ws_elems, s));
#undef RET
    return hipSuccess;
}

}  // namespace

// ---- The allocation-free loss / gradient (matvis_mlp_loss_grad_noalloc) ----
// Its workspace is one file-scope device array of kNoAllocRows rows' worth of
// activations (33.6 MB), which every GPU the library runs on holds until the
// process ends.  Host code never uses the array's name as an address: its
// device address is looked up once per device (hipGetSymbolAddress, with that
// device current) and kept in noalloc_ptr.
static constexpr int64_t kNoAllocRows = 4096;
static constexpr int64_t kNoAllocFloats = 8388800;  // Work::floats_for(kNoAllocRows), checked below
static __device__ __align__(256) float scratch[kNoAllocFloats];

static constexpr int kMaxDevices = 64;
static std::mutex noalloc_mu;
static float *noalloc_ptr[kMaxDevices] = {};

static hipError_t noalloc_scratch(float **p) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(noalloc_mu);
    if (!noalloc_ptr[dev]) {
        void *q = nullptr;
        e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        noalloc_ptr[dev] = (float *)q;
    }
    *p = noalloc_ptr[dev];
    return hipSuccess;
}

// Weight images of forward calls in flight: a few static slots per device (module memory),
// taken for the length of a call, which ends after its stream is done with them; a call
// that finds none free allocates, which costs some 10 us more.
constexpr int kImgSlots = 4;
static __device__ __attribute__((aligned(16))) __bf16 forward_images[kImgSlots][mlp::kImgElems];
static unsigned img_busy[kMaxDevices] = {};

struct ForwardImage {
    __bf16 *p = nullptr;
    int dev = -1, slot = -1;
    hipError_t take() {
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < kMaxDevices) {
            std::lock_guard<std::mutex> lock(noalloc_mu);
            for (int i = 0; i < kImgSlots && slot < 0; i++)
                if (!(img_busy[dev] >> i & 1)) slot = i;
            if (slot >= 0) {
                void *q = nullptr;
                e = hipGetSymbolAddress(&q, HIP_SYMBOL(forward_images));
                if (e != hipSuccess) {
                    slot = -1;
                    return e;
                }
                img_busy[dev] |= 1u << slot;
                p = (__bf16 *)q + (size_t)slot * mlp::kImgElems;
                return hipSuccess;
            }
        }
        return hipMalloc(&p, sizeof(__bf16) * mlp::kImgElems);
    }
    ~ForwardImage() {
        if (slot < 0) {
            if (p) (void)hipFree(p);
            return;
        }
        std::lock_guard<std::mutex> lock(noalloc_mu);
        img_busy[dev] &= ~(1u << slot);
    }
};

extern "C" {

matvis_status matvis_mlp_forward(const float *params, const float *x, int64_t n, float *out, void *stream) {
    if (!params || (n > 0 && (!x || !out)) || n < 0) return MATVIS_EINVAL;
    if ((uintptr_t)params % 16 || (uintptr_t)out % 16) return MATVIS_EINVAL;  // read / written as float4
    if (n == 0) return MATVIS_OK;
    hipStream_t s = (hipStream_t)stream;
    ForwardImage img;
    CK(img.take());
    hipError_t e = mlp::pack_weights(params, img.p, s);
    if (e == hipSuccess) e = mlp::infer_plain(params, img.p, x, n, out, s);
    const hipError_t sync = hipStreamSynchronize(s);  // the image is given back after this, also on an error
    CK(e);
    CK(sync);
    return MATVIS_OK;
}

matvis_status matvis_mlp_loss_grad(const float *params, const float *x, const float *y, int64_t n, int32_t fp32_math,
                                   float *grad, float *loss, void *stream) {
    if (!params || !x || !y || !grad || !loss || n <= 0 || n > (1 << 24)) return MATVIS_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (!fp32_math) {
        float *base = nullptr;
        CK(hipMalloc(&base, sizeof(float) * train_floats(n)));
        hipError_t e = loss_grad_bf16(params, x, y, n, grad, loss, base, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        (void)hipFree(base);
        CK(e);
        return MATVIS_OK;
    }
    Work w;
    CK(w.alloc(n));
    CK(loss_grad_impl(params, x, y, grad, loss, w, s));
    CK(hipStreamSynchronize(s));
    return MATVIS_OK;
}

matvis_status matvis_mlp_loss_grad_noalloc(const float *params, const float *x, const float *y, int64_t n,
                                           int32_t fp32_math, float *grad, float *loss, void *stream) {
    if (!params || !x || !y || !grad || !loss || n <= 0) return MATVIS_EINVAL;
    if (n > kNoAllocRows) {
        fprintf(stderr,
                "matvis_mlp_loss_grad_noalloc: n = %lld rows exceeds the static workspace of %lld rows "
                "(use matvis_mlp_loss_grad)\n",
                (long long)n, (long long)kNoAllocRows);
        return MATVIS_EINVAL;
    }
    if (Work::floats_for(kNoAllocRows) != kNoAllocFloats || train_floats(n) > kNoAllocFloats) {  // layout and array size out of step
        fprintf(stderr, "matvis_mlp_loss_grad_noalloc: workspace layout needs %lld floats, array holds %lld\n",
                (long long)Work::floats_for(kNoAllocRows), (long long)kNoAllocFloats);
        return MATVIS_EUNSUPPORTED;
    }
    float *base = nullptr;
    CK(noalloc_scratch(&base));
    if (!fp32_math) {
        CK(loss_grad_bf16(params, x, y, n, grad, loss, base, (hipStream_t)stream));
        return MATVIS_OK;
    }
    Work w;
    w.bind(base, n);
    CK(loss_grad_impl(params, x, y, grad, loss, w, (hipStream_t)stream));
    return MATVIS_OK;
}

matvis_status matvis_mlp_adam(float *params, const float *grad, float *m1, float *m2, int64_t step, float lr,
                              void *stream) {
    if (!params || !grad || !m1 || !m2 || step < 1) return MATVIS_EINVAL;
    CK(mlp::adam(params, grad, m1, m2, kNParams, step, lr, (hipStream_t)stream));
    return MATVIS_OK;
}

matvis_status matvis_beam_samples(const void *grid, int32_t n_chan, int32_t n_feed, int32_t n_ax, int32_t n_za,
                                  int32_t n_az, double dza_rad, double daz_rad, int32_t bicubic, const double *za,
                                  const double *az, const int32_t *chan, int64_t n, float *out,
                                  const double *chan_freq_hz, double nu_min_hz, double nu_max_hz, float *x,
                                  void *stream) {
    if (!grid || (n > 0 && (!za || !az || !chan || !out)) || n < 0) return MATVIS_EINVAL;
    if (x && (!chan_freq_hz || !std::isfinite(nu_min_hz) || !std::isfinite(nu_max_hz) || !(nu_max_hz > nu_min_hz)))
        return MATVIS_EINVAL;
    if (n_chan <= 0 || n_feed < 1 || n_feed > 2 || n_ax < 1 || n_ax > 2 || n_za < 3 || n_az < 3) return MATVIS_EINVAL;
    if (!(dza_rad > 0) || !(daz_rad > 0)) return MATVIS_EINVAL;
    // validate the channel indices here so that no kernel reads outside the grid
    std::vector<int32_t> h((size_t)n);
    CK(hipMemcpy(h.data(), chan, sizeof(int32_t) * n, hipMemcpyDeviceToHost));
    for (int32_t c : h)
        if (c < 0 || c >= n_chan) return MATVIS_EINVAL;
    CK(mlp::beam_samples(grid, n_feed, n_ax, n_za, n_az, dza_rad, daz_rad, bicubic, za, az, chan, n, out,
                         chan_freq_hz, nu_min_hz, nu_max_hz, x, (hipStream_t)stream));
    return MATVIS_OK;
}

matvis_status matvis_train_surrogate(float *params, const float *x, const float *y, int64_t n, int32_t batch,
                                     int32_t epochs, float lr0, float lr1, uint64_t seed, int32_t fp32_math,
                                     float *loss_history, void *stream) {
    if (!params || !x || !y || n <= 0 || n > (1 << 30) || batch <= 0 || batch > (1 << 24) || epochs <= 0 ||
        !(lr0 > 0) || !(lr1 > 0))
        return MATVIS_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const int64_t bsz = std::min<int64_t>(batch, n);
    const int64_t nb = n / bsz;  // whole batches only
    std::vector<int32_t> order[2];  // this epoch's and the next one's
    std::vector<float> lh;
    try {
        order[0].resize((size_t)n);
        if (epochs > 1) order[1].resize((size_t)n);
        lh.resize((size_t)std::min<int64_t>(nb, 4096));
    } catch (const std::bad_alloc &) {
        return MATVIS_ENOMEM;
    }
    std::iota(order[0].begin(), order[0].end(), 0);
    std::mt19937_64 rng(seed);
    std::shuffle(order[0].begin(), order[0].end(), rng);
    Work w;
    if (fp32_math) CK(w.alloc(bsz));
    // one block: the row buffers (bf16 mode) or a batch's gradient and samples (check
    // mode), then the moments, the losses and the order
    const int64_t head = fp32_math ? Work::round_a(kNParams) + Work::round_a(bsz * 3) + Work::round_a(bsz * kOut)
                                   : train_floats(bsz);
    const int64_t moments = Work::round_a(kNParams);
    float *base = nullptr;
    CK(hipMalloc(&base, sizeof(float) * (head + 2 * moments + 4096 + n)));
    float *grad = base, *xb = grad + Work::round_a(kNParams), *yb = xb + Work::round_a(bsz * 3);  // check mode
    float *m1 = base + head, *m2 = m1 + moments, *lossd = m2 + moments;
    int32_t *perm_d = (int32_t *)(lossd + 4096);
    const mlp::TrainBufs tb = fp32_math ? mlp::TrainBufs{} : train_bind(base, bsz);
    hipError_t e = hipMemsetAsync(m1, 0, sizeof(float) * 2 * moments, s);
    if (e == hipSuccess && !fp32_math) e = mlp::train_pack(params, tb.images, s);
    int64_t step = 0;
    for (int ep = 0; ep < epochs && e == hipSuccess; ep++) {
        if (ep > 0) e = hipStreamSynchronize(s);  // the previous epoch's order has been uploaded
        if (e != hipSuccess) break;
        const std::vector<int32_t> &perm = order[ep & 1];
        e = hipMemcpyAsync(perm_d, perm.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, s);
        const float lr = epochs > 1 ? lr0 * std::pow(lr1 / lr0, (float)ep / (float)(epochs - 1)) : lr0;
        for (int64_t b = 0; b < nb && e == hipSuccess; b++) {
            if (!fp32_math) {
                e = mlp::train_step(tb, params, x, y, perm_d + b * bsz, bsz, nullptr, lossd + (b % 4096), params, m1,
                                    m2, ++step, lr, s);
                continue;
            }
            e = mlp::gather_rows(x, 3, perm_d + b * bsz, bsz, xb, s);
            if (e == hipSuccess) e = mlp::gather_rows(y, kOut, perm_d + b * bsz, bsz, yb, s);
            if (e == hipSuccess) e = loss_grad_impl(params, xb, yb, grad, lossd + (b % 4096), w, s);
            if (e == hipSuccess) e = mlp::adam(params, grad, m1, m2, kNParams, ++step, lr, s);
        }
        if (ep + 1 < epochs) {  // the next epoch's order, while the GPU works
            std::vector<int32_t> &next = order[(ep + 1) & 1];
            std::copy(perm.begin(), perm.end(), next.begin());
            std::shuffle(next.begin(), next.end(), rng);
        }
        if (e == hipSuccess && loss_history) {
            const int64_t k = std::min<int64_t>(nb, 4096);
            e = hipMemcpyAsync(lh.data(), lossd, sizeof(float) * k, hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            double sum = 0.0;
            for (int64_t i = 0; i < k; i++) sum += lh[i];
            loss_history[ep] = (float)(sum / (double)k);
        }
    }
    const hipError_t done = hipStreamSynchronize(s);  // also after an error: the block is in use until then
    if (e == hipSuccess) e = done;
    (void)hipFree(base);
    CK(e);
    return MATVIS_OK;
}

}  // extern "C"
