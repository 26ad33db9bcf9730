// C-ABI host side of the droplet-shape surrogate.  Declarations and the contract
// of every call: sclmlp.h.  Kernels: mlp_kernels.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <mutex>
#include <string>
#include <vector>

#include "mlp_kernels.hpp"
#include "sclmlp.h"

using namespace sclmlp;

namespace {

thread_local std::string g_err;

sclbm_status fail(sclbm_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

#define HIP_TRY(expr)                                                                                   \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess) return fail(SCLBM_EHIP, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                                          __FILE__, __LINE__);                                          \
    } while (0)

#define HIP_LAUNCHED()                                                                                  \
    do {                                                                                                \
        hipError_t e_ = hipGetLastError();                                                              \
        if (e_ != hipSuccess) return fail(SCLBM_EHIP, "kernel launch: %s (%s:%d)", hipGetErrorString(e_), \
                                          __FILE__, __LINE__);                                          \
    } while (0)

#define TRY(expr)                            \
    do {                                     \
        sclbm_status s_ = (expr);            \
        if (s_ != SCLBM_OK) return s_;       \
    } while (0)

constexpr size_t kAlign = 256;
size_t round_up(size_t v, size_t a = kAlign) { return (v + a - 1) / a * a; }

// Slices of the batch whose weight gradients are summed separately.  Up to kSmallBatch rows 32 x 32
// tiles give 800 wavefronts and need none; above, a wavefront takes 64 x 64 (half the operand
// traffic) and the batch is cut into slices of about 1024 rows, three at 2049 rows and at most 8, to
// have enough of them (8192 rows: all gradients 30 us and their sum 5.5; one 64 x 64 tile per
// LDS-staging workgroup, layer after layer, with the row sums after each, took 287).
constexpr int64_t kSmallBatch = 2048;
int grad_slices(int64_t mpad) { return mpad <= kSmallBatch ? 1 : int(std::min<int64_t>(8, (mpad + 1023) / 1024)); }

// Byte offsets of every buffer inside the workspace for batches of up to mmax rows.
struct Layout {
    size_t p, g, m1, m2, norm, wf[3], wtf[3], w4, x, xt, h[3], ht[3], dz[2], dzt[3], dy, partial, part, loss, bad, zeroed, total;
};

Layout make_layout(int64_t mmax) {
    Layout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = round_up(off + bytes);
        return o;
    };
    const size_t pb = sizeof(float) * NPARAM;
    L.p = take(pb);
    L.g = take(pb);
    L.m1 = take(pb);
    L.m2 = take(pb);
    L.norm = take(sizeof(float) * (2 * NIN + 2 * NOUT));
    for (int l = 0; l < 3; ++l) L.wf[l] = take(sizeof(bf16) * NHID * (l == 0 ? NIN : NHID));
    for (int l = 0; l < 3; ++l) L.wtf[l] = l == 0 ? 0 : take(sizeof(bf16) * NHID * NHID);
    L.w4 = take(sizeof(bf16) * NOUT * NHID);
    L.loss = take(sizeof(double));
    L.bad = take(sizeof(unsigned));
    L.zeroed = off;
    const size_t m = (size_t)mmax;
    L.x = take(sizeof(bf16) * m * NIN);
    for (int l = 0; l < 3; ++l) L.h[l] = take(sizeof(bf16) * m * NHID);
    // the pre-activation gradients over the units take the place of activations whose last
    // reader has run (dZ3 that of H3, which its kernel reads in the same place), and the
    // slices of the weight gradients that of X and all of them
    L.dz[0] = L.h[2];
    L.dz[1] = L.h[1];
    L.part = L.x;
    off = std::max(off, round_up(L.part + sizeof(float) * grad_slices(mmax) * OFF_W4));
    L.xt = take(sizeof(bf16) * m * NIN);
    for (int l = 0; l < 3; ++l) {
        L.ht[l] = take(sizeof(bf16) * m * NHID);
        L.dzt[l] = take(sizeof(bf16) * m * NHID);
    }
    L.dy = take(sizeof(float) * m * NOUT);
    L.partial = take(sizeof(double) * 4 * (m / OUT_ROWS));
    L.total = off;
    return L;
}

int64_t padded_rows(int64_t n) { return (n + ROW_ALIGN - 1) / ROW_ALIGN * ROW_ALIGN; }

}  // namespace

struct sclmlp_ctx {
    int64_t max_batch = 0, mmax = 0;
    char *ws = nullptr;
    Layout lay{};
    hipStream_t stream = nullptr;
    int device = 0;
    int64_t step = 0;
    hipEvent_t inputs = nullptr, results = nullptr;  // order against another stream (no timing)
    std::mutex ordering;  // held from an event's record to its wait: threads may share a context

    template <class T>
    T *at(size_t off) const { return reinterpret_cast<T *>(ws + off); }
    float *P() const { return at<float>(lay.p); }
    float *G() const { return at<float>(lay.g); }
    float *in_shift() const { return at<float>(lay.norm); }
    float *in_scale() const { return at<float>(lay.norm) + NIN; }
    float *out_shift() const { return at<float>(lay.norm) + 2 * NIN; }
    float *out_scale() const { return at<float>(lay.norm) + 2 * NIN + NOUT; }
    bf16 *wf(int l) const { return at<bf16>(lay.wf[l]); }
    bf16 *wtf(int l) const { return at<bf16>(lay.wtf[l]); }
    bf16 *w4() const { return at<bf16>(lay.w4); }
    bf16 *h(int l) const { return at<bf16>(lay.h[l]); }
    bf16 *ht(int l) const { return at<bf16>(lay.ht[l]); }
    bf16 *dz(int l) const { return at<bf16>(lay.dz[l]); }
    bf16 *dzt(int l) const { return at<bf16>(lay.dzt[l]); }
};

namespace {

// One hidden layer over mpad rows: forward, or with MASK the gradient of the layer below.
// Up to kSmallBatch rows a wavefront takes one 32 x 32 tile and a workgroup of its own (256 rows: 128
// of them, 4.1 us a layer; 64 x 64 tiles staged through LDS, 32 workgroups, took 8.6).  Above, four
// wavefronts to a workgroup: 64 x 32 each up to twice that, where 64 x 64 would leave fewer than a wavefront
// per SIMD, then 64 x 64, which reads each operand half as often (8192 rows: 11 us).
template <int K, bool MASK>
sclbm_status layer(const sclmlp_ctx *c, const LayerArgs &g) {
    if (g.Mpad <= kSmallBatch)
        k_layer<K, 1, 1, MASK, 1><<<g.Mpad / 32 * (NHID / 32), 64, 0, c->stream>>>(g);
    else if (g.Mpad <= 2 * kSmallBatch)
        k_layer<K, 2, 1, MASK, 2><<<g.Mpad / 128 * (NHID / 64), 256, 0, c->stream>>>(g);
    else
        k_layer<K, 2, 2, MASK, 2><<<g.Mpad / 128 * (NHID / 128), 256, 0, c->stream>>>(g);
    HIP_LAUNCHED();
    return SCLBM_OK;
}

AdamArgs adam_args(const sclmlp_ctx *c) {
    AdamArgs a{};
    a.p = c->P();
    a.g = c->G();
    a.m = c->at<float>(c->lay.m1);
    a.v = c->at<float>(c->lay.m2);
    for (int l = 0; l < 3; ++l) {
        a.w[l] = c->wf(l);
        a.wt[l] = l == 0 ? nullptr : c->wtf(l);
    }
    a.w4 = c->w4();
    return a;
}

sclbm_status refresh_copies(sclmlp_ctx *c) {
    AdamArgs a = adam_args(c);
    a.update = 0;
    k_adam<<<ADAM_BLOCKS, 256, 0, c->stream>>>(a);
    HIP_LAUNCHED();
    return SCLBM_OK;
}

sclbm_status use_device(const sclmlp_ctx *c) {
    HIP_TRY(hipSetDevice(c->device));
    return SCLBM_OK;
}

}  // namespace

extern "C" {

sclbm_status sclmlp_workspace_bytes(int64_t max_batch, size_t *bytes) {
    if (!bytes) return fail(SCLBM_EINVAL, "null output");
    if (max_batch < 1 || max_batch > (1 << 24)) return fail(SCLBM_EINVAL, "max_batch must be in [1, 2^24]");
    *bytes = make_layout(padded_rows(max_batch)).total;
    return SCLBM_OK;
}

sclbm_status sclmlp_create(int64_t max_batch, void *dev_workspace, size_t bytes, void *hip_stream, sclmlp_ctx **out) {
    if (!out) return fail(SCLBM_EINVAL, "null output");
    *out = nullptr;
    size_t need = 0;
    TRY(sclmlp_workspace_bytes(max_batch, &need));
    if (!dev_workspace) return fail(SCLBM_EINVAL, "null workspace");
    if (reinterpret_cast<uintptr_t>(dev_workspace) % kAlign) return fail(SCLBM_EINVAL, "workspace not 256-byte aligned");
    if (bytes < need) return fail(SCLBM_ESIZE, "workspace has %zu bytes, needs %zu", bytes, need);
    sclmlp_ctx *c = new sclmlp_ctx;
    c->max_batch = max_batch;
    c->mmax = padded_rows(max_batch);
    c->ws = static_cast<char *>(dev_workspace);
    c->lay = make_layout(c->mmax);
    c->stream = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipGetDevice(&c->device);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->inputs, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->results, hipEventDisableTiming);
    if (e == hipSuccess) e = hipMemsetAsync(c->ws, 0, c->lay.zeroed, c->stream);
    if (e == hipSuccess) {
        std::vector<float> norm(2 * NIN + 2 * NOUT, 0.0f);
        for (int i = 0; i < NIN; ++i) norm[NIN + i] = 1.0f;
        for (int j = 0; j < NOUT; ++j) norm[2 * NIN + NOUT + j] = 1.0f;
        e = hipMemcpyAsync(c->in_shift(), norm.data(), norm.size() * sizeof(float), hipMemcpyHostToDevice, c->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    }
    if (e != hipSuccess) {
        sclmlp_destroy(c);
        return fail(SCLBM_EHIP, "create: %s", hipGetErrorString(e));
    }
    *out = c;
    return SCLBM_OK;
}

sclbm_status sclmlp_destroy(sclmlp_ctx *ctx) {
    if (ctx) {
        if (ctx->inputs) (void)hipEventDestroy(ctx->inputs);  // teardown: nothing to do on failure
        if (ctx->results) (void)hipEventDestroy(ctx->results);
    }
    delete ctx;
    return SCLBM_OK;
}

sclbm_status sclmlp_after_stream(sclmlp_ctx *c, void *hip_stream) {
    if (!c) return fail(SCLBM_EINVAL, "null context");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (s == c->stream) return SCLBM_OK;
    TRY(use_device(c));
    std::lock_guard<std::mutex> lock(c->ordering);
    HIP_TRY(hipEventRecord(c->inputs, s));
    HIP_TRY(hipStreamWaitEvent(c->stream, c->inputs, 0));
    return SCLBM_OK;
}

sclbm_status sclmlp_before_stream(sclmlp_ctx *c, void *hip_stream) {
    if (!c) return fail(SCLBM_EINVAL, "null context");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (s == c->stream) return SCLBM_OK;
    TRY(use_device(c));
    std::lock_guard<std::mutex> lock(c->ordering);
    HIP_TRY(hipEventRecord(c->results, c->stream));
    HIP_TRY(hipStreamWaitEvent(s, c->results, 0));
    return SCLBM_OK;
}

sclbm_status sclmlp_set_params(sclmlp_ctx *c, const float *params) {
    if (!c || !params) return fail(SCLBM_EINVAL, "null argument");
    for (int i = 0; i < NPARAM; ++i)
        if (!std::isfinite(params[i])) return fail(SCLBM_EINVAL, "parameter %d is not finite", i);
    TRY(use_device(c));
    HIP_TRY(hipMemcpyAsync(c->P(), params, sizeof(float) * NPARAM, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipMemsetAsync(c->at<float>(c->lay.m1), 0, sizeof(float) * NPARAM, c->stream));
    HIP_TRY(hipMemsetAsync(c->at<float>(c->lay.m2), 0, sizeof(float) * NPARAM, c->stream));
    TRY(refresh_copies(c));
    HIP_TRY(hipStreamSynchronize(c->stream));
    c->step = 0;
    return SCLBM_OK;
}

sclbm_status sclmlp_get_params(sclmlp_ctx *c, float *params) {
    if (!c || !params) return fail(SCLBM_EINVAL, "null argument");
    TRY(use_device(c));
    HIP_TRY(hipMemcpyAsync(params, c->P(), sizeof(float) * NPARAM, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return SCLBM_OK;
}

sclbm_status sclmlp_get_grads(sclmlp_ctx *c, float *grads) {
    if (!c || !grads) return fail(SCLBM_EINVAL, "null argument");
    TRY(use_device(c));
    HIP_TRY(hipMemcpyAsync(grads, c->G(), sizeof(float) * NPARAM, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return SCLBM_OK;
}

sclbm_status sclmlp_set_normalization(sclmlp_ctx *c, const float *in_shift, const float *in_scale,
                                      const float *out_shift, const float *out_scale) {
    if (!c || !in_shift || !in_scale || !out_shift || !out_scale) return fail(SCLBM_EINVAL, "null argument");
    std::vector<float> norm(2 * NIN + 2 * NOUT);
    for (int i = 0; i < NIN; ++i) {
        if (!std::isfinite(in_shift[i]) || !std::isfinite(in_scale[i]) || in_scale[i] == 0.0f)
            return fail(SCLBM_EINVAL, "input normalisation entry %d invalid", i);
        norm[i] = in_shift[i];
        norm[NIN + i] = in_scale[i];
    }
    for (int j = 0; j < NOUT; ++j) {
        if (!std::isfinite(out_shift[j]) || !std::isfinite(out_scale[j]) || out_scale[j] == 0.0f)
            return fail(SCLBM_EINVAL, "output normalisation entry %d invalid", j);
        norm[2 * NIN + j] = out_shift[j];
        norm[2 * NIN + NOUT + j] = out_scale[j];
    }
    TRY(use_device(c));
    HIP_TRY(hipMemcpyAsync(c->in_shift(), norm.data(), norm.size() * sizeof(float), hipMemcpyHostToDevice,
                           c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return SCLBM_OK;
}

sclbm_status sclmlp_predict(sclmlp_ctx *c, const float *dev_windows, int64_t n, float *dev_out) {
    if (!c) return fail(SCLBM_EINVAL, "null context");
    if (n < 0 || n > c->max_batch) return fail(SCLBM_EINVAL, "n = %lld outside [0, %lld]", (long long)n,
                                              (long long)c->max_batch);
    if (n == 0) return SCLBM_OK;
    if (!dev_windows || !dev_out) return fail(SCLBM_EINVAL, "null buffer");
    TRY(use_device(c));
    ForwardArgs f{};
    f.win = dev_windows;
    f.n = (int)n;
    f.ashift = c->in_shift();
    f.ascale = c->in_scale();
    const int boff[3] = {OFF_B1, OFF_B2, OFF_B3};
    for (int l = 0; l < 3; ++l) {
        f.W[l] = c->wf(l);
        f.bias[l] = c->P() + boff[l];
    }
    f.W4 = c->w4();
    f.b4 = c->P() + OFF_B4;
    f.oshift = c->out_shift();
    f.oscale = c->out_scale();
    f.out = dev_out;
    const int blocks = int((n + FW_M - 1) / FW_M);
    if (reinterpret_cast<uintptr_t>(dev_windows) % 16 == 0)
        k_forward<true><<<blocks, FW_T, 0, c->stream>>>(f);
    else
        k_forward<false><<<blocks, FW_T, 0, c->stream>>>(f);
    HIP_LAUNCHED();
    return SCLBM_OK;
}

namespace {

// Forward and backward pass, all gradients into the context; with adam->update also the Adam step.
sclbm_status backward(sclmlp_ctx *c, const float *dev_windows, const float *dev_targets, const int32_t *dev_index,
                      const int32_t *dev_sym, int64_t n, int64_t ndata, double *dev_loss, const AdamArgs &adam) {
    if (!c) return fail(SCLBM_EINVAL, "null context");
    if (n < 1 || n > c->max_batch) return fail(SCLBM_EINVAL, "n = %lld outside [1, %lld]", (long long)n,
                                              (long long)c->max_batch);
    if (ndata < 1 || ndata > INT32_MAX) return fail(SCLBM_EINVAL, "ndata must be in [1, 2^31)");
    if (!dev_index && ndata < n) return fail(SCLBM_EINVAL, "without an index ndata must be >= n");
    if (!dev_windows || !dev_targets) return fail(SCLBM_EINVAL, "null buffer");
    TRY(use_device(c));
    const int Mp = (int)padded_rows(n), nbo = Mp / OUT_ROWS;
    float *P = c->P();
    bf16 *x = c->at<bf16>(c->lay.x), *xt = c->at<bf16>(c->lay.xt);
    float *dy = c->at<float>(c->lay.dy);
    double *partial = c->at<double>(c->lay.partial);

    k_prep<<<Mp / PREP_ROWS, PREP_T, 0, c->stream>>>(dev_windows, dev_index, dev_sym, (int)n, (int)ndata, c->in_shift(),
                                                  c->in_scale(), x, xt, Mp, c->at<unsigned>(c->lay.bad));
    HIP_LAUNCHED();
    TRY((layer<NIN, false>(c, {x, c->wf(0), P + OFF_B1, nullptr, c->h(0), c->ht(0), Mp})));
    TRY((layer<NHID, false>(c, {c->h(0), c->wf(1), P + OFF_B2, nullptr, c->h(1), c->ht(1), Mp})));
    TRY((layer<NHID, false>(c, {c->h(1), c->wf(2), P + OFF_B3, nullptr, c->h(2), c->ht(2), Mp})));
    k_out<<<nbo, 256, 0, c->stream>>>(c->h(2), c->w4(), P + OFF_B4, (int)n, c->out_shift(), c->out_scale(), dev_targets,
                                      dev_index, dev_sym, (int)ndata, dy, partial, c->dz(0), c->dzt(2), Mp);
    HIP_LAUNCHED();
    // dZ2, then dZ1 (of which only the parameter gradients are taken)
    TRY((layer<NHID, true>(c, {c->dz(0), c->wtf(2), nullptr, c->ht(1), c->dz(1), c->dzt(1), Mp})));
    TRY((layer<NHID, true>(c, {c->dz(1), c->wtf(1), nullptr, c->ht(0), nullptr, c->dzt(0), Mp})));

    GradArgs g{};
    const bf16 *prev[3] = {xt, c->ht(0), c->ht(1)};
    for (int l = 0; l < 3; ++l) {
        g.dzT[l] = c->dzt(l);
        g.prevT[l] = prev[l];
    }
    g.hT3 = c->ht(2);
    g.dY = dy;
    g.partial = partial;
    g.npartial = nbo;
    g.n = (int)n;
    g.Mpad = Mp;
    g.loss = dev_loss ? dev_loss : c->at<double>(c->lay.loss);
    g.ad = adam;
    if (Mp <= kSmallBatch) {
        constexpr int tiles = (NHID / 64) * (NIN / 64 + 2 * (NHID / 64));
        g.slices = 1;
        g.per = Mp / 16;
        if (adam.update)
            k_grad<1, 1, true><<<tiles + GRAD_SUMS + 1, 256, 0, c->stream>>>(g);
        else
            k_grad<1, 1, false><<<tiles + GRAD_SUMS + 1, 256, 0, c->stream>>>(g);
        HIP_LAUNCHED();
        return SCLBM_OK;
    }
    constexpr int tiles = (NHID / 256) * (NIN / 64 + 2 * (NHID / 64));
    g.slices = grad_slices(Mp);
    g.per = (Mp / 16 + g.slices - 1) / g.slices;
    g.slices = (Mp / 16 + g.per - 1) / g.per;  // no empty slice
    g.part = c->at<float>(c->lay.part);
    k_grad<2, 2, false><<<tiles * g.slices + GRAD_SUMS + 1, 256, 0, c->stream>>>(g);
    HIP_LAUNCHED();
    if (adam.update) {
        AdamArgs a = adam;
        a.part = g.part;
        a.slices = g.slices;
        k_adam<<<ADAM_BLOCKS, 256, 0, c->stream>>>(a);
    } else {
        k_sum<<<(OFF_W4 / 4 + 255) / 256, 256, 0, c->stream>>>(g.part, g.slices, adam.g);
    }
    HIP_LAUNCHED();
    return SCLBM_OK;
}

// The next Adam step's arguments.
sclbm_status adam_next(const sclmlp_ctx *c, float lr, float beta1, float beta2, float eps, AdamArgs &a) {
    if (!c) return fail(SCLBM_EINVAL, "null context");
    if (!(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps > 0.0f))
        return fail(SCLBM_EINVAL, "Adam hyper-parameters out of range");
    const int64_t t = c->step + 1;
    a = adam_args(c);
    a.update = 1;
    a.lr = lr;
    a.beta1 = beta1;
    a.beta2 = beta2;
    a.eps = eps;
    a.bc1 = (float)(1.0 - std::pow((double)beta1, (double)t));
    a.bc2 = (float)(1.0 - std::pow((double)beta2, (double)t));
    return SCLBM_OK;
}

}  // namespace

sclbm_status sclmlp_gradients(sclmlp_ctx *c, const float *dev_windows, const float *dev_targets,
                              const int32_t *dev_index, const int32_t *dev_sym, int64_t n, int64_t ndata,
                              double *dev_loss) {
    if (!c) return fail(SCLBM_EINVAL, "null context");
    return backward(c, dev_windows, dev_targets, dev_index, dev_sym, n, ndata, dev_loss, adam_args(c));
}

sclbm_status sclmlp_adam(sclmlp_ctx *c, float lr, float beta1, float beta2, float eps) {
    AdamArgs a;
    TRY(adam_next(c, lr, beta1, beta2, eps, a));
    TRY(use_device(c));
    k_adam<<<ADAM_BLOCKS, 256, 0, c->stream>>>(a);
    HIP_LAUNCHED();
    c->step += 1;
    return SCLBM_OK;
}

sclbm_status sclmlp_train_step(sclmlp_ctx *c, const float *dev_windows, const float *dev_targets,
                               const int32_t *dev_index, const int32_t *dev_sym, int64_t n, int64_t ndata, float lr,
                               float beta1, float beta2, float eps, double *dev_loss) {
    AdamArgs a;
    TRY(adam_next(c, lr, beta1, beta2, eps, a));
    TRY(backward(c, dev_windows, dev_targets, dev_index, dev_sym, n, ndata, dev_loss, a));
    c->step += 1;
    return SCLBM_OK;
}

sclbm_status sclmlp_get_step(const sclmlp_ctx *c, int64_t *step) {
    if (!c || !step) return fail(SCLBM_EINVAL, "null argument");
    *step = c->step;
    return SCLBM_OK;
}

sclbm_status sclmlp_bad_rows(sclmlp_ctx *c, int64_t *count) {
    if (!c || !count) return fail(SCLBM_EINVAL, "null argument");
    TRY(use_device(c));
    unsigned v = 0;
    HIP_TRY(hipMemcpyAsync(&v, c->at<unsigned>(c->lay.bad), sizeof v, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    *count = v;
    return SCLBM_OK;
}

const char *sclmlp_last_error(void) { return g_err.c_str(); }

}  // extern "C"
