// C ABI of the learned sampling proposal (forward, training step, sampling).
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "mlp_internal.hpp"
#include "pump.h"

using namespace pump;

// Staging for pump_mlp_sample_noalloc (draws in host memory): the uniforms,
// the normals and the drawn states pass through this array instead of
// buffers allocated per call.  One copy per GPU, held until the process
// ends: kNoallocFloats floats (8 MiB).  Host code never names the array
// itself: its device address comes from hipGetSymbolAddress, once per device
// (noalloc_staging below), since the host-side symbol is only a stand-in.
constexpr size_t kNoallocFloats = (size_t)2 << 20;
static __device__ __align__(256) float scratch[kNoallocFloats];

struct pump_mlp {
    hipStream_t stream = nullptr;
    int device = 0;                 // the device current at create
    float* staging = nullptr;       // that device's address of `scratch`
    bool own_stream = false;
    int max_batch = 0, maxBp = 0;
    MlpDev d{};
    float* Y = nullptr;             // outputs [maxBp][kOutPad]
    float* loss_h = nullptr;        // pinned; the kernels write the mean loss here
    float *xbuf = nullptr, *zbuf = nullptr;
    int t = 0;
    std::string err;
};

namespace {

int mfail(pump_mlp* m, int code, const std::string& msg) {
    if (m) m->err = msg;
    return code;
}

#define MCHK(call)                                                                     \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess)                                                          \
            return mfail(m, PUMP_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

int round32(int b) { return (b + 31) / 32 * 32; }

// Y = MLP(cond rows X).
void forward(pump_mlp* m, const float* X, int B) {
    launch_mlp_forward(m->stream, m->d, X, B, m->Y, kOutPad, kOutPad, B);
}

// Do the arrays share memory?
bool overlap(const float* a, size_t na, const float* b, size_t nb) {
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa < pb + nb * sizeof(float) && pb < pa + na * sizeof(float);
}

// Device address of `scratch` on the current device, looked up on the first
// call per device and kept for the life of the process.
constexpr int kMaxDevices = 64;
std::mutex g_staging_mu;
float* g_staging[kMaxDevices] = {};

hipError_t noalloc_staging(int dev, float** out) {
    *out = nullptr;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_staging_mu);
    if (!g_staging[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_staging[dev] = static_cast<float*>(p);
    }
    *out = g_staging[dev];
    return hipSuccess;
}

const float* stage(pump_mlp* m, const float* src, float* buf, size_t n, int mem, hipError_t* e) {
    *e = hipSuccess;
    if (mem == PUMP_MEM_DEVICE) return src;
    *e = hipMemcpyAsync(buf, src, n * sizeof(float), hipMemcpyHostToDevice, m->stream);
    return buf;
}

}  // namespace

extern "C" {

int pump_mlp_create(int32_t max_batch, void* hip_stream, pump_mlp** out) {
    if (!out) return PUMP_E_ARG;
    *out = nullptr;
    if (max_batch < 1 || max_batch > (1 << 20)) return PUMP_E_ARG;
    pump_mlp* m = new pump_mlp();
    if (hip_stream) {
        m->stream = (hipStream_t)hip_stream;
    } else {
        if (hipStreamCreate(&m->stream) != hipSuccess) { delete m; return PUMP_E_HIP; }
        m->own_stream = true;
    }
    m->max_batch = max_batch;
    m->maxBp = round32(max_batch);
    // this device's staging address for pump_mlp_sample_noalloc (the
    // device current now is the one whose memory the context uses)
    if (hipGetDevice(&m->device) != hipSuccess ||
        noalloc_staging(m->device, &m->staging) != hipSuccess) {
        if (m->own_stream) (void)hipStreamDestroy(m->stream);
        delete m;
        return PUMP_E_HIP;
    }
    MlpDev& d = m->d;
    int off = 0;
    for (int l = 0; l < kLayers; ++l) {
        d.off_W[l] = off;
        off += mlp_out(l) * mlp_in(l);
        d.off_b[l] = off;
        off += mlp_out(l);
    }
    d.n_params = off;
    const size_t Bp = (size_t)m->maxBp;
    bool ok = true;
    auto A = [&](hipError_t e) { ok = ok && e == hipSuccess; };
    auto alloc = [&](auto** p, size_t n) { A(hipMalloc((void**)p, n * sizeof(**p))); };
    alloc(&d.params, (size_t)off);
    alloc(&d.m1, (size_t)off);
    alloc(&d.m2, (size_t)off);
    alloc(&d.grads, (size_t)off);
    for (int l = 0; l < kLayers; ++l) {
        alloc(&d.Wb[l], (size_t)mlp_out_p(l) * mlp_in_p(l));
        alloc(&d.WbT[l], (size_t)mlp_out_p(l) * mlp_in_p(l));
        alloc(&d.HT[l], Bp * mlp_in_p(l));
        alloc(&d.GT[l], Bp * mlp_out_p(l));
    }
    alloc(&d.bpart, (Bp / 16) * kBiasTotal);
    alloc(&d.lpart, Bp / 16);
    alloc(&m->Y, Bp * kOutPad);
    alloc(&m->xbuf, Bp * kIn);
    alloc(&m->zbuf, Bp * kDState);
    A(hipHostMalloc((void**)&m->loss_h, 16, hipHostMallocDefault));
    if (!ok) {
        pump_mlp_destroy(m);
        return PUMP_E_HIP;
    }
    *out = m;
    return PUMP_OK;
}

int pump_mlp_destroy(pump_mlp* m) {
    if (!m) return PUMP_OK;
    if (m->stream) (void)hipStreamSynchronize(m->stream);
    const MlpDev& d = m->d;
    void* ptrs[] = {d.params, d.m1, d.m2, d.grads, d.bpart, d.lpart, m->Y, m->xbuf, m->zbuf};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    for (int l = 0; l < kLayers; ++l) {
        void* q[] = {d.Wb[l], d.WbT[l], d.HT[l], d.GT[l]};
        for (void* p : q)
            if (p) (void)hipFree(p);
    }
    if (m->loss_h) (void)hipHostFree(m->loss_h);
    if (m->own_stream && m->stream) (void)hipStreamDestroy(m->stream);
    delete m;
    return PUMP_OK;
}

int pump_mlp_num_params(void) {
    int n = 0;
    for (int l = 0; l < kLayers; ++l) n += mlp_out(l) * mlp_in(l) + mlp_out(l);
    return n;
}

int pump_mlp_set_params(pump_mlp* m, const float* params, int64_t n) {
    if (!m || !params) return PUMP_E_ARG;
    if (n != m->d.n_params) return mfail(m, PUMP_E_ARG, "parameter count mismatch");
    MCHK(hipMemcpyAsync(m->d.params, params, (size_t)n * 4, hipMemcpyHostToDevice, m->stream));
    MCHK(hipMemsetAsync(m->d.m1, 0, (size_t)n * 4, m->stream));
    MCHK(hipMemsetAsync(m->d.m2, 0, (size_t)n * 4, m->stream));
    launch_refresh_bf16(m->stream, m->d);
    m->t = 0;
    MCHK(hipStreamSynchronize(m->stream));
    return PUMP_OK;
}

int pump_mlp_get_params(pump_mlp* m, float* params, int64_t n) {
    if (!m || !params) return PUMP_E_ARG;
    if (n != m->d.n_params) return mfail(m, PUMP_E_ARG, "parameter count mismatch");
    MCHK(hipMemcpyAsync(params, m->d.params, (size_t)n * 4, hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return PUMP_OK;
}

int pump_mlp_get_state(pump_mlp* m, float* params, float* m1, float* m2, int64_t n, int32_t* t) {
    if (!m || !params || !m1 || !m2 || !t) return PUMP_E_ARG;
    if (n != m->d.n_params) return mfail(m, PUMP_E_ARG, "parameter count mismatch");
    MCHK(hipMemcpyAsync(params, m->d.params, (size_t)n * 4, hipMemcpyDeviceToHost, m->stream));
    MCHK(hipMemcpyAsync(m1, m->d.m1, (size_t)n * 4, hipMemcpyDeviceToHost, m->stream));
    MCHK(hipMemcpyAsync(m2, m->d.m2, (size_t)n * 4, hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    *t = m->t;
    return PUMP_OK;
}

int pump_mlp_set_state(pump_mlp* m, const float* params, const float* m1, const float* m2,
                       int64_t n, int32_t t) {
    if (!m || !params || !m1 || !m2) return PUMP_E_ARG;
    if (n != m->d.n_params) return mfail(m, PUMP_E_ARG, "parameter count mismatch");
    if (t < 0) return mfail(m, PUMP_E_ARG, "negative step count");
    MCHK(hipMemcpyAsync(m->d.params, params, (size_t)n * 4, hipMemcpyHostToDevice, m->stream));
    MCHK(hipMemcpyAsync(m->d.m1, m1, (size_t)n * 4, hipMemcpyHostToDevice, m->stream));
    MCHK(hipMemcpyAsync(m->d.m2, m2, (size_t)n * 4, hipMemcpyHostToDevice, m->stream));
    launch_refresh_bf16(m->stream, m->d);
    m->t = t;
    MCHK(hipStreamSynchronize(m->stream));
    return PUMP_OK;
}

int pump_mlp_adam_step(pump_mlp* m, const float* grads, int64_t n, float lr, int32_t mem) {
    if (!m || !grads) return PUMP_E_ARG;
    if (n != m->d.n_params) return mfail(m, PUMP_E_ARG, "parameter count mismatch");
    if (!(lr > 0.0f)) return mfail(m, PUMP_E_ARG, "learning rate must be positive");
    if (mem == PUMP_MEM_DEVICE) {
        MCHK(hipMemcpyAsync(m->d.grads, grads, (size_t)n * 4, hipMemcpyDeviceToDevice, m->stream));
    } else {
        MCHK(hipMemcpyAsync(m->d.grads, grads, (size_t)n * 4, hipMemcpyHostToDevice, m->stream));
    }
    m->t += 1;
    launch_adam(m->stream, m->d, lr, m->t);
    MCHK(hipStreamSynchronize(m->stream));
    MCHK(hipGetLastError());
    return PUMP_OK;
}

int pump_mlp_forward(pump_mlp* m, const float* cond, int32_t B, float* out, int32_t mem) {
    if (!m || !cond || !out) return PUMP_E_ARG;
    if (B < 1 || B > m->max_batch) return mfail(m, PUMP_E_ARG, "batch out of range");
    hipError_t e;
    const float* X = stage(m, cond, m->xbuf, (size_t)B * kIn, mem, &e);
    MCHK(e);
    // Device rows are written where the caller wants them, unless that memory
    // holds condition rows, which other workgroups may still have to read; those
    // and host rows go through a packed copy.
    const bool direct = mem == PUMP_MEM_DEVICE && !overlap(X, (size_t)B * kIn, out, (size_t)B * kOut);
    launch_mlp_forward(m->stream, m->d, X, B, direct ? out : m->Y, kOut, kOut, B);
    if (!direct)
        MCHK(hipMemcpyAsync(out, m->Y, (size_t)B * kOut * 4,
                            mem == PUMP_MEM_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                            m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    MCHK(hipGetLastError());
    return PUMP_OK;
}

int pump_mlp_loss_grad(pump_mlp* m, const float* cond, const float* target, int32_t B,
                       float* loss, float* grads, int32_t mem) {
    if (!m || !cond || !target) return PUMP_E_ARG;
    if (B < 1 || B > m->max_batch) return mfail(m, PUMP_E_ARG, "batch out of range");
    hipError_t e;
    const float* X = stage(m, cond, m->xbuf, (size_t)B * kIn, mem, &e);
    MCHK(e);
    const float* Z = stage(m, target, m->zbuf, (size_t)B * kDState, mem, &e);
    MCHK(e);
    const int Bp = round32(B);
    launch_mlp_grad(m->stream, m->d, X, Z, B, Bp, m->loss_h);
    if (grads)
        MCHK(hipMemcpyAsync(grads, m->d.grads, (size_t)m->d.n_params * 4,
                            mem == PUMP_MEM_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                            m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    MCHK(hipGetLastError());
    if (loss) *loss = *m->loss_h;
    return PUMP_OK;
}

int pump_mlp_train_step(pump_mlp* m, const float* cond, const float* target, int32_t B, float lr,
                        float* loss, int32_t mem) {
    if (!m || !cond || !target) return PUMP_E_ARG;
    if (B < 1 || B > m->max_batch) return mfail(m, PUMP_E_ARG, "batch out of range");
    if (!(lr > 0.0f)) return mfail(m, PUMP_E_ARG, "learning rate must be positive");
    hipError_t e;
    const float* X = stage(m, cond, m->xbuf, (size_t)B * kIn, mem, &e);
    MCHK(e);
    const float* Z = stage(m, target, m->zbuf, (size_t)B * kDState, mem, &e);
    MCHK(e);
    const int Bp = round32(B);
    launch_mlp_grad(m->stream, m->d, X, Z, B, Bp, m->loss_h);
    m->t += 1;
    launch_adam(m->stream, m->d, lr, m->t);
    if (loss) {
        MCHK(hipStreamSynchronize(m->stream));
        *loss = *m->loss_h;
    }
    MCHK(hipGetLastError());
    return PUMP_OK;
}

int pump_mlp_condition(pump_mlp* m, const float* x_init, const float* goal, const float* boxes,
                       const int32_t* n_obs, int32_t q, int32_t max_boxes_in, float* cond) {
    if (!m || !x_init || !goal || !boxes || !n_obs || !cond) return PUMP_E_ARG;
    if (q < 1 || max_boxes_in < 1) return mfail(m, PUMP_E_ARG, "bad sizes");
    launch_condition(m->stream, x_init, goal, boxes, n_obs, q, max_boxes_in, cond);
    MCHK(hipStreamSynchronize(m->stream));
    MCHK(hipGetLastError());
    return PUMP_OK;
}

int pump_mlp_sample(pump_mlp* m, const float* cond, int32_t q, const float* u, const float* eps,
                    int32_t n, float* out, int32_t mem) {
    if (!m || !cond || !u || !eps || !out) return PUMP_E_ARG;
    if (q < 1 || q > m->max_batch || n < 1) return mfail(m, PUMP_E_ARG, "bad sizes");
    hipError_t e;
    const float* X = stage(m, cond, m->xbuf, (size_t)q * kIn, mem, &e);
    MCHK(e);
    forward(m, X, q);
    const float* U = u;
    const float* EPS = eps;
    float* O = out;
    float *du = nullptr, *de = nullptr, *dout = nullptr;
    if (mem != PUMP_MEM_DEVICE) {
        const size_t total = (size_t)q * n;
        MCHK(hipMalloc((void**)&du, total * 4));
        MCHK(hipMalloc((void**)&de, total * kDState * 4));
        MCHK(hipMalloc((void**)&dout, total * kDState * 4));
        MCHK(hipMemcpyAsync(du, u, total * 4, hipMemcpyHostToDevice, m->stream));
        MCHK(hipMemcpyAsync(de, eps, total * kDState * 4, hipMemcpyHostToDevice, m->stream));
        U = du;
        EPS = de;
        O = dout;
    }
    launch_sample(m->stream, m->Y, kOutPad, q, n, U, EPS, O);
    if (mem != PUMP_MEM_DEVICE) {
        const size_t total = (size_t)q * n;
        MCHK(hipMemcpyAsync(out, dout, total * kDState * 4, hipMemcpyDeviceToHost, m->stream));
    }
    MCHK(hipStreamSynchronize(m->stream));
    if (du) (void)hipFree(du);
    if (de) (void)hipFree(de);
    if (dout) (void)hipFree(dout);
    MCHK(hipGetLastError());
    return PUMP_OK;
}

int pump_mlp_sample_noalloc(pump_mlp* m, const float* cond, int32_t q, const float* u,
                            const float* eps, int32_t n, float* out, int32_t mem) {
    if (!m || !cond || !u || !eps || !out) return PUMP_E_ARG;
    if (q < 1 || q > m->max_batch || n < 1) return mfail(m, PUMP_E_ARG, "bad sizes");
    const size_t total = (size_t)q * (size_t)n;
    if (mem != PUMP_MEM_DEVICE && total * (1 + 2 * kDState) > kNoallocFloats)
        return mfail(m, PUMP_E_CAPACITY,
                     "q * n = " + std::to_string(total) + " draws exceed the no-alloc staging (" +
                         std::to_string(kNoallocFloats / (1 + 2 * kDState)) + " draws)");
    if (!m->staging) return mfail(m, PUMP_E_STATE, "no staging address for this device");
    hipError_t e;
    const float* X = stage(m, cond, m->xbuf, (size_t)q * kIn, mem, &e);
    MCHK(e);
    forward(m, X, q);
    const float* U = u;
    const float* EPS = eps;
    float* O = out;
    if (mem != PUMP_MEM_DEVICE) {
        // the uniforms, the normals and the draws in the staging array:
        // every word the kernel reads is copied in first, every word it
        // writes is copied out, so nothing needs clearing
        float* su = m->staging;
        float* se = su + total;
        float* so = se + total * kDState;
        MCHK(hipMemcpyAsync(su, u, total * 4, hipMemcpyHostToDevice, m->stream));
        MCHK(hipMemcpyAsync(se, eps, total * kDState * 4, hipMemcpyHostToDevice, m->stream));
        U = su;
        EPS = se;
        O = so;
    }
    launch_sample(m->stream, m->Y, kOutPad, q, n, U, EPS, O);
    if (mem != PUMP_MEM_DEVICE)
        MCHK(hipMemcpyAsync(out, O, total * kDState * 4, hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    MCHK(hipGetLastError());
    return PUMP_OK;
}

const char* pump_mlp_last_error(const pump_mlp* m) { return m ? m->err.c_str() : ""; }

}  // extern "C"
