// Open-loop actuation controller (App. "MPC controller architecture"; Sec. 5.3):
// N phase-shifted sinusoids of the simulation time -> one bias-free fully
// connected layer -> tanh, one actuation per output element per step.
//
//   s_k(t)    = sin(omega (t0 + t) dt + 2 pi k / N)
//   act[t][e] = scale tanh(sum_k W[k][e] s_k(t))
//
// The N signals share one frequency and differ only in phase, so
//   sum_k W[k][e] s_k(t) = A_e sin(omega tau) + B_e cos(omega tau),
//   A_e = sum_k W[k][e] cos(2 pi k / N),   B_e = sum_k W[k][e] sin(2 pi k / N)
// (sin(x + p) = sin x cos p + cos x sin p): each thread forms its element's A, B
// once and then spends two FMAs per step on the layer.  The backward accumulates
// the two sums  sum_t zbar_t sin(omega tau_t)  and  sum_t zbar_t cos(omega tau_t)
// and maps them back to the N weights with the same phase table.
//
// Both kernels stream: WAVES wavefronts share 64 output elements, each walking every
// WAVES-th batch of steps, so every row access of act / act_grad is one coalesced 256 B
// (FP32) wavefront access; the (sin, cos) table of a chunk of steps is computed once per
// workgroup (FP64, rounded to the dtype) into LDS and read as broadcasts.  The backward
// issues the loads of a batch of steps before using any of them, so each wave keeps
// several HBM reads in flight.  Forward: reads W once, writes n_steps rows.  Backward:
// recomputes the layer from W (cheaper than re-reading act), reads n_steps rows of
// act_grad, and adds its N sums per element to W_grad (the wavefronts' sums in order).
//
// WAVES = 1 with four element groups per workgroup for large layers, where one thread per
// element fills the card and the weights are read once; 8 for small ones, which are
// bound by one thread's chain: the FP64 sines (phases and steps side by side, the weights
// on their way meanwhile), then a tanh per step.
#include <hip/hip_runtime.h>

#include <cmath>

#include "gsim.h"
#include "gsim_host.h"

namespace {

constexpr int CTRL_CHUNK = 128;  // steps per LDS table
constexpr int CTRL_BATCH = 8;    // steps a wavefront takes at a time
constexpr int CTRL_SPLIT = 8;    // wavefronts per 64 elements of a small layer
constexpr int MAXN = GSIM_CTRL_MAX_SIGNALS;

struct CtrlArgs {
    int n_signals;
    double omega, dt, scale;
    int64_t n, t0, n_steps;
};

template <typename T>
struct SC {
    T s, c;
};

// Threads of a workgroup: one group of 64 elements with WAVES wavefronts, or four groups.
template <int WAVES>
constexpr int ctrl_block() {
    return WAVES == 1 ? 256 : 64 * WAVES;
}

// (sin, cos) of omega tau for steps tc .. tc + CTRL_CHUNK - 1 of the call.
template <typename T>
__device__ __forceinline__ void ctrl_table(const CtrlArgs& a, int64_t tc, SC<T>* tab, int from) {
    for (int t = (int)threadIdx.x - from; t < CTRL_CHUNK && tc + t < a.n_steps; t += blockDim.x - from) {
        if (t < 0) continue;
        const double x = a.omega * ((double)(a.t0 + tc + t) * a.dt);
        tab[t].s = (T)sin(x);
        tab[t].c = (T)cos(x);
    }
}

// The phase table cos / sin(2 pi k / N) (FP64 rounded to T) and the first chunk's step
// table into LDS, then this thread's A, B from its weights.  Contains a barrier: every
// thread calls it.
template <typename T>
__device__ __forceinline__ void ctrl_coeffs(const CtrlArgs& a, const T* __restrict__ W, int64_t e, bool live,
                                            SC<T>* tab, T* cp, T* sp, T& A, T& B) {
    const double two_pi = 6.283185307179586476925287;
    T w[MAXN];
#pragma unroll
    for (int k = 0; k < MAXN; ++k) w[k] = live && k < a.n_signals ? W[(int64_t)k * a.n + e] : T(0);
    if (threadIdx.x < 64) {
        if ((int)threadIdx.x < a.n_signals) {
            const double p = two_pi * (double)threadIdx.x / (double)a.n_signals;
            cp[threadIdx.x] = (T)cos(p);
            sp[threadIdx.x] = (T)sin(p);
        }
    } else {
        ctrl_table<T>(a, 0, tab, 64);
    }
    __syncthreads();
    A = T(0);
    B = T(0);
#pragma unroll
    for (int k = 0; k < MAXN; ++k)
        if (k < a.n_signals) {
            A = fma(w[k], cp[k], A);
            B = fma(w[k], sp[k], B);
        }
}

// tanh of the layer at a step's (sin, cos).
template <typename T>
__device__ __forceinline__ T ctrl_layer(T A, T B, SC<T> q) {
    return tanh(fma(A, q.s, B * q.c));
}

template <typename T, int WAVES>
__global__ __launch_bounds__(ctrl_block<WAVES>()) void k_ctrl_fwd(CtrlArgs a, const T* __restrict__ W,
                                                                  T* __restrict__ act) {
    __shared__ SC<T> tab[CTRL_CHUNK];
    __shared__ T cp[MAXN], sp[MAXN];
    const int wave = WAVES == 1 ? 0 : (int)threadIdx.x >> 6;
    const int64_t e = WAVES == 1 ? (int64_t)blockIdx.x * 256 + threadIdx.x : (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const bool live = e < a.n;
    const T scale = (T)a.scale;
    T A, B;
    ctrl_coeffs<T>(a, W, e, live, tab, cp, sp, A, B);
    for (int64_t tc = 0; tc < a.n_steps; tc += CTRL_CHUNK) {
        if (tc > 0) {
            __syncthreads();  // the previous chunk's table is no longer read
            ctrl_table<T>(a, tc, tab, 0);
            __syncthreads();
        }
        const int nt = (int)(a.n_steps - tc < CTRL_CHUNK ? a.n_steps - tc : CTRL_CHUNK);
        if (live)
            for (int t = wave; t < nt; t += WAVES) act[(tc + t) * a.n + e] = scale * ctrl_layer(A, B, tab[t]);
    }
}

template <typename T, int WAVES>
__global__ __launch_bounds__(ctrl_block<WAVES>()) void k_ctrl_bwd(CtrlArgs a, const T* __restrict__ W,
                                                                  const T* __restrict__ g, T* __restrict__ gW) {
    __shared__ SC<T> tab[CTRL_CHUNK];
    __shared__ T cp[MAXN], sp[MAXN];
    __shared__ T sum[2][WAVES == 1 ? 1 : 64 * WAVES];
    const int wave = WAVES == 1 ? 0 : (int)threadIdx.x >> 6;
    const int64_t e = WAVES == 1 ? (int64_t)blockIdx.x * 256 + threadIdx.x : (int64_t)blockIdx.x * 64 + (threadIdx.x & 63);
    const bool live = e < a.n;
    const T scale = (T)a.scale;
    T A, B;
    ctrl_coeffs<T>(a, W, e, live, tab, cp, sp, A, B);
    T gA = T(0), gB = T(0);
    for (int64_t tc = 0; tc < a.n_steps; tc += CTRL_CHUNK) {
        if (tc > 0) {
            __syncthreads();
            ctrl_table<T>(a, tc, tab, 0);
            __syncthreads();
        }
        const int nt = (int)(a.n_steps - tc < CTRL_CHUNK ? a.n_steps - tc : CTRL_CHUNK);
        if (live)
            for (int t0 = wave * CTRL_BATCH; t0 < nt; t0 += WAVES * CTRL_BATCH) {
                T gv[CTRL_BATCH];
#pragma unroll
                for (int j = 0; j < CTRL_BATCH; ++j)
                    gv[j] = t0 + j < nt ? g[(tc + t0 + j) * a.n + e] : T(0);
#pragma unroll
                for (int j = 0; j < CTRL_BATCH; ++j)
                    if (t0 + j < nt) {
                        const SC<T> q = tab[t0 + j];
                        const T y = ctrl_layer(A, B, q);
                        const T dz = gv[j] * scale * (T(1) - y * y);
                        gA += dz * q.s;
                        gB += dz * q.c;
                    }
            }
    }
    if constexpr (WAVES > 1) {  // the wavefronts' sums, in order
        sum[0][threadIdx.x] = gA;
        sum[1][threadIdx.x] = gB;
        __syncthreads();
        const int l = threadIdx.x & 63;
        gA = sum[0][l];
        gB = sum[1][l];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            gA += sum[0][64 * w + l];
            gB += sum[1][64 * w + l];
        }
    }
    if (live)  // the signals are shared over the wavefronts
#pragma unroll
        for (int k = 0; k < MAXN; ++k)
            if (k % WAVES == wave && k < a.n_signals) gW[(int64_t)k * a.n + e] += gA * cp[k] + gB * sp[k];
}

int check_ctrl(int dtype, const gsim_controller* c, int64_t n, int64_t t0, int64_t n_steps, CtrlArgs& a) {
    if (dtype != GSIM_F32 && dtype != GSIM_F64) return gsim::fail(GSIM_E_INVALID, "dtype must be GSIM_F32 or GSIM_F64");
    if (!c) return gsim::fail(GSIM_E_INVALID, "NULL controller");
    if (c->n_signals < 1 || c->n_signals > MAXN)
        return gsim::fail(GSIM_E_INVALID, "n_signals must be in [1, %d]", MAXN);
    if (n < 0 || t0 < 0 || n_steps < 0) return gsim::fail(GSIM_E_INVALID, "n, t0 and n_steps must be >= 0");
    if (!std::isfinite(c->omega) || !std::isfinite(c->dt) || !std::isfinite(c->scale))
        return gsim::fail(GSIM_E_INVALID, "omega, dt and scale must be finite");
    a.n_signals = c->n_signals;
    a.omega = c->omega;
    a.dt = c->dt;
    a.scale = c->scale;
    a.n = n;
    a.t0 = t0;
    a.n_steps = n_steps;
    return GSIM_OK;
}

// CTRL_SPLIT wavefronts per 64 elements, or one.  Up to 16384 elements (one group of 64 per
// compute unit) the split is never slower.  Each further such share puts another workgroup
// on every compute unit, whose wavefronts compete, while a call of few steps leaves most of
// the eight without one (they take the steps, backward eight at a time): so the split needs
// more steps the more shares, and no number of steps makes up for a fourth share in FP64 or
// a fifth in FP32.  Measured (8 signals, one / eight wavefronts, us): float32, 600 elements, 60
// steps forward 11.1 / 4.4, backward 13.8 / 5.7; 32000, 60 steps 12.7 / 6.4, 13.1 / 7.0, 1 step
// 3.5 / 4.1, 5.0 / 5.3; 48000, 8 steps 4.5 / 4.9, 5.7 / 8.9, 32 steps 8.4 / 6.3, 9.1 / 9.1; 65000, 60
// steps 13.5 / 9.9, 14.6 / 12.4, 24 steps 7.4 / 7.3, 9.1 / 11.2; 200000, 60 steps 19.4 / 23.3, 22.5 /
// 35.7.  float64, 32000, 24 steps 12.6 / 9.3, 14.7 / 13.3, 12 steps 8.3 / 6.9, 10.2 / 13.2; 48000, 60
// steps 27.2 / 23.1, 31.0 / 27.7, 24 steps 13.1 / 12.7, 14.8 / 19.1; 65000, 60 steps 28.4 / 30.0,
// 32.0 / 37.8, 300 steps 113 / 109, 131 / 130.
template <typename T>
bool ctrl_split(int64_t n, int64_t steps, bool backward) {
    const bool f32 = sizeof(T) == 4;
    const int64_t more = (n - 1) / 16384;  // shares beyond the first
    return more < (f32 ? 4 : 3) && steps >= more * (f32 ? (backward ? 16 : 8) : (backward ? 32 : 12));
}
#define CTRL_LAUNCH(K, T, BACKWARD, ...)                                                                          \
    do {                                                                                                          \
        if (ctrl_split<T>(n, n_steps, BACKWARD))                                                                  \
            hipLaunchKernelGGL((K<T, CTRL_SPLIT>), dim3((unsigned)((n + 63) / 64)), dim3(64 * CTRL_SPLIT), 0,      \
                               (hipStream_t)stream, a, __VA_ARGS__);                                              \
        else                                                                                                      \
            hipLaunchKernelGGL((K<T, 1>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, a, \
                               __VA_ARGS__);                                                                      \
    } while (0)

int launched(const char* what) {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GSIM_OK : gsim::hip_fail(e, what);
}

}  // namespace

extern "C" {

int gsim_controller_forward(int dtype, const gsim_controller* ctrl, const void* W, int64_t n, int64_t t0,
                            int64_t n_steps, void* act, void* stream) {
    CtrlArgs a;
    int rc = check_ctrl(dtype, ctrl, n, t0, n_steps, a);
    if (rc) return rc;
    if (n == 0 || n_steps == 0) return GSIM_OK;
    if (!W || !act) return gsim::fail(GSIM_E_INVALID, "NULL W or act");
    if (dtype == GSIM_F32) CTRL_LAUNCH(k_ctrl_fwd, float, false, (const float*)W, (float*)act);
    else CTRL_LAUNCH(k_ctrl_fwd, double, false, (const double*)W, (double*)act);
    return launched("controller forward launch");
}

int gsim_controller_backward(int dtype, const gsim_controller* ctrl, const void* W, const void* act_grad, int64_t n,
                             int64_t t0, int64_t n_steps, void* W_grad, void* stream) {
    CtrlArgs a;
    int rc = check_ctrl(dtype, ctrl, n, t0, n_steps, a);
    if (rc) return rc;
    if (n == 0 || n_steps == 0) return GSIM_OK;
    if (!W || !act_grad || !W_grad) return gsim::fail(GSIM_E_INVALID, "NULL W, act_grad or W_grad");
    if (dtype == GSIM_F32) CTRL_LAUNCH(k_ctrl_bwd, float, true, (const float*)W, (const float*)act_grad, (float*)W_grad);
    else CTRL_LAUNCH(k_ctrl_bwd, double, true, (const double*)W, (const double*)act_grad, (double*)W_grad);
    return launched("controller backward launch");
}

}  // extern "C"
