// EvolveGCN's weight recurrence (Section "EvolveGCN") over all timesteps in one launch, and its adjoint:
//     a_t = W_{t-1} (U_x + U_h) + b,   (W_t, C_t) = LSTM cell(a_t, C_{t-1}),   t = 1 .. T,  C_0 = 0
// (the weight matrix is the LSTM's input and its hidden state at once, so the two products share their left operand).
//
// The matrices are F x F', a few kilobytes: launched step by step through the dense transform and the cell kernel the chain
// of launches was all the time there was (8 steps of 32 x 32, forward and back: 112 launches, 560 us of kernels).  A row of W_t
// depends on the same row of W_{t-1} only, so a wavefront takes a row through all steps by itself: lane l holds columns l
// (and l + 64) of U in registers, the row's elements are broadcast through scalar registers, the four gates of an element meet
// by lane shuffles, and no step waits for any other wavefront (about 0.5 us per step forward, 1.2 us back).  Gradients of U and b
// are sums over rows: every wavefront leaves its part, a second kernel adds them in row order.
#include <algorithm>

#include "common.hpp"

namespace {

using namespace dgnn;

constexpr int kStepsPerLaunch = 64;      // addresses of upstream gradients that travel in the kernel arguments
struct Upstream { const float *dw[kStepsPerLaunch]; };

// Gate pre-activations of one row: lane l holds columns l and, with F2 = 32, l + 64.  F2 = 16: one column per lane.
template <int F2>
struct Row {
    static constexpr int kCols = 4 * F2 / kWave;                 // columns per lane
    float u[kCols][F2], b[kCols];

    __device__ __forceinline__ void load(const float *__restrict__ u_x, const float *__restrict__ u_h, const float *__restrict__ bias, int lane) {
#pragma unroll
        for (int q = 0; q < kCols; ++q) {
#pragma unroll
            for (int k = 0; k < F2; ++k) u[q][k] = u_x[k * 4 * F2 + q * kWave + lane] + u_h[k * 4 * F2 + q * kWave + lane];
            b[q] = bias ? bias[q * kWave + lane] : 0.0f;
        }
    }
    // w: element k of the row in lane k.  Gates (input, forget, cell, output) of element k come out in lane k < F2.
    __device__ __forceinline__ void gates(float w, int lane, float (&a)[4]) const {
        float acc[kCols];
#pragma unroll
        for (int q = 0; q < kCols; ++q) acc[q] = b[q];
#pragma unroll
        for (int k = 0; k < F2; ++k) {
            const float s = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), k));
#pragma unroll
            for (int q = 0; q < kCols; ++q) acc[q] = fmaf(s, u[q][k], acc[q]);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) a[g] = __shfl(acc[g * F2 / kWave], (g * F2) % kWave + (lane % F2), kWave);
    }
    // The other way: gradients of the four gates of element k in lane k < F2 -> per column.
    __device__ __forceinline__ void columns(const float (&d)[4], int lane, float (&c)[kCols]) const {
#pragma unroll
        for (int q = 0; q < kCols; ++q) {
            c[q] = 0.0f;
#pragma unroll
            for (int g = q * kWave / F2; g < (q + 1) * kWave / F2; ++g) {
                const float v = __shfl(d[g], lane % F2, kWave);
                if ((q * kWave + lane) / F2 == g) c[q] = v;
            }
        }
    }
};

template <int F2>
__global__ __launch_bounds__(kWave) void evolve_kernel(const float *__restrict__ w0, const float *__restrict__ u_x, const float *__restrict__ u_h,
                                                       const float *__restrict__ bias, int T, int f, float *__restrict__ w, float *__restrict__ c) {
    const int row = blockIdx.x, lane = threadIdx.x, k = lane % F2;
    Row<F2> r;
    r.load(u_x, u_h, bias, lane);
    const int at = row * F2 + k;
    const int64_t frame = (int64_t)f * F2;
    float wv = w0[at], cv = 0.0f;
    if (lane < F2) c[at] = 0.0f;
    for (int t = 0; t < T; ++t) {
        float a[4];
        r.gates(wv, lane, a);
        cv = sigmoidf(a[1]) * cv + sigmoidf(a[0]) * tanhf(a[2]);
        wv = sigmoidf(a[3]) * tanhf(cv);
        if (lane < F2) {
            w[t * frame + at] = wv;
            c[(t + 1) * frame + at] = cv;
        }
    }
}

// Steps t_hi-1 .. t_lo of the walk back; carry: dL/dW_{t_lo} and dL/dC_{t_lo} of the row go on in `state` ([2][f][F2]), read
// unless `first`; partial [f][F2 + 1][4 F2]: the row's part of dL/dU and, behind it, of dL/db, added to unless `first`.
template <int F2>
__global__ __launch_bounds__(kWave) void evolve_backward_kernel(const float *__restrict__ w0, const float *__restrict__ u_x,
                                                                const float *__restrict__ u_h, const float *__restrict__ bias, int f, int t_lo,
                                                                int t_hi, const float *__restrict__ w, const float *__restrict__ c, Upstream up,
                                                                float *__restrict__ state, float *__restrict__ partial, int first) {
    constexpr int kCols = Row<F2>::kCols;
    constexpr int G4 = 4 * F2;
    constexpr int kParts = kWave / F2, kPer = G4 / kParts;        // lanes k, k + F2, ... share the columns of row k of U
    const int row = blockIdx.x, lane = threadIdx.x, k = lane % F2, part = lane / F2;
    Row<F2> r;
    r.load(u_x, u_h, bias, lane);
    float ut[kPer];                                               // U[k][part * kPer + j]
#pragma unroll
    for (int j = 0; j < kPer; ++j) ut[j] = u_x[k * G4 + part * kPer + j] + u_h[k * G4 + part * kPer + j];
    const int at = row * F2 + k;
    const int64_t frame = (int64_t)f * F2;
    float *mine = partial + (int64_t)row * (F2 + 1) * G4;
    float du[kCols][F2], db[kCols], dh = 0.0f, dc = 0.0f;
#pragma unroll
    for (int q = 0; q < kCols; ++q) {
        db[q] = first ? 0.0f : mine[F2 * G4 + q * kWave + lane];
#pragma unroll
        for (int j = 0; j < F2; ++j) du[q][j] = first ? 0.0f : mine[j * G4 + q * kWave + lane];
    }
    if (!first) { dh = state[at]; dc = state[frame + at]; }
    for (int t = t_hi - 1; t >= t_lo; --t) {
        const float wp = t == 0 ? w0[at] : w[(t - 1) * frame + at], cp = c[t * frame + at];
        dh += as_global(up.dw[t - t_lo])[at];
        float a[4], d[4];
        r.gates(wp, lane, a);
        const float i = sigmoidf(a[0]), fg = sigmoidf(a[1]), g = tanhf(a[2]), o = sigmoidf(a[3]);
        const float tc = tanhf(fg * cp + i * g);
        const float e = dh * o * (1.0f - tc * tc) + dc;
        d[0] = e * g * i * (1.0f - i);
        d[1] = e * cp * fg * (1.0f - fg);
        d[2] = e * i * (1.0f - g * g);
        d[3] = dh * tc * o * (1.0f - o);
        dc = e * fg;
        float col[kCols];
        r.columns(d, lane, col);
#pragma unroll
        for (int q = 0; q < kCols; ++q) db[q] += col[q];
        // dL/dU += (row of W_{t-1})^T da
#pragma unroll
        for (int j = 0; j < F2; ++j) {
            const float s = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wp), j));
#pragma unroll
            for (int q = 0; q < kCols; ++q) du[q][j] = fmaf(s, col[q], du[q][j]);
        }
        // dL/dW_{t-1} = da U^T: the lanes of element k take kPer columns each
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            float v = 0.0f;
#pragma unroll
            for (int p = 0; p < kParts; ++p) {
                const int cc = p * kPer + j;
                const float s = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(col[cc / kWave]), cc % kWave));
                v = part == p ? s : v;
            }
            acc = fmaf(v, ut[j], acc);
        }
#pragma unroll
        for (int x = F2; x < kWave; x <<= 1) acc += __shfl_xor(acc, x, kWave);
        dh = acc;
    }
    if (lane < F2) { state[at] = dh; state[frame + at] = dc; }
#pragma unroll
    for (int q = 0; q < kCols; ++q) {
        mine[F2 * G4 + q * kWave + lane] = db[q];
#pragma unroll
        for (int j = 0; j < F2; ++j) mine[j * G4 + q * kWave + lane] = du[q][j];
    }
}

// The rows' parts in row order; W_{t-1} feeds both products, so U_x and U_h have the same gradient.
__global__ __launch_bounds__(256) void evolve_reduce_kernel(const float *__restrict__ partial, int f, int elems, int u_elems, const float *__restrict__ dh,
                                                            float *__restrict__ du_x, float *__restrict__ du_h, float *__restrict__ db,
                                                            float *__restrict__ dw0, int w_elems) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < elems) {
        float s = 0.0f;
#pragma unroll 16
        for (int r = 0; r < f; ++r) s += partial[(int64_t)r * elems + e];
        if (e < u_elems) { du_x[e] = s; du_h[e] = s; } else db[e - u_elems] = s;
    }
    if (e < w_elems) dw0[e] = dh[e];
}

}  // namespace

extern "C" int dgnn_evolve_weights(const float *w0, const float *u_x, const float *u_h, const float *bias, int32_t T, int32_t f, int32_t f2,
                                   float *w, float *c, void *stream) {
    if (!w0 || !u_x || !u_h || !w || !c) return DGNN_ERR_NULL;
    if (T <= 0 || !supported_width(f) || (f2 != 16 && f2 != 32)) return DGNN_ERR_SHAPE;
    if (w == w0 || w == c) return DGNN_ERR_ALIAS;
    hipStream_t s = (hipStream_t)stream;
    if (f2 == 16) hipLaunchKernelGGL(evolve_kernel<16>, dim3((unsigned)f), dim3(kWave), 0, s, w0, u_x, u_h, bias, T, f, w, c);
    else hipLaunchKernelGGL(evolve_kernel<32>, dim3((unsigned)f), dim3(kWave), 0, s, w0, u_x, u_h, bias, T, f, w, c);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

extern "C" int dgnn_evolve_weights_backward_workspace(int32_t f, int32_t f2, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (!supported_width(f) || (f2 != 16 && f2 != 32)) return DGNN_ERR_SHAPE;
    *bytes = ((size_t)f * (f2 + 1) * 4 * f2 + 2 * (size_t)f * f2) * sizeof(float);
    return DGNN_OK;
}

extern "C" int dgnn_evolve_weights_backward(const float *w0, const float *u_x, const float *u_h, const float *bias, int32_t T, int32_t f, int32_t f2,
                                            const float *w, const float *c, const float *const *dw, float *dw0, float *du_x, float *du_h,
                                            float *db, void *ws, size_t ws_bytes, void *stream) {
    if (!w0 || !u_x || !u_h || !w || !c || !dw || !dw0 || !du_x || !du_h || !db || !ws) return DGNN_ERR_NULL;
    if (T <= 0 || !supported_width(f) || (f2 != 16 && f2 != 32)) return DGNN_ERR_SHAPE;
    for (int t = 0; t < T; ++t)
        if (!dw[t]) return DGNN_ERR_NULL;
    size_t need = 0;
    dgnn_evolve_weights_backward_workspace(f, f2, &need);
    if (ws_bytes < need) return DGNN_ERR_CAPACITY;
    hipStream_t s = (hipStream_t)stream;
    float *partial = static_cast<float *>(ws), *state = partial + (size_t)f * (f2 + 1) * 4 * f2;
    for (int hi = T; hi > 0; hi -= kStepsPerLaunch) {
        const int lo = std::max(0, hi - kStepsPerLaunch);
        Upstream up;
        for (int t = lo; t < hi; ++t) up.dw[t - lo] = dw[t];
        if (f2 == 16)
            hipLaunchKernelGGL(evolve_backward_kernel<16>, dim3((unsigned)f), dim3(kWave), 0, s, w0, u_x, u_h, bias, f, lo, hi, w, c, up, state, partial, hi == T);
        else
            hipLaunchKernelGGL(evolve_backward_kernel<32>, dim3((unsigned)f), dim3(kWave), 0, s, w0, u_x, u_h, bias, f, lo, hi, w, c, up, state, partial, hi == T);
        DGNN_RETURN_IF_LAUNCH_FAILED();
    }
    const int elems = (f2 + 1) * 4 * f2, w_elems = f * f2;
    hipLaunchKernelGGL(evolve_reduce_kernel, dim3((unsigned)((std::max(elems, w_elems) + 255) / 256)), dim3(256), 0, s, partial, f, elems, f2 * 4 * f2, state, du_x,
                       du_h, db, dw0, w_elems);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}
