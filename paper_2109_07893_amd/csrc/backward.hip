// Gradient propagation through the GCN operation of Eqn (2) (Section "Gradient Checkpoint": after a block
// has been run forward again, gradients travel through it in the reverse direction).  With
//     H = X W,   P = A~ H,   Z = max(P, 0)
// and G_Z = dL/dZ arriving from the layer above (or from the adjoint of the M-transform):
//     G_P = G_Z where Z > 0, else 0              relu_backward_kernel (can fold a row scale in)
//     G_H = A~^T G_P                              the aggregation kernel on the transposed snapshot
//     dW  = X^T G_H                               wgrad_kernel + wgrad_reduce_kernel   (this file)
//         = (A~ X)^T G_P                          the same, with the mask folded in: no aggregation going back
//     dX  = G_H W^T                               the X W kernels with W read transposed
//
// dW = X^T G_H contracts over the N rows, so it reads both matrices once (HBM-bound, 2 s N F bytes) and
// leaves an F x F' result.  The rows are dealt out in steps of 16 to "row workers"; a worker keeps its
// part of the F x F' accumulator in MFMA registers for its whole share of the rows.  In a 32x32xK MFMA
// lane (i, h) supplies A[i][k-slice h] and B[k-slice h][i]; with A = X^T and B = G_H both operands of a
// lane are elements of column i of a 32-column tile, taken from the rows of the k-slice, which are plain
// strided loads (whole 128-byte or 64-byte runs per row across the lanes), no transposition needed.
// The workers of a workgroup add up their results in LDS, pair by pair, so that one partial result per workgroup goes to the workspace;
// a second kernel adds these up, all in a fixed order: the result repeats bit for bit (no floating-point atomics).  With one
// partial result per worker, 2048 or 512 of them, they were as many bytes as a frame: us per call (both kernels), 60 K x 128 bf16
// 21.6 -> 17.7, 16 x 50 K x 64 fp32 131 -> 119, 4 x 2^20 x 32 fp32 masked 283 -> 280.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace {

using namespace dgnn;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// One gradient of a launch; blockIdx.y says which.  z (may be null): only rows' elements with z > 0 let g through.
struct Item {
    const void *x, *g, *z;
    float *dw;
};
constexpr int kMaxBatch = 32;
struct Batch { Item item[kMaxBatch]; };

constexpr int kThreads = 256;        // of the elementwise kernel
constexpr int kWavesPerBlock = 8;    // of the weight gradient: a partial result for eight wavefronts
constexpr int kStepRows = 16;        // rows per step: eight fp32 MFMAs of depth 2, or one bf16 MFMA of depth 16
constexpr int kMaxBlocks = 512;      // bounds the workspace; two workgroups per compute unit, where registers allow them

// How the 32x32 tiles of the F x F' accumulator are shared out inside a workgroup: a wavefront holds
// TI x TJ tiles (at most four), GROUPS wavefronts cover all tiles, and the remaining factor of the eight
// wavefronts splits the rows (RS row workers per workgroup).
template <int FIN, int FOUT>
struct Split {
    static constexpr int NI = (FIN + 31) / 32, NJ = (FOUT + 31) / 32;
    static constexpr int TILES = NI * NJ;
    static constexpr int TPW = TILES < 4 ? TILES : 4;
    static constexpr int TI = (NI >= 2 && NJ >= 2) ? 2 : (NI < TPW ? NI : TPW);
    static constexpr int TJ = TPW / TI;
    static constexpr int GI = NI / TI, GJ = NJ / TJ;
    static constexpr int GROUPS = GI * GJ;
    static constexpr int RS = kWavesPerBlock / GROUPS;
    static_assert(TI * TJ == TPW && GI * TI == NI && GJ * TJ == NJ && RS * GROUPS == kWavesPerBlock, "tile split");
};

// MASKED: G is taken where Z > 0 only (the gradient through the ReLU, which then needs no pass of its own).
// The gradient is the sum over `items` items from the first one on, n rows each, whose steps are one line: worker `me` takes steps
// me, me + workers, ... of it.  LINE: there are several; the worker then adds up its steps of each item on their own, as a call per
// item does (one sum over all of its steps: 12 x 60 K x 128 bf16 1.4e-7 -> 2.4e-7 away from 64 bits while partial results met in fp32).
template <int FIN, int FOUT, bool BF16, bool MASKED, bool LINE>
__device__ __forceinline__ void wgrad(const Item *__restrict__ first, int items, int64_t n, int64_t n_steps, float *__restrict__ partial) {
    using S = Split<FIN, FOUT>;
    typedef typename std::conditional<BF16, uint16_t, float>::type Elem;
    typedef typename std::conditional<BF16, uint32_t, float>::type Raw;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int i = lane & 31, hh = lane >> 5;
    const int group = wave % S::GROUPS, rs = wave / S::GROUPS;
    const Elem *x = static_cast<const Elem *>(as_global(first->x));
    const Elem *g = static_cast<const Elem *>(as_global(first->g));
    const Elem *z = static_cast<const Elem *>(as_global(first->z));
    int item = 0;
    auto open_item = [&] {
        x = static_cast<const Elem *>(as_global(first[item].x));
        g = static_cast<const Elem *>(as_global(first[item].g));
        z = static_cast<const Elem *>(as_global(first[item].z));
    };
    const int it0 = (group / S::GJ) * S::TI, jt0 = (group % S::GJ) * S::TJ;
    const int64_t workers = (int64_t)gridDim.x * S::RS;
    const int64_t me = (int64_t)blockIdx.x * S::RS + rs;

    floatx16 acc[S::TI][S::TJ];
#pragma unroll
    for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
        for (int tj = 0; tj < S::TJ; ++tj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ti][tj][v] = 0.0f;
    floatx16 behind[LINE ? S::TI : 1][LINE ? S::TJ : 1];       // the items behind the worker
    auto close_item = [&] {
        if constexpr (LINE) {
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
                for (int tj = 0; tj < S::TJ; ++tj)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        behind[ti][tj][v] += acc[ti][tj][v];
                        acc[ti][tj][v] = 0.0f;
                    }
        }
    };
    if constexpr (LINE) {
#pragma unroll
        for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
            for (int tj = 0; tj < S::TJ; ++tj)
#pragma unroll
                for (int v = 0; v < 16; ++v) behind[ti][tj][v] = 0.0f;
    }

    // Row of the k-slice element e of this lane inside a step: depth-2 MFMAs take rows (2 e + h), the
    // depth-16 MFMA takes rows (8 h + e).
    auto row_of = [&](int64_t step, int e) { return step * kStepRows + (BF16 ? 8 * hh + e : 2 * e + hh); };
    // Loads are unconditional (addresses clamped into the matrices); what lies outside is zeroed when used.
    Raw xa_next[S::TI][8], gb_next[S::TJ][8], zb_next[MASKED ? S::TJ : 1][8];
    auto fetch = [&](int64_t step) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t row = std::min<int64_t>(row_of(step, e), n - 1);
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti) xa_next[ti][e] = x[row * FIN + std::min((it0 + ti) * 32 + i, FIN - 1)];
#pragma unroll
            for (int tj = 0; tj < S::TJ; ++tj) {
                const int64_t at = row * FOUT + std::min((jt0 + tj) * 32 + i, FOUT - 1);
                gb_next[tj][e] = g[at];
                if (MASKED) zb_next[tj][e] = z[at];
            }
        }
    };
    // What was fetched, the rows of `step`, is multiplied while fetch_next() is under way.
    auto take = [&](int64_t step, auto fetch_next) {
        Raw xa[S::TI][8], gb[S::TJ][8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool row_ok = row_of(step, e) < n;
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti) xa[ti][e] = (row_ok && (it0 + ti) * 32 + i < FIN) ? xa_next[ti][e] : Raw(0);
#pragma unroll
            for (int tj = 0; tj < S::TJ; ++tj) {
                bool ok = row_ok && (jt0 + tj) * 32 + i < FOUT;
                if constexpr (MASKED && BF16) ok = ok && zb_next[tj][e] - 1u < 0x7f80u;      // a positive bf16: sign clear, not zero, no NaN
                if constexpr (MASKED && !BF16) ok = ok && zb_next[tj][e] > 0.0f;
                gb[tj][e] = ok ? gb_next[tj][e] : Raw(0);
            }
        }
        fetch_next();
        __builtin_amdgcn_sched_barrier(0);                  // the loads must stay ahead of the multiplications
        if constexpr (BF16) {
            bf16x8 a[S::TI], b[S::TJ];
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti) {
                const uintx4 p = {xa[ti][0] | (xa[ti][1] << 16), xa[ti][2] | (xa[ti][3] << 16), xa[ti][4] | (xa[ti][5] << 16),
                                  xa[ti][6] | (xa[ti][7] << 16)};
                a[ti] = __builtin_bit_cast(bf16x8, p);
            }
#pragma unroll
            for (int tj = 0; tj < S::TJ; ++tj) {
                const uintx4 p = {gb[tj][0] | (gb[tj][1] << 16), gb[tj][2] | (gb[tj][3] << 16), gb[tj][4] | (gb[tj][5] << 16),
                                  gb[tj][6] | (gb[tj][7] << 16)};
                b[tj] = __builtin_bit_cast(bf16x8, p);
            }
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
                for (int tj = 0; tj < S::TJ; ++tj)
                    acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ti], b[tj], acc[ti][tj], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
                    for (int tj = 0; tj < S::TJ; ++tj)
                        acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[ti][e], gb[tj][e], acc[ti][tj], 0, 0, 0);
        }
    };
    // One item: without the line's bookkeeping beside every step (720 K x 128 bf16: 105 / 87 us), but in fp32 under a mask the compiler makes
    // more of the counted loop (60 K x 128, twelve gradients 345 / 380; of 16 columns 165 / 150).
    if constexpr (!LINE && (BF16 || !MASKED || FIN == 16)) {
        if (me < n_steps) fetch(me);
        for (int64_t step = me; step < n_steps; step += workers) take(step, [&] { fetch(std::min(step + workers, n_steps - 1)); });
    } else {
        int64_t at = me, left = me < n_steps * items ? (n_steps * items - me + workers - 1) / workers : 0;    // step within the item; this worker's
        auto advance = [&] {
            bool turned = false;
            for (; at >= n_steps; at -= n_steps, turned = true) item = uniform(item + 1);
            if (turned) open_item();
            return turned;
        };
        if (left > 0) {
            advance();
            fetch(at);
        }
        for (; left > 0; --left) {
            bool turned = false;
            take(at, [&] {
                if (left > 1) {
                    at += workers;
                    turned = advance();
                }
                fetch(at);
            });
            if (turned) close_item();
        }
        if constexpr (LINE) {
            close_item();
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
                for (int tj = 0; tj < S::TJ; ++tj) acc[ti][tj] = behind[ti][tj];
        }
    }

    // ---- the workgroup's workers: the upper half hands its sums to the lower half until one is left
    constexpr int kTile = 16 * kWave;                       // values of a 32x32 tile, lane by lane
    __shared__ float s_acc[(S::RS > 1 ? S::RS / 2 : 1) * S::GROUPS * S::TPW * kTile];
#pragma unroll
    for (int half = S::RS / 2; half > 0; half /= 2) {
        float *slot = &s_acc[((rs % half) * S::GROUPS + group) * S::TPW * kTile + lane];
        if (rs >= half && rs < 2 * half)
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
                for (int tj = 0; tj < S::TJ; ++tj)
#pragma unroll
                    for (int v = 0; v < 16; ++v) slot[(ti * S::TJ + tj) * kTile + v * kWave] = acc[ti][tj][v];
        __syncthreads();
        if (rs < half)
#pragma unroll
            for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
                for (int tj = 0; tj < S::TJ; ++tj)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[ti][tj][v] += slot[(ti * S::TJ + tj) * kTile + v * kWave];
        if (half > 1) __syncthreads();
    }
    if (rs > 0) return;

    // register v of lane (i, h) holds element (8 (v / 4) + 4 h + v % 4, i) of its 32x32 tile
    float *mine = partial + blockIdx.x * (int64_t)(FIN * FOUT);
#pragma unroll
    for (int ti = 0; ti < S::TI; ++ti)
#pragma unroll
        for (int tj = 0; tj < S::TJ; ++tj)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = (it0 + ti) * 32 + 8 * (v / 4) + 4 * hh + v % 4;
                const int c = (jt0 + tj) * 32 + i;
                if (r < FIN && c < FOUT) mine[r * FOUT + c] = acc[ti][tj][v];
            }
}

// `items` items of every gradient of the launch
template <int FIN, int FOUT, bool BF16, bool MASKED, bool LINE>
__global__ __launch_bounds__(kWavesPerBlock *kWave) void wgrad_kernel(Batch batch, int items, int64_t n, int64_t n_steps, float *__restrict__ partial) {
    wgrad<FIN, FOUT, BF16, MASKED, LINE>(&batch.item[blockIdx.y * items], items, n, n_steps, partial + (int64_t)blockIdx.y * gridDim.x * FIN * FOUT);
}

// dw[e] = (accumulate ? dw[e] : 0) + sum over the workers' partial results: sixteen wavefronts take a slice of
// the workers each (in worker order), then the sixteen slice sums are added in slice order: a fixed order.  In 64 bits and rounded
// once per item: a line of items has one such sum where calls have one each, whose roundings average out, and with fp32 additions it
// was the further off on positive numbers (12 x 60 K x 128 bf16: 6.2e-8 from 64 bits in calls, 6.6e-8 as a line; now 5.8e-8 and
// 3.2e-8; 6 x 200 K 4.7e-8 and 6.0e-8, now 3.6e-8 and 1.9e-8), in the same time (116 / 115 us).
// `items` of them in a row have one dw; apart: each with partial results of its own, added to dw one after the other.
constexpr int kReduceSlices = 16;
template <bool APART>
__global__ __launch_bounds__(kReduceSlices *kWave) void wgrad_reduce_kernel(Batch batch, int items, const float *__restrict__ partial, int workers, int elems,
                                                                            int accumulate) {
    float *__restrict__ dw = as_global(batch.item[blockIdx.y * items].dw);
    partial += (int64_t)blockIdx.y * workers * elems;
    __shared__ double s_sum[kReduceSlices][kWave];
    const int lane = threadIdx.x & (kWave - 1), slice = threadIdx.x / kWave;
    const int e = blockIdx.x * kWave + lane;
    const int per = (workers + kReduceSlices - 1) / kReduceSlices;
    const int p0 = slice * per, p1 = min(p0 + per, workers);
    auto sum_of = [&](const float *__restrict__ from) {
        double sum = 0.0;
        if (e < elems) {
#pragma unroll 8
            for (int p = p0; p < p1; ++p) sum += from[(int64_t)p * elems + e];
        }
        s_sum[slice][lane] = sum;
        __syncthreads();
        double total = s_sum[0][lane];
#pragma unroll
        for (int s = 1; s < kReduceSlices; ++s) total += s_sum[s][lane];
        return total;
    };
    if constexpr (!APART) {
        const double total = sum_of(partial);
        if (slice == 0 && e < elems) dw[e] = (float)(accumulate ? dw[e] + total : total);
    } else {
        float out = accumulate && e < elems ? dw[e] : 0.0f;
        for (int k = 0; k < items; ++k) {
            if (k) __syncthreads();
            const double total = sum_of(partial + (int64_t)k * workers * elems);
            out = (float)(accumulate || k ? out + total : total);
        }
        if (slice == 0 && e < elems) dw[e] = out;
    }
}

// out = (Z > 0 ? G : 0) * row_scale[row]; one 16-byte piece per lane.
template <bool BF16>
__global__ __launch_bounds__(kThreads) void relu_backward_kernel(const uintx4 *__restrict__ g, const uintx4 *__restrict__ z,
                                                                 const float *__restrict__ row_scale, uintx4 *__restrict__ out,
                                                                 int64_t pieces, int pieces_per_row) {
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= pieces) return;
    const uintx4 gv = __builtin_nontemporal_load(g + p), zv = __builtin_nontemporal_load(z + p);   // streams: read once
    const float sc = row_scale ? row_scale[p / pieces_per_row] : 1.0f;
    uintx4 o;
    if (BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // a bf16 is positive when its sign bit is clear and it is not a zero
            const uint32_t zl = zv[e] & 0xffffu, zh = zv[e] >> 16;
            const float gl = __uint_as_float(gv[e] << 16), gh = __uint_as_float(gv[e] & 0xffff0000u);
            const float ol = (zl != 0u && zl < 0x8000u) ? gl * sc : 0.0f;
            const float oh = (zh != 0u && zh < 0x8000u) ? gh * sc : 0.0f;
            o[e] = f32_to_bf16(ol) | (f32_to_bf16(oh) << 16);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = __float_as_uint(__uint_as_float(zv[e]) > 0.0f ? __uint_as_float(gv[e]) * sc : 0.0f);
    }
    __builtin_nontemporal_store(o, out + p);
}

// `count` gradients, each the sum over `items` items (count = 1 where items > 1)
template <int FIN, int FOUT, bool BF16, bool MASKED>
int launch_wgrad(int count, int items, const Batch &b, int64_t n, int accumulate, float *partial, hipStream_t s) {
    using S = Split<FIN, FOUT>;
    const int64_t n_steps = (n + kStepRows - 1) / kStepRows;
    auto workgroups = [](int64_t steps) { return (steps + S::RS - 1) / S::RS; };
    // the gradients of a launch share the workspace (one partial result per workgroup) and the device
    const int64_t most = std::min<int64_t>(resident_workgroups(wgrad_kernel<FIN, FOUT, BF16, MASKED, false>, kWavesPerBlock * kWave, 256), kMaxBlocks);
    // Items of one sum: with partial results of their own where the workspace has room for all of them, which is then bit for bit
    // a call per item; otherwise their steps are one line and a workgroup leaves one result for all of them.  On large items the
    // results would be as many bytes as the items are (60 K x 128 bf16: 31 MB of rows, 17 MB of results; a checkpointed step over 24
    // such timesteps, twelve of them to a line instead of a launch pair each, 2497 -> 2297 us).
    const int64_t alone = std::min<int64_t>(workgroups(n_steps), most);
    const int apart = items > 1 && alone * items <= kMaxBlocks;
    const int64_t blocks = apart ? alone : std::min<int64_t>(workgroups(n_steps * items), std::max<int64_t>(1, most / count));
    const bool line = items > 1 && !apart;
    // (items under a mask are never taken together)
    hipLaunchKernelGGL((line ? wgrad_kernel<FIN, FOUT, BF16, MASKED, !MASKED> : wgrad_kernel<FIN, FOUT, BF16, MASKED, false>),
                       dim3((unsigned)blocks, (unsigned)(apart ? items : count)), dim3(kWavesPerBlock * kWave), 0, s, b, apart ? 1 : items, n, n_steps, partial);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    constexpr int elems = FIN * FOUT;
    hipLaunchKernelGGL((apart ? wgrad_reduce_kernel<true> : wgrad_reduce_kernel<false>), dim3((elems + kWave - 1) / kWave, (unsigned)count),
                       dim3(kReduceSlices * kWave), 0, s, b, items, partial, (int)blocks, elems, accumulate);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

template <int FIN, bool BF16, bool MASKED>
int wgrad_out(int32_t f_out, int count, int items, const Batch &b, int64_t n, int accumulate, float *partial, hipStream_t s) {
    switch (f_out) {
        case 16: return launch_wgrad<FIN, 16, BF16, MASKED>(count, items, b, n, accumulate, partial, s);
        case 32: return launch_wgrad<FIN, 32, BF16, MASKED>(count, items, b, n, accumulate, partial, s);
        case 64: return launch_wgrad<FIN, 64, BF16, MASKED>(count, items, b, n, accumulate, partial, s);
        case 128: return launch_wgrad<FIN, 128, BF16, MASKED>(count, items, b, n, accumulate, partial, s);
        default: return DGNN_ERR_SHAPE;
    }
}

template <bool BF16, bool MASKED>
int wgrad_in(int32_t f_in, int32_t f_out, int count, int items, const Batch &b, int64_t n, int accumulate, float *partial, hipStream_t s) {
    switch (f_in) {
        case 16: return wgrad_out<16, BF16, MASKED>(f_out, count, items, b, n, accumulate, partial, s);
        case 32: return wgrad_out<32, BF16, MASKED>(f_out, count, items, b, n, accumulate, partial, s);
        case 64: return wgrad_out<64, BF16, MASKED>(f_out, count, items, b, n, accumulate, partial, s);
        case 128: return wgrad_out<128, BF16, MASKED>(f_out, count, items, b, n, accumulate, partial, s);
        default: return DGNN_ERR_SHAPE;
    }
}

}  // namespace

extern "C" int dgnn_weight_grad_workspace(int32_t f_in, int32_t f_out, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (!supported_width(f_in) || !supported_width(f_out)) return DGNN_ERR_SHAPE;
    // one F x F' partial per workgroup
    *bytes = (size_t)kMaxBlocks * (size_t)f_in * (size_t)f_out * sizeof(float);
    return DGNN_OK;
}

extern "C" int dgnn_weight_grad_batch(int32_t count, const dgnn_weight_grad_item *items, int64_t n, int32_t f_in, int32_t f_out,
                                      int32_t accumulate, dgnn_dtype dt, void *ws, size_t ws_bytes, void *stream) {
    if (!items || !ws) return DGNN_ERR_NULL;
    for (int k = 0; k < count; ++k)
        if (!items[k].x || !items[k].g || !items[k].dw) return DGNN_ERR_NULL;
    if (n <= 0 || count <= 0 || !supported_width(f_in) || !supported_width(f_out)) return DGNN_ERR_SHAPE;
    if (dt != DGNN_F32 && dt != DGNN_BF16) return DGNN_ERR_SHAPE;
    if (!fits_index(n)) return DGNN_ERR_OVERFLOW;
    const bool masked = items[0].z != nullptr;
    for (int k = 0; k < count; ++k) {
        if ((items[k].z != nullptr) != masked) return DGNN_ERR_SHAPE;
        if (!aligned16(items[k].x) || !aligned16(items[k].g) || !aligned16(items[k].z)) return DGNN_ERR_ALIGN;
    }
    if (!aligned16(ws)) return DGNN_ERR_ALIGN;
    size_t need = 0;
    dgnn_weight_grad_workspace(f_in, f_out, &need);
    if (ws_bytes < need) return DGNN_ERR_CAPACITY;
    hipStream_t s = (hipStream_t)stream;
    float *partial = static_cast<float *>(ws);
    for (int done = 0; done < count;) {
        // items that follow each other with one dw are one sum (under a mask, which no caller has them under, one after the other);
        // gradients of their own go together up to the next such run
        auto same = [&](int k) { return k >= 0 && k + 1 < count && items[k].dw == items[k + 1].dw; };
        const bool sum = !masked && same(done), goes_on = same(done - 1);      // (a run longer than a launch)
        int m = 1;
        while (m < kMaxBatch && done + m < count && (sum ? same(done + m - 1) : !goes_on && !same(done + m - 1) && !same(done + m))) ++m;
        Batch b;
        for (int k = 0; k < m; ++k) b.item[k] = Item{items[done + k].x, items[done + k].g, items[done + k].z, items[done + k].dw};
        const int gradients = sum ? 1 : m, each = sum ? m : 1;
        const int acc = accumulate || goes_on ? 1 : 0;
        const int rc = dt == DGNN_BF16 ? (masked ? wgrad_in<true, true>(f_in, f_out, gradients, each, b, n, acc, partial, s) : wgrad_in<true, false>(f_in, f_out, gradients, each, b, n, acc, partial, s))
                                       : (masked ? wgrad_in<false, true>(f_in, f_out, gradients, each, b, n, acc, partial, s) : wgrad_in<false, false>(f_in, f_out, gradients, each, b, n, acc, partial, s));
        if (rc != DGNN_OK) return rc;
        done += m;
    }
    return DGNN_OK;
}

extern "C" int dgnn_weight_grad(const void *x, const void *g, int64_t n, int32_t f_in, int32_t f_out, float *dw,
                                int32_t accumulate, dgnn_dtype dt, void *ws, size_t ws_bytes, void *stream) {
    const dgnn_weight_grad_item item{x, g, nullptr, dw};
    return dgnn_weight_grad_batch(1, &item, n, f_in, f_out, accumulate, dt, ws, ws_bytes, stream);
}

extern "C" int dgnn_relu_backward(const void *g, const void *z, const float *row_scale, void *out, int64_t n, int32_t f,
                                  dgnn_dtype dt, void *stream) {
    if (!g || !z || !out) return DGNN_ERR_NULL;
    if (n <= 0 || !supported_width(f)) return DGNN_ERR_SHAPE;
    if (dt != DGNN_F32 && dt != DGNN_BF16) return DGNN_ERR_SHAPE;
    if (!fits_index(n)) return DGNN_ERR_OVERFLOW;
    if (!aligned16(g) || !aligned16(z) || !aligned16(out)) return DGNN_ERR_ALIGN;
    const int pieces_per_row = f * (dt == DGNN_F32 ? 4 : 2) / 16;
    const int64_t pieces = n * pieces_per_row;
    const unsigned blocks = (unsigned)((pieces + kThreads - 1) / kThreads);
    hipStream_t s = (hipStream_t)stream;
    if (dt == DGNN_BF16)
        hipLaunchKernelGGL(relu_backward_kernel<true>, dim3(blocks), dim3(kThreads), 0, s, static_cast<const uintx4 *>(g),
                           static_cast<const uintx4 *>(z), row_scale, static_cast<uintx4 *>(out), pieces, pieces_per_row);
    else
        hipLaunchKernelGGL(relu_backward_kernel<false>, dim3(blocks), dim3(kThreads), 0, s, static_cast<const uintx4 *>(g),
                           static_cast<const uintx4 *>(z), row_scale, static_cast<uintx4 *>(out), pieces, pieces_per_row);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}
