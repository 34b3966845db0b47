// The LSTM of the CD-GCN layer (Section "CD-GCN") over a series of timesteps in one launch, and its adjoint.
//
// The recurrence runs per vertex, a = [Y_t | h_{t-1}] [W_x ; W_h] + b and the cell, so a wavefront that owns 32 vertices can
// walk all timesteps by itself: [W_x ; W_h] is staged in LDS once per workgroup, h_{t-1} is in the tile buffer when it is
// needed, c stays in the registers (rounded to the storage type after every step).  Per step a wavefront forms the TRANSPOSED
// gate tiles on the matrix cores (W^T as the A operand, the rows of [Y | h] as the B operand): column C = g * hidden + k of the
// pre-activations is gate g of state element k, it lies in the 32-column tile C / 32, and lane (i, h) holds, for vertex i, the
// columns c of a tile with (c / 4) % 2 == h, four consecutive ones per four accumulator registers.  hidden is a multiple of 8,
// so the four gates of a state element sit in the same lane: lane (i, h) owns state elements 8 m + 4 h + r of vertex i, and the
// cell works on the accumulators.
//
// Going back the same wavefront recomputes the gates of timestep t, turns the accumulators into da and multiplies them by the
// rows of [W_x ; W_h] that are wanted, W da^T, straight from the registers: a lane's accumulators are half of the contraction
// indices of its vertex, the other lane half holds the other half, which is how a matrix instruction splits its k.  That gives
// dL/dh_{t-1}, which stays on chip for the next step, and dL/dY1 under the ReLU's mask; da leaves for the weight gradients,
// which contract over vertices and timesteps and are one product afterwards.
//
// fp32 products are formed on the bf16 matrix cores (below): 262 144 vertices, 4 steps, 64 + 32 columns, forward 292 -> 200 us, back
// 503 -> 405, against the fp32 matrix instruction, which alone takes 164 and 328 of these.  What is left in fp32 is the cell
// (exponentials) and the vector instructions of the parts, at two wavefronts per SIMD, and the traffic: 0.8 and 1.3 GB.  bf16 is
// bound by the cell (and, up to 64 columns of Y, the tile staging); what the series saves is the traffic and the launches of the state: h and c in, c out, dh and dc both ways.
#include <algorithm>
#include <initializer_list>
#include <type_traits>

#include "common.hpp"

namespace {

using namespace dgnn;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The nonlinearities from the hardware exponential and reciprocal (1 ulp each): sig(x) = 1 / (1 + 2^(-x log2 e)), tanh(x) = 2 sig(2x) - 1;
// absolute error a few 1e-7.  They compete with the matrix cores for issue slots: library versions take as many as the products.
__device__ __forceinline__ float fast_sigmoid(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
__device__ __forceinline__ float fast_tanh(float x) { return 2.0f * fast_sigmoid(2.0f * x) - 1.0f; }

// What the two storage types do differently: the LDS image of W, the operands' fetch, the rounding on the way out.
template <bool BF16> struct Store;
template <> struct Store<false> {
    typedef float Elem;
    static constexpr int kPiece = 4;                   // elements per 16-byte piece
    static constexpr int kTilePad = 4;                 // elements of padding per tile row
    static __device__ __forceinline__ floatx4 load4(const float *p) { return *reinterpret_cast<const floatx4 *>(p); }
    static __device__ __forceinline__ void store4(float *p, floatx4 v) { *reinterpret_cast<floatx4 *>(p) = v; }
    static __device__ __forceinline__ floatx4 rounded(floatx4 v) { return v; }
    static __device__ __forceinline__ float product(float v) { return -v; }          // of what the products below leave
};
template <> struct Store<true> {
    typedef uint16_t Elem;
    static constexpr int kPiece = 8;
    static constexpr int kTilePad = 8;
    static __device__ __forceinline__ floatx4 load4(const uint16_t *p) {
        const uint2 r = *reinterpret_cast<const uint2 *>(p);
        return floatx4{bf16_to_f32(r.x & 0xffffu), __uint_as_float(r.x & 0xffff0000u), bf16_to_f32(r.y & 0xffffu), __uint_as_float(r.y & 0xffff0000u)};
    }
    static __device__ __forceinline__ void store4(uint16_t *p, floatx4 v) {
        *reinterpret_cast<uint2 *>(p) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
    }
    static __device__ __forceinline__ float product(float v) { return v; }
    static __device__ __forceinline__ floatx4 rounded(floatx4 v) {
        const uint32_t lo = pack_bf16(v[0], v[1]), hi = pack_bf16(v[2], v[3]);
        return floatx4{__uint_as_float(lo << 16), __uint_as_float(lo & 0xffff0000u), __uint_as_float(hi << 16), __uint_as_float(hi & 0xffff0000u)};
    }
};

// ---- fp32 products on the bf16 matrix cores (the splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", 2019).  An fp32 number is the sum of three bf16 numbers, each the rounded rest
// of the ones before it (8 + 8 + 8 bits), and of the nine products of two such sums the six largest are formed, 2.6 times as fast as the fp32 matrix
// instruction forms the one.  The second part is at most 2^-8 of a number in [1, 2), the third 2^-17, so what is left out is up to 2^-24 of the
// product (1.7 x 2^-25 met with random numbers), no more than rounding the product would take.  That holds for numbers from 2^-110 on: the matrix
// cores keep denormal numbers, but bf16 has none below 2^-133, so smaller ones enter with an absolute error of up to 2^-134.
// From kSplitBelow on a wavefront's step takes the fp32 instruction: there a smaller product could pass fp32 ahead of the largest, with the
// other sign, and the sum would be no number where the product is infinite.  Below, the at most 128 products of a sum, 2^120 each, stay
// in fp32 whatever their order.
constexpr int kParts = 3;
constexpr uint32_t kSplitBelow = 0x5d800000u;          // 2^60
constexpr uint32_t kRoundsFinite = 0x7f7f7fffu;        // the largest fp32 that rounds to a finite bf16

// Whether all numbers noted are to be split: the largest pattern of either sign (half an instruction each per number).
struct Largest {
    int above = 0;
    uint32_t below = 0;
    __device__ __forceinline__ void note(uint32_t bits) {
        above = max(above, (int)bits);
        below = max(below, bits);
    }
    __device__ __forceinline__ bool odd() const { return above >= (int)kSplitBelow || below >= (kSplitBelow | 0x80000000u); }
};

__device__ __forceinline__ void split(const float (&v)[8], bf16x8 (&part)[kParts]) {
    float rest[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) rest[e] = v[e];
#pragma unroll
    for (int k = 0; k < kParts; ++k) {
        uintx4 p;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = pack_bf16(rest[2 * e], rest[2 * e + 1]);
            if (k + 1 < kParts) {
                rest[2 * e] -= __uint_as_float(p[e] << 16);
                rest[2 * e + 1] -= __uint_as_float(p[e] & 0xffff0000u);
            }
        }
        part[k] = __builtin_bit_cast(bf16x8, p);
    }
}

// Two passes over the contraction: first the five smaller products of every step, then the largest, (part of a, part of b) in turn.
// The matrix cores cut what they add towards minus infinity, a few thousandths of the last place per instruction, and sums over all
// vertices see that.  With the smaller products ahead it counts for a sixth of the instructions, and from the middle of the second pass on
// the sum is carried with the other sign, so that the cuts of its two halves meet (the bias gradient of 40 K vertices and four steps,
// error against 64 bits: 2.3e-7 with the fp32 instruction, 4.9e-7 with all products step by step, 2.8e-7 with them in two passes).
// The result has the other sign.
constexpr int kSmaller = 5;
constexpr int kTermA[kSmaller] = {2, 0, 1, 1, 0}, kTermB[kSmaller] = {0, 2, 1, 0, 1};

template <int N>
__device__ __forceinline__ void smaller_products(floatx16 (&acc)[N], const bf16x8 (&a)[N][kParts], const bf16x8 (&b)[kParts]) {
#pragma unroll
    for (int k = 0; k < kSmaller; ++k)
#pragma unroll
        for (int g = 0; g < N; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g][kTermA[k]], b[kTermB[k]], acc[g], 0, 0, 0);
}

// The operand of the second pass' step s of `steps`.
__device__ __forceinline__ bf16x8 first_part(const float (&v)[8], int s, int steps) {
    const uint32_t sign = s < steps / 2 ? 0u : 0x80008000u;
    return __builtin_bit_cast(bf16x8, uintx4{pack_bf16(v[0], v[1]) ^ sign, pack_bf16(v[2], v[3]) ^ sign, pack_bf16(v[4], v[5]) ^ sign, pack_bf16(v[6], v[7]) ^ sign});
}
template <int N>
__device__ __forceinline__ void turn_sign(floatx16 (&acc)[N]) {
#pragma unroll
    for (int g = 0; g < N; ++g)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[g][v] = -acc[g][v];
}

// [W_x ; W_h] transposed in LDS, k contiguous: in bf16 as it is, in fp32 its three parts one after the other.
template <int FY, int HID, bool BF16>
struct Weights {
    static constexpr int G4 = 4 * HID, NT = G4 / 32, K = FY + HID;
    static constexpr int kLd = K + 8, kImage = G4 * kLd, kSize = BF16 ? kImage : kParts * kImage;
    typedef typename Store<BF16>::Elem Elem;
    // whether this thread has met a number that is not to be split (its parts are put together again: at())
    static __device__ __forceinline__ bool stage(uint16_t *s_w, const Elem *__restrict__ w_x, const Elem *__restrict__ w_h, int tid, int threads) {
        bool odd = false;
        for (int idx = tid; idx < K * G4; idx += threads) {
            const int k = idx / G4, col = idx % G4;
            const Elem v = k < FY ? w_x[idx] : w_h[idx - FY * G4];
            if constexpr (BF16) {
                s_w[col * kLd + k] = v;
            } else {
                const uint32_t bits = __float_as_uint(v) & 0x7fffffffu;
                const bool whole = bits >= 0x7f800000u;            // an infinity, or no number: the first part is all of it
                odd |= bits >= kSplitBelow;
                float rest = v;
#pragma unroll
                for (int part = 0; part < kParts; ++part) {
                    const uint32_t p = bits > kRoundsFinite && !whole ? __float_as_uint(rest) >> 16 : f32_to_bf16(rest);
                    s_w[part * kImage + col * kLd + k] = (uint16_t)p;
                    rest = whole ? 0.0f : rest - __uint_as_float(p << 16);
                }
            }
        }
        return odd;
    }
    // fp32: element [k][col], put together again
    static __device__ __forceinline__ float at(const uint16_t *s_w, int k, int col) {
        float v = 0.0f;
#pragma unroll
        for (int part = kParts - 1; part >= 0; --part) v += bf16_to_f32(s_w[part * kImage + col * kLd + k]);
        return v;
    }
};

// Where the lanes' rows of Y come straight from memory in operand layout (16 bytes of a row per lane) instead of through the tile
// buffer, which then holds h or c only.  128 + 64 columns of bf16: W takes 100 KB of the LDS, whole tiles of [Y | h] leave room for four
// wavefronts, one per SIMD, which multiply and then evaluate the cell with nothing beside it; without Y there are eight.  200 K
// vertices, 6 steps: four wavefronts 315 us, eight 221.  With c kept for every step the buffer carries both states, and stays.
template <int FY, int HID, bool BF16, bool KEEP_C> constexpr bool kDirectY = BF16 && FY == 128 && HID == 64 && !KEEP_C;

// acc[g] = transposed tile g of [Y | h] [W_x ; W_h] for the 32 vertices in `tile` (rows of LDT elements).  In bf16 step s of the
// contraction takes the 16 columns from 16 s on, the lane half h the second eight of them; with `y` the first FY / 16 steps'
// operands are given, and the tile holds the columns behind them.
template <int FY, int HID, int LDT>
__device__ __forceinline__ void gate_tiles(const uint16_t *s_w, const uint16_t *tile, int i, int hh, floatx16 (&acc)[4 * HID / 32], const uintx4 *y = nullptr) {
    typedef Weights<FY, HID, true> W;
    constexpr int KS = W::K / 16;
#pragma unroll
    for (int g = 0; g < W::NT; ++g)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[g][v] = 0.0f;
    bf16x8 a[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        a[s] = y && s < FY / 16 ? __builtin_bit_cast(bf16x8, y[s < FY / 16 ? s : 0])
                                : *reinterpret_cast<const bf16x8 *>(&tile[i * LDT + 16 * s + 8 * hh - (y ? FY : 0)]);
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int g = 0; g < W::NT; ++g) {
            const bf16x8 wv = *reinterpret_cast<const bf16x8 *>(&s_w[(g * 32 + i) * W::kLd + 16 * s + 8 * hh]);
            acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, a[s], acc[g], 0, 0, 0);
        }
}

// Eight fp32 columns of a row of the tile buffer, from 16 s + 8 h on: a lane's operand of step s.
__device__ __forceinline__ void operand(const float *row, int s, int hh, float (&v)[8]) {
    const floatx4 lo = *reinterpret_cast<const floatx4 *>(&row[16 * s + 8 * hh]), hi = *reinterpret_cast<const floatx4 *>(&row[16 * s + 8 * hh + 4]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = lo[e];
        v[4 + e] = hi[e];
    }
}

// The same in fp32, with the other sign: Y's columns lie in the tile buffer, those of h in the lanes (step by step, as operands).
// odd: some number is not to be split.
template <int FY, int HID, int LDT>
__device__ __forceinline__ void gate_tiles_f32(const uint16_t *s_w, const float *tile, const float (&h)[HID / 16][8], bool odd, int i, int hh,
                                               floatx16 (&acc)[4 * HID / 32]) {
    typedef Weights<FY, HID, false> W;
#pragma unroll
    for (int g = 0; g < W::NT; ++g)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[g][v] = 0.0f;
    if (!odd) {
        auto weights = [&](int s, int g, int part) { return *reinterpret_cast<const bf16x8 *>(&s_w[part * W::kImage + (g * 32 + i) * W::kLd + 16 * s + 8 * hh]); };
#pragma unroll
        for (int s = 0; s < W::K / 16; ++s) {
            float v[8];
            if (s < FY / 16) operand(&tile[i * LDT], s, hh, v);
            bf16x8 a[W::NT][kParts], b[kParts];
#pragma unroll
            for (int g = 0; g < W::NT; ++g)
#pragma unroll
                for (int part = 0; part < kParts; ++part) a[g][part] = weights(s, g, part);
            split(s < FY / 16 ? v : h[s < FY / 16 ? 0 : s - FY / 16], b);
            smaller_products(acc, a, b);
            __builtin_amdgcn_sched_barrier(0);           // the operands of all steps at once would not fit the registers
        }
#pragma unroll
        for (int s = 0; s < W::K / 16; ++s) {
            float v[8];
            if (s < FY / 16) operand(&tile[i * LDT], s, hh, v);
            const bf16x8 b = first_part(s < FY / 16 ? v : h[s < FY / 16 ? 0 : s - FY / 16], s, W::K / 16);
            if (s == W::K / 16 / 2) turn_sign(acc);
#pragma unroll
            for (int g = 0; g < W::NT; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(weights(s, g, 0), b, acc[g], 0, 0, 0);
        }
    } else {
        auto product = [&](int k, float v) {             // rare: few registers rather than few trips
#pragma unroll
            for (int g = 0; g < W::NT; ++g) acc[g] = __builtin_amdgcn_mfma_f32_32x32x2f32(W::at(s_w, k, g * 32 + i), v, acc[g], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll 1
        for (int k = 0; k < FY / 2; ++k) {
            const int at = 16 * (k / 8) + 8 * hh + k % 8;
            product(at, tile[i * LDT + at]);
        }
#pragma unroll
        for (int s = 0; s < HID / 16; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) product(FY + 16 * s + 8 * hh + e, h[s][e]);
        turn_sign(acc);
    }
}

__device__ __forceinline__ uint2 read_transposed(const uint16_t *p) {
    typedef short shortx4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) shortx4 LdsShortx4;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsShortx4 *)p));
}

// register of gate g, state elements 8 m + 4 h + r: tile and first of four registers
template <int HID> constexpr int gate_tile(int g, int m) { return (g * HID + 8 * m) / 32; }
template <int HID> constexpr int gate_reg(int g, int m) { return 4 * (((g * HID + 8 * m) % 32) / 8); }

// The rows of the 32 vertices of a tile in one of a step's tensors, `bytes` each, behind a buffer descriptor: what lies behind the last
// vertex is 0 or dropped, without a mask or an address per access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rows(const void *step, int64_t tile, int64_t n, int bytes) {
    const int rows = (int)max((int64_t)0, min((int64_t)32, n - tile * 32));
    return buffer_of(static_cast<const char *>(step) + tile * 32 * bytes, rows * bytes / 4);
}

// h_1 .. h_T from h_0, c_0; KEEP_C: c_t of every step is kept (c [T][n][HID]), else c is the state after the last step
// (and may be c_0's array: a wavefront reads its vertices before it writes them).
template <int FY, int HID, bool BF16, bool KEEP_C, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void lstm_series_kernel(const void *__restrict__ yv_, const void *__restrict__ h0_,
                                                                   const void *__restrict__ wx_, const void *__restrict__ wh_,
                                                                   const float *__restrict__ bias, const void *c0_, void *c_,
                                                                   void *__restrict__ h_, int64_t n, int64_t n_tiles, int T) {
    typedef Store<BF16> S;
    typedef typename S::Elem Elem;
    typedef Weights<FY, HID, BF16> W;
    constexpr int P = S::kPiece;
    // The widest step is the faster with an address and a mask per piece, all others behind buffer descriptors (bf16, 200 K vertices, 6 steps,
    // 128 + 64 columns with c kept 285 / 309 us, without 252 / 255; 64 + 64 198.9 / 196.3; these without c kept: one step of 2^20 174 / 157, six of
    // 20 K 48 / 49.5, eight of 1000 57 / 60)
    constexpr bool BY_ADDRESS = BF16 && FY == 128;
    constexpr bool DIRECT = kDirectY<FY, HID, BF16, KEEP_C>;
    // the tile buffer: [Y | h], or h alone where Y's operands come straight from memory; in fp32, where W's parts take 80 KB, the lanes
    // hold h's operands while the buffer holds Y, and it carries h (and c beside it) between the steps
    constexpr int LDT = (!BF16 ? (KEEP_C ? 2 * HID : FY) : DIRECT ? HID : W::K) + S::kTilePad;
    constexpr int H_COL = !BF16 ? (KEEP_C ? HID : 0) : DIRECT ? 0 : FY;
    constexpr int Y_PIECES = 32 * FY / P / kWave, S_PIECES = 32 * HID / P / kWave;     // 16-byte pieces per lane of a tile
    static_assert(DIRECT || LDT >= H_COL + HID, "the tile buffer also carries c beside h");
    static_assert(BF16 || LDT >= FY, "... and Y");
    __shared__ __attribute__((aligned(16))) uint16_t s_w[W::kSize];
    __shared__ __attribute__((aligned(16))) float s_bias[W::G4];
    __shared__ __attribute__((aligned(16))) Elem s_tile[WAVES][32 * LDT];
    const Elem *y = static_cast<const Elem *>(yv_), *h0 = static_cast<const Elem *>(h0_), *c0 = static_cast<const Elem *>(c0_);
    Elem *c = static_cast<Elem *>(c_), *h = static_cast<Elem *>(h_);

    const int tid = threadIdx.x;
    bool odd_w = W::stage(s_w, static_cast<const Elem *>(wx_), static_cast<const Elem *>(wh_), tid, WAVES * kWave);
    for (int idx = tid; idx < W::G4; idx += WAVES * kWave) s_bias[idx] = bias ? bias[idx] : 0.0f;
    const int lane = tid & (kWave - 1), wave = BY_ADDRESS ? tid / kWave : uniform(tid / kWave);
    const int i = lane & 31, hh = lane >> 5;
    Elem *tile_lds = s_tile[wave];
    const int64_t stride = (int64_t)gridDim.x * WAVES;
    const int64_t first = (int64_t)blockIdx.x * WAVES + wave;
    if (BF16) __syncthreads(); else odd_w = __syncthreads_or(odd_w);      // W is in LDS; from here on every wavefront is on its own
    constexpr int Y_BYTES = FY * sizeof(Elem), S_BYTES = HID * sizeof(Elem);
    const uintx4 zero = {0u, 0u, 0u, 0u};
    // the rows of the next step (or of the next tile, with its state) travel while this one is multiplied
    uintx4 yv[Y_PIECES], hv[S_PIECES], cv[S_PIECES];
    auto fetch_y = [&](int64_t tile, int t) {
        if constexpr (DIRECT) {
            const int64_t row = tile * 32 + i;
#pragma unroll
            for (int q = 0; q < Y_PIECES; ++q) yv[q] = row < n ? *reinterpret_cast<const uintx4 *>(y + (t * n + row) * FY + 16 * q + 8 * hh) : zero;
        } else if constexpr (BY_ADDRESS) {
#pragma unroll
            for (int q = 0; q < Y_PIECES; ++q) {
                const int64_t piece = tile * (32 * FY / P) + q * kWave + lane;
                yv[q] = (tile < n_tiles && piece * P < n * FY) ? reinterpret_cast<const uintx4 *>(y + t * n * FY)[piece] : zero;
            }
        } else {
            const __amdgpu_buffer_rsrc_t rows = tile_rows(y + t * n * FY, tile, n, Y_BYTES);
#pragma unroll
            for (int q = 0; q < Y_PIECES; ++q) yv[q] = __builtin_amdgcn_raw_buffer_load_b128(rows, (q * kWave + lane) * 16, 0, 0);
        }
    };
    auto fetch_state = [&](int64_t tile) {
        if constexpr (BY_ADDRESS) {
#pragma unroll
            for (int q = 0; q < S_PIECES; ++q) {
                const int64_t piece = tile * (32 * HID / P) + q * kWave + lane;
                const bool ok = tile < n_tiles && piece * P < n * HID;
                hv[q] = ok ? reinterpret_cast<const uintx4 *>(h0)[piece] : zero;
                cv[q] = ok ? reinterpret_cast<const uintx4 *>(c0)[piece] : zero;
            }
        } else {
            const __amdgpu_buffer_rsrc_t of_h = tile_rows(h0, tile, n, S_BYTES), of_c = tile_rows(c0, tile, n, S_BYTES);
#pragma unroll
            for (int q = 0; q < S_PIECES; ++q) {
                hv[q] = __builtin_amdgcn_raw_buffer_load_b128(of_h, (q * kWave + lane) * 16, 0, 0);
                cv[q] = __builtin_amdgcn_raw_buffer_load_b128(of_c, (q * kWave + lane) * 16, 0, 0);
            }
        }
    };
    auto put = [&](int col, const uintx4 (&v)[S_PIECES]) {           // a tile of HID columns: registers -> LDS
#pragma unroll
        for (int q = 0; q < S_PIECES; ++q) {
            const int e = (q * kWave + lane) * P;
            *reinterpret_cast<uintx4 *>(&tile_lds[(e / HID) * LDT + col + e % HID]) = v[q];
        }
    };
    auto flush = [&](int col, Elem *dst, int64_t tile) {             // ... LDS -> memory, whole lines
        if constexpr (BY_ADDRESS) {
#pragma unroll
            for (int q = 0; q < S_PIECES; ++q) {
                const int e = (q * kWave + lane) * P;
                const int64_t piece = tile * (32 * HID / P) + q * kWave + lane;
                if (piece * P < n * HID) reinterpret_cast<uintx4 *>(dst)[piece] = *reinterpret_cast<const uintx4 *>(&tile_lds[(e / HID) * LDT + col + e % HID]);
            }
            return;
        }
        const __amdgpu_buffer_rsrc_t rows = tile_rows(dst, tile, n, S_BYTES);
#pragma unroll
        for (int q = 0; q < S_PIECES; ++q) {
            const int e = (q * kWave + lane) * P;
            __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const uintx4 *>(&tile_lds[(e / HID) * LDT + col + e % HID]), rows, e * (int)sizeof(Elem), 0, 0);
        }
    };
    constexpr bool kStateAhead = !(BF16 && HID == 64);     // the widest step has no registers left for it
    fetch_y(first, 0);
    if (kStateAhead) fetch_state(first);
    for (int64_t tile = first; tile < n_tiles; tile += stride) {
        if (!kStateAhead) fetch_state(tile);
        if (BF16 && !DIRECT) put(FY, hv);
        put(0, cv);
        wave_lds_sync();
        floatx4 cell[HID / 8];                          // c of this lane's state elements
#pragma unroll
        for (int m = 0; m < HID / 8; ++m) cell[m] = S::load4(&tile_lds[i * LDT + 8 * m + 4 * hh]);
        wave_lds_sync();
        if (DIRECT || !BF16) {
            put(H_COL, hv);
            wave_lds_sync();
        }
#pragma unroll 1
        for (int t = 0; t < T; ++t) {
            auto fetch_next = [&]() {
                if (t + 1 < T) fetch_y(tile, t + 1);
                else {
                    fetch_y(tile + stride, 0);
                    if (kStateAhead) fetch_state(tile + stride);
                }
            };
            floatx16 acc[W::NT];
            if constexpr (DIRECT) {
                gate_tiles<FY, HID, LDT>(s_w, tile_lds, i, hh, acc, yv);
                fetch_next();                           // into the operands' registers, while the cell is evaluated
            } else if constexpr (!BF16) {
                float hop[HID / 16][8];
                Largest top;
#pragma unroll
                for (int q = 0; q < HID / 16; ++q) {
                    operand(&tile_lds[i * LDT + H_COL], q, hh, hop[q]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) top.note(__float_as_uint(hop[q][e]));
                }
                wave_lds_sync();
#pragma unroll
                for (int q = 0; q < Y_PIECES; ++q) {
                    const int e = (q * kWave + lane) * P;
                    *reinterpret_cast<uintx4 *>(&tile_lds[(e / FY) * LDT + e % FY]) = yv[q];
#pragma unroll
                    for (int k = 0; k < 4; ++k) top.note(yv[q][k]);
                }
                fetch_next();
                wave_lds_sync();
                gate_tiles_f32<FY, HID, LDT>(s_w, tile_lds, hop, odd_w || __ballot(top.odd()), i, hh, acc);
            } else {
#pragma unroll
                for (int q = 0; q < Y_PIECES; ++q) {
                    const int e = (q * kWave + lane) * P;
                    *reinterpret_cast<uintx4 *>(&tile_lds[(e / FY) * LDT + e % FY]) = yv[q];
                }
                fetch_next();
                wave_lds_sync();
                gate_tiles<FY, HID, LDT>(s_w, tile_lds, i, hh, acc);
            }
            wave_lds_sync();                            // every lane has its operands
#pragma unroll
            for (int m = 0; m < HID / 8; ++m) {
                const int k0 = 8 * m + 4 * hh;
                floatx4 h_new;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float ai = S::product(acc[gate_tile<HID>(0, m)][gate_reg<HID>(0, m) + r]) + s_bias[k0 + r];
                    const float af = S::product(acc[gate_tile<HID>(1, m)][gate_reg<HID>(1, m) + r]) + s_bias[HID + k0 + r];
                    const float ag = S::product(acc[gate_tile<HID>(2, m)][gate_reg<HID>(2, m) + r]) + s_bias[2 * HID + k0 + r];
                    const float ao = S::product(acc[gate_tile<HID>(3, m)][gate_reg<HID>(3, m) + r]) + s_bias[3 * HID + k0 + r];
                    cell[m][r] = fast_sigmoid(af) * cell[m][r] + fast_sigmoid(ai) * fast_tanh(ag);
                    h_new[r] = fast_sigmoid(ao) * fast_tanh(cell[m][r]);
                }
                S::store4(&tile_lds[i * LDT + H_COL + k0], h_new);
                cell[m] = S::rounded(cell[m]);          // as a launch per step would hand it on: results do not depend on how many share one
                if (KEEP_C) S::store4(&tile_lds[i * LDT + k0], cell[m]);
            }
            wave_lds_sync();
            flush(H_COL, h + t * n * HID, tile);
            if (KEEP_C) flush(0, c + t * n * HID, tile);
            wave_lds_sync();                            // Y's columns are written again
        }
        if (!KEEP_C) {
#pragma unroll
            for (int m = 0; m < HID / 8; ++m) S::store4(&tile_lds[i * LDT + 8 * m + 4 * hh], cell[m]);
            wave_lds_sync();
            flush(0, c, tile);
            wave_lds_sync();
        }
    }
}

// The walk back over T steps.  Y1 = the last HID columns of Y (as many as the state is wide); out: da [T][n][4 HID], dy1 [T][n][HID]
// = dL/dY1 where Y1 > 0.  dh, dc [n][HID] fp32: dL/dh and dL/dc behind the last step (read if `carried`), then in front of the first.
template <int FY, int HID, bool BF16, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void lstm_series_backward_kernel(
    const void *__restrict__ y_, const void *__restrict__ h0_, const void *__restrict__ h_, const void *__restrict__ wx_, const void *__restrict__ wh_,
    const float *__restrict__ bias, const void *__restrict__ c0_, const void *__restrict__ c_, const void *__restrict__ gh_, void *__restrict__ da_,
    void *__restrict__ dy1_, float *__restrict__ dh_state, float *__restrict__ dc_state, int carried, int64_t n, int64_t n_tiles, int T) {
    typedef Store<BF16> S;
    typedef typename S::Elem Elem;
    typedef Weights<FY, HID, BF16> W;
    constexpr int P = S::kPiece, NT = W::NT, G4 = W::G4;
    constexpr int LDT = (BF16 ? W::K : FY > 2 * HID ? FY : 2 * HID) + S::kTilePad;     // fp32: h's operands are held by the lanes, as going forward
    static_assert(W::K >= 2 * HID, "c and the incoming gradient, halves of da");
    constexpr int Y_PIECES = 32 * FY / P / kWave, S_PIECES = 32 * HID / P / kWave, HALF_PIECES = 2 * S_PIECES;
    constexpr int ROWS = 2 * HID, N2 = ROWS / 32;               // rows of [W_x ; W_h] that da meets: those of Y1, then W_h
    constexpr int LDR = G4 + 8;                                 // bf16: these rows once more, columns contiguous
    static_assert(FY >= HID && ROWS % 32 == 0, "whole tiles of output columns");
    __shared__ __attribute__((aligned(16))) uint16_t s_w[W::kSize];
    __shared__ __attribute__((aligned(16))) Elem s_wr[BF16 ? ROWS * LDR : 1];
    __shared__ __attribute__((aligned(16))) float s_bias[G4];
    __shared__ __attribute__((aligned(16))) Elem s_tile[WAVES][32 * LDT];
    const Elem *y = static_cast<const Elem *>(y_), *h0 = static_cast<const Elem *>(h0_), *h = static_cast<const Elem *>(h_);
    const Elem *c0 = static_cast<const Elem *>(c0_), *c = static_cast<const Elem *>(c_), *gh = static_cast<const Elem *>(gh_);
    Elem *da = static_cast<Elem *>(da_), *dy1 = static_cast<Elem *>(dy1_);

    const int tid = threadIdx.x;
    bool odd_w = W::stage(s_w, static_cast<const Elem *>(wx_), static_cast<const Elem *>(wh_), tid, WAVES * kWave);
    if (BF16)
        for (int idx = tid; idx < ROWS * G4; idx += WAVES * kWave) {
            const int k = FY - HID + idx / G4;
            s_wr[(idx / G4) * LDR + idx % G4] = k < FY ? static_cast<const Elem *>(wx_)[k * G4 + idx % G4] : static_cast<const Elem *>(wh_)[(k - FY) * G4 + idx % G4];
        }
    for (int idx = tid; idx < G4; idx += WAVES * kWave) s_bias[idx] = bias ? bias[idx] : 0.0f;
    const int lane = tid & (kWave - 1), wave = uniform(tid / kWave);
    const int i = lane & 31, hh = lane >> 5;
    Elem *tile_lds = s_tile[wave];
    const int64_t stride = (int64_t)gridDim.x * WAVES;
    if (BF16) __syncthreads(); else odd_w = __syncthreads_or(odd_w);
    // fp32: rows of W from its transposed parts, by the LDS's transposing read: four lanes name 16 elements of a column's image, 16
    // lanes the four columns of a read, and lane k of them gets element k of each
    const int from = (4 * hh + (lane & 15) / 4) * W::kLd + FY - HID + (lane & 16) + (lane & 3) * 4;
    constexpr int Y_BYTES = FY * sizeof(Elem), S_BYTES = HID * sizeof(Elem);
    uintx4 yv[Y_PIECES], hv[S_PIECES], cv[S_PIECES], gv[S_PIECES];
    auto fetch = [&](int64_t tile, int t) {
        const __amdgpu_buffer_rsrc_t of_y = tile_rows(y + t * n * FY, tile, n, Y_BYTES), of_h = tile_rows(t > 0 ? h + (t - 1) * n * HID : h0, tile, n, S_BYTES);
#pragma unroll
        for (int q = 0; q < Y_PIECES; ++q) yv[q] = __builtin_amdgcn_raw_buffer_load_b128(of_y, (q * kWave + lane) * 16, 0, 0);
#pragma unroll
        for (int q = 0; q < S_PIECES; ++q) hv[q] = __builtin_amdgcn_raw_buffer_load_b128(of_h, (q * kWave + lane) * 16, 0, 0);
    };
    auto fetch_rest = [&](int64_t tile, int t) {        // what the cell takes, behind the gates
        const __amdgpu_buffer_rsrc_t of_c = tile_rows(t > 0 ? c + (t - 1) * n * HID : c0, tile, n, S_BYTES), of_g = tile_rows(gh + t * n * HID, tile, n, S_BYTES);
#pragma unroll
        for (int q = 0; q < S_PIECES; ++q) {
            cv[q] = __builtin_amdgcn_raw_buffer_load_b128(of_c, (q * kWave + lane) * 16, 0, 0);
            gv[q] = __builtin_amdgcn_raw_buffer_load_b128(of_g, (q * kWave + lane) * 16, 0, 0);
        }
    };
    auto put = [&](int col, const uintx4 (&v)[S_PIECES]) {
#pragma unroll
        for (int q = 0; q < S_PIECES; ++q) {
            const int e = (q * kWave + lane) * P;
            *reinterpret_cast<uintx4 *>(&tile_lds[(e / HID) * LDT + col + e % HID]) = v[q];
        }
    };
    const int64_t first = (int64_t)blockIdx.x * WAVES + wave;
    fetch(first, T - 1);
    for (int64_t tile = first; tile < n_tiles; tile += stride) {
        const int64_t vertex = tile * 32 + i;
        floatx4 dh[HID / 8], dc[HID / 8];               // what the step behind sent back, for this lane's state elements
#pragma unroll
        for (int m = 0; m < HID / 8; ++m) {
            dh[m] = dc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
            if (carried && vertex < n) {
                dh[m] = *reinterpret_cast<const floatx4 *>(&dh_state[vertex * HID + 8 * m + 4 * hh]);
                dc[m] = *reinterpret_cast<const floatx4 *>(&dc_state[vertex * HID + 8 * m + 4 * hh]);
            }
        }
#pragma unroll 1
        for (int t = T - 1; t >= 0; --t) {
            // ---- [Y | h_{t-1}] and the gates
            float hop[HID / 16][8];
            Largest top;
            if (!BF16) {
                put(0, hv);
                wave_lds_sync();
#pragma unroll
                for (int q = 0; q < HID / 16; ++q) {
                    operand(reinterpret_cast<const float *>(&tile_lds[i * LDT]), q, hh, hop[q]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) top.note(__float_as_uint(hop[q][e]));
                }
                wave_lds_sync();
            }
#pragma unroll
            for (int q = 0; q < Y_PIECES; ++q) {
                const int e = (q * kWave + lane) * P;
                *reinterpret_cast<uintx4 *>(&tile_lds[(e / FY) * LDT + e % FY]) = yv[q];
#pragma unroll
                for (int k = 0; k < 4; ++k) top.note(yv[q][k]);
            }
            if (BF16) put(FY, hv);
            fetch_rest(tile, t);
            wave_lds_sync();
            floatx16 acc[NT];
            if constexpr (BF16) gate_tiles<FY, HID, LDT>(s_w, tile_lds, i, hh, acc);
            else gate_tiles_f32<FY, HID, LDT>(s_w, tile_lds, hop, odd_w || __ballot(top.odd()), i, hh, acc);
            uint32_t through = 0;                       // where Y1 > 0 among the columns this lane will form
#pragma unroll
            for (int m = 0; m < HID / 8; ++m) {
                const floatx4 v = S::load4(&tile_lds[i * LDT + FY - HID + 8 * m + 4 * hh]);
#pragma unroll
                for (int r = 0; r < 4; ++r) through |= v[r] > 0.0f ? 1u << (4 * m + r) : 0u;
            }
            wave_lds_sync();
            put(0, cv);
            put(HID, gv);
            wave_lds_sync();
            // ---- the cell's adjoint on the accumulators:
            // dc = dh o (1 - tanh(c_t)^2) + dc_t, da_i = dc g i (1 - i), da_f = dc c_{t-1} f (1 - f), da_g = dc i (1 - g^2),
            // da_o = dh tanh(c_t) o (1 - o), dc_{t-1} = dc f
#pragma unroll
            for (int m = 0; m < HID / 8; ++m) {
                const int k0 = 8 * m + 4 * hh;
                const floatx4 c_old = S::load4(&tile_lds[i * LDT + k0]), g_h = S::load4(&tile_lds[i * LDT + HID + k0]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    constexpr int kI = 0, kF = 1, kG = 2, kO = 3;
                    const float gi = fast_sigmoid(S::product(acc[gate_tile<HID>(kI, m)][gate_reg<HID>(kI, m) + r]) + s_bias[k0 + r]);
                    const float gf = fast_sigmoid(S::product(acc[gate_tile<HID>(kF, m)][gate_reg<HID>(kF, m) + r]) + s_bias[HID + k0 + r]);
                    const float gg = fast_tanh(S::product(acc[gate_tile<HID>(kG, m)][gate_reg<HID>(kG, m) + r]) + s_bias[2 * HID + k0 + r]);
                    const float go = fast_sigmoid(S::product(acc[gate_tile<HID>(kO, m)][gate_reg<HID>(kO, m) + r]) + s_bias[3 * HID + k0 + r]);
                    const float tc = fast_tanh(gf * c_old[r] + gi * gg);
                    const float d_h = g_h[r] + dh[m][r];
                    const float d = d_h * go * (1.0f - tc * tc) + dc[m][r];
                    acc[gate_tile<HID>(kI, m)][gate_reg<HID>(kI, m) + r] = d * gg * gi * (1.0f - gi);
                    acc[gate_tile<HID>(kF, m)][gate_reg<HID>(kF, m) + r] = d * c_old[r] * gf * (1.0f - gf);
                    acc[gate_tile<HID>(kG, m)][gate_reg<HID>(kG, m) + r] = d * gi * (1.0f - gg * gg);
                    acc[gate_tile<HID>(kO, m)][gate_reg<HID>(kO, m) + r] = d_h * tc * go * (1.0f - go);
                    dc[m][r] = d * gf;
                }
                if (!BF16) __builtin_amdgcn_sched_barrier(0);            // a few elements at a time: registers
            }
            // ---- [dY1 | dh_{t-1}]^T = W da^T
            floatx16 out[N2];
#pragma unroll
            for (int j = 0; j < N2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) out[j][v] = 0.0f;
            if constexpr (BF16) {
#pragma unroll
                for (int g = 0; g < NT; ++g)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {       // eight of this lane's columns: 32 g + 16 p + 4 h + r and 8 further
                        uintx4 b;
#pragma unroll
                        for (int e = 0; e < 4; ++e) b[e] = pack_bf16(acc[g][8 * p + 2 * e], acc[g][8 * p + 2 * e + 1]);
#pragma unroll
                        for (int j = 0; j < N2; ++j) {
                            const Elem *src = &s_wr[(j * 32 + i) * LDR + g * 32 + 16 * p + 4 * hh];
                            const uint2 lo = *reinterpret_cast<const uint2 *>(src), hi = *reinterpret_cast<const uint2 *>(src + 8);
                            const uintx4 a = {lo.x, lo.y, hi.x, hi.y};
                            out[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), out[j], 0, 0, 0);
                        }
                    }
            } else {
                Largest most;
#pragma unroll
                for (int g = 0; g < NT; ++g)
#pragma unroll
                    for (int v = 0; v < 16; ++v) most.note(__float_as_uint(acc[g][v]));
                const bool odd = odd_w || __ballot(most.odd());
                auto columns = [&](int g, int p, float (&v)[8]) {          // the same as above
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = acc[g][8 * p + e];
                };
                auto rows_of_w = [&](int g, int p, int j, int part) {
                    const uint16_t *src = &s_w[from + part * W::kImage + (32 * g + 16 * p) * W::kLd + 32 * j];
                    const uint2 lo = read_transposed(src), hi = read_transposed(src + 8 * W::kLd);
                    return __builtin_bit_cast(bf16x8, uintx4{lo.x, lo.y, hi.x, hi.y});
                };
                if (!odd) {
#pragma unroll
                    for (int g = 0; g < NT; ++g)
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            float v[8];
                            columns(g, p, v);
                            bf16x8 a[N2][kParts], b[kParts];
#pragma unroll
                            for (int j = 0; j < N2; ++j)
#pragma unroll
                                for (int part = 0; part < kParts; ++part) a[j][part] = rows_of_w(g, p, j, part);
                            split(v, b);
                            smaller_products(out, a, b);
                            __builtin_amdgcn_sched_barrier(0);
                        }
#pragma unroll
                    for (int g = 0; g < NT; ++g)
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            float v[8];
                            columns(g, p, v);
                            const bf16x8 b = first_part(v, 2 * g + p, 2 * NT);
                            if (g == NT / 2 && p == 0) turn_sign(out);
#pragma unroll
                            for (int j = 0; j < N2; ++j) out[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows_of_w(g, p, j, 0), b, out[j], 0, 0, 0);
                        }
                } else {
#pragma unroll
                    for (int g = 0; g < NT; ++g)
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            float v[8];
                            columns(g, p, v);
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
#pragma unroll
                                for (int j = 0; j < N2; ++j)
                                    out[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(W::at(s_w, FY - HID + j * 32 + i, 32 * g + 16 * p + 4 * hh + e % 4 + 8 * (e / 4)),
                                                                                  v[e], out[j], 0, 0, 0);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
                    turn_sign(out);
                }
            }
            // ---- da leaves in two halves of two gates each (a whole tile of it does not fit the buffer)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                wave_lds_sync();
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int m = 0; m < HID / 8; ++m) {
                        const floatx16 &src = acc[gate_tile<HID>(2 * half + g, m)];
                        const int q = gate_reg<HID>(2 * half + g, m);
                        S::store4(&tile_lds[i * LDT + g * HID + 8 * m + 4 * hh], floatx4{src[q], src[q + 1], src[q + 2], src[q + 3]});
                    }
                wave_lds_sync();
                const __amdgpu_buffer_rsrc_t rows = tile_rows(da + t * n * G4, tile, n, G4 * (int)sizeof(Elem));
#pragma unroll
                for (int q = 0; q < HALF_PIECES; ++q) {
                    const int e = (q * kWave + lane) * P;
                    const int r = e / (2 * HID), col = e % (2 * HID);
                    __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const uintx4 *>(&tile_lds[r * LDT + col]), rows,
                                                           (r * G4 + half * 2 * HID + col) * (int)sizeof(Elem), 0, 0);
                }
            }
            wave_lds_sync();
            // ---- dY1 under the ReLU, dh_{t-1}
#pragma unroll
            for (int m = 0; m < HID / 8; ++m) {
                floatx4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = (through >> (4 * m + r)) & 1u ? S::product(out[(8 * m) / 32][4 * (((8 * m) % 32) / 8) + r]) : 0.0f;
                    dh[m][r] = S::product(out[(HID + 8 * m) / 32][4 * (((HID + 8 * m) % 32) / 8) + r]);
                }
                S::store4(&tile_lds[i * LDT + 8 * m + 4 * hh], v);
            }
            // the next step's rows, as early as there are registers for them
            if (t > 0) fetch(tile, t - 1);
            else fetch(tile + stride, T - 1);
            wave_lds_sync();
            const __amdgpu_buffer_rsrc_t of_dy1 = tile_rows(dy1 + t * n * HID, tile, n, S_BYTES);
#pragma unroll
            for (int q = 0; q < S_PIECES; ++q) {
                const int e = (q * kWave + lane) * P;
                __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const uintx4 *>(&tile_lds[(e / HID) * LDT + e % HID]), of_dy1, e * (int)sizeof(Elem), 0, 0);
            }
            wave_lds_sync();
        }
        if (vertex < n) {
#pragma unroll
            for (int m = 0; m < HID / 8; ++m) {
                *reinterpret_cast<floatx4 *>(&dh_state[vertex * HID + 8 * m + 4 * hh]) = dh[m];
                *reinterpret_cast<floatx4 *>(&dc_state[vertex * HID + 8 * m + 4 * hh]) = dc[m];
            }
        }
    }
}

// ---- dW_x = Y^T da, dW_h = H^T da, db = column sums of da over all rows (timesteps times vertices) in one pass over da.
// As the weight gradient of the dense transform (both operands of a lane are plain strided loads, partial results per
// workgroup, a second kernel adds them in order), with [Y | h_{t-1}] taken from two tensors: row r's state is row r - n of the
// states after each step, h_0 for the first n rows.  A wavefront owns the 32 columns `wave` of da and all columns of [Y | h].
// fp32 is bound by the matrix cores and what is issued beside them (1 M rows, widths 64 + 32 and 128: 25.8 GFLOP, 168 us at the
// rate of a large product, 0.94 GB): with addresses, clamps and masks formed per row 406 us, with uniform bases 258 us, 100 TFLOP/s.
constexpr int kGradWaves = 4;
constexpr int kGradBlocks = 512;
constexpr int kStepRows = 16;

template <int FY, int HID, bool BF16>
__global__ __launch_bounds__(kGradWaves *kWave) void lstm_wgrad_kernel(const void *__restrict__ y_, const void *__restrict__ h0_, const void *__restrict__ h_,
                                                                      const void *__restrict__ da_, int64_t n, int64_t rows,
                                                                      float *__restrict__ partial) {
    typedef typename std::conditional<BF16, uint16_t, float>::type Elem;
    typedef typename std::conditional<BF16, uint32_t, float>::type Raw;
    constexpr int G4 = 4 * HID, K = FY + HID, NI = (K + 31) / 32, NJ = G4 / 32, RS = kGradWaves / NJ;   // RS: row workers per workgroup
    const Elem *y = static_cast<const Elem *>(y_), *h0 = static_cast<const Elem *>(h0_), *h = static_cast<const Elem *>(h_), *da = static_cast<const Elem *>(da_);
    static_assert(FY % 32 == 0, "a tile of 32 columns of [Y | h] comes from one tensor");
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int i = lane & 31, hh = lane >> 5;
    const int tj = wave % NJ, rs = wave / NJ;
    const int64_t workers = (int64_t)gridDim.x * RS, me = (int64_t)blockIdx.x * RS + rs;
    floatx16 acc[NI];
    float bsum = 0.0f;
#pragma unroll
    for (int ti = 0; ti < NI; ++ti)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[ti][v] = 0.0f;
    auto row_in_step = [&](int e) { return BF16 ? 8 * hh + e : 2 * e + hh; };
    auto add_to_bias = [&](auto g) { bsum += ((g(0) + g(1)) + (g(2) + g(3))) + ((g(4) + g(5)) + (g(6) + g(7))); };     // a chain of an eighth of the rows
    auto multiply = [&](const Raw (&xa)[NI][8], const Raw (&gb)[8]) {
        if constexpr (BF16) {
            const uintx4 pb = {gb[0] | (gb[1] << 16), gb[2] | (gb[3] << 16), gb[4] | (gb[5] << 16), gb[6] | (gb[7] << 16)};
            add_to_bias([&](int e) { return bf16_to_f32(gb[e]); });
#pragma unroll
            for (int ti = 0; ti < NI; ++ti) {
                const uintx4 pa = {xa[ti][0] | (xa[ti][1] << 16), xa[ti][2] | (xa[ti][3] << 16), xa[ti][4] | (xa[ti][5] << 16), xa[ti][6] | (xa[ti][7] << 16)};
                acc[ti] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, pa), __builtin_bit_cast(bf16x8, pb), acc[ti], 0, 0, 0);
            }
        } else {
            add_to_bias([&](int e) { return gb[e]; });
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int ti = 0; ti < NI; ++ti) acc[ti] = __builtin_amdgcn_mfma_f32_32x32x2f32(xa[ti][e], gb[e], acc[ti], 0, 0, 0);
        }
    };
    // Steps whose 16 rows are all there and take their states from one tensor: the bases are uniform (scalar), a lane's offsets
    // the same in every step.  The step in which the rows' states change from h_0 to h is left out of the count, and follows
    // with the last, ragged one.  (Columns beyond K only reach rows of the product that are not stored.)
    const int64_t full = rows / kStepRows, change = (n < rows && n % kStepRows != 0 && n / kStepRows < full) ? n / kStepRows : full;
    const int64_t whole = full - (change < full ? 1 : 0);
    Raw xa_next[NI][8], gb_next[8];
    auto fetch = [&](int64_t w) {
        const int64_t r0 = (w + (w >= change ? 1 : 0)) * kStepRows;
        const Elem *yb = y + r0 * FY, *hb = r0 >= n ? h + (r0 - n) * HID : h0 + r0 * HID, *gb = da + r0 * G4 + tj * 32;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int r = row_in_step(e);
#pragma unroll
            for (int ti = 0; ti < NI; ++ti) xa_next[ti][e] = ti * 32 < FY ? yb[r * FY + ti * 32 + i] : hb[r * HID + std::min(ti * 32 - FY + i, HID - 1)];
            gb_next[e] = gb[r * G4 + i];
        }
    };
    if (me < whole) fetch(me);
    for (int64_t w = me; w < whole; w += workers) {
        Raw xa[NI][8], gb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma unroll
            for (int ti = 0; ti < NI; ++ti) xa[ti][e] = xa_next[ti][e];
            gb[e] = gb_next[e];
        }
        fetch(std::min(w + workers, whole - 1));
        __builtin_amdgcn_sched_barrier(0);             // the next step's loads stay ahead of the multiplications
        multiply(xa, gb);
    }
    for (int k = 0; k < 2; ++k) {
        const int64_t step = k == 0 ? change : full;   // both only where there are such rows, one worker each
        if (k == 0 ? change == full : rows % kStepRows == 0) continue;
        if (me != k % workers) continue;
        Raw xa[NI][8], gb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t at = step * kStepRows + row_in_step(e), row = std::min<int64_t>(at, rows - 1);
            const Elem *hp = row >= n ? h + (row - n) * HID : h0 + row * HID;
#pragma unroll
            for (int ti = 0; ti < NI; ++ti) {
                const Raw v = ti * 32 < FY ? y[row * FY + ti * 32 + i] : hp[std::min(ti * 32 - FY + i, HID - 1)];
                xa[ti][e] = at < rows ? v : Raw(0);
            }
            const Raw g = da[row * G4 + tj * 32 + i];
            gb[e] = at < rows ? g : Raw(0);
        }
        multiply(xa, gb);
    }
    float *mine = partial + me * (int64_t)((K + 1) * G4);
#pragma unroll
    for (int ti = 0; ti < NI; ++ti)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = ti * 32 + 8 * (v / 4) + 4 * hh + v % 4;
            if (r < K) mine[r * G4 + tj * 32 + i] = acc[ti][v];
        }
    bsum += __shfl_xor(bsum, 32, kWave);
    if (hh == 0) mine[K * G4 + tj * 32 + i] = bsum;
}

// The partial results in worker order: sixteen wavefronts take a slice of the workers each, then the slices are added in order.  In 64
// bits and rounded once: added in fp32 they were most of the error of a sum over all vertices (40 K vertices, 4 steps, 64 + 32
// columns fp32, against 64 bits: db 6.5e-8 -> 3.0e-8, dW_x 6.9e-8 -> 3.2e-8, dW_h 9.4e-8 -> 7.0e-8, of which h's own error is 6.1e-8), in the
// same time (2^18 vertices, both kernels 301 / 295 us: what bounds it is the partial results' way from memory).
constexpr int kReduceSlices = 16;
__global__ __launch_bounds__(kReduceSlices *kWave) void lstm_wgrad_reduce_kernel(const float *__restrict__ partial, int workers, int x_elems, int h_elems,
                                                                                int b_elems, float *__restrict__ dw_x, float *__restrict__ dw_h,
                                                                                float *__restrict__ db, int accumulate) {
    __shared__ double s_sum[kReduceSlices][kWave];
    const int lane = threadIdx.x & (kWave - 1), slice = threadIdx.x / kWave;
    const int elems = x_elems + h_elems + b_elems, e = blockIdx.x * kWave + lane;
    const int per = (workers + kReduceSlices - 1) / kReduceSlices;
    const int p0 = slice * per, p1 = min(p0 + per, workers);
    double sum = 0.0;
    if (e < elems) {
#pragma unroll 8
        for (int p = p0; p < p1; ++p) sum += partial[(int64_t)p * elems + e];
    }
    s_sum[slice][lane] = sum;
    __syncthreads();
    if (slice == 0 && e < elems) {
        double total = s_sum[0][lane];
#pragma unroll
        for (int k = 1; k < kReduceSlices; ++k) total += s_sum[k][lane];
        float *dst = e < x_elems ? dw_x + e : e < x_elems + h_elems ? dw_h + (e - x_elems) : db + (e - x_elems - h_elems);
        *dst = (float)(accumulate ? *dst + total : total);
    }
}

bool series_shape_ok(int32_t f_y, int32_t hidden, dgnn_dtype dt) {
    if (dt == DGNN_F32) return (hidden == 16 || hidden == 32) && (f_y == hidden || f_y == 2 * hidden);
    if (dt == DGNN_BF16) return (hidden == 32 || hidden == 64) && (f_y == hidden || f_y == 2 * hidden);
    return false;
}
bool backward_shape_ok(int32_t f_y, int32_t hidden, dgnn_dtype dt) {
    return f_y == 2 * hidden && (dt == DGNN_F32 ? hidden == 16 || hidden == 32 : dt == DGNN_BF16 && hidden == 32);
}

template <int FY, int HID, bool BF16, int WAVES, int KEEP_WAVES = WAVES>
int launch_series(const void *y, const void *h0, const void *w_x, const void *w_h, const float *bias, const void *c0, void *c, void *h, int64_t n,
                  int T, bool keep_c, hipStream_t s) {
    const int64_t n_tiles = (n + 31) / 32;
    auto run = [&](auto kernel, int waves) {
        const int64_t needed = (n_tiles + waves - 1) / waves, resident = resident_workgroups(kernel, waves * kWave, 256);
        hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(needed, resident)), dim3(waves * kWave), 0, s, y, h0, w_x, w_h, bias, c0, c, h, n, n_tiles, T);
    };
    if (keep_c) run(lstm_series_kernel<FY, HID, BF16, true, KEEP_WAVES>, KEEP_WAVES); else run(lstm_series_kernel<FY, HID, BF16, false, WAVES>, WAVES);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

template <int FY, int HID, bool BF16, int WAVES>
int launch_backward(const void *y, const void *h0, const void *h, const void *w_x, const void *w_h, const float *bias, const void *c0, const void *c,
                    const void *g_h, void *da, void *dy1, float *dh, float *dc, int carried, int64_t n, int T, hipStream_t s) {
    const int64_t n_tiles = (n + 31) / 32, needed = (n_tiles + WAVES - 1) / WAVES;
    const int64_t resident = resident_workgroups(lstm_series_backward_kernel<FY, HID, BF16, WAVES>, WAVES * kWave, 256);
    hipLaunchKernelGGL((lstm_series_backward_kernel<FY, HID, BF16, WAVES>), dim3((unsigned)std::min(needed, resident)), dim3(WAVES * kWave), 0, s, y, h0, h,
                       w_x, w_h, bias, c0, c, g_h, da, dy1, dh, dc, carried, n, n_tiles, T);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

template <int FY, int HID, bool BF16>
int launch_grad(const void *y, const void *h0, const void *h, const void *da, int64_t n, int64_t rows, float *dw_x, float *dw_h, float *db, int accumulate,
                float *partial, hipStream_t s) {
    constexpr int RS = kGradWaves / (4 * HID / 32);
    const int64_t n_steps = (rows + kStepRows - 1) / kStepRows;
    const int64_t blocks = std::min<int64_t>({(n_steps + RS - 1) / RS, resident_workgroups(lstm_wgrad_kernel<FY, HID, BF16>, kGradWaves * kWave, 512), (int64_t)kGradBlocks});
    hipLaunchKernelGGL((lstm_wgrad_kernel<FY, HID, BF16>), dim3((unsigned)blocks), dim3(kGradWaves * kWave), 0, s, y, h0, h, da, n, rows, partial);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    const int x = FY * 4 * HID, hh = HID * 4 * HID, b = 4 * HID;
    hipLaunchKernelGGL(lstm_wgrad_reduce_kernel, dim3((x + hh + b + kWave - 1) / kWave), dim3(kReduceSlices * kWave), 0, s, partial, (int)(blocks * RS), x, hh, b,
                       dw_x, dw_h, db, accumulate);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

}  // namespace

extern "C" int dgnn_lstm_series(const void *y, int32_t f_y, const void *h0, const void *w_x, const void *w_h, const float *bias, const void *c0,
                                void *c, int32_t keep_c, void *h, int64_t n, int32_t T, int32_t hidden, dgnn_dtype dt, void *stream) {
    if (!y || !h0 || !w_x || !w_h || !c0 || !c || !h) return DGNN_ERR_NULL;
    if (n <= 0 || T <= 0 || !series_shape_ok(f_y, hidden, dt)) return DGNN_ERR_SHAPE;
    if (!fits_index(n)) return DGNN_ERR_OVERFLOW;
    for (const void *p : {y, h0, c0, (const void *)c, (const void *)h})
        if (!aligned16(p)) return DGNN_ERR_ALIGN;
    if (h == h0 || h == c || h == y || c == y || c == h0 || h == c0 || (keep_c && c == c0)) return DGNN_ERR_ALIAS;
    hipStream_t s = (hipStream_t)stream;
    const bool keep = keep_c != 0;
    if (dt == DGNN_F32) {
        if (hidden == 32) return f_y == 32 ? launch_series<32, 32, false, 8>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s)
                                           : launch_series<64, 32, false, 8>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s);
        return f_y == 16 ? launch_series<16, 16, false, 8>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s)
                         : launch_series<32, 16, false, 8>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s);
    }
    if (hidden == 32) return f_y == 32 ? launch_series<32, 32, true, 8>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s)
                                       : launch_series<64, 32, true, 8>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s);
    return f_y == 64 ? launch_series<64, 64, true, 8>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s)
                     : launch_series<128, 64, true, 8, 4>(y, h0, w_x, w_h, bias, c0, c, h, n, T, keep, s);
}

extern "C" int dgnn_lstm_step(const void *y, int32_t f_y, const void *h_prev, const void *w_x, const void *w_h,
                              const float *bias, void *c, void *h_next, int64_t n, int32_t hidden, dgnn_dtype dt,
                              void *stream) {
    return dgnn_lstm_series(y, f_y, h_prev, w_x, w_h, bias, c, c, 0, h_next, n, 1, hidden, dt, stream);
}

extern "C" int dgnn_lstm_series_backward(const void *y, int32_t f_y, const void *h0, const void *h, const void *w_x, const void *w_h, const float *bias,
                                         const void *c0, const void *c, const void *g_h, void *da, void *dy1, float *dh, float *dc, int32_t carried,
                                         int64_t n, int32_t T, int32_t hidden, dgnn_dtype dt, void *stream) {
    if (!y || !h0 || !h || !w_x || !w_h || !c0 || !c || !g_h || !da || !dy1 || !dh || !dc) return DGNN_ERR_NULL;
    if (n <= 0 || T <= 0 || !backward_shape_ok(f_y, hidden, dt)) return DGNN_ERR_SHAPE;
    if (!fits_index(n)) return DGNN_ERR_OVERFLOW;
    for (const void *p : {y, h0, h, c0, c, g_h, (const void *)da, (const void *)dy1, (const void *)dh, (const void *)dc})
        if (!aligned16(p)) return DGNN_ERR_ALIGN;
    for (const void *p : {y, h0, h, c0, c, g_h})
        if (p == da || p == dy1 || p == dh || p == dc) return DGNN_ERR_ALIAS;
    if (da == dy1 || dh == dc) return DGNN_ERR_ALIAS;
    hipStream_t s = (hipStream_t)stream;
    if (dt == DGNN_BF16) return launch_backward<64, 32, true, 8>(y, h0, h, w_x, w_h, bias, c0, c, g_h, da, dy1, dh, dc, carried, n, T, s);
    return hidden == 32 ? launch_backward<64, 32, false, 8>(y, h0, h, w_x, w_h, bias, c0, c, g_h, da, dy1, dh, dc, carried, n, T, s)
                        : launch_backward<32, 16, false, 8>(y, h0, h, w_x, w_h, bias, c0, c, g_h, da, dy1, dh, dc, carried, n, T, s);
}

extern "C" int dgnn_lstm_weight_grad_workspace(int32_t f_y, int32_t hidden, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (!backward_shape_ok(f_y, hidden, DGNN_F32) && !backward_shape_ok(f_y, hidden, DGNN_BF16)) return DGNN_ERR_SHAPE;
    const int rs = kGradWaves / (4 * hidden / 32);
    *bytes = (size_t)kGradBlocks * rs * (f_y + hidden + 1) * 4 * hidden * sizeof(float);
    return DGNN_OK;
}

extern "C" int dgnn_lstm_weight_grad(const void *y, int32_t f_y, const void *h0, const void *h, const void *da, int64_t n, int32_t T, int32_t hidden,
                                     float *dw_x, float *dw_h, float *db, int32_t accumulate, dgnn_dtype dt, void *ws, size_t ws_bytes, void *stream) {
    if (!y || !h0 || !h || !da || !dw_x || !dw_h || !db || !ws) return DGNN_ERR_NULL;
    if (n <= 0 || T <= 0 || !backward_shape_ok(f_y, hidden, dt)) return DGNN_ERR_SHAPE;
    if (!fits_index(n)) return DGNN_ERR_OVERFLOW;
    size_t need = 0;
    dgnn_lstm_weight_grad_workspace(f_y, hidden, &need);
    if (ws_bytes < need) return DGNN_ERR_CAPACITY;
    hipStream_t s = (hipStream_t)stream;
    float *partial = static_cast<float *>(ws);
    const int64_t rows = (int64_t)T * n;
    if (dt == DGNN_BF16) return launch_grad<64, 32, true>(y, h0, h, da, n, rows, dw_x, dw_h, db, accumulate, partial, s);
    return hidden == 32 ? launch_grad<64, 32, false>(y, h0, h, da, n, rows, dw_x, dw_h, db, accumulate, partial, s)
                        : launch_grad<32, 16, false>(y, h0, h, da, n, rows, dw_x, dw_h, db, accumulate, partial, s);
}
