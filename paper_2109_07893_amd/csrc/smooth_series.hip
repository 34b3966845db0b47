// The smoothed snapshots of a whole series from its first snapshot and the graph differences (Section "Smoothening the Input
// Graphs"): S_t holds every entry of A_{t-l+1} .. A_t with the number of these snapshots that hold it as its value, S_1 = A_1;
// S_2 .. S_{steps+1} in four launches.  No raw snapshot is formed.
//
// One step after the other (dgnn_delta_rebuild for A_t, dgnn_csr_combine for S_t) is nine launches a step and reads S_{t-1},
// A_t and A_{t-l} twice.  Here, as in dgnn_delta_rebuild_series, a workgroup keeps a stretch of the series in LDS, the entries
// between two keys (row, column); with each entry goes a word of history, bit j: present j snapshots ago.  A step's lists
// set the newest bit, entries whose history runs empty leave, added ones that are still remembered come back.
//   smooth_dinv_kernel   rows: the stored entries of a row sum up to the degrees of the last l snapshots (less the extra self
//                        loops), which the first row pointers and the lists' entries per row give without any S_t;
//   smooth_merge_kernel  twice: where a stretch begins in S_t depends on how many entries the others remember, so a first
//                        launch walks the steps and counts only, smooth_scan_kernel turns the counts into places, and a second
//                        one walks them again and writes.  (Keeping the first launch's result in memory and moving it to its
//                        place afterwards would be 16 bytes per entry and step instead.)
// What bounds it: as for the series of raw snapshots, the chain of steps inside a workgroup, and the issue of its instructions
// once the workgroups no longer fit the chip at once.
#include <algorithm>

#include "common.hpp"

namespace {

using namespace dgnn;

constexpr int kSteps = DGNN_SERIES_STEPS;
constexpr int kRowTile = 256;                // rows (and threads) per workgroup of the row kernel
constexpr int kThreads = 512;
constexpr int kPerThread = 4;
constexpr int kCap = kThreads * kPerThread;  // entries of a stretch that LDS holds
constexpr int kTile = kCap * 3 / 4;          // entries of A_1 per stretch: it may grow by a third before it is cut further
constexpr int kVmcntZero = 0x0F70;           // s_waitcnt operand: every vector memory access has completed
constexpr int kHalf = kThreads / 2;          // half of the workgroup takes the added entries, the other half the deleted ones
constexpr int kAddsKept = 2;                 // added entries per thread and step, at most
constexpr int kScanThreads = 1024;

struct Smooth {
    int n, nnz1, steps, cap, life, stretches;
    float diag;
    const int32_t *rowptr1, *colidx1;
    int32_t *counts, *d_status;              // [steps][stretches]; [steps]
    dgnn_smooth_step s[kSteps];
};

// dinv_t[r] = (sum of row r of S_t)^(-1/2) for all steps
__global__ __launch_bounds__(kRowTile) void smooth_dinv_kernel(Smooth P) {
    __shared__ int s_net[kSteps][kRowTile];
    __shared__ int s_bound[kSteps][4];       // of the tile: added begin, deleted begin, added end, deleted end
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int r0 = blockIdx.x * kRowTile, r1 = min(r0 + kRowTile, P.n), r = r0 + tid;
    const int deg1 = r < P.n ? P.rowptr1[r + 1] - P.rowptr1[r] : 0;
    for (int s = 0; s < P.steps; ++s) s_net[s][tid] = 0;
    for (int q = tid; q < 4 * P.steps; q += kRowTile) {
        const dgnn_smooth_step &st = P.s[q >> 2];
        const int32_t *rows = (q & 1) ? st.del_row : st.add_row;
        const int len = (int)((q & 1) ? st.n_del : st.n_add);
        s_bound[q >> 2][q & 3] = lower4(0, len, (uint64_t)((q & 2) ? r1 : r0), [=](int i) { return (uint64_t)(uint32_t)rows[i]; });
    }
    block_lds_sync();
    for (int s = wave; s < P.steps; s += kRowTile / kWave) {            // a wavefront per step, four loads of a lane in flight
        const dgnn_smooth_step &st = P.s[s];
        const int a0 = s_bound[s][0], d0 = s_bound[s][1], na = max(s_bound[s][2] - a0, 0), nd = max(s_bound[s][3] - d0, 0);
#pragma unroll 1
        for (int j0 = lane; j0 < na + nd; j0 += 4 * kWave) {
            int row[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = j0 + k * kWave;
                row[k] = j < na ? st.add_row[a0 + j] : j < na + nd ? st.del_row[d0 + j - na] : -1;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned q = (unsigned)(row[k] - r0);
                if (q < (unsigned)kRowTile) atomicAdd(&s_net[s][q], j0 + k * kWave < na ? 1 : -1);
            }
        }
    }
    block_lds_sync();
    if (r >= P.n) return;
    int deg = deg1, oldest = deg1, sum = deg1;                          // of A_t, of A_{t-l}, of the window's snapshots
    for (int s = 0; s < P.steps; ++s) {
        deg += s_net[s][tid];
        sum += deg;
        if (s + 1 >= P.life) {
            sum -= oldest;
            if (s + 1 < P.steps) oldest += s_net[s + 1 - P.life][tid];
        }
        float total = (float)sum;
        if (P.diag != 0.0f) total = (float)(sum - min(s + 2, P.life)) + P.diag;      // every snapshot holds the diagonal
        if (P.s[s].dinv) P.s[s].dinv[r] = total > 0.0f ? 1.0f / sqrtf(total) : 0.0f;
    }
}

template <bool WRITE>
__global__ __launch_bounds__(kThreads) void smooth_merge_kernel(Smooth P) {
    __shared__ __attribute__((aligned(16))) uint64_t s_key[kCap];
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kCap];
    // per entry: deleted << 31 | present again << 10 | new entries that go right before it; then the exclusive sums of
    // kept << 20 | present again << 10 | new ones before it ([kCap]: the total)
    __shared__ __attribute__((aligned(16))) uint32_t s_mark[kCap + 4];
    __shared__ int s_seg[kSteps][4];           // the keys' parts of the lists: added begin, deleted begin, added end, deleted end
    __shared__ int s_start[kSteps];            // where the keys at hand begin in S_t (first launch: how many have been counted)
    __shared__ int s_now[kSteps];              // entries of S_t between the keys at hand
    __shared__ uint32_t s_wave[kThreads / kWave];
    __shared__ int s_rows[3];
    static_assert(kCap < 1 << 12 && kAddsKept * kHalf < 1 << 10, "three sums share a word");

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int e0 = blockIdx.x * kTile, e1 = min(e0 + kTile, P.nnz1);
    // rows of the first and last entry and of the one after (the next stretch's first key), searched side by side
    if (wave < 3) {
        const int row = wave_find_row(P.rowptr1, P.n, min(wave == 0 ? e0 : wave == 1 ? e1 - 1 : e1, P.nnz1 - 1), lane);
        if (lane == 0) s_rows[wave] = max(row, 0);
    }
    if (tid < P.steps) s_start[tid] = WRITE ? P.counts[(int64_t)tid * P.stretches + blockIdx.x] : 0;
    block_lds_sync();
    const int row_first = s_rows[0], row_last = s_rows[1];
    const uint64_t k_hi = e1 == P.nnz1 ? ~0ull : ((uint64_t)(uint32_t)s_rows[2] << 32) | (uint32_t)P.colidx1[e1];
    const uint32_t remembered = P.life >= 32 ? ~0u : (1u << P.life) - 1;
    const bool adds = uniform(wave) < kHalf / kWave;
    const int half_tid = adds ? tid : tid - kHalf;

    // first position in the LDS keys that is not below `key`: four ways per round, the offsets constants
    auto place_of = [&](uint64_t key) {
        int at = 0;
#pragma unroll
        for (int b = kCap / 4; b >= 2; b /= 4) {
            const uint64_t k1 = s_key[at + b - 1], k2 = s_key[at + 2 * b - 1], k3 = s_key[at + 3 * b - 1];
            at += (k1 < key ? b : 0) + (k2 < key ? b : 0) + (k3 < key ? b : 0);
        }
        at += s_key[at] < key ? 1 : 0;
        return at + (s_key[min(at, kCap - 1)] < key ? 1 : 0);
    };
    static_assert(kCap == 2048, "place_of takes rounds of 512, 128, 32, 8, 2 keys");

    // The stretch is walked as one piece; keys among which more is remembered than the LDS holds are halved until it fits
    // (a piece that fails writes nothing that the pieces it is cut into do not write again).
    uint64_t lo = e0 == 0 ? 0 : ((uint64_t)(uint32_t)row_first << 32) | (uint32_t)P.colidx1[e0], hi = k_hi;
    int ea = e0, eb = e1;                      // the entries of A_1 in [lo, hi)
    for (;;) {
        __syncthreads();                       // what the last piece left in LDS has been read
        for (int q = tid; q < 4 * P.steps; q += kThreads) {
            const dgnn_smooth_step &st = P.s[q >> 2];
            const int len = (int)((q & 1) ? st.n_del : st.n_add);
            const uint64_t key = (q & 2) ? hi : lo;
            s_seg[q >> 2][q & 3] = key == 0 ? 0 : key == ~0ull ? len : lower_key((q & 1) ? st.del_row : st.add_row, (q & 1) ? st.del_col : st.add_col, 0, len, key);
        }
        for (int p = eb - ea + tid; p < kCap; p += kThreads) s_key[p] = ~0ull;    // beyond the piece: above every key
        {   // keys of the piece in A_1: a thread finds the row of its first entry and walks on
            constexpr int kOwn = kTile / kThreads;
            const int p0 = ea + tid * kOwn;
            if (p0 < eb) {
                int a = row_first, b = row_last;                        // last row whose pointer is <= p0
                while (a < b) {
                    const int mid = a + ((b - a + 1) >> 1);
                    if (P.rowptr1[mid] <= p0) a = mid; else b = mid - 1;
                }
                int row = a, end = P.rowptr1[row + 1];
#pragma unroll
                for (int k = 0; k < kOwn; ++k) {
                    const int p = p0 + k;
                    if (p < eb) {
                        while (p >= end && row < row_last) end = P.rowptr1[++row + 1];
                        s_key[p - ea] = ((uint64_t)(uint32_t)row << 32) | (uint32_t)P.colidx1[p];
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            s_mark[tid * kPerThread + k] = 0;
            s_hist[tid * kPerThread + k] = 1;
        }
        block_lds_sync();
        // rows that begin in the piece
        const int row_a = min((int64_t)(lo >> 32), (int64_t)P.n) + ((uint32_t)lo > 0 ? 1 : 0);
        const int row_b = min(min((int64_t)(hi >> 32), (int64_t)P.n) - ((uint32_t)hi > 0 ? 0 : 1), (int64_t)P.n - 1);
        const bool last_key = hi - lo <= 1;                             // cannot be cut: for lists that keep the preconditions it fits
        int cnt = eb - ea;
        // list entries of kGroup steps are fetched at once, a group ahead (as in the series of raw snapshots)
        constexpr int kGroup = 4;
        uint32_t row_next[kGroup], col_next[kGroup], row_now[kGroup], col_now[kGroup];
        auto fetch = [&](int first) {
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                const int s = min(first + q, P.steps - 1);
                const dgnn_smooth_step &st = P.s[s];
                const int from = uniform(s_seg[s][adds ? 0 : 1]), len = max(uniform(s_seg[s][adds ? 2 : 3]) - from, 0);
                row_next[q] = __builtin_amdgcn_raw_buffer_load_b32(buffer_of((adds ? st.add_row : st.del_row) + from, len), half_tid * 4, 0, 0);
                col_next[q] = __builtin_amdgcn_raw_buffer_load_b32(buffer_of((adds ? st.add_col : st.del_col) + from, len), half_tid * 4, 0, 0);
            }
        };
        fetch(0);
        bool fits = true;
#pragma unroll 1
        for (int s = 0; s < P.steps; ++s) {
            if (s % kGroup == 0) {
#pragma unroll
                for (int q = 0; q < kGroup; ++q) { row_now[q] = row_next[q]; col_now[q] = col_next[q]; }
                fetch(s + kGroup);
            }
            const dgnn_smooth_step &st = P.s[s];
            const int a0 = uniform(s_seg[s][0]), d0 = uniform(s_seg[s][1]), nd = max(uniform(s_seg[s][3]) - d0, 0);
            int na = max(uniform(s_seg[s][2]) - a0, 0);
            if (na > kAddsKept * kHalf || cnt + na > kCap) {
                fits = last_key;
                if (!fits) break;
                na = min(na, min(kAddsKept * kHalf, kCap - cnt));
            }
            uint32_t row_own = row_now[0], col_own = col_now[0];
#pragma unroll
            for (int q = 1; q < kGroup; ++q) {
                row_own = s % kGroup == q ? row_now[q] : row_own;
                col_own = s % kGroup == q ? col_now[q] : col_own;
            }
            const uint64_t list_first = ((uint64_t)row_own << 32) | col_own;
            block_lds_sync();                                           // keys, history and cleared marks are there
            uint64_t a_key[kAddsKept];
            int a_slot[kAddsKept];                                      // the entry it goes before, or -1
            if (adds) {
#pragma unroll
                for (int k = 0; k < kAddsKept; ++k) {
                    const int j = half_tid + k * kHalf;
                    a_slot[k] = -1;
                    if (j < na) {
                        a_key[k] = list_first;
                        if (k > 0) {                                    // rare: a step this full pays for its loads on the spot
                            a_key[k] = ((uint64_t)(uint32_t)st.add_row[a0 + j] << 32) | (uint32_t)st.add_col[a0 + j];
                            __builtin_amdgcn_s_waitcnt(kVmcntZero);
                        }
                        const int p = place_of(a_key[k]);
                        const bool again = p < cnt && s_key[p] == a_key[k];
                        a_slot[k] = again ? -1 : p;
                        if (p < cnt) atomicAdd(&s_mark[p], again ? 1u << 10 : 1u);
                    }
                }
            } else {
                for (int j = half_tid; j < nd; j += kHalf) {
                    uint64_t key = list_first;
                    if (j != half_tid) {
                        key = ((uint64_t)(uint32_t)st.del_row[d0 + j] << 32) | (uint32_t)st.del_col[d0 + j];
                        __builtin_amdgcn_s_waitcnt(kVmcntZero);
                    }
                    const int p = place_of(key);
                    if (p < cnt && s_key[p] == key) atomicOr(&s_mark[p], 1u << 31);
                }
            }
            block_lds_sync();
            // ---- a step further in every entry's history, and the exclusive sums
            uint32_t v[kPerThread], sum = 0;
            {
                const uintx4 m = *reinterpret_cast<const uintx4 *>(&s_mark[tid * kPerThread]);
                uintx4 h = *reinterpret_cast<const uintx4 *>(&s_hist[tid * kPerThread]);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t again = (m[q] >> 10) & 1u, here = m[q] >> 31 ? again : (h[q] & 1u) | again;
                    h[q] = ((h[q] << 1) | here) & remembered;
                    v[q] = tid * kPerThread + q < cnt ? (h[q] != 0 ? 1u << 20 : 0) | (m[q] & 0xfffffu) : 0;
                    sum += v[q];
                }
                *reinterpret_cast<uintx4 *>(&s_hist[tid * kPerThread]) = h;
            }
            static_assert(kPerThread == 4, "one 16-byte access per thread");
            const uint32_t incl = (uint32_t)wave_scan_add((int)sum, lane);
            if (lane == kWave - 1) s_wave[wave] = incl;
            block_lds_sync();
            uint32_t run = incl - sum, total = 0;
#pragma unroll
            for (int w = 0; w < kThreads / kWave; ++w) {
                const uint32_t t = s_wave[w];
                if (w < wave) run += t;
                total += t;
            }
            {
                uintx4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) { o[q] = run; run += v[q]; }
                *reinterpret_cast<uintx4 *>(&s_mark[tid * kPerThread]) = o;
            }
            if (tid == 0) s_mark[kCap] = total;
            block_lds_sync();
            // ---- new places: old entries by the sums; new ones by their rank in the list, less those before them that were
            // still remembered, behind the kept entries before their slot
            uint64_t key[kPerThread];
            uint32_t hist[kPerThread];
            int pos[kPerThread], a_pos[kAddsKept];
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {
                const int p = tid + k * kThreads;
                pos[k] = kCap;
                if (p < cnt) {
                    const uint32_t before = s_mark[p], own = s_mark[p + 1] - before;
                    key[k] = s_key[p];
                    hist[k] = s_hist[p];
                    if (own >> 20) pos[k] = (int)((before >> 20) + (before & 0x3ffu) + (own & 0x3ffu));
                }
            }
#pragma unroll
            for (int k = 0; k < kAddsKept; ++k) {
                a_pos[k] = kCap;
                if (adds && a_slot[k] >= 0) {
                    const uint32_t before = s_mark[min(a_slot[k], cnt)];
                    a_pos[k] = half_tid + k * kHalf - (int)((before >> 10) & 0x3ffu) + (int)(before >> 20);
                }
            }
            block_lds_sync();
            const int cnt_before = cnt;
            cnt = uniform(min((int)(total >> 20) + na - (int)((total >> 10) & 0x3ffu), kCap));
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {
                if (pos[k] < kCap) { s_key[pos[k]] = key[k]; s_hist[pos[k]] = hist[k]; }
                s_mark[tid * kPerThread + k] = 0;
            }
#pragma unroll
            for (int k = 0; k < kAddsKept; ++k)
                if (a_pos[k] < kCap) { s_key[a_pos[k]] = a_key[k]; s_hist[a_pos[k]] = 1; }
            for (int p = cnt + tid; p < cnt_before; p += kThreads) s_key[p] = ~0ull;
            if (tid == 0) s_now[s] = cnt;
            if (WRITE) {
                block_lds_sync();
                const int start = uniform(s_start[s]);
                const bool placed = start >= 0 && start < P.cap;        // unless S_t does not fit its arrays
                const int room = placed ? min(cnt, P.cap - start) : 0;
                const __amdgpu_buffer_rsrc_t out_col = buffer_of(st.colidx + (placed ? start : 0), room), out_val = buffer_of(st.val + (placed ? start : 0), room);
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    const int p = tid + k * kThreads;
                    const uint64_t entry = s_key[p];
                    const float value = P.diag != 0.0f && (uint32_t)entry == (uint32_t)(entry >> 32) ? P.diag : (float)__popc(s_hist[p]);
                    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)entry, out_col, p * 4, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(value), out_val, p * 4, 0, 0);
                }
                for (int r = row_a + tid; r <= row_b; r += kThreads) st.rowptr[r] = start + place_of((uint64_t)(uint32_t)r << 32);
            }
        }
        if (!fits) {                           // the lower half of the keys first
            if (eb - ea >= 2) {
                eb = ea + (eb - ea) / 2;
                __syncthreads();
                const int row = wave_find_row(P.rowptr1, P.n, eb, lane);
                hi = ((uint64_t)(uint32_t)max(uniform(row), 0) << 32) | (uint32_t)P.colidx1[eb];
            } else {
                hi = lo + (hi - lo) / 2;
                if (eb > ea) {
                    const int row = wave_find_row(P.rowptr1, P.n, ea, lane);
                    if ((((uint64_t)(uint32_t)max(uniform(row), 0) << 32) | (uint32_t)P.colidx1[ea]) >= hi) eb = ea;
                }
            }
            continue;
        }
        block_lds_sync();
        if (tid < P.steps) s_start[tid] += s_now[tid];
        if (hi == k_hi) break;
        lo = hi;
        hi = k_hi;
        ea = eb;
        eb = e1;
    }
    if (!WRITE && tid < P.steps) P.counts[(int64_t)tid * P.stretches + blockIdx.x] = s_start[tid];
}

// counts of a step -> where each stretch begins in S_t, a workgroup per step; the number of stored entries goes into the last
// row pointer
__global__ __launch_bounds__(kScanThreads) void smooth_scan_kernel(Smooth P) {
    constexpr int kWaves = kScanThreads / kWave;
    __shared__ int s_wave[kWaves];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    int32_t *counts = P.counts + (int64_t)blockIdx.x * P.stretches;
    int carry = 0;
    for (int base = 0; base < P.stretches; base += 4 * kScanThreads) {
        const int i = base + 4 * tid;
        int v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = i + q < P.stretches ? counts[i + q] : 0;
        const int mine = (v[0] + v[1]) + (v[2] + v[3]);
        const int incl = wave_scan_add(mine, lane);
        if (lane == kWave - 1) s_wave[wave] = incl;
        __syncthreads();
        int before = carry, total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int t = s_wave[w];
            if (w < wave) before += t;
            total += t;
        }
        int run = before + incl - mine;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i + q < P.stretches) counts[i + q] = run;
            run += v[q];
        }
        carry += total;
        __syncthreads();
    }
    if (tid == 0) {
        P.s[blockIdx.x].rowptr[P.n] = carry;
        if (P.d_status) P.d_status[blockIdx.x] = carry > P.cap ? DGNN_BAD_CAPACITY : 0;
    }
}

int64_t stretch_count(int64_t nnz) { return (nnz + kTile - 1) / kTile; }

}  // namespace

extern "C" int dgnn_smooth_series_workspace(int64_t nnz_first, int32_t steps, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (nnz_first <= 0 || steps < 0 || steps > kSteps) return DGNN_ERR_SHAPE;
    if (!fits_index(nnz_first)) return DGNN_ERR_OVERFLOW;
    *bytes = std::max<size_t>(16, (size_t)stretch_count(nnz_first) * steps * sizeof(int32_t));
    return DGNN_OK;
}

extern "C" int dgnn_smooth_series(int64_t n, const int32_t *rowptr_first, const int32_t *colidx_first, int64_t nnz_first, int32_t steps,
                                  const dgnn_smooth_step *step, int32_t life, float diag_value, int64_t capacity, int32_t *d_status,
                                  void *ws, size_t ws_bytes, void *stream) {
    if (!rowptr_first || !colidx_first || !ws || (steps > 0 && !step)) return DGNN_ERR_NULL;
    if (n <= 0 || nnz_first <= 0 || steps < 0 || steps > kSteps || life < 1 || life > 32 || capacity < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz_first)) return DGNN_ERR_OVERFLOW;
    int64_t most = nnz_first;
    bool dinv = false;
    for (int k = 0; k < steps; ++k) {
        const dgnn_smooth_step &st = step[k];
        if (!st.rowptr || !st.colidx || !st.val) return DGNN_ERR_NULL;
        if (st.n_add < 0 || st.n_del < 0) return DGNN_ERR_SHAPE;
        if ((st.n_add > 0 && (!st.add_row || !st.add_col)) || (st.n_del > 0 && (!st.del_row || !st.del_col))) return DGNN_ERR_NULL;
        most += st.n_add;
        if (!fits_index(most) || !fits_index(st.n_del)) return DGNN_ERR_OVERFLOW;
        // all steps are written by the same launches: every snapshot needs arrays of its own
        if (st.rowptr == rowptr_first || st.colidx == colidx_first) return DGNN_ERR_ALIAS;
        for (int j = 0; j < k; ++j)
            if (st.rowptr == step[j].rowptr || st.colidx == step[j].colidx || st.val == step[j].val) return DGNN_ERR_ALIAS;
        dinv |= st.dinv != nullptr;
    }
    if (!aligned16(ws)) return DGNN_ERR_ALIGN;
    const int64_t stretches = stretch_count(nnz_first);
    if (ws_bytes < (size_t)stretches * steps * sizeof(int32_t)) return DGNN_ERR_CAPACITY;
    if (steps == 0) return DGNN_OK;
    hipStream_t s = (hipStream_t)stream;
    Smooth P;
    P.n = (int)n;
    P.nnz1 = (int)nnz_first;
    P.steps = steps;
    P.cap = (int)std::min<int64_t>(capacity, 2147483647LL);
    P.life = life;
    P.stretches = (int)stretches;
    P.diag = diag_value;
    P.rowptr1 = rowptr_first;
    P.colidx1 = colidx_first;
    P.counts = (int32_t *)ws;
    P.d_status = d_status;
    for (int k = 0; k < steps; ++k) P.s[k] = step[k];
    if (dinv) {
        hipLaunchKernelGGL(smooth_dinv_kernel, dim3((unsigned)((n + kRowTile - 1) / kRowTile)), dim3(kRowTile), 0, s, P);
        DGNN_RETURN_IF_LAUNCH_FAILED();
    }
    hipLaunchKernelGGL(smooth_merge_kernel<false>, dim3((unsigned)stretches), dim3(kThreads), 0, s, P);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(smooth_scan_kernel, dim3((unsigned)steps), dim3(kScanThreads), 0, s, P);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(smooth_merge_kernel<true>, dim3((unsigned)stretches), dim3(kThreads), 0, s, P);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}
