// A whole series of snapshots from its first one and the graph differences (Section "Graph-difference Based Input
// Transfer"), for callers that have the difference lists of several steps at hand: A_2 .. A_{S+1} in two launches.
//
// Rebuilding step by step reads A_{t-1} back from memory for every A_t and pays two launches per step.  Here a workgroup
// keeps a stretch of the series: the entries between two keys (row, column), taken from A_1 at every kTile-th entry.  The
// lists are sorted by the same key, so the stretch of step t is the stretch of step t-1 minus and plus its own parts of the
// two lists, whatever happens elsewhere; it stays in LDS from step to step, is read once and written once per step.  Where
// it begins in A_t follows from the list positions of its first key:
//     start_t = start_1 + sum over the steps so far of (#added before the key - #deleted before the key).
//   series_rowptr_kernel  tiles of rows: row pointers and dinv of every step from per-row counts of the lists;
//   series_merge_kernel   the column indices.  Per step and workgroup: a list entry finds its place among the keys in LDS,
//                         a deleted one marks the entry it names, an added one counts at the entry it precedes; one prefix
//                         sum over (kept, added before) gives all new places.
// What bounds it: the chain of steps inside a workgroup, 2.3 us each (a search of six LDS trips, the scan, the placing, five
// barriers: the latency of some six hundred dependent instructions), while the workgroups fit the chip at once (up to about
// a million entries); beyond that the issue of those instructions, 0.2 M entries per us.  Seven steps over 11 thousand entries
// take 32 us against 89 us rebuilt one after the other, fifteen steps over 1.7 M entries 125 against 221 us.
#include <algorithm>

#include "common.hpp"

namespace {

using namespace dgnn;

constexpr int kSteps = DGNN_SERIES_STEPS;    // steps of one launch: what fits the kernel arguments and the LDS counters
constexpr int kRowTile = 256;                // rows (and threads) per workgroup of the row-pointer kernel
constexpr int kCountLd = kRowTile + 4;
constexpr int kThreads = 512;                // of the merge: a step is a chain of instructions, so few entries per thread
constexpr int kPerThread = 4;
constexpr int kCap = kThreads * kPerThread;  // entries of a stretch that LDS holds
constexpr int kTile = kCap * 3 / 4;          // entries of A_1 per stretch: it may grow by a third before it leaves the LDS
constexpr int kVmcntZero = 0x0F70;           // s_waitcnt operand: every vector memory access has completed
constexpr int kHalf = kThreads / 2;          // half of the workgroup places the added entries, the other half the deleted ones
constexpr int kAddsKept = 2;                 // added entries per thread and step, at most, on the LDS path

struct Series {
    int n, nnz1, steps, cap;
    const int32_t *rowptr1, *colidx1;
    dgnn_series_step s[kSteps];
};

// rowptr_t[r] = rowptr_1[r] + sum over the steps so far of (#added - #deleted with row < r); all steps of the launch.
__global__ __launch_bounds__(kRowTile) void series_rowptr_kernel(Series P) {
    __shared__ __attribute__((aligned(16))) int s_cnt[kSteps][kCountLd];   // net entries per row, then their exclusive sums
    __shared__ int s_bound[kSteps][4];                                     // of the tile: added begin, deleted begin, added end, deleted end
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int r0 = blockIdx.x * kRowTile, r1 = min(r0 + kRowTile, P.n);
    const int r = r0 + tid;
    const int rp0 = P.rowptr1[min(r, P.n)], rp1 = P.rowptr1[min(r + 1, P.n)];
    for (int i = tid; i < P.steps * kCountLd; i += kRowTile) (&s_cnt[0][0])[i] = 0;
    for (int q = tid; q < 4 * P.steps; q += kRowTile) {
        const dgnn_series_step &st = P.s[q >> 2];
        const int32_t *rows = (q & 1) ? st.del_row : st.add_row;
        const int len = (int)((q & 1) ? st.n_del : st.n_add);
        s_bound[q >> 2][q & 3] = lower4(0, len, (uint64_t)((q & 2) ? r1 : r0), [=](int i) { return (uint64_t)(uint32_t)rows[i]; });
    }
    block_lds_sync();
    for (int s = wave; s < P.steps; s += kRowTile / kWave) {            // a wavefront per step, four loads of a lane in flight
        const dgnn_series_step &st = P.s[s];
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
                if (q < (unsigned)kRowTile) atomicAdd(&s_cnt[s][q], j0 + k * kWave < na ? 1 : -1);
            }
        }
    }
    block_lds_sync();
    for (int s = wave; s < P.steps; s += kRowTile / kWave) {
        int4 v = *reinterpret_cast<const int4 *>(&s_cnt[s][4 * lane]);
        const int sum = v.x + v.y + v.z + v.w;
        const int incl = wave_scan_add(sum, lane);
        int run = incl - sum;
        int4 o;
        o.x = run; run += v.x;
        o.y = run; run += v.y;
        o.z = run; run += v.z;
        o.w = run; run += v.w;
        *reinterpret_cast<int4 *>(&s_cnt[s][4 * lane]) = o;
        if (lane == kWave - 1) s_cnt[s][kRowTile] = run;
    }
    block_lds_sync();
    if (r >= P.n) return;
    int acc = rp0, next = rp1;
    for (int s = 0; s < P.steps; ++s) {
        const int base = s_bound[s][0] - s_bound[s][1];
        acc += base + s_cnt[s][tid];
        next += base + s_cnt[s][tid + 1];
        P.s[s].rowptr[r] = acc;
        if (P.s[s].dinv) P.s[s].dinv[r] = 1.0f / sqrtf((float)(next - acc));
        if (r == P.n - 1) P.s[s].rowptr[P.n] = next;
    }
}

__global__ __launch_bounds__(kThreads) void series_merge_kernel(Series P) {
    __shared__ __attribute__((aligned(16))) uint64_t s_key[kCap];
    // per entry: kept << 16 | added entries that go right before it; then the exclusive sums of that ([kCap]: the total)
    __shared__ __attribute__((aligned(16))) uint32_t s_mark[kCap + 4];
    __shared__ int s_seg[kSteps][4];           // the stretch's parts of the lists: added begin, deleted begin, added end, deleted end
    __shared__ int s_start[kSteps];            // where the stretch begins in A_t
    __shared__ uint32_t s_wave[kThreads / kWave];
    __shared__ int s_rows[3];

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int e0 = blockIdx.x * kTile, e1 = min(e0 + kTile, P.nnz1);
    // rows of the first and last entry and of the one after (the next stretch's first key), searched side by side
    if (wave < 3) {
        const int row = wave_find_row(P.rowptr1, P.n, min(wave == 0 ? e0 : wave == 1 ? e1 - 1 : e1, P.nnz1 - 1), lane);
        if (lane == 0) s_rows[wave] = max(row, 0);
    }
    block_lds_sync();
    const int row_first = s_rows[0], row_last = s_rows[1];
    const uint64_t k_lo = e0 == 0 ? 0 : ((uint64_t)(uint32_t)row_first << 32) | (uint32_t)P.colidx1[e0];
    const uint64_t k_hi = e1 == P.nnz1 ? ~0ull : ((uint64_t)(uint32_t)s_rows[2] << 32) | (uint32_t)P.colidx1[e1];
    for (int q = tid; q < 4 * P.steps; q += kThreads) {
        const dgnn_series_step &st = P.s[q >> 2];
        const int len = (int)((q & 1) ? st.n_del : st.n_add);
        const uint64_t key = (q & 2) ? k_hi : k_lo;
        s_seg[q >> 2][q & 3] = key == 0 ? 0 : key == ~0ull ? len : lower_key((q & 1) ? st.del_row : st.add_row, (q & 1) ? st.del_col : st.add_col, 0, len, key);
    }
    for (int p = e1 - e0 + tid; p < kCap; p += kThreads) s_key[p] = ~0ull;    // beyond the stretch: above every key
    {   // keys of the stretch in A_1: a thread finds the row of its first entry and walks on
        constexpr int kOwn = kTile / kThreads;
        const int p0 = e0 + tid * kOwn;
        if (p0 < e1) {
            int lo = row_first, hi = row_last;                          // last row whose pointer is <= p0
            while (lo < hi) {
                const int mid = lo + ((hi - lo + 1) >> 1);
                if (P.rowptr1[mid] <= p0) lo = mid; else hi = mid - 1;
            }
            int row = lo, end = P.rowptr1[row + 1];
#pragma unroll
            for (int k = 0; k < kOwn; ++k) {
                const int p = p0 + k;
                if (p < e1) {
                    while (p >= end && row < row_last) end = P.rowptr1[++row + 1];
                    s_key[p - e0] = ((uint64_t)(uint32_t)row << 32) | (uint32_t)P.colidx1[p];
                }
            }
        }
    }
    block_lds_sync();
    if (wave == 0) {
        const int mine = lane < P.steps ? s_seg[lane][0] - s_seg[lane][1] : 0;
        const int incl = wave_scan_add(mine, lane);
        if (lane < P.steps) s_start[lane] = e0 + incl;
    }
#pragma unroll
    for (int k = 0; k < kPerThread; ++k) s_mark[tid * kPerThread + k] = 0;
    int cnt = e1 - e0;
    // Loads and stores are counted together and complete in order, so a list entry fetched one step ahead is waited for
    // together with the stores of the step in between, a trip to memory per step.  Therefore the lists of kGroup steps are
    // fetched at once, a group ahead.
    constexpr int kGroup = 4;
    const bool adds = uniform(wave) < kHalf / kWave;
    const int half_tid = adds ? tid : tid - kHalf;
    uint32_t row_next[kGroup], col_next[kGroup], row_now[kGroup], col_now[kGroup];
    auto fetch = [&](int first) {
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            const int s = min(first + q, P.steps - 1);
            const dgnn_series_step &st = P.s[s];
            const int from = uniform(s_seg[s][adds ? 0 : 1]), len = max(uniform(s_seg[s][adds ? 2 : 3]) - from, 0);
            row_next[q] = __builtin_amdgcn_raw_buffer_load_b32(buffer_of((adds ? st.add_row : st.del_row) + from, len), half_tid * 4, 0, 0);
            col_next[q] = __builtin_amdgcn_raw_buffer_load_b32(buffer_of((adds ? st.add_col : st.del_col) + from, len), half_tid * 4, 0, 0);
        }
    };
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
    fetch(0);
    int s = 0;
#pragma unroll 1
    for (; s < P.steps; ++s) {
        if (s % kGroup == 0) {
#pragma unroll
            for (int q = 0; q < kGroup; ++q) { row_now[q] = row_next[q]; col_now[q] = col_next[q]; }
            fetch(s + kGroup);
        }
        const dgnn_series_step &st = P.s[s];
        const int a0 = uniform(s_seg[s][0]), d0 = uniform(s_seg[s][1]), na = max(uniform(s_seg[s][2]) - a0, 0), nd = max(uniform(s_seg[s][3]) - d0, 0);
        if (na > kAddsKept * kHalf || cnt + na > kCap) break;           // too much for the LDS: the rest goes through memory
        uint32_t row_first = row_now[0], col_first = col_now[0];
#pragma unroll
        for (int q = 1; q < kGroup; ++q) {
            row_first = s % kGroup == q ? row_now[q] : row_first;
            col_first = s % kGroup == q ? col_now[q] : col_first;
        }
        const uint64_t list_first = ((uint64_t)row_first << 32) | col_first;
        block_lds_sync();                                               // keys and cleared marks are there (and s_start, the first time)
        uint64_t a_key[kAddsKept];
        int a_slot[kAddsKept];
        if (adds) {
#pragma unroll
            for (int k = 0; k < kAddsKept; ++k) {
                const int j = half_tid + k * kHalf;
                a_slot[k] = 0;
                if (j < na) {
                    a_key[k] = list_first;
                    if (k > 0) {                                        // rare: a step this full pays for its loads on the spot
                        a_key[k] = ((uint64_t)(uint32_t)st.add_row[a0 + j] << 32) | (uint32_t)st.add_col[a0 + j];
                        __builtin_amdgcn_s_waitcnt(kVmcntZero);
                    }
                    a_slot[k] = place_of(a_key[k]);
                    if (a_slot[k] < cnt) atomicAdd(&s_mark[a_slot[k]], 1u);
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
                if (p < cnt && s_key[p] == key) atomicOr(&s_mark[p], 1u << 16);
            }
        }
        block_lds_sync();
        // ---- exclusive sums of (kept << 16 | added before); an entry of a stretch of at most 2^15 fits either half
        uint32_t v[kPerThread], sum = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; k += 4) {
            const uintx4 m = *reinterpret_cast<const uintx4 *>(&s_mark[tid * kPerThread + k]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[k + q] = tid * kPerThread + k + q < cnt ? m[q] ^ (1u << 16) : 0;      // "deleted" -> "kept"
                sum += v[k + q];
            }
        }
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
#pragma unroll
        for (int k = 0; k < kPerThread; k += 4) {
            uintx4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) { o[q] = run; run += v[k + q]; }
            *reinterpret_cast<uintx4 *>(&s_mark[tid * kPerThread + k]) = o;
        }
        if (tid == 0) s_mark[kCap] = total;
        block_lds_sync();
        // ---- new places: old entries by the sums, added ones by their rank and the kept entries before their slot
        uint64_t key[kPerThread];
        int pos[kPerThread], a_pos[kAddsKept];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int p = tid + k * kThreads;
            pos[k] = kCap;
            if (p < cnt) {
                const uint32_t before = s_mark[p], own = s_mark[p + 1] - before;
                key[k] = s_key[p];
                if (own >> 16) pos[k] = (int)((before >> 16) + (before & 0xffffu) + (own & 0xffffu));
            }
        }
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k) {
            const int j = half_tid + k * kHalf;
            a_pos[k] = kCap;
            if (adds && j < na) a_pos[k] = j + (int)(s_mark[min(a_slot[k], cnt)] >> 16);
        }
        block_lds_sync();
        const int cnt_before = cnt;
        cnt = uniform(min((int)(total >> 16) + na, kCap));
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            if (pos[k] < kCap) s_key[pos[k]] = key[k];
            s_mark[tid * kPerThread + k] = 0;
        }
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k)
            if (a_pos[k] < kCap) s_key[a_pos[k]] = a_key[k];
        for (int p = cnt + tid; p < cnt_before; p += kThreads) s_key[p] = ~0ull;
        block_lds_sync();
        const int start = uniform(s_start[s]);
        const bool placed = start >= 0 && start < P.cap;                // always, for lists that keep the preconditions
        const __amdgpu_buffer_rsrc_t out = buffer_of(st.colidx + (placed ? start : 0), placed ? min(cnt, P.cap - start) : 0);
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int p = tid + k * kThreads;
            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)s_key[p], out, p * 4, 0, 0);
        }
    }
    // ---- a stretch that outgrew the LDS: the remaining steps from memory, every place from searches alone:
    // an old entry moves by the list entries before it, an added one comes behind the kept entries before it
    int from = s == 0 ? e0 : s_start[s - 1];
    for (; s < P.steps; ++s) {
        __syncthreads();                                                // what this workgroup stored last is visible to all of it
        const dgnn_series_step &st = P.s[s];
        const int32_t *rp = s == 0 ? P.rowptr1 : P.s[s - 1].rowptr, *ci = s == 0 ? P.colidx1 : P.s[s - 1].colidx;
        const int a0 = s_seg[s][0], d0 = s_seg[s][1], a1 = max(s_seg[s][2], a0), d1 = max(s_seg[s][3], d0);
        const int start = s_start[s];
        cnt = max(min(cnt, P.cap - from), 0);
        for (int i = tid; i < cnt; i += kThreads) {
            int lo = 0, hi = P.n - 1;
            while (lo < hi) {
                const int mid = lo + ((hi - lo + 1) >> 1);
                if (rp[mid] <= from + i) lo = mid; else hi = mid - 1;
            }
            const int32_t c = ci[from + i];
            const uint64_t key = ((uint64_t)(uint32_t)lo << 32) | (uint32_t)c;
            const int d = lower_key(st.del_row, st.del_col, d0, d1, key), a = lower_key(st.add_row, st.add_col, a0, a1, key);
            if (d < d1 && st.del_row[d] == lo && st.del_col[d] == c) continue;
            const int to = start + i - (d - d0) + (a - a0);
            if ((unsigned)to < (unsigned)P.cap) st.colidx[to] = c;
        }
        for (int j = a0 + tid; j < a1; j += kThreads) {
            const int row = st.add_row[j], c = st.add_col[j];
            if ((unsigned)row >= (unsigned)P.n) continue;
            const int lo = min(max(rp[row], from), from + cnt), hi = min(max(rp[row + 1], lo), from + cnt);
            const int i = lower_bound(ci, lo, hi, c) - from;
            const int d = lower_key(st.del_row, st.del_col, d0, d1, ((uint64_t)(uint32_t)row << 32) | (uint32_t)c);
            const int to = start + i - (d - d0) + (j - a0);
            if ((unsigned)to < (unsigned)P.cap) st.colidx[to] = c;
        }
        cnt += (a1 - a0) - (d1 - d0);
        from = start;
    }
}

}  // namespace

extern "C" int dgnn_delta_rebuild_series(int64_t n, const int32_t *rowptr_first, const int32_t *colidx_first, int64_t nnz_first,
                                         int32_t steps, const dgnn_series_step *step, int64_t cap, void *stream) {
    if (!rowptr_first || !colidx_first || (steps > 0 && !step)) return DGNN_ERR_NULL;
    if (n <= 0 || nnz_first <= 0 || steps < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz_first)) return DGNN_ERR_OVERFLOW;
    int64_t nnz = nnz_first;
    for (int k = 0; k < steps; ++k) {
        const dgnn_series_step &st = step[k];
        if (!st.rowptr || !st.colidx) return DGNN_ERR_NULL;
        if (st.n_add < 0 || st.n_del < 0) return DGNN_ERR_SHAPE;
        if ((st.n_add > 0 && (!st.add_row || !st.add_col)) || (st.n_del > 0 && (!st.del_row || !st.del_col))) return DGNN_ERR_NULL;
        if (!fits_index(nnz + st.n_add)) return DGNN_ERR_OVERFLOW;
        nnz += st.n_add - st.n_del;
        if (nnz < 0) return DGNN_ERR_SHAPE;
        if (nnz > cap) return DGNN_ERR_CAPACITY;
        // all steps are written by the same launches: every snapshot needs arrays of its own
        if (st.rowptr == rowptr_first || st.colidx == colidx_first) return DGNN_ERR_ALIAS;
        for (int j = std::max(0, k - kSteps); j < k; ++j)
            if (st.rowptr == step[j].rowptr || st.colidx == step[j].colidx) return DGNN_ERR_ALIAS;
    }
    hipStream_t s = (hipStream_t)stream;
    Series P;
    P.n = (int)n;
    P.cap = (int)std::min<int64_t>(cap, 2147483647LL);
    P.rowptr1 = rowptr_first;
    P.colidx1 = colidx_first;
    nnz = nnz_first;
    for (int done = 0; done < steps; done += P.steps) {
        P.steps = std::min(steps - done, kSteps);
        P.nnz1 = (int)nnz;
        for (int k = 0; k < P.steps; ++k) P.s[k] = step[done + k];
        hipLaunchKernelGGL(series_rowptr_kernel, dim3((unsigned)((n + kRowTile - 1) / kRowTile)), dim3(kRowTile), 0, s, P);
        DGNN_RETURN_IF_LAUNCH_FAILED();
        if (nnz > 0) {
            hipLaunchKernelGGL(series_merge_kernel, dim3((unsigned)((nnz + kTile - 1) / kTile)), dim3(kThreads), 0, s, P);
            DGNN_RETURN_IF_LAUNCH_FAILED();
        }
        for (int k = 0; k < P.steps; ++k) nnz += P.s[k].n_add - P.s[k].n_del;
        P.rowptr1 = P.s[P.steps - 1].rowptr;
        P.colidx1 = P.s[P.steps - 1].colidx;
    }
    return DGNN_OK;
}
