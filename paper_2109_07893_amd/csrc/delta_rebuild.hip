// On-GPU reconstruction of a snapshot from the previous one and a graph difference
// (Section "Graph-difference Based Input Transfer"): common = A_prev \ deleted,
// A_next = common U added, both kept as CSR of A + I with ascending duplicate-free rows.
//
// Because both difference lists arrive sorted by (row, col), no global prefix scan is needed:
//   rowptr_next[r] = rowptr_prev[r] + #added with row < r - #deleted with row < r
// and "#entries with row < r" is a lower bound in a sorted list.  Every tile is independent:
//   1. rowptr_kernel  (tiles of rows)         new row pointers, dinv = (row length)^(-1/2), and what the merge
//                                             has to know about the row in which each of its ranges begins
//                                             (in the workspace);
//   2. merge_kernel   (ranges of old entries) streams A_prev's column indices once: deleted entries
//      are struck out, added entries slotted in, a prefix sum per sub-tile gives the positions.
//      Ranges hold equal numbers of old entries, so hub rows of power-law graphs are spread over
//      many wavefronts, and an old entry costs one coalesced read and one coalesced write.
#include <algorithm>

#include "common.hpp"

namespace {

using namespace dgnn;

constexpr int kRowThreads = 256;
constexpr int kRowsPerThread = 4;          // rowptr_kernel moves a thread's rows as one 16-byte access: keep at 4
constexpr int kRowTile = kRowThreads * kRowsPerThread;
constexpr int kHeavyList = 8 * kRowTile;     // list entries per row tile beyond which counting walks no more (16: 21.2 instead of 19.4 us, see count_by_search)

constexpr int kPerLane = 8;                  // old entries per lane and sub-tile of the merge
constexpr int kSub = kWave * kPerLane;       // old entries per sub-tile, at most
constexpr int kWavesAtOnce = 4096;           // see merge_range_length
constexpr int kLongestShare = kSub * 13;     // ... entries
constexpr unsigned kLdsOfTwelve = 12800, kMergeLds = 6676, kMergeLdsUpdates = 8736;      // bytes: a twelfth of a CU's, and what the merge declares
constexpr int kBufferReach = (1 << 29) - 2;  // words behind a place that a store through a buffer descriptor can name (31 bits of bytes)

// The row in which a range of the merge begins: its extent in A_prev (rp, rp1) and in A_next (rn, rn1), and the stretch
// of the added list that belongs to it (as, ae); the deleted list's stretch follows from these.
struct RangeStart { int rp, rp1, rn, rn1, as, ae, row, pad; };

__device__ __forceinline__ void report(int32_t *status, int code) {
    if (!status) return;
    int old = *status;
    while (old == 0 || code < old) {
        int seen = atomicCAS(status, old, code);
        if (seen == old) break;
        old = seen;
    }
}

constexpr int kListPerThread = 4;           // consecutive list entries per thread and round of the walk below

// Per-row counts of a sorted row list restricted to [lo, hi), accumulated into LDS counters by
// run boundaries: the last element of a run adds (j + 1), the first subtracts j.
// A thread takes kListPerThread consecutive entries and their two neighbours, all loaded before any is looked at,
// so that a tile's usual stretch of a list costs one trip to memory.
__device__ __forceinline__ void count_runs(const int32_t *__restrict__ rows, int lo, int hi, int r0, int nr, int *cnt, int tid) {
#pragma unroll 1
    for (int base = lo; base < hi; base += kRowThreads * kListPerThread) {
        const int j0 = base + tid * kListPerThread;
        int r[kListPerThread + 2];        // rows[j0 - 1 .. j0 + kListPerThread]; -1 stands for "outside [lo, hi)"
#pragma unroll
        for (int k = 0; k < kListPerThread + 2; ++k) {
            const int j = j0 - 1 + k;
            r[k] = (j >= lo && j < hi) ? rows[j] : -1;
        }
#pragma unroll
        for (int k = 0; k < kListPerThread; ++k) {
            const int j = j0 + k;
            const unsigned q = (unsigned)(r[k + 1] - r0);
            if (j < hi && q < (unsigned)nr) {
                if (r[k + 2] != r[k + 1]) atomicAdd(&cnt[q], j + 1);     // last of its run
                if (r[k] != r[k + 1]) atomicSub(&cnt[q], j);             // first of its run
            }
        }
    }
}

// The lists that change a snapshot's rows: added entries and deleted ones.
constexpr int kLists = 2;

// The same counts from lower bounds, for every list that `heavy` names: thread t finds where each of its rows begins inside
// [lo, hi).  All searches of a thread advance in lock step, so the whole costs as many trips to memory as one search (one search
// after the other, each starting where the last had ended, was what the kernel took: R-MAT, 2^19 vertices, 8.9 M entries,
// 3 % churn with value updates 46.5 us, then 19.4).
__device__ __forceinline__ void count_by_search(const int32_t *const (&rows)[kLists], const int (&lo)[kLists], const int (&hi)[kLists],
                                                const bool (&heavy)[kLists], int r0, int nr, int (*cnt)[kRowTile], int tid) {
    int pos[kLists][kRowsPerThread + 1], longest = 0;
#pragma unroll
    for (int l = 0; l < kLists; ++l) {
        if (heavy[l]) longest = max(longest, hi[l] - lo[l]);
#pragma unroll
        for (int k = 0; k <= kRowsPerThread; ++k) pos[l][k] = lo[l];
    }
    auto key = [&](int k) { return r0 + min(tid * kRowsPerThread + k, nr); };
#pragma unroll 1
    for (int step = 1 << (31 - __clz(longest)); step > 0; step >>= 1) {
        int v[kLists][kRowsPerThread + 1];
#pragma unroll
        for (int l = 0; l < kLists; ++l)
            if (heavy[l])
#pragma unroll
                for (int k = 0; k <= kRowsPerThread; ++k) v[l][k] = rows[l][pos[l][k] + min(step, hi[l] - pos[l][k]) - 1];   // (a sum with step itself may pass 2^31)
#pragma unroll
        for (int l = 0; l < kLists; ++l)
            if (heavy[l])
#pragma unroll
                for (int k = 0; k <= kRowsPerThread; ++k)
                    if (step <= hi[l] - pos[l][k] && v[l][k] < key(k)) pos[l][k] += step;      // entries before pos have smaller rows
    }
#pragma unroll
    for (int l = 0; l < kLists; ++l)
        if (heavy[l])
#pragma unroll
            for (int k = 0; k < kRowsPerThread; ++k) cnt[l][tid * kRowsPerThread + k] = pos[l][k + 1] - pos[l][k];
}

// How many entries of each ascending list a[l][0 .. len[l]) lie below key[l]: 64-ary searches of the wavefront, in lock step.
template <int LISTS>
__device__ __forceinline__ void wave_count_below(const int32_t *const (&a)[LISTS], const int (&len)[LISTS], const int (&key)[LISTS], int lane, int (&below)[LISTS]) {
    int hi[LISTS];
    bool more = false;
#pragma unroll
    for (int l = 0; l < LISTS; ++l) {
        below[l] = 0;
        hi[l] = len[l];
        more |= len[l] > 0;
    }
    while (more) {
        int v[LISTS];
#pragma unroll
        for (int l = 0; l < LISTS; ++l) {
            const int at = below[l] + lane * ((hi[l] - below[l] + kWave - 1) / kWave);
            v[l] = at < hi[l] ? a[l][at] : key[l];
        }
        more = false;
#pragma unroll
        for (int l = 0; l < LISTS; ++l) {
            const int step = (hi[l] - below[l] + kWave - 1) / kWave, m = __popcll(__ballot(v[l] < key[l]));
            const int from = below[l];
            below[l] = m ? from + (m - 1) * step + 1 : from;
            hi[l] = m ? min(from + m * step, hi[l]) : from;
            more |= hi[l] > below[l];
        }
    }
}

// VEC: rowptr_prev, rowptr_next and dinv are 16-byte aligned, so a thread moves its four rows with one access each.
template <bool VEC>
__global__ __launch_bounds__(kRowThreads) void rowptr_kernel(
    int n, const int32_t *__restrict__ rowptr_prev,
    const int32_t *__restrict__ add_row, int n_add, const int32_t *__restrict__ del_row, int n_del,
    int32_t *__restrict__ rowptr_next, float *__restrict__ dinv,
    int range_len, int n_ranges, RangeStart *__restrict__ range_start, int32_t *status) {
    __shared__ int s_cnt[kLists][kRowTile];     // entries per row of the added and deleted lists
    __shared__ int s_bound[4];
    __shared__ int s_wsum[kLists][kRowThreads / kWave];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int r0 = blockIdx.x * kRowTile;
    const int r1 = min(r0 + kRowTile, n);
    const int nr = r1 - r0;
    const int r_own = r0 + tid * kRowsPerThread;          // this thread's rows: r_own .. r_own + 3
    const bool whole = r_own + kRowsPerThread <= n;       // all four exist

    if (blockIdx.x == 0 && tid == 0 && status) *status = 0;
    // the pointers of the thread's rows and the one after, on their way while the searches run
    int rp[kRowsPerThread + 1];
    if (VEC && whole) {
        const int4 v = *reinterpret_cast<const int4 *>(rowptr_prev + r_own);
        rp[0] = v.x; rp[1] = v.y; rp[2] = v.z; rp[3] = v.w;
        rp[4] = rowptr_prev[r_own + kRowsPerThread];
    } else {
#pragma unroll
        for (int k = 0; k <= kRowsPerThread; ++k) rp[k] = r_own + k <= n ? rowptr_prev[r_own + k] : 0;
    }
    {   // how many list entries have a row below r0 / below r1: one 64-ary search per wavefront and list
        const int found = wave_find_row(wave < 2 ? add_row : del_row, wave < 2 ? n_add : n_del, ((wave & 1) ? r1 : r0) - 1, lane);
        if (lane == 0) s_bound[wave] = found + 1;
    }
    for (int i = tid; i < kRowTile; i += kRowThreads)
#pragma unroll
        for (int l = 0; l < kLists; ++l) s_cnt[l][i] = 0;
    __syncthreads();
    // A tile of hub rows can own a very long stretch of a list; walking it would leave the whole chip
    // waiting for this workgroup, so there the counts come from one lower bound per row instead.
    const int32_t *const rows[kLists] = {add_row, del_row};
    const int lo[kLists] = {s_bound[0], s_bound[2]}, hi[kLists] = {s_bound[1], s_bound[3]};
    bool heavy[kLists], any_heavy = false;
#pragma unroll
    for (int l = 0; l < kLists; ++l) {
        heavy[l] = hi[l] - lo[l] > kHeavyList;
        any_heavy |= heavy[l];
        if (!heavy[l]) count_runs(rows[l], lo[l], hi[l], r0, nr, s_cnt[l], tid);
    }
    if (any_heavy) count_by_search(rows, lo, hi, heavy, r0, nr, s_cnt, tid);
    __syncthreads();

    int ca[kRowsPerThread], cd[kRowsPerThread];
    int sum[kLists] = {0, 0}, inc[kLists];
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
        ca[k] = s_cnt[0][tid * kRowsPerThread + k];
        cd[k] = s_cnt[1][tid * kRowsPerThread + k];
        sum[0] += ca[k];
        sum[1] += cd[k];
    }
#pragma unroll
    for (int l = 0; l < kLists; ++l) {
        inc[l] = wave_scan_add(sum[l], lane);
        if (lane == kWave - 1) s_wsum[l][wave] = inc[l];
    }
    __syncthreads();
    int oa = lo[0] + inc[0] - sum[0], od = lo[1] + inc[1] - sum[1];      // exclusive offsets of this thread's first row
    for (int w = 0; w < wave; ++w) { oa += s_wsum[0][w]; od += s_wsum[1][w]; }

    int rn[kRowsPerThread];
    float dv[kRowsPerThread];
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
        const int r = r_own + k;
        const int p = rp[k], q = rp[k + 1];
        rn[k] = p + oa - od;
        dv[k] = 1.0f / sqrtf((float)(q - p + ca[k] - cd[k]));
        if (r < r1) {
            // ranges of the merge that begin inside this row (few rows hold a multiple of the range length; a hub
            // row several): what the merge needs to know about the row, so that it starts without a search
            for (int g = max((p + range_len - 1) / range_len, 0); g < n_ranges && (int64_t)g * range_len < q; ++g)
                range_start[g] = RangeStart{p, q, p + oa - od, q + oa + ca[k] - od - cd[k], oa, oa + ca[k], r, 0};
        }
        oa += ca[k];
        od += cd[k];
    }
    if (VEC && whole) {
        *reinterpret_cast<int4 *>(rowptr_next + r_own) = make_int4(rn[0], rn[1], rn[2], rn[3]);
        if (dinv) *reinterpret_cast<float4 *>(dinv + r_own) = make_float4(dv[0], dv[1], dv[2], dv[3]);
    } else {
#pragma unroll
        for (int k = 0; k < kRowsPerThread; ++k)
            if (r_own + k < r1) {
                rowptr_next[r_own + k] = rn[k];
                if (dinv) dinv[r_own + k] = dv[k];
            }
    }
    if (r1 == n && tid == 0) rowptr_next[n] = rowptr_prev[n] + n_add - n_del;
}

// How many entries of a list sorted by (row, column) come before (row, col): a 64-ary search of the wavefront.
__device__ __forceinline__ int wave_count_before(const int32_t *__restrict__ rows, const int32_t *__restrict__ cols, int len, int row, int col, int lane) {
    int lo = 0, hi = len;
    while (hi > lo) {
        const int step = (hi - lo + kWave - 1) / kWave, at = lo + lane * step;
        const bool in = at < hi;
        const int r = in ? rows[at] : 0, c = in ? cols[at] : 0;
        const int m = __popcll(__ballot(in && (r < row || (r == row && c < col))));
        if (m == 0) break;                       // the first one does not: lo come before
        hi = min(lo + m * step, hi);
        lo += (m - 1) * step + 1;
    }
    return lo;
}

// For K stretches [pos, hi) of an ascending LDS array at once (hi >= pos): moves pos to the first element >= key.  Element p of the
// array is a[p + 1]; a[0] is only read.  All searches advance in lock step, five trips to the LDS where no stretch of the
// wavefront is longer than 31 elements.
template <int K>
__device__ __forceinline__ void lds_bound(const int *a, int (&pos)[K], const int (&hi)[K], const int (&key)[K]) {
    auto round = [&](int step) {
        int to[K], v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            to[k] = min(pos[k] + step, hi[k]);
            v[k] = a[to[k]];                     // the element before it; where nothing is left, the move is none
        }
#pragma unroll
        for (int k = 0; k < K; ++k) pos[k] = v[k] < key[k] ? to[k] : pos[k];
    };
    bool far = false;
#pragma unroll
    for (int k = 0; k < K; ++k) far |= hi[k] - pos[k] > 31;
    if (__ballot(far))
#pragma unroll 1
        for (int step = kSub; step >= 32; step >>= 1) round(step);
#pragma unroll
    for (int step = 16; step > 0; step >>= 1) round(step);
}

// One wavefront streams a contiguous range of old entries in sub-tiles of kSub entries.
// The work per OLD entry is a load, a position from a prefix sum, and a store; everything that
// needs a search is done per DIFFERENCE entry, of which there are few:
//   - the sub-tile's column indices are staged in LDS; each deleted entry that falls into the
//     sub-tile finds its old entry there by binary search and marks it dead, each added entry
//     finds the old entry it goes in front of (its slot) and counts itself there;
//   - where the row of a difference entry lies inside the sub-tile comes from the row pointers of A_prev, which
//     the wavefront streams beside the column indices: the pointers of the rows that meet the sub-tile (from the
//     row that holds its first entry on) are staged in LDS as well, fetched one sub-tile ahead like the column
//     indices, so a list entry (row, col) looks its row's extent up there and no load depends on another;
//   - both lists are consumed in order through two cursors, so the lists are never searched
//     (except once, where a range begins in the middle of a row); where a range's first row lies in A_prev,
//     in A_next and in the lists comes from rowptr_kernel;
//   - one prefix sum over (alive, added-before) gives every old entry and every slot its place
//     relative to the sub-tile's first output position; that position follows from rowptr_next
//     at the start of the range and simply advances by what each sub-tile wrote.
// Lane l owns entries l, l + 64, ... of the sub-tile, so loads and stores coalesce; the column
// indices of the next sub-tile are fetched while this one is placed.
// What bounds it is the instructions beside these two streams, so the accesses go through buffer descriptors: no branch and no
// 64-bit address per access, and what lies outside is 0 or dropped; the loads in flight can then be counted, so that a sub-tile waits
// for its own and not for the last one's stores.  us per rebuild, this form and its ranges against a branch per access, a search per list and
// 16384 ranges or ranges of 8192: R-MAT, 4.2 M entries 24.7 -> 18.8, 17 M 54.2 -> 41.2, 140 M 350 -> 333, 280 M 665 -> 657
// (the merge alone 545: 4.1 TB/s of column indices);
// with values and updates for nearly all 8.5 M entries 101 -> 77, for a tenth of 9 M 59 -> 48.
// VALUES: every stored entry carries a value, which travels with its column index (same position); added
// entries bring theirs.  UPDATES (with VALUES): a third list, sorted like the other two, names surviving entries
// that get a new value; it is consumed through a cursor of its own, each entry finds its old entry in the staged
// columns as a deleted entry does and leaves the new value there.  An entry that names nothing stored is passed over.
// The list may be long: AHEAD batches of 64 of its entries are fetched ahead, eight where most entries have an update, as in the first steps of a
// smoothed series (figures in rebuild()); the place of a range's first update is found here, where it is wanted once, and not per row in
// rowptr_kernel.
// FAR: a sub-tile may leave more entries than a buffer's offsets reach (kBufferReach): positions are kept whole, and the stores
// find their addresses themselves.
template <bool VALUES, int AHEAD, bool FAR>
__global__ __launch_bounds__(kWave) void merge_kernel(
    int n, const int32_t *__restrict__ rowptr_prev, const int32_t *__restrict__ colidx_prev, int nnz_prev, int range_len,
    const int32_t *__restrict__ add_row, const int32_t *__restrict__ add_col, int n_add,
    const int32_t *__restrict__ del_row, const int32_t *__restrict__ del_col, int n_del,
    const RangeStart *__restrict__ range_start,
    int32_t *__restrict__ colidx_next, int cap_next,
    const float *__restrict__ val_prev, const float *__restrict__ add_val, float *__restrict__ val_next,
    const int32_t *__restrict__ upd_row, const int32_t *__restrict__ upd_col, const float *__restrict__ upd_val, int n_upd) {
    constexpr bool UPDATES = AHEAD > 0;
    constexpr int kBatches = UPDATES ? AHEAD : 1;
    constexpr int kWindow = 2 * kWave;      // row pointers fetched ahead for every sub-tile; more are fetched when rows are short
    constexpr int kMaxWindow = kSub + kWave;
    constexpr unsigned kDropped = 0x80000000u;   // an offset that no buffer here reaches
    __shared__ int s_col[1 + kSub];              // from s_col[1] on
    __shared__ __align__(16) int s_mark[kSub + kWave];   // bit 0: deleted; bit 1: new value in s_newval; bits 2..: added entries that go right before this slot
    // Until the prefix sums are taken: s_rows[k] = rowptr_prev[first_row + k], the rows that meet the sub-tile.
    // From then on: s_start[p] / 4 = outputs (kept + added) that precede slot p's block; its low bits are the mark's of entry p - 1 (FAR:
    // the outputs, and the marks stay where they are).
    __shared__ __align__(16) int s_shared[kMaxWindow + 4];
    __shared__ float s_newval[UPDATES ? kSub : 1];
    int *const s_rows = s_shared;
    int *const s_start = s_shared + 3;           // (16-byte alignment from s_start[1] on)
    static_assert(kMaxWindow >= kWindow + kWave, "the window must be able to grow");

    const int lane = threadIdx.x;
    const int e_begin = (int)((int64_t)blockIdx.x * range_len);
    const int e_end = (int)min((int64_t)e_begin + range_len, (int64_t)nnz_prev);
    constexpr int kNone = 0x7fffffff;    // a pointer "beyond everything"

    // the range's column indices and values
    const __amdgpu_buffer_rsrc_t col_in = buffer_of(colidx_prev + e_begin, e_end - e_begin);
    const __amdgpu_buffer_rsrc_t val_in = buffer_of(VALUES ? val_prev + e_begin : nullptr, VALUES ? e_end - e_begin : 0);
    auto word = [](__amdgpu_buffer_rsrc_t from, int at) { return (int)__builtin_amdgcn_raw_buffer_load_b32(from, at * 4, 0, 0); };
    int c_next[kPerLane];
    float v_next[VALUES ? kPerLane : 1];
    auto fetch_entries = [&](int e) {
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            c_next[j] = word(col_in, e - e_begin + lane + j * kWave);
            if (VALUES) v_next[j] = __int_as_float(word(val_in, e - e_begin + lane + j * kWave));
        }
    };
    fetch_entries(e_begin);

    // ---- start of the range: its row, the list cursors, the first output position
    int a_cur, d_cur;   // first added / deleted entry not yet placed
    int u_cur = 0;      // first value update not yet looked at
    int base;           // output position of the next entry to be written
    int first_row;      // the row that holds the sub-tile's first entry
    // the pointers of rows first_row + lane and first_row + 64 + lane, for the next sub-tile (behind the last row: the number of entries)
    int w0, w1;
    auto fetch_window = [&](int row) {
        w0 = rowptr_prev[row + min(lane, n - row)];
        w1 = rowptr_prev[row + min(kWave + lane, n - row)];
    };
    {
        const RangeStart st = range_start[blockIdx.x];                     // the row that holds entry e_begin
        const int c_at = colidx_prev[e_begin], c_before = colidx_prev[max(e_begin - 1, 0)];
        const int rp = st.rp, rp1 = st.rp1, rn = st.rn, rn1 = st.rn1, as = st.as, ae = st.ae;
        const int ds = rp + as - rn, de = rp1 + ae - rn1;
        first_row = uniform(min(max(st.row, 0), n - 1));
        fetch_window(first_row);
        a_cur = as;
        d_cur = ds;
        if (rp < e_begin) {   // the range begins inside the row: skip what earlier ranges place
            // (both lists at once, 64 entries a trip: most ranges of a hub row start here)
            const bool in_a = as >= 0 && as < ae && ae <= n_add, in_d = ds >= 0 && ds < de && de <= n_del;
            const int32_t *list[2] = {add_col + (in_a ? as : 0), del_col + (in_d ? ds : 0)};
            int len[2] = {in_a ? ae - as : 0, in_d ? de - ds : 0}, key[2] = {c_before, c_at}, below[2];
            wave_count_below<2>(list, len, key, lane, below);
            a_cur += below[0];
            d_cur += below[1];
        }
        if (UPDATES) u_cur = uniform(wave_count_before(upd_row, upd_col, n_upd, st.row, rp < e_begin ? c_at : 0, lane));
        a_cur = uniform(min(max(a_cur, 0), n_add));
        d_cur = uniform(min(max(d_cur, 0), n_del));
        base = uniform(rn + (e_begin - rp) - (d_cur - ds) + (a_cur - as));
    }
    // The 64 list entries at each cursor (row, column) are fetched ahead of use, for every sub-tile anew: it consumes only some of
    // them, but the others are in the caches, and sliding them down costs more.  An entry that does not exist reads as 0.
    constexpr int kVmcntZero = 0x0F70;   // s_waitcnt operand: every vector memory load has returned, other counters untouched
    auto at_cursor = [&](const void *list, int len, int cur) {
        const bool some = cur < len;
        return word(buffer_of(some ? (const int32_t *)list + cur : nullptr, some ? min(len - cur, kWave) : 0), lane);
    };
    int pa_row, pa_col, pd_row, pd_col, pu_row[kBatches], pu_col[kBatches];
    float pa_val = 0.0f, pu_val[kBatches];
    auto load_added = [&] {
        pa_row = at_cursor(add_row, n_add, a_cur);
        pa_col = at_cursor(add_col, n_add, a_cur);
        if (VALUES) pa_val = __int_as_float(at_cursor(add_val, n_add, a_cur));
    };
    auto load_deleted = [&] {
        pd_row = at_cursor(del_row, n_del, d_cur);
        pd_col = at_cursor(del_col, n_del, d_cur);
    };
    auto load_batch = [&](int b) {
        const int from = u_cur + min(b * kWave, n_upd - u_cur);
        pu_row[b] = at_cursor(upd_row, n_upd, from);
        pu_col[b] = at_cursor(upd_col, n_upd, from);
        pu_val[b] = __int_as_float(at_cursor(upd_val, n_upd, from));
    };
    auto load_updates = [&] {
#pragma unroll
        for (int b = 0; b < kBatches; ++b) load_batch(b);
    };
    load_added();
    load_deleted();
    if (UPDATES) load_updates();

    for (int e = e_begin; e < e_end; e += kSub) {
        const int e_stop = min(e + kSub, e_end);
        const int cnt = e_stop - e;
        int c_[kPerLane];
        float v_[VALUES ? kPerLane : 1];
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            c_[j] = c_next[j];
            if (VALUES) v_[j] = v_next[j];
            s_col[1 + lane + j * kWave] = c_[j];
            s_mark[lane + j * kWave] = 0;
        }
        s_mark[kSub + lane] = 0;
        if (cnt < kSub) {                            // behind the last entry nothing is kept
            wave_lds_sync();
            for (int p = cnt + lane; p < kSub; p += kWave) s_mark[p] = 1;
        }
        // ---- the rows that meet the sub-tile: their pointers go to LDS; `below` counts the staged pointers that are
        // <= e_stop, so the row that holds entry e_stop (the next sub-tile's first) is first_row + below - 1
        s_rows[lane] = w0;
        s_rows[kWave + lane] = w1;
        int n_win = kWindow;
        int last = __builtin_amdgcn_readlane(w1, kWave - 1);
        int below = __popcll(__ballot(w0 <= e_stop)) + __popcll(__ballot(w1 <= e_stop));
#pragma unroll 1
        while (last < e_stop && n_win + kWave <= kMaxWindow) {      // short rows: the sub-tile reaches beyond the window
            const int v = rowptr_prev[first_row + min(n_win + lane, n - first_row)];
            s_rows[n_win + lane] = v;
            below += __popcll(__ballot(v <= e_stop));
            last = __builtin_amdgcn_readlane(v, kWave - 1);
            n_win += kWave;
        }
        const int row0 = first_row;                  // the window staged now starts here
        first_row = min(first_row + max(below, 1) - 1, n - 1);
        // fetched while this sub-tile is placed; behind the range's last one too, so that the loads in flight can be counted
        fetch_entries(e_stop);
        fetch_window(first_row);
        wave_lds_sync();

        // where a list entry's row lies in A_prev, from the staged pointers: rows outside the window do not meet the sub-tile
        auto extent = [&](int row, int &lo, int &hi) {
            const unsigned k = (unsigned)(row - row0);
            lo = hi = kNone;
            if (k < (unsigned)(n_win - 1)) {
                lo = s_rows[k];
                hi = s_rows[k + 1];
            }
        };
        // the stretch of the sub-tile in which the entry of a row is looked for, if the row has entries here
        auto stretch = [&](bool exists, int row, int &r_lo, int &r_hi, int &lo, int &hi) {
            extent(row, r_lo, r_hi);
            const bool here = exists && r_lo < e_stop && r_hi > e;
            lo = here ? max(r_lo - e, 0) : 0;
            hi = here ? min(r_hi - e, cnt) : 0;
            return here;
        };
        // ---- of the first 64 entries of every list, which are in registers: where they belong.  A sub-tile with more than that
        // of one list is rare and pays for its loads on the spot.
        constexpr int kSearches = UPDATES ? 3 : 2;
        int r_lo[kSearches], r_hi[kSearches], at[kSearches], hi[kSearches], key[kSearches];
        bool here[kSearches];
        const int a_tile = a_cur;
        here[0] = stretch(d_cur + lane < n_del, pd_row, r_lo[0], r_hi[0], at[0], hi[0]);
        here[1] = stretch(a_cur + lane < n_add, pa_row, r_lo[1], r_hi[1], at[1], hi[1]);
        key[0] = pd_col;
        key[1] = pa_col + 1;                         // behind an equal one
        if constexpr (UPDATES) {
            here[2] = stretch(u_cur + lane < n_upd, pu_row[0], r_lo[2], r_hi[2], at[2], hi[2]);
            key[2] = pu_col[0];
        }
        lds_bound<kSearches>(s_col, at, hi, key);

        // ---- deleted entries: mark the old entry dead
        auto strike = [&](bool here, int p, int hi) {
            const bool owned = here && p < hi && s_col[1 + p] == pd_col;
            if (owned) atomicOr(&s_mark[p], 1);
            return __popcll(__ballot(owned));
        };
        auto search_one = [&](int lo, int hi, int key) {
            int p[1] = {lo}, h[1] = {hi}, k[1] = {key};
            lds_bound<1>(s_col, p, h, k);
            return p[0];
        };
        int d_got = strike(here[0], at[0], hi[0]);
#pragma unroll 1
        while (d_got == kWave) {
            d_cur += kWave;
            load_deleted();
            __builtin_amdgcn_s_waitcnt(kVmcntZero);
            int r0, r1, lo, h;
            const bool in = stretch(d_cur + lane < n_del, pd_row, r0, r1, lo, h);
            d_got = strike(in, search_one(lo, h, pd_col), h);
        }
        d_cur += d_got;
        // ---- value updates: leave the new value at the old entry.  An entry is done with once its place in A_prev's
        // order lies before the end of this sub-tile, whether something is stored there or not.
        if constexpr (UPDATES) {
            auto touch = [&](int b, bool here, int r_lo, int r_hi, int p, int hi) {
                const bool exists = u_cur + lane < n_upd;
                bool done = exists && pu_row[b] < row0;           // a row before the sub-tile's first: nothing left to find
                if (here && p < hi) {
                    done = true;
                    if (s_col[1 + p] == pu_col[b]) {
                        s_newval[p] = pu_val[b];
                        atomicOr(&s_mark[p], 2);
                    }
                } else if (exists && r_lo < e_stop) {
                    done |= r_hi <= e_stop;                       // beyond the sub-tile's part of an unfinished row: later
                }
                return __popcll(__ballot(done));
            };
            auto find_and_touch = [&](int b) {
                int r0, r1, lo, h;
                const bool in = stretch(u_cur + lane < n_upd, pu_row[b], r0, r1, lo, h);
                return touch(b, in, r0, r1, search_one(lo, h, pu_col[b]), h);
            };
            int u_got = touch(0, here[2], r_lo[2], r_hi[2], at[2], hi[2]);
#pragma unroll
            for (int b = 1; b < kBatches; ++b)
                if (u_got == kWave) {
                    u_cur += kWave;
                    u_got = find_and_touch(b);
                }
                else break;
#pragma unroll 1
            while (u_got == kWave) {
                u_cur += kWave;
                load_batch(0);
                __builtin_amdgcn_s_waitcnt(kVmcntZero);
                u_got = find_and_touch(0);
            }
            u_cur += u_got;
        }
        // ---- added entries: count at the slot (old entry they precede; a row's end if none)
        auto slot = [&](bool here, int r_hi, int &q, int hi) {
            const bool owned = here && (q < hi || r_hi <= e_stop);        // beyond the sub-tile's part of an unfinished row: later
            if (owned) atomicAdd(&s_mark[q], 4); else q = -2 - lane;
            return __popcll(__ballot(owned));
        };
        int q_first = at[1];                      // slot, column and value of the first 64, kept for the write below
        const int c_first = pa_col;
        const float av_first = pa_val;
        int a_got = slot(here[1], r_hi[1], q_first, hi[1]);
#pragma unroll 1
        while (a_got == kWave) {
            a_cur += kWave;
            load_added();
            __builtin_amdgcn_s_waitcnt(kVmcntZero);
            int r0, r1, lo, h;
            const bool in = stretch(a_cur + lane < n_add, pa_row, r0, r1, lo, h);
            int q = search_one(lo, h, pa_col + 1);
            a_got = slot(in, r1, q, h);
        }
        a_cur += a_got;
        // the list entries at the new cursors, for the next sub-tile
        load_added();
        load_deleted();
        if (UPDATES) load_updates();
        wave_lds_sync();

        // ---- prefix sums: s_start[p] = kept entries before p + added entries of slots before p (the staged row
        // pointers are not needed any more; their place is taken)
        int written;
        {
            int mk[kPerLane], sum = 0;
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                mk[j] = s_mark[lane * kPerLane + j];
                sum += (mk[j] >> 2) + (~mk[j] & 1);
            }
            const int inc = wave_scan_add(sum, lane);
            int run = inc - sum;
            if (lane == 0) s_start[0] = 0;
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                run += (mk[j] >> 2) + (~mk[j] & 1);
                s_start[lane * kPerLane + j + 1] = FAR ? run : (run << 2) | (mk[j] & 3);
            }
            written = uniform(__builtin_amdgcn_readlane(inc, kWave - 1) + (s_mark[kSub] >> 2));
        }
        wave_lds_sync();

        // the entries from one before `base` on: a kept entry's place is one before what precedes the next slot
        const int room = (unsigned)base < (unsigned)cap_next ? min(cap_next - base, kBufferReach) + 1 : 0;
        const __amdgpu_buffer_rsrc_t col_out = buffer_of(colidx_next + (int64_t)base - 1, room);
        const __amdgpu_buffer_rsrc_t val_out = buffer_of(VALUES ? val_next + (int64_t)base - 1 : nullptr, VALUES ? room : 0);
        auto put = [&](unsigned offset, int c, float v) {
            __builtin_amdgcn_raw_buffer_store_b32(c, col_out, offset, 0, 0);
            if (VALUES) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), val_out, offset, 0, 0);
        };
        auto put_far = [&](bool kept, int place, int c, float v) {       // place: from 1 on, as above
            const unsigned pos = (unsigned)base + (unsigned)place - 1u;
            if (kept && pos < (unsigned)cap_next) {
                colidx_next[pos] = c;
                if (VALUES) val_next[pos] = v;
            }
        };
        // ---- old entries
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const int p = lane + j * kWave;
            const unsigned s = (unsigned)s_start[p + 1], mark = FAR ? (unsigned)s_mark[p] : s;
            float v = VALUES ? v_[j] : 0.0f;
            if (UPDATES) v = (mark & 2u) ? s_newval[p] : v;
            if (FAR) put_far(!(mark & 1u), (int)s, c_[j], v);
            else put((s & ~3u) | (s << 31), c_[j], v);         // the deleted ones are dropped
        }
        // ---- added entries: their slot, then the rank among the adds of the same slot (they are consecutive).
        // The first 64 kept their slot and column from the search above; more than 64 per sub-tile are rare.
        int q_carry = -1, rank_carry = 0;
        auto place = [&](int j, int q, int c, float v) {
            const int q_left = __shfl_up(q, 1, kWave);
            const bool head = lane == 0 ? q != q_carry : q != q_left;
            const unsigned long long true_heads = __ballot(head);
            const unsigned long long upto = (true_heads | 1ull) & (~0ull >> (kWave - 1 - lane));
            const int run_start = 63 - __clzll(upto);
            int rank = lane - run_start;
            if (run_start == 0 && !(true_heads & 1ull)) rank += rank_carry;   // run continues from the previous 64
            if (FAR) put_far(j < a_cur, s_start[max(q, 0)] + rank + 1, c, v);
            else put(j < a_cur ? ((unsigned)s_start[max(q, 0)] & ~3u) + 4u * (unsigned)(rank + 1) : kDropped, c, v);
            q_carry = __shfl(q, kWave - 1, kWave);
            rank_carry = __shfl(rank, kWave - 1, kWave) + 1;
        };
        if (a_tile < a_cur) place(a_tile + lane, q_first, c_first, av_first);
#pragma unroll 1
        for (int j0 = a_tile + kWave; j0 < a_cur; j0 += kWave) {
            // these search again; the extent of an entry's row comes from the row pointers themselves, two loads that
            // depend on the entry's, which a sub-tile this full can afford
            const int j = j0 + lane;
            int lo = 0, h = 0, c = 0;
            float v = 0.0f;
            bool there = false;
            if (j < a_cur) {
                const int r = add_row[j];
                c = add_col[j];
                if (VALUES) v = add_val[j];
                if ((unsigned)r < (unsigned)n) {
                    there = true;
                    h = max(min(rowptr_prev[r + 1] - e, cnt), 0);
                    lo = min(max(rowptr_prev[r] - e, 0), h);
                }
            }
            const int q = search_one(lo, h, c + 1);
            place(j, there ? q : -2 - lane, c, v);
        }
        base += written;
        wave_lds_sync();           // LDS is rewritten by the next sub-tile
    }
}

// Surviving entries whose value changes, for an update list in no particular order: one thread per listed entry
// finds it in its (new) row and overwrites the value.  Entries that are not there are skipped.  cap: entries that the arrays hold;
// row pointers that came out of lists which break the preconditions can point anywhere.
__global__ __launch_bounds__(256) void update_values_kernel(int n, const int32_t *__restrict__ rowptr, int cap,
                                                            const int32_t *__restrict__ colidx,
                                                            const int32_t *__restrict__ upd_row,
                                                            const int32_t *__restrict__ upd_col,
                                                            const float *__restrict__ upd_val, int n_upd,
                                                            float *__restrict__ val) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_upd) return;
    const int r = upd_row[j], c = upd_col[j];
    if ((unsigned)r >= (unsigned)n) return;
    const int lo = max(rowptr[r], 0), hi = min(rowptr[r + 1], cap);
    const int p = lower_bound(colidx, lo, hi, c);
    if (p < hi && colidx[p] == c) val[p] = upd_val[j];
}

// One thread per difference entry (added first, then deleted), then one per row of A_prev.
__global__ __launch_bounds__(256) void validate_kernel(
    int n, const int32_t *__restrict__ rowptr_prev, const int32_t *__restrict__ colidx_prev,
    const int32_t *__restrict__ add_row, const int32_t *__restrict__ add_col, int n_add,
    const int32_t *__restrict__ del_row, const int32_t *__restrict__ del_col, int n_del, int32_t *status) {
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)n_add + n_del) {
        int64_t r = g - n_add - n_del;
        if (r < n && rowptr_prev[r + 1] <= rowptr_prev[r]) report(status, DGNN_BAD_EMPTY_ROW);
        return;
    }
    const bool is_add = g < n_add;
    const int j = is_add ? (int)g : (int)(g - n_add);
    const int32_t *rows = is_add ? add_row : del_row;
    const int32_t *cols = is_add ? add_col : del_col;
    const int r = rows[j], c = cols[j];
    if (r < 0 || r >= n || c < 0 || c >= n) { report(status, DGNN_BAD_INDEX_RANGE); return; }
    if (j > 0) {
        int pr = rows[j - 1], pc = cols[j - 1];
        if (pr > r || (pr == r && pc >= c)) report(status, DGNN_BAD_DELTA_ORDER);
    }
    if (r == c) { report(status, DGNN_BAD_DIAGONAL); return; }
    int lo = rowptr_prev[r], hi = rowptr_prev[r + 1];
    if (lo < 0 || hi < lo) return;
    int q = lower_bound(colidx_prev, lo, hi, c);
    bool present = q < hi && colidx_prev[q] == c;
    if (is_add && present) report(status, DGNN_BAD_ADD_PRESENT);
    if (!is_add && !present) report(status, DGNN_BAD_DEL_ABSENT);
}

// One thread per row: its pointers, then its columns one after the other (rows are short on average; a hub row
// keeps one thread busy for its length, which a check that runs once per uploaded snapshot can afford).
__global__ __launch_bounds__(256) void csr_validate_kernel(int n, const int32_t *__restrict__ rowptr,
                                                           const int32_t *__restrict__ colidx, int nnz, int require_diagonal,
                                                           int32_t *status) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int lo = rowptr[r], hi = rowptr[r + 1];
    if ((r == 0 && lo != 0) || (r == n - 1 && hi != nnz) || lo < 0 || hi < lo || hi > nnz) {
        report(status, DGNN_BAD_ROWPTR);
        return;                                             // the row's extent cannot be trusted
    }
    bool diagonal = false;
    int prev = -1;
    for (int e = lo; e < hi; ++e) {
        const int c = colidx[e];
        if (c < 0 || c >= n) { report(status, DGNN_BAD_INDEX_RANGE); return; }
        if (c <= prev) { report(status, DGNN_BAD_ROW_ORDER); return; }
        diagonal |= c == r;
        prev = c;
    }
    if (require_diagonal && !diagonal) report(status, DGNN_BAD_NO_DIAGONAL);
}

// One thread per entry of a value-update list that is declared sorted: indices in range, strictly ascending by (row, col).
__global__ __launch_bounds__(256) void validate_updates_kernel(int n, const int32_t *__restrict__ upd_row,
                                                               const int32_t *__restrict__ upd_col, int n_upd, int32_t *status) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n_upd) return;
    const int r = upd_row[j], c = upd_col[j];
    if (r < 0 || r >= n || c < 0 || c >= n) { report(status, DGNN_BAD_INDEX_RANGE); return; }
    if (j > 0) {
        const int pr = upd_row[j - 1], pc = upd_col[j - 1];
        if (pr > r || (pr == r && pc >= c)) report(status, DGNN_BAD_DELTA_ORDER);
    }
}

__global__ __launch_bounds__(64) void reset_status_kernel(int32_t *status) { *status = 0; }

__global__ __launch_bounds__(256) void dinv_kernel(int n, const int32_t *__restrict__ rowptr, float *__restrict__ dinv) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < n) dinv[r] = 1.0f / sqrtf((float)(rowptr[r + 1] - rowptr[r]));
}

}  // namespace

extern "C" int dgnn_csr_validate(int64_t n, const int32_t *rowptr, const int32_t *colidx, int64_t nnz, int require_diagonal,
                                 int32_t *d_status, void *stream) {
    if (!rowptr || !d_status || (nnz > 0 && !colidx)) return DGNN_ERR_NULL;
    if (n <= 0 || nnz < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz)) return DGNN_ERR_OVERFLOW;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(reset_status_kernel, dim3(1), dim3(64), 0, s, d_status);     // a fill kernel: capturable
    DGNN_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(csr_validate_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (int)n, rowptr, colidx, (int)nnz,
                       require_diagonal, d_status);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

extern "C" const char *dgnn_strerror(int code) {
    switch (code) {
        case DGNN_OK: return "ok";
        case DGNN_ERR_NULL: return "a required pointer is NULL";
        case DGNN_ERR_SHAPE: return "bad size, feature width, window or dtype";
        case DGNN_ERR_CAPACITY: return "output buffer or workspace too small";
        case DGNN_ERR_OVERFLOW: return "n or nnz does not fit in int32";
        case DGNN_ERR_ALIAS: return "output aliases an input";
        case DGNN_ERR_HIP: return "HIP runtime error";
        case DGNN_ERR_ALIGN: return "feature pointer not 16-byte aligned";
        default: return "unknown dgnn status";
    }
}

extern "C" int dgnn_csr_dinv(int64_t n, const int32_t *rowptr, float *dinv, void *stream) {
    if (!rowptr || !dinv) return DGNN_ERR_NULL;
    if (n <= 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n)) return DGNN_ERR_OVERFLOW;
    hipLaunchKernelGGL(dinv_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       (int)n, rowptr, dinv);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

extern "C" int dgnn_delta_h2d(const int32_t *h_add_row, const int32_t *h_add_col, int64_t n_add,
                              const int32_t *h_del_row, const int32_t *h_del_col, int64_t n_del,
                              int32_t *d_add_row, int32_t *d_add_col, int32_t *d_del_row, int32_t *d_del_col,
                              void *stream) {
    if (n_add < 0 || n_del < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n_add) || !fits_index(n_del)) return DGNN_ERR_OVERFLOW;
    if (n_add > 0 && (!h_add_row || !h_add_col || !d_add_row || !d_add_col)) return DGNN_ERR_NULL;
    if (n_del > 0 && (!h_del_row || !h_del_col || !d_del_row || !d_del_col)) return DGNN_ERR_NULL;
    hipStream_t s = (hipStream_t)stream;
    const void *src[4] = {h_add_row, h_add_col, h_del_row, h_del_col};
    void *dst[4] = {d_add_row, d_add_col, d_del_row, d_del_col};
    const int64_t cnt[4] = {n_add, n_add, n_del, n_del};
    for (int k = 0; k < 4; ++k) {
        if (cnt[k] == 0) continue;
        if (hipMemcpyAsync(dst[k], src[k], (size_t)cnt[k] * sizeof(int32_t), hipMemcpyHostToDevice, s) != hipSuccess)
            return DGNN_ERR_HIP;
    }
    return DGNN_OK;
}

namespace {

// The workspace holds a record per range of any snapshot of at most nnz_prev entries, so that one sized for the largest snapshot of a
// block serves every step: 40 bytes per 8192 entries, never less than 16386 times, as callers are told.
constexpr int64_t kRoomEntries = 8192, kRoomBytes = 40, kLeastRoom = 16385;
int64_t workspace_records(int64_t nnz_prev) { return std::max<int64_t>(kLeastRoom, (nnz_prev + kRoomEntries - 1) / kRoomEntries) + 1; }
static_assert(kLeastRoom * kRoomBytes >= kWavesAtOnce * (int64_t)sizeof(RangeStart), "records of one generation fit");

// Entries per wavefront of the merge, a multiple of the sub-tile.  Up to 27 M stored entries all wavefronts are one generation that the
// device holds at once (16 on a CU, as registers and LDS allow every variant), so that no range pays for its start a second time.  Beyond, ranges are
// as short as their records fit the workspace, so that wavefronts end together; with updates, whose place a range has to search for, no shorter than
// eight sub-tiles, nine where the updates are many.  A generation of eight sub-tiles, 16 KB of entries, is slower than its neighbours and takes
// nine (uniform, with values: 14.5 M entries, 7 / 8 / 9 sub-tiles 59.3 / 65.2 / 59.3; 16 M 8 / 9 75.2 / 69.6).  us per rebuild, uniform graphs, by
// sub-tiles to a range (* one generation): without values 14 M 4: 36.3, 7*: 33.9, 13: 38.4;
// 22 M 4: 49.6, 11*: 48.0; 27 M 4: 59.4, 13*: 56.7; 31 M 3: 78.1, 9: 82.0, 13: 82.3, 15*: 81.2; 56 M 6: 131.4, 13: 133.8; R-MAT 40 M 4: 93.9, 13: 105.8;
// with values 31 M 3: 126, 13: 138; 56 M 6: 225, 13: 236; with an update for 3 entries of 10, 30 M 4: 187, 9: 171, 13: 193, 15*: 169; 56 M 9: 306, 13: 324.
bool few_updates(int64_t nnz_prev, int64_t n_upd) { return n_upd <= nnz_prev / 5; }
int64_t merge_range_length(int64_t nnz_prev, int64_t n_upd) {
    auto dealt = [&](int64_t ranges) { return ((nnz_prev + ranges - 1) / ranges + kSub - 1) / kSub * kSub; };
    const int64_t generation = dealt(kWavesAtOnce);
    if (generation <= kLongestShare) return generation == 8 * kSub ? 9 * kSub : generation;
    const int64_t least = dealt(workspace_records(nnz_prev) * kRoomBytes / (int64_t)sizeof(RangeStart));
    return n_upd > 0 ? std::max<int64_t>(least, (few_updates(nnz_prev, n_upd) ? 8 : 9) * kSub) : least;
}

}  // namespace

extern "C" int dgnn_delta_rebuild_workspace(int64_t n, int64_t nnz_prev, int64_t n_add, int64_t n_del, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (n <= 0 || nnz_prev < 0 || n_add < 0 || n_del < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz_prev + n_add)) return DGNN_ERR_OVERFLOW;
    *bytes = round_up((size_t)workspace_records(nnz_prev) * kRoomBytes, 256);   // the row every range of the merge begins in
    return DGNN_OK;
}

namespace {

struct Values {
    const float *prev;
    const float *add;
    float *next;
    // value updates the merge consumes (sorted by (row, col)); n_upd = 0: none
    const int32_t *upd_row;
    const int32_t *upd_col;
    const float *upd_val;
    int64_t n_upd;
};

int rebuild(int64_t n, const int32_t *rowptr_prev, const int32_t *colidx_prev, int64_t nnz_prev,
            const int32_t *add_row, const int32_t *add_col, int64_t n_add,
            const int32_t *del_row, const int32_t *del_col, int64_t n_del,
            int32_t *rowptr_next, int32_t *colidx_next, int64_t cap_next, int64_t *nnz_next, float *dinv_next,
            const Values *vals, void *ws, size_t ws_bytes, uint32_t flags, int32_t *d_status, void *stream) {
    if (!rowptr_prev || !colidx_prev || !rowptr_next || !colidx_next || !ws) return DGNN_ERR_NULL;
    if (n_add < 0 || n_del < 0) return DGNN_ERR_SHAPE;
    if (n_add > 0 && (!add_row || !add_col)) return DGNN_ERR_NULL;
    if (n_del > 0 && (!del_row || !del_col)) return DGNN_ERR_NULL;
    if (vals && (!vals->prev || !vals->next || (n_add > 0 && !vals->add))) return DGNN_ERR_NULL;
    if (n <= 0 || nnz_prev <= 0 || (flags & ~(vals ? DGNN_VALIDATE | DGNN_UPDATES_SORTED : DGNN_VALIDATE))) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz_prev + n_add)) return DGNN_ERR_OVERFLOW;
    const int64_t nnz_new = nnz_prev + n_add - n_del;
    if (nnz_new < 0) return DGNN_ERR_SHAPE;
    if (cap_next < nnz_new) return DGNN_ERR_CAPACITY;
    const int64_t n_upd = vals ? vals->n_upd : 0;
    size_t need = 0;
    int rc = dgnn_delta_rebuild_workspace(n, nnz_prev, n_add, n_del, &need);
    if (rc != DGNN_OK) return rc;
    if (ws_bytes < need) return DGNN_ERR_CAPACITY;
    if (rowptr_next == rowptr_prev || colidx_next == colidx_prev) return DGNN_ERR_ALIAS;
    if (vals && vals->next == vals->prev) return DGNN_ERR_ALIAS;
    if (nnz_next) *nnz_next = nnz_new;

    hipStream_t s = (hipStream_t)stream;
    char *wsb = static_cast<char *>(ws);
    RangeStart *range_start = reinterpret_cast<RangeStart *>(wsb);
    const int cap = (int)min(cap_next, (int64_t)2147483647LL);
    const int64_t range_len = merge_range_length(nnz_prev, n_upd);
    const int n_ranges = (int)((nnz_prev + range_len - 1) / range_len);

    const dim3 row_grid((unsigned)((n + kRowTile - 1) / kRowTile));
    if (aligned16(rowptr_prev) && aligned16(rowptr_next) && aligned16(dinv_next))
        hipLaunchKernelGGL(rowptr_kernel<true>, row_grid, dim3(kRowThreads), 0, s, (int)n, rowptr_prev, add_row, (int)n_add, del_row,
                           (int)n_del, rowptr_next, dinv_next, (int)range_len, n_ranges, range_start, d_status);
    else
        hipLaunchKernelGGL(rowptr_kernel<false>, row_grid, dim3(kRowThreads), 0, s, (int)n, rowptr_prev, add_row, (int)n_add, del_row,
                           (int)n_del, rowptr_next, dinv_next, (int)range_len, n_ranges, range_start, d_status);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    if ((flags & DGNN_VALIDATE) && d_status) {
        int64_t work = n_add + n_del + n;
        hipLaunchKernelGGL(validate_kernel, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, s,
                           (int)n, rowptr_prev, colidx_prev, add_row, add_col, (int)n_add, del_row, del_col,
                           (int)n_del, d_status);
        DGNN_RETURN_IF_LAUNCH_FAILED();
        if (n_upd > 0) {
            hipLaunchKernelGGL(validate_updates_kernel, dim3((unsigned)((n_upd + 255) / 256)), dim3(256), 0, s, (int)n, vals->upd_row,
                               vals->upd_col, (int)n_upd, d_status);
            DGNN_RETURN_IF_LAUNCH_FAILED();
        }
    }
    const dim3 grid((unsigned)n_ranges);
    // (a sub-tile leaves no more than its own entries and all that is added)
    const bool far = n_add > kBufferReach - kSub;
    // Many generations with values: twelve wavefronts on a CU instead of 16 or 20, by LDS that nobody uses.  With more of them at work the
    // lists' lines, of which a sub-tile takes a part, are gone from the L2 when the next one comes for the rest: R-MAT, 69 M entries, without
    // updates 306 / 292 us (all that fit / twelve), one for 50 entries 324 / 313, for 10 342 / 328, 280 M 1180 / 1120, 1250 / 1202, 1323 / 1274.
    // Where updates are many it is their chain of batches that counts: one for 3 of 10 entries, 44 M 246 / 267, 69 M 382 / 406.
    const unsigned lds = n_ranges > kWavesAtOnce && few_updates(nnz_prev, n_upd) ? kLdsOfTwelve : 0;
    // Eight batches ahead from three updates for five entries on: fewer of them are fetched in vain (us with one / eight: 8.5 M entries, for 3 of
    // 10 entries 49.5 / 61.2, 5 of 10 56.1 / 64.7, 7 of 10 63.8 / 67.1, all 77.5 / 70.9; 17 M 99 / 117, 117 / 123, 132 / 125, 166 / 140).
    if (vals && n_upd > 0)
        hipLaunchKernelGGL((far ? merge_kernel<true, 1, true> : n_upd > nnz_prev * 3 / 5 ? merge_kernel<true, 8, false> : merge_kernel<true, 1, false>), grid,
                           dim3(kWave), lds ? lds - kMergeLdsUpdates : 0, s, (int)n, rowptr_prev, colidx_prev,
                           (int)nnz_prev, (int)range_len, add_row, add_col, (int)n_add, del_row, del_col, (int)n_del, range_start, colidx_next, cap,
                           vals->prev, vals->add, vals->next, vals->upd_row, vals->upd_col, vals->upd_val, (int)n_upd);
    else if (vals)
        hipLaunchKernelGGL((far ? merge_kernel<true, 0, true> : merge_kernel<true, 0, false>), grid, dim3(kWave), lds ? lds - kMergeLds : 0, s, (int)n, rowptr_prev, colidx_prev, (int)nnz_prev,
                           (int)range_len, add_row, add_col, (int)n_add, del_row, del_col, (int)n_del, range_start, colidx_next, cap,
                           vals->prev, vals->add, vals->next, nullptr, nullptr, nullptr, 0);
    else
        hipLaunchKernelGGL((far ? merge_kernel<false, 0, true> : merge_kernel<false, 0, false>), grid, dim3(kWave), 0, s, (int)n, rowptr_prev, colidx_prev, (int)nnz_prev,
                           (int)range_len, add_row, add_col, (int)n_add, del_row, del_col, (int)n_del, range_start, colidx_next, cap,
                           nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

}  // namespace

extern "C" int dgnn_delta_rebuild(int64_t n,
                                  const int32_t *rowptr_prev, const int32_t *colidx_prev, int64_t nnz_prev,
                                  const int32_t *add_row, const int32_t *add_col, int64_t n_add,
                                  const int32_t *del_row, const int32_t *del_col, int64_t n_del,
                                  int32_t *rowptr_next, int32_t *colidx_next, int64_t cap_next, int64_t *nnz_next,
                                  float *dinv_next,
                                  void *ws, size_t ws_bytes, uint32_t flags, int32_t *d_status, void *stream) {
    return rebuild(n, rowptr_prev, colidx_prev, nnz_prev, add_row, add_col, n_add, del_row, del_col, n_del, rowptr_next,
                   colidx_next, cap_next, nnz_next, dinv_next, nullptr, ws, ws_bytes, flags, d_status, stream);
}

extern "C" int dgnn_delta_rebuild_weighted(int64_t n,
                                           const int32_t *rowptr_prev, const int32_t *colidx_prev, const float *val_prev,
                                           int64_t nnz_prev,
                                           const int32_t *add_row, const int32_t *add_col, const float *add_val, int64_t n_add,
                                           const int32_t *del_row, const int32_t *del_col, int64_t n_del,
                                           const int32_t *upd_row, const int32_t *upd_col, const float *upd_val, int64_t n_upd,
                                           int32_t *rowptr_next, int32_t *colidx_next, float *val_next, int64_t cap_next,
                                           int64_t *nnz_next,
                                           void *ws, size_t ws_bytes, uint32_t flags, int32_t *d_status, void *stream) {
    if (n_upd < 0) return DGNN_ERR_SHAPE;
    if (n_upd > 0 && (!upd_row || !upd_col || !upd_val)) return DGNN_ERR_NULL;
    if (!fits_index(n_upd)) return DGNN_ERR_OVERFLOW;
    const bool folded = (flags & DGNN_UPDATES_SORTED) && n_upd > 0;      // the merge takes the updates itself
    const Values vals{val_prev, add_val, val_next, upd_row, upd_col, upd_val, folded ? n_upd : 0};
    const int rc = rebuild(n, rowptr_prev, colidx_prev, nnz_prev, add_row, add_col, n_add, del_row, del_col, n_del,
                           rowptr_next, colidx_next, cap_next, nnz_next, nullptr, &vals, ws, ws_bytes, flags, d_status, stream);
    if (rc != DGNN_OK || n_upd == 0 || folded) return rc;
    hipLaunchKernelGGL(update_values_kernel, dim3((unsigned)((n_upd + 255) / 256)), dim3(256), 0, (hipStream_t)stream, (int)n,
                       rowptr_next, (int)std::min<int64_t>(cap_next, 2147483647LL), colidx_next, upd_row, upd_col, upd_val, (int)n_upd, val_next);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}
