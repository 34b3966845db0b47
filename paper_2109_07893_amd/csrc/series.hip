// A whole series of snapshots from its first one and the graph differences, for callers that have the difference lists of
// several steps at hand: the raw ones A_2 .. A_{S+1} (Section "Graph-difference Based Input Transfer") in one
// or two launches, the smoothed ones S_2 .. S_{S+1} (Section "Smoothening the Input Graphs") in four.  S_t holds every entry of A_{t-l+1} .. A_t
// with the number of these snapshots that hold it as its value; l = 1 would be A_t.
//
// One step after the other reads A_{t-1} back from memory for every A_t, S_{t-1}, A_t and A_{t-l} for every S_t, and pays two
// (nine) launches per step.  Here a workgroup takes a stretch of the keys (row, column), between two entries of A_1, through
// the whole series at once, whatever happens elsewhere (the lists are sorted by the same key):
//   - it forms the sorted union of its entries over ALL steps in LDS: A_1's, and everything the lists add.  The entry an added
//     one precedes is searched, counted there, and a prefix sum over the counts places old and new ones; an added entry ranks
//     itself among the others of its slot.  (An entry that is added twice gets two places; the second stays empty.)
//   - with each entry goes a word, bit t: A_{t+1} holds it.  An entry of A_1 begins with all bits set, an added one with none,
//     and a list that names it in step s turns the bits from s + 1 on;
//   - A_t (S_t) is then the entries with bit t (any of the l bits up to t) set, in order: per step and 64 entries a ballot,
//     and, once the ballots of all steps have been counted, a store at the place the counts give.  Entries never move.
// Where a stretch begins in A_t follows from the list positions of its first key,
//     start_t = start_1 + sum over the steps so far of (#added before the key - #deleted before the key);
// in S_t it depends on how many entries the others remember: a first launch only counts, series_scan_kernel turns the counts
// into places, and a second one writes.
// Row pointers and normalisation of the raw snapshots come from tiles of rows, which count the lists' entries per row, in the
// same launch; the row sums of S_t are the row lengths of the last l snapshots less the extra self loops, so its normalisation
// comes from the same counts; its row pointers from the ballots, by the stretch in which the row begins.
// What bounds it: the set-up of a stretch (searches through its LDS keys, a prefix sum, eleven barriers: 6 us of dependent
// instructions, three workgroups per CU at a time, 9 us per million entries), then the stores, per step 14 vector instructions
// for 64 entries.  Seven steps over 11 thousand entries 13 us, fifteen over 1.7 M entries 80 us (rebuilt one after the other 94
// and 234 us); moving a stretch's entries to their new places in every step instead took 32 and 125 us.  Five smoothed snapshots
// of 4.4 M entries 162 us, 340 us when the entries moved, 940 us one after the other.
#include <algorithm>
#include <cstddef>

#include "common.hpp"

namespace {

using namespace dgnn;

constexpr int kSteps = DGNN_SERIES_STEPS;    // steps of one launch: a word of bits per entry, the first for A_1
constexpr int kThreads = 512, kWaves = kThreads / kWave;
constexpr int kPerThread = 4;
constexpr int kCap = kThreads * kPerThread;  // entries of a stretch's union
constexpr int kChunks = kCap / kWave;        // of 64 entries, dealt to the wavefronts in turn
constexpr int kAddsKept = 2;                 // added entries per thread, all steps together
constexpr int kDelsKept = 1;                 // deleted ones; further ones are read again where they are needed
constexpr int kAddCap = kAddsKept * kThreads;
constexpr int kRowTile = 256;                // rows per workgroup of the row part
constexpr int kCountLd = kRowTile + 4;
constexpr int kLeastTile = 256;
constexpr int kScanThreads = 1024;

enum Mode { kRaw, kCount, kWrite };          // raw snapshots; smoothed ones, counting and writing

struct Series {
    int n, nnz1, steps, cap, life, tile, stretches, row_tiles, found;
    float diag;
    const int32_t *rowptr1, *colidx1;
    int32_t *bounds;                         // [stretches + 1][2 steps + 2], valid if `found`: places in the lists, row and column of the entry
    int32_t *counts, *d_status;              // [steps][stretches]; [steps]
    dgnn_smooth_step s[kSteps];
};

// The difference lists, copied to LDS by wavefront-uniform (scalar) loads: the lanes of a search take different steps, and
// vector loads from the kernel arguments are not cached.
struct Lists {
    const int32_t *row[kSteps][2], *col[kSteps][2];      // added, deleted
    int len[kSteps][2];
    void *out[kSteps][2];                                // colidx, val
};
__device__ __forceinline__ void copy_lists(const Series &P, Lists &lists, int lane, int first, int stride) {
    for (int s = first; s < P.steps; s += stride) {
        const dgnn_smooth_step &st = P.s[s];
        if (lane < 2) {
            lists.out[s][lane] = lane ? (void *)st.val : (void *)st.colidx;
            lists.row[s][lane] = lane ? st.del_row : st.add_row;
            lists.col[s][lane] = lane ? st.del_col : st.add_col;
            lists.len[s][lane] = (int)(lane ? st.n_del : st.n_add);
        }
    }
}

struct RowPart {
    Lists lists;
    alignas(16) int net[kSteps][kCountLd];   // entries per row, added less deleted, then (raw) their exclusive sums
    int bound[kSteps][4];                    // of the tile: added begin, deleted begin, added end, deleted end
};
struct StretchPart {
    Lists lists;
    uint64_t key[kCap];
    uint32_t bits[kCap];
    union {
        struct {
            alignas(16) int before[kCap + 4];   // added entries per slot, then their exclusive sums
            uint64_t added[kAddCap];         // by slot
        } build;
        struct {
            uint64_t held[kSteps][kChunks];  // ballots
            int place[kSteps][kChunks];      // their counts, then the exclusive sums
        } write;
    };
    int seg[kSteps][4];                      // the keys' parts of the lists: added begin, deleted begin, added end, deleted end
    int first_add[32], first_del[32];        // exclusive sums of the parts' lengths
    int start[kSteps];                       // where the keys at hand begin in the snapshot (kCount: how many have been counted)
    int sums[kWaves];
    int bound[2][2], total_add, total_del;   // row and column at either end
};
static_assert(kSteps < 32, "a word of bits, and places for the ends of the parts");
static_assert(offsetof(RowPart, net) % 16 == 0 && kCountLd % 4 == 0 && offsetof(StretchPart, build.before) % 16 == 0, "taken four words at a time");

// Row pointers and dinv of every raw snapshot, or dinv of every smoothed one, for a tile of rows.
template <Mode MODE>
__device__ __forceinline__ void rows_of_series(const Series &P, RowPart &L, int tile) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int r0 = tile * kRowTile, r1 = min(r0 + kRowTile, P.n), r = r0 + tid;
    const int rp0 = P.rowptr1[min(r, P.n)], rp1 = P.rowptr1[min(r + 1, P.n)];
    for (int i = tid; i < P.steps * kCountLd; i += kThreads) (&L.net[0][0])[i] = 0;
    copy_lists(P, L.lists, lane, uniform(wave), kWaves);
    block_lds_sync();
    for (int q = tid; q < 4 * P.steps; q += kThreads) {
        const int32_t *rows = as_global(L.lists.row[q >> 2][q & 1]);
        const int len = L.lists.len[q >> 2][q & 1];
        L.bound[q >> 2][q & 3] = lower4(0, len, (uint64_t)((q & 2) ? r1 : r0), [=](int i) { return (uint64_t)(uint32_t)rows[i]; });
    }
    block_lds_sync();
    for (int s = wave; s < P.steps; s += kWaves) {                      // a wavefront per step, four loads of a lane in flight
        const dgnn_smooth_step &st = P.s[s];
        const int32_t *add_row = as_global(st.add_row), *del_row = as_global(st.del_row);
        const int a0 = L.bound[s][0], d0 = L.bound[s][1], na = max(L.bound[s][2] - a0, 0), nd = max(L.bound[s][3] - d0, 0);
#pragma unroll 1
        for (int j0 = lane; j0 < na + nd; j0 += 4 * kWave) {
            int row[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int j = j0 + k * kWave;
                row[k] = j < na ? add_row[a0 + j] : j < na + nd ? del_row[d0 + j - na] : -1;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned q = (unsigned)(row[k] - r0);
                if (q < (unsigned)kRowTile) atomicAdd(&L.net[s][q], j0 + k * kWave < na ? 1 : -1);
            }
        }
    }
    block_lds_sync();
    if (MODE == kRaw) {
        for (int s = wave; s < P.steps; s += kWaves) {
            int4 v = *reinterpret_cast<const int4 *>(&L.net[s][4 * lane]);
            const int sum = v.x + v.y + v.z + v.w;
            const int incl = wave_scan_add(sum, lane);
            int run = incl - sum;
            int4 o;
            o.x = run; run += v.x;
            o.y = run; run += v.y;
            o.z = run; run += v.z;
            o.w = run; run += v.w;
            *reinterpret_cast<int4 *>(&L.net[s][4 * lane]) = o;
            if (lane == kWave - 1) L.net[s][kRowTile] = run;
        }
        block_lds_sync();
    }
    if (tid >= kRowTile || r >= P.n) return;
    if (MODE == kRaw) {
        // rowptr_t[r] = rowptr_1[r] + sum over the steps so far of (#added - #deleted with row < r)
        int acc = rp0, next = rp1;
        for (int s = 0; s < P.steps; ++s) {
            const int base = L.bound[s][0] - L.bound[s][1];
            acc += base + L.net[s][tid];
            next += base + L.net[s][tid + 1];
            as_global(P.s[s].rowptr)[r] = acc;
            if (P.s[s].dinv) as_global(P.s[s].dinv)[r] = 1.0f / sqrtf((float)(next - acc));
            if (r == P.n - 1) as_global(P.s[s].rowptr)[P.n] = next;
        }
    } else {
        int deg = rp1 - rp0, oldest = deg, sum = deg;                   // of A_t, of A_{t-l}, of the window's snapshots
        for (int s = 0; s < P.steps; ++s) {
            deg += L.net[s][tid];
            sum += deg;
            if (s + 1 >= P.life) {
                sum -= oldest;
                if (s + 1 < P.steps) oldest += L.net[s + 1 - P.life][tid];
            }
            float total = (float)sum;
            if (P.diag != 0.0f) total = (float)(sum - min(s + 2, P.life)) + P.diag;      // every snapshot holds the diagonal
            if (P.s[s].dinv) as_global(P.s[s].dinv)[r] = total > 0.0f ? 1.0f / sqrtf(total) : 0.0f;
        }
    }
}

// The first entry of a sorted list that is not below `key`, looked for around `guess` first (lists favour no part of the
// snapshot very much, so the place is known to within a few times the square root of the length).
__device__ __forceinline__ int lower_key_near(const int32_t *row, const int32_t *col, int len, uint64_t key, int guess) {
    auto get = [=](int i) { return ((uint64_t)(uint32_t)row[i] << 32) | (uint32_t)col[i]; };
    const int reach = 2 * (int)sqrtf((float)len) + 2;
    int lo = max(guess - reach, 0), hi = min(guess + reach, len);
    const uint64_t at_lo = lo > 0 ? get(lo - 1) : 0, at_hi = hi < len ? get(hi) : ~0ull;
    if (lo > 0 && at_lo >= key) { hi = lo - 1; lo = 0; }
    else if (hi < len && at_hi < key) { lo = hi + 1; hi = len; }
    return lower4(lo, hi, key, get);
}

// Where `key`, in front of entry e of A_1, lies in the lists: lane 2 s in the added ones of step s, lane 2 s + 1 in the deleted
// ones.
__device__ __forceinline__ int list_place(const Series &P, const Lists &lists, uint64_t key, int e, int lane) {
    if (lane >= 2 * P.steps) return 0;
    const int len = lists.len[lane >> 1][lane & 1];
    if (key == 0 || key == ~0ull) return key == 0 ? 0 : len;
    return lower_key_near(as_global(lists.row[lane >> 1][lane & 1]), as_global(lists.col[lane >> 1][lane & 1]), len, key,
                          (int)((int64_t)len * e / P.nnz1));
}

__device__ __forceinline__ uint64_t key_of_entry(const Series &P, int e, int lane, int &row) {
    row = max(uniform(wave_find_row(as_global(P.rowptr1), P.n, e, lane)), 0);
    return ((uint64_t)(uint32_t)row << 32) | (uint32_t)as_global(P.colidx1)[e];
}

// The key in front of stretch b (the end behind the last one), and the row of its entry.
__device__ __forceinline__ uint64_t bound_key(const Series &P, int b, int lane, int &row) {
    const int e = (int)min((int64_t)b * P.tile, (int64_t)P.nnz1);
    row = e == 0 ? 0 : P.n - 1;
    return e > 0 && e < P.nnz1 ? key_of_entry(P, e, lane, row) : e == 0 ? 0 : ~0ull;
}

// The bounds of all stretches beforehand: a workgroup that finds its own spends half its time on these searches, which is
// hidden behind nothing once there are more workgroups than fit the chip.
__global__ __launch_bounds__(kWave) void series_bounds_kernel(Series P) {
    __shared__ Lists lists;
    const int lane = threadIdx.x;
    copy_lists(P, lists, lane, 0, 1);
    wave_lds_sync();
    int row;
    const uint64_t key = bound_key(P, blockIdx.x, lane, row);
    const int at = list_place(P, lists, key, (int)min((int64_t)blockIdx.x * P.tile, (int64_t)P.nnz1), lane), words = 2 * P.steps + 2;
    if (lane < words) as_global(P.bounds)[(int64_t)blockIdx.x * words + lane] = lane == words - 2 ? row : lane == words - 1 ? (int)(uint32_t)key : at;
}

template <Mode MODE>
__device__ __forceinline__ void stretch_of_series(const Series &P, StretchPart &L, int stretch) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid / kWave);
    const int32_t *rowptr1 = as_global(P.rowptr1), *colidx1 = as_global(P.colidx1);
    const int e0 = stretch * P.tile, e1 = min(e0 + P.tile, P.nnz1);
    copy_lists(P, L.lists, lane, (wave + kWaves - 2) % kWaves, kWaves);
    const int words = 2 * P.steps + 2;
    if (wave < 2) {                            // wavefront 0: where the stretch begins, 1: where it ends
        int at = 0;
        if (P.found) {
            at = lane < words ? as_global(P.bounds)[(int64_t)(stretch + wave) * words + lane] : 0;
            if (lane < words - 2) L.seg[lane >> 1][(lane & 1) + 2 * wave] = at;
        } else {                               // the list places follow below
            int row;
            const uint64_t key = bound_key(P, stretch + wave, lane, row);
            at = lane == words - 2 ? row : (int)(uint32_t)key;
        }
        if (lane >= words - 2 && lane < words) L.bound[wave][lane - (words - 2)] = at;
    }
    if (MODE != kRaw && tid < P.steps) L.start[tid] = MODE == kWrite ? as_global(P.counts)[(int64_t)tid * P.stretches + stretch] : 0;
    block_lds_sync();
    const int row_first = uniform(L.bound[0][0]), row_last = uniform(L.bound[1][0]);
    const uint64_t k_lo = e0 == 0 ? 0 : ((uint64_t)(uint32_t)row_first << 32) | (uint32_t)uniform(L.bound[0][1]);
    const uint64_t k_hi = e1 == P.nnz1 ? ~0ull : ((uint64_t)(uint32_t)row_last << 32) | (uint32_t)uniform(L.bound[1][1]);

    // first position among the LDS keys that is not below `key`: four ways per round, the offsets constants
    auto place_of = [&](uint64_t key) {
        int at = 0;
#pragma unroll
        for (int b = kCap / 4; b >= 2; b /= 4) {
            const uint64_t k1 = L.key[at + b - 1], k2 = L.key[at + 2 * b - 1], k3 = L.key[at + 3 * b - 1];
            at += (k1 < key ? b : 0) + (k2 < key ? b : 0) + (k3 < key ? b : 0);
        }
        at += L.key[at] < key ? 1 : 0;
        return at + (L.key[min(at, kCap - 1)] < key ? 1 : 0);
    };
    static_assert(kCap == 2048, "place_of takes rounds of 512, 128, 32, 8, 2 keys");
    // entry j of all steps' parts of one side (0 added, 1 deleted) in a row, and its step
    auto entry_of = [&](int side, int j, int &s) {
        const int *first = side ? L.first_del : L.first_add;
        s = 0;
#pragma unroll
        for (int b = 16; b >= 1; b /= 2) s += first[s + b] <= j ? b : 0;
        const int at = L.seg[s][side] + j - first[s];
        const int32_t *row = as_global(L.lists.row[s][side]), *col = as_global(L.lists.col[s][side]);
        return ((uint64_t)(uint32_t)row[at] << 32) | (uint32_t)col[at];
    };

    // The stretch is taken as one piece; keys among which more is added than the LDS holds are halved until it fits.
    uint64_t lo = k_lo, hi = k_hi;
    int ea = e0, eb = e1;                      // the entries of A_1 in [lo, hi)
    bool sought = !P.found;
    for (;;) {
        if (sought) {
            if (wave < 2) {
                const int at = list_place(P, L.lists, wave ? hi : lo, wave ? eb : ea, lane);
                if (lane < 2 * P.steps) L.seg[lane >> 1][(lane & 1) + 2 * wave] = at;
            }
            block_lds_sync();
        }
        sought = true;                         // the next piece's parts are looked for
        // ---- A_1's entries and the row pointers of their rows, on their way while the lists' parts are put in a row
        const int p0 = tid * kPerThread, rows = row_last - row_first + 2;
        const bool staged = rows <= kCap;
        uint32_t own_col[kPerThread], pointer[kPerThread];
        {
            const __amdgpu_buffer_rsrc_t cols = buffer_of(colidx1 + ea, eb - ea), pointers = buffer_of(rowptr1 + row_first, staged ? rows : 0);
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) own_col[k] = __builtin_amdgcn_raw_buffer_load_b32(cols, (p0 + k) * 4, 0, 0);
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) pointer[k] = __builtin_amdgcn_raw_buffer_load_b32(pointers, (tid + k * kThreads) * 4, 0, 0);
        }
        if (wave < 2) {                                                 // wavefront 0: added, 1: deleted
            const int len = lane < P.steps ? max(L.seg[lane][2 + wave] - L.seg[lane][wave], 0) : 0;
            const int incl = wave_scan_add(len, lane);
            if (lane < 32) (wave ? L.first_del : L.first_add)[lane] = lane < P.steps ? incl - len : 0x7fffffff;
            if (lane == kWave - 1) (wave ? L.total_del : L.total_add) = incl;
        } else if (MODE == kRaw && wave == 2) {
            const int moved = lane < P.steps ? L.seg[lane][0] - L.seg[lane][1] : 0;
            const int incl = wave_scan_add(moved, lane);
            if (lane < P.steps) L.start[lane] = ea + incl;
        }
        block_lds_sync();
        int adds = uniform(L.total_add);
        const int dels = uniform(L.total_del), old = eb - ea;
        if (adds > kAddCap || old + adds > kCap) {
            if (hi - lo > 1) {                                          // the lower half of the keys first
                int row;
                if (old >= 2) {
                    eb = ea + old / 2;
                    hi = key_of_entry(P, eb, lane, row);
                } else {
                    hi = lo + (hi - lo) / 2;
                    if (eb > ea && key_of_entry(P, ea, lane, row) >= hi) eb = ea;
                }
                continue;
            }
            adds = min(adds, min(kAddCap, kCap - old));                 // one key: it fits for lists that keep the preconditions
        }
        // ---- list entries: the first threads take added ones, the last ones deleted ones
        const int a_tid = tid, d_tid = kThreads - 1 - tid;
        uint64_t a_key[kAddsKept], d_key[kDelsKept];
        int a_step[kAddsKept], d_step[kDelsKept];
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k)
            if (a_tid + k * kThreads < adds) a_key[k] = entry_of(0, a_tid + k * kThreads, a_step[k]);
#pragma unroll
        for (int k = 0; k < kDelsKept; ++k)
            if (d_tid + k * kThreads < dels) d_key[k] = entry_of(1, d_tid + k * kThreads, d_step[k]);
        // ---- A_1's keys: a thread finds the row of its first entry, in the row pointers in LDS if they fit, and walks on
        int *pointers = reinterpret_cast<int *>(L.bits);
        if (staged) {
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) pointers[tid + k * kThreads] = (int)pointer[k];
        }
        block_lds_sync();
        uint64_t own[kPerThread];
        auto keys = [&](auto pointer_of) {
            int row = row_first, end = 0;
            if (ea + p0 < eb) {
                int b = row_last;                                       // last row whose pointer is <= ea + p0
                while (row < b) {
                    const int mid = row + ((b - row + 1) >> 1);
                    if (pointer_of(mid) <= ea + p0) row = mid; else b = mid - 1;
                }
                end = pointer_of(row + 1);
            }
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {
                own[k] = ~0ull;                                         // beyond the piece: above every key
                if (ea + p0 + k < eb) {
                    while (ea + p0 + k >= end && row < row_last) end = pointer_of(++row + 1);
                    own[k] = ((uint64_t)(uint32_t)row << 32) | own_col[k];
                }
                L.key[p0 + k] = own[k];
                L.build.before[p0 + k] = 0;
            }
        };
        if (staged) keys([&](int row) { return pointers[row - row_first]; });
        else keys([&](int row) { return rowptr1[row]; });
        block_lds_sync();
        // ---- where the lists' entries lie among them: at a_at; new ones count themselves at the entry they precede
        int a_at[kAddsKept], a_rank[kAddsKept], d_at[kDelsKept];
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k) {
            a_rank[k] = -1;
            if (a_tid + k * kThreads < adds) {
                a_at[k] = place_of(a_key[k]);
                if (a_at[k] >= old || L.key[a_at[k]] != a_key[k]) a_rank[k] = atomicAdd(&L.build.before[a_at[k]], 1);
            }
        }
#pragma unroll
        for (int k = 0; k < kDelsKept; ++k) {
            d_at[k] = -1;
            if (d_tid + k * kThreads < dels) {
                const int p = place_of(d_key[k]);
                if (p < old && L.key[p] == d_key[k]) d_at[k] = p;
            }
        }
        block_lds_sync();
        {
            int4 v = *reinterpret_cast<const int4 *>(&L.build.before[p0]);
            const int sum = (v.x + v.y) + (v.z + v.w);
            const int incl = wave_scan_add(sum, lane);
            if (lane == kWave - 1) L.sums[wave] = incl;
            block_lds_sync();
            int run = incl - sum;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) run += w < wave ? L.sums[w] : 0;
            int4 o;
            o.x = run; run += v.x;
            o.y = run; run += v.y;
            o.z = run; run += v.z;
            o.w = run; run += v.w;
            *reinterpret_cast<int4 *>(&L.build.before[p0]) = o;
            if (tid == kThreads - 1) L.build.before[kCap] = run;
        }
        static_assert(kPerThread == 4, "one 16-byte access per thread");
        block_lds_sync();
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k)
            if (a_rank[k] >= 0) L.build.added[L.build.before[a_at[k]] + a_rank[k]] = a_key[k];
        const int held = old + uniform(L.build.before[kCap]);           // entries of the union
        block_lds_sync();
        // ---- their places in the union; an entry that is added several times lives at the first of its places
        int to[kPerThread], a_to[kAddsKept];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) to[k] = p0 + k < old ? p0 + k + L.build.before[p0 + k + 1] : kCap;
#pragma unroll
        for (int k = 0; k < kDelsKept; ++k)
            if (d_at[k] >= 0) d_at[k] += L.build.before[d_at[k] + 1];
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k) {
            a_to[k] = kCap;
            if (a_rank[k] >= 0) {
                const int b = L.build.before[a_at[k]], e = L.build.before[a_at[k] + 1], mine = b + a_rank[k];
                int less = 0, same = 0;
                for (int i = b; i < e; ++i) {
                    const uint64_t other = L.build.added[i];
                    less += other < a_key[k] ? 1 : 0;
                    same += other == a_key[k] && i < mine ? 1 : 0;
                }
                a_at[k] += b + less;
                a_to[k] = a_at[k] + same;
            } else if (a_tid + k * kThreads < adds) {
                a_at[k] += L.build.before[a_at[k] + 1];
            }
        }
#pragma unroll
        for (int k = 0; k < kPerThread; ++k)                            // (every search among A_1's keys is behind the last barriers)
            if (to[k] < kCap) { L.key[to[k]] = own[k]; L.bits[to[k]] = ~0u; }
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k)
            if (a_to[k] < kCap) { L.key[a_to[k]] = a_key[k]; L.bits[a_to[k]] = 0; }
        for (int p = held + tid; p < kCap; p += kThreads) { L.key[p] = ~0ull; L.bits[p] = 0; }
        block_lds_sync();
        // ---- the lists turn the bits of the entries they name
#pragma unroll
        for (int k = 0; k < kAddsKept; ++k)
            if (a_tid + k * kThreads < adds) atomicXor(&L.bits[a_at[k]], ~0u << (a_step[k] + 1));
        auto deleted = [&](uint64_t key, int s) {                       // not one of A_1's
            const int p = place_of(key);
            if (p < held && L.key[p] == key) atomicXor(&L.bits[p], ~0u << (s + 1));
        };
#pragma unroll
        for (int k = 0; k < kDelsKept; ++k)
            if (d_tid + k * kThreads < dels) {
                if (d_at[k] >= 0) atomicXor(&L.bits[d_at[k]], ~0u << (d_step[k] + 1));
                else deleted(d_key[k], d_step[k]);
            }
#pragma unroll 1
        for (int j = d_tid + kDelsKept * kThreads; j < dels; j += kThreads) {
            int s;
            const uint64_t key = entry_of(1, j, s);
            deleted(key, s);
        }
        block_lds_sync();
        // ---- ballots of all steps, 64 entries each; lane s keeps those of step s
        const uint32_t window = MODE == kRaw ? 1u : P.life >= 32 ? ~0u : (1u << P.life) - 1;
        uint32_t col[kPerThread], bits[kPerThread];
        bool self[kPerThread];
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int p = (wave + k * kWaves) * kWave + lane;
            const uint64_t key = L.key[p];
            col[k] = (uint32_t)key;
            bits[k] = L.bits[p];
            self[k] = MODE == kWrite && P.diag != 0.0f && (uint32_t)(key >> 32) == col[k];
        }
        // the window's bits as of step s, the newest the highest of them: bits s + 2 - l .. s + 1, none before A_1
        auto seen_at = [&](int s) {
            const int from = s + 2 - P.life;
            return MODE == kRaw ? 2u << s : from >= 0 ? window << from : (2u << (s + 1)) - 1;
        };
        {
            int count[kPerThread], held_lo[kPerThread], held_hi[kPerThread];
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) count[k] = held_lo[k] = held_hi[k] = 0;
#pragma unroll 1
            for (int s = 0; s < P.steps; ++s) {
                const uint32_t seen = seen_at(s);
                const bool mine = lane == s;
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    const uint64_t h = __ballot((bits[k] & seen) != 0);
                    count[k] = mine ? __builtin_popcountll(h) : count[k];
                    if (MODE == kWrite) {
                        held_lo[k] = mine ? (int)(uint32_t)h : held_lo[k];
                        held_hi[k] = mine ? (int)(uint32_t)(h >> 32) : held_hi[k];
                    }
                }
            }
            if (lane < P.steps) {
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    L.write.place[lane][wave + k * kWaves] = count[k];
                    if (MODE == kWrite) L.write.held[lane][wave + k * kWaves] = ((uint64_t)(uint32_t)held_hi[k] << 32) | (uint32_t)held_lo[k];
                }
            }
        }
        block_lds_sync();
        for (int s = wave; s < P.steps; s += kWaves) {
            const int v = lane < kChunks ? L.write.place[s][lane] : 0;
            const int incl = wave_scan_add(v, lane);
            if (lane < kChunks) L.write.place[s][lane] = incl - v;
            if (lane == kWave - 1) L.seg[s][0] = incl;                  // entries of the piece in the snapshot of step s
        }
        block_lds_sync();
        if (MODE != kCount) {
            // where the piece's entries of step s go, how many bytes of them, and this wavefront's places there, in lane s
            const int own_step = min(lane, P.steps - 1), start = L.start[own_step];
            const bool placed = start >= 0 && start < P.cap;            // always, unless a smoothed snapshot does not fit its arrays
            const int bytes = placed ? min(L.seg[own_step][0], P.cap - start) * 4 : 0;
            const uint64_t out_col = (uint64_t)L.lists.out[own_step][0] + (placed ? (uint64_t)start * 4 : 0);
            const uint64_t out_val = (uint64_t)L.lists.out[own_step][1] + (placed ? (uint64_t)start * 4 : 0);
            int place[kPerThread];
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) place[k] = L.write.place[own_step][wave + k * kWaves] * 4;
#pragma unroll 1
            for (int s = 0; s < P.steps; ++s) {
                auto buffer = [&](uint64_t at) {
                    const uint64_t base = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(at >> 32), s) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)at, s);
                    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, __builtin_amdgcn_readlane(bytes, s), 0x00027000);
                };
                const __amdgpu_buffer_rsrc_t to_col = buffer(out_col), to_val = buffer(out_val);
                const uint32_t seen = seen_at(s);
#pragma unroll
                for (int k = 0; k < kPerThread; ++k) {
                    if ((wave + k * kWaves) * kWave >= held) break;
                    const uint32_t b = bits[k] & seen;
                    const uint64_t h = __ballot(b != 0);
                    const int before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(h >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)h, 0));
                    const int at = before * 4 + __builtin_amdgcn_readlane(place[k], s);
                    const int offset = b != 0 ? at : -4;                // outside the buffer: not stored
                    __builtin_amdgcn_raw_buffer_store_b32(col[k], to_col, offset, 0, 0);
                    if (MODE == kWrite) {
                        const float value = self[k] ? P.diag : (float)__popc(b);
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(value), to_val, offset, 0, 0);
                    }
                }
            }
        }
        if (MODE == kWrite) {                                           // rows that begin among these keys
            const int row_a = (int)min((int64_t)(lo >> 32), (int64_t)P.n) + ((uint32_t)lo > 0 ? 1 : 0);
            const int row_b = (int)min(min((int64_t)(hi >> 32), (int64_t)P.n) - ((uint32_t)hi > 0 ? 0 : 1), (int64_t)P.n - 1);
            for (int r = row_a + tid; r <= row_b; r += kThreads) {
                const int u = place_of((uint64_t)(uint32_t)r << 32);
#pragma unroll 1
                for (int s = 0; s < P.steps; ++s) {
                    int at = L.seg[s][0];
                    if (u < kCap) at = L.write.place[s][u / kWave] + __popcll(L.write.held[s][u / kWave] & ((1ull << (u % kWave)) - 1));
                    as_global(P.s[s].rowptr)[r] = L.start[s] + at;
                }
            }
        }
        block_lds_sync();                                               // all has been read that the next piece overwrites
        if (MODE != kRaw && tid < P.steps) L.start[tid] += L.seg[tid][0];
        if (hi == k_hi) break;
        lo = hi;
        hi = k_hi;
        ea = eb;
        eb = e1;
        block_lds_sync();
    }
    if (MODE == kCount && tid < P.steps) as_global(P.counts)[(int64_t)tid * P.stretches + stretch] = L.start[tid];
}

// The first row_tiles workgroups take rows, the others stretches.
template <Mode MODE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6, 8))) void series_kernel(Series P) {
    constexpr size_t kBytes = MODE == kWrite || sizeof(StretchPart) > sizeof(RowPart) ? sizeof(StretchPart) : sizeof(RowPart);
    __shared__ __attribute__((aligned(16))) char lds[kBytes];
    if (MODE != kWrite && (int)blockIdx.x < P.row_tiles)
        rows_of_series<MODE>(P, *reinterpret_cast<RowPart *>(lds), blockIdx.x);
    else
        stretch_of_series<MODE>(P, *reinterpret_cast<StretchPart *>(lds), blockIdx.x - (MODE != kWrite ? P.row_tiles : 0));
}

// counts of a step -> where each stretch begins in S_t, a workgroup per step; the number of stored entries goes into the last
// row pointer
__global__ __launch_bounds__(kScanThreads) void series_scan_kernel(Series P) {
    constexpr int kScanWaves = kScanThreads / kWave;
    __shared__ int s_wave[kScanWaves];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    int32_t *counts = as_global(P.counts) + (int64_t)blockIdx.x * P.stretches;
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
        for (int w = 0; w < kScanWaves; ++w) {
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
        as_global(P.s[blockIdx.x].rowptr)[P.n] = carry;
        if (P.d_status) as_global(P.d_status)[blockIdx.x] = carry > P.cap ? DGNN_BAD_CAPACITY : 0;
    }
}

// Entries of A_1 per stretch: as few as still give every CU three workgroups, as many as leave the LDS room for what the lists
// add, with a quarter to spare for lists that favour some stretches.
int tile_of(int64_t nnz, int64_t added) {
    const double grow = (double)added / (double)nnz;
    const double most = 0.75 * std::min(kCap / (1.0 + grow), kAddCap / std::max(grow, 1e-9));
    return (int)std::max<int64_t>(16, std::min<int64_t>((int64_t)most, std::max<int64_t>(kLeastTile, nnz / 768)));
}
int stretches_of(int64_t nnz, int tile) { return (int)((nnz + tile - 1) / tile); }
size_t bounds_bytes(int stretches, int steps) { return round_up((size_t)(stretches + 1) * (2 * steps + 2) * sizeof(int32_t), (size_t)256); }
// More stretches than the chip holds at once: their bounds are found by a launch of their own.
constexpr int kOwnBounds = 768;

int raw_workspace(int64_t nnz, int32_t steps, const dgnn_series_step *step, size_t *bytes) {
    *bytes = 16;
    for (int done = 0; done < steps; done += kSteps) {
        const int m = std::min(steps - done, kSteps);
        int64_t added = 0, net = 0;
        for (int k = done; k < done + m; ++k) { added += step[k].n_add; net += step[k].n_add - step[k].n_del; }
        if (nnz > 0) {
            const int stretches = stretches_of(nnz, tile_of(nnz, added));
            if (stretches > kOwnBounds) *bytes = std::max(*bytes, bounds_bytes(stretches, m));
        }
        nnz += net;
    }
    return DGNN_OK;
}
size_t smooth_workspace(int64_t nnz, int64_t added, int steps) {
    const int stretches = stretches_of(nnz, tile_of(nnz, added));
    return bounds_bytes(stretches, steps) + std::max<size_t>(16, (size_t)stretches * steps * sizeof(int32_t));
}
int launch_bounds(Series &P, hipStream_t s) {
    P.found = 1;
    hipLaunchKernelGGL(series_bounds_kernel, dim3((unsigned)(P.stretches + 1)), dim3(kWave), 0, s, P);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

}  // namespace

extern "C" int dgnn_delta_rebuild_series_workspace(int64_t nnz_first, int32_t steps, const dgnn_series_step *step, size_t *bytes) {
    if (!bytes || (steps > 0 && !step)) return DGNN_ERR_NULL;
    if (nnz_first <= 0 || steps < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(nnz_first)) return DGNN_ERR_OVERFLOW;
    return raw_workspace(nnz_first, steps, step, bytes);
}

extern "C" int dgnn_delta_rebuild_series(int64_t n, const int32_t *rowptr_first, const int32_t *colidx_first, int64_t nnz_first,
                                         int32_t steps, const dgnn_series_step *step, int64_t cap, void *ws, size_t ws_bytes, void *stream) {
    if (!rowptr_first || !colidx_first || (steps > 0 && !step)) return DGNN_ERR_NULL;
    if (n <= 0 || nnz_first <= 0 || steps < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz_first)) return DGNN_ERR_OVERFLOW;
    int64_t nnz = nnz_first;
    for (int k = 0; k < steps; ++k) {
        const dgnn_series_step &st = step[k];
        if (!st.rowptr || !st.colidx) return DGNN_ERR_NULL;
        if (nnz == 0) return DGNN_ERR_SHAPE;             // a step from a snapshot without entries, which the single call refuses too
        if (st.n_add < 0 || st.n_del < 0) return DGNN_ERR_SHAPE;
        if ((st.n_add > 0 && (!st.add_row || !st.add_col)) || (st.n_del > 0 && (!st.del_row || !st.del_col))) return DGNN_ERR_NULL;
        if (!fits_index(nnz + st.n_add)) return DGNN_ERR_OVERFLOW;
        nnz += st.n_add - st.n_del;
        if (nnz < 0) return DGNN_ERR_SHAPE;
        if (nnz > cap) return DGNN_ERR_CAPACITY;
        // all steps are written by the same launch: every snapshot needs arrays of its own
        if (st.rowptr == rowptr_first || st.colidx == colidx_first) return DGNN_ERR_ALIAS;
        for (int j = std::max(0, k - kSteps); j < k; ++j)
            if (st.rowptr == step[j].rowptr || st.colidx == step[j].colidx) return DGNN_ERR_ALIAS;
    }
    size_t needed = 0;
    raw_workspace(nnz_first, steps, step, &needed);
    if (!ws) return DGNN_ERR_NULL;
    if (!aligned16(ws)) return DGNN_ERR_ALIGN;
    if (ws_bytes < needed) return DGNN_ERR_CAPACITY;
    hipStream_t s = (hipStream_t)stream;
    Series P{};
    P.n = (int)n;
    P.cap = (int)std::min<int64_t>(cap, 2147483647LL);
    P.life = 1;
    P.bounds = (int32_t *)ws;
    P.row_tiles = (int)((n + kRowTile - 1) / kRowTile);
    P.rowptr1 = rowptr_first;
    P.colidx1 = colidx_first;
    nnz = nnz_first;
    for (int done = 0; done < steps; done += P.steps) {
        P.steps = std::min(steps - done, kSteps);
        P.nnz1 = (int)nnz;
        int64_t added = 0;
        for (int k = 0; k < P.steps; ++k) {
            const dgnn_series_step &st = step[done + k];
            P.s[k] = dgnn_smooth_step{st.add_row, st.add_col, st.del_row, st.del_col, st.n_add, st.n_del, st.rowptr, st.colidx, nullptr, st.dinv};
            added += st.n_add;
        }
        P.tile = nnz > 0 ? tile_of(nnz, added) : 1;
        P.stretches = stretches_of(nnz, P.tile);
        P.found = 0;
        if (P.stretches > kOwnBounds) {
            const int rc = launch_bounds(P, s);
            if (rc != DGNN_OK) return rc;
        }
        hipLaunchKernelGGL(series_kernel<kRaw>, dim3((unsigned)(P.row_tiles + P.stretches)), dim3(kThreads), 0, s, P);
        DGNN_RETURN_IF_LAUNCH_FAILED();
        for (int k = 0; k < P.steps; ++k) nnz += P.s[k].n_add - P.s[k].n_del;
        P.rowptr1 = P.s[P.steps - 1].rowptr;
        P.colidx1 = P.s[P.steps - 1].colidx;
    }
    return DGNN_OK;
}

extern "C" int dgnn_smooth_series_workspace(int64_t nnz_first, int64_t added, int32_t steps, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (nnz_first <= 0 || added < 0 || steps < 0 || steps > kSteps) return DGNN_ERR_SHAPE;
    if (!fits_index(nnz_first + added)) return DGNN_ERR_OVERFLOW;
    *bytes = smooth_workspace(nnz_first, added, steps);
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
    if (ws_bytes < smooth_workspace(nnz_first, most - nnz_first, steps)) return DGNN_ERR_CAPACITY;
    if (steps == 0) return DGNN_OK;
    hipStream_t s = (hipStream_t)stream;
    Series P{};
    P.n = (int)n;
    P.nnz1 = (int)nnz_first;
    P.steps = steps;
    P.cap = (int)std::min<int64_t>(capacity, 2147483647LL);
    P.life = life;
    P.tile = tile_of(nnz_first, most - nnz_first);
    P.stretches = stretches_of(nnz_first, P.tile);
    P.row_tiles = dinv ? (int)((n + kRowTile - 1) / kRowTile) : 0;
    P.diag = diag_value;
    P.rowptr1 = rowptr_first;
    P.colidx1 = colidx_first;
    P.bounds = (int32_t *)ws;
    P.counts = (int32_t *)((char *)ws + bounds_bytes(P.stretches, steps));
    P.d_status = d_status;
    for (int k = 0; k < steps; ++k) P.s[k] = step[k];
    const int rc = launch_bounds(P, s);
    if (rc != DGNN_OK) return rc;
    hipLaunchKernelGGL(series_kernel<kCount>, dim3((unsigned)(P.row_tiles + P.stretches)), dim3(kThreads), 0, s, P);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(series_scan_kernel, dim3((unsigned)steps), dim3(kScanThreads), 0, s, P);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(series_kernel<kWrite>, dim3((unsigned)P.stretches), dim3(kThreads), 0, s, P);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}
