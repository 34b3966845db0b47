// Sparse factor of the GCN operation, Eqn (1) and Eqn (2): Z = sigma?(A~ H) with
// A~ = D^(-1/2) (A + I) D^(-1/2).  The snapshot is unweighted, so a stored entry (u, v) weighs
// dinv[u] * dinv[v] and the kernel needs no value array:
//     Z[u] = dinv[u] * sum_{v in row u} dinv[v] * H[v].
//
// The work is a gather of whole H rows (one 16-byte piece per lane, a lane group per row of H).  On large snapshots it is bound by
// the rate at which L2 misses are served; where the rows lie in the L2s, by the vector memory units of the CUs (2.5 - 3.5 cycles
// per cache line touched), so lines other than those of H count.  It is split by ENTRIES, not by rows, and every wavefront is
// an independent stream:
//   - a wavefront owns a contiguous range of stored entries and walks it in sub-tiles (up to 65536 sub-tiles: one per wavefront,
//     which then takes 64 registers in fp32, 73 with factors, 81 - 88 in bf16, where one that walks on takes 94 - 154).  The row that
//     holds the range's first entry is found once, mostly by two scalar loads and one look at 64 row pointers; afterwards rows
//     simply follow on;
//   - the sub-tile's columns go to LDS as byte offsets, a lane group reads four of them at once; the rows with entries are listed
//     in LDS, their starts become a bit mask (one 32-bit word per lane group);
//   - every lane group takes 32 consecutive entries, keeps eight gathers in flight, each replaced as it is used, and where
//     the mask has a bit puts its running sum away: a row that began inside the group's 32 entries is stored at once, a piece cut
//     on the left is parked in LDS.  Where no group has a row start, an entry costs four additions, an address and a load;
//   - the group where a cut row begins adds the parked pieces in entry order; a row still open goes on in group 0 of the next
//     sub-tile; only rows cut by the range itself leave a "left" or "right" carry in the workspace, which a second small
//     kernel adds up, again in entry order;
//   - where a range has several sub-tiles, columns and row pointers of the next one are fetched while this one is summed.
// Hub rows of power-law graphs are thereby spread over as many wavefronts as they have ranges,
// short rows share a wavefront, and every sum has a fixed order: no floating-point atomics,
// results repeat bit for bit.
// Against the form with a search per lane group, a branch per entry and workgroup barriers, us per aggregation: uniform 50 K
// vertices x 64 fp32 25.1 -> 16.2 (with slices of columns, see slices_of), 100 K 55.5 -> 47.5, R-MAT 2^16 x 64 20.7 -> 18.8, 2^18 x 128 bf16
// 125 -> 97, 2^19 x 32 with values 131 -> 99.  Where misses bound it, more wavefronts wait for the same fabric: R-MAT 2^23 x 32 2292 / 2286, but
// with values 2326 -> 2360, and uniform graphs of 135 K - 2 M vertices with rows of 256 and 512 bytes take 2 - 5 % longer (200 K x 64 126.7 ->
// 129.3, 500 K 246 -> 256, x 128 491 -> 516, 2 M 986 -> 1005): the same bytes pass the L2s, a request is away for 1130 cycles
// instead of 1040.  Eight wavefronts per CU instead of up to 32 give that back (500 K 248) and take more from power-law graphs, whose hot
// rows come from the L2s (2^18 x 64 92 -> 107); nothing that a call is given tells the two apart.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace {

using namespace dgnn;

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kBatch = 8;            // gathers issued together by a lane group
// Entries a lane group walks per sub-tile (one mask word; half of one where the groups are so many that the sub-tile's rows would
// take the LDS of half the wavefronts).
constexpr int per_group(int lanes_per_row) { return lanes_per_row == 2 ? 16 : 32; }
constexpr int kMaxRange = 2048;      // entries streamed by one wavefront, at most: many short-lived wavefronts stream
                                     // faster than few long-lived ones (8192: +2.5 % on the largest workloads)
constexpr int kTargetWaves = 65536;  // ranges shrink on small inputs so that about this many wavefronts exist (16384: +4 %)
constexpr int kLongestRange = 8192;  // what a caller with little room for records may stretch a range to
constexpr int kXcds = 8;             // accelerator dies of an MI355X, each with its own L2
constexpr int kXcdChunk = 16;        // consecutive ranges that go to the same XCD
constexpr int kVmcntZero = 0x0F70;   // s_waitcnt operand: all vector memory loads returned, other counters untouched

// What a range leaves for the carry kernel: the row that begins in it and goes on behind it, or -1.  How far that row reaches,
// and with it whose left carries are its pieces, follows from the row pointers.
struct RangeRec { int32_t open_row, pad0, pad1, pad2; };

// One aggregation of a launch, which may take those of several timesteps: the first kernel finds it by its place in the launch's
// line of units (see Line), the second by blockIdx.y.
struct Item {
    const int32_t *rowptr, *colidx;
    const float *dinv, *vals;
    const char *h;
    char *z;
    RangeRec *recs;
    float *carry;
    int32_t nnz, range_len, n_ranges, gather_dinv;   // gather_dinv: rows of h are scaled as they are gathered
    float rows_per_entry;
};
constexpr int kMaxBatch = 32;        // what fits the kernel arguments comfortably
struct Batch { Item item[kMaxBatch]; };

struct RowRef { uint32_t at; float du; };   // a row that holds entries: where its result begins (FAR: its number), and its dinv

// ---- 16-byte feature pieces: 4 fp32 or 8 bf16, accumulated in fp32 -------------------------
template <bool BF16> struct Piece;
template <> struct Piece<false> {
    static constexpr int kVals = 4;
    typedef floatx4 Raw;
    template <bool SCALE> static __device__ __forceinline__ void add(float (&acc)[4], float s, Raw v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = SCALE ? fmaf(s, v[e], acc[e]) : acc[e] + v[e];
    }
    static __device__ __forceinline__ Raw pack(const float (&acc)[4]) { return Raw{acc[0], acc[1], acc[2], acc[3]}; }
};
template <> struct Piece<true> {
    static constexpr int kVals = 8;
    typedef uintx4 Raw;
    template <bool SCALE> static __device__ __forceinline__ void add(float (&acc)[8], float s, Raw v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float lo = __uint_as_float(v[e] << 16), hi = __uint_as_float(v[e] & 0xffff0000u);
            acc[2 * e] = SCALE ? fmaf(s, lo, acc[2 * e]) : acc[2 * e] + lo;
            acc[2 * e + 1] = SCALE ? fmaf(s, hi, acc[2 * e + 1]) : acc[2 * e + 1] + hi;
        }
    }
    static __device__ __forceinline__ Raw pack(const float (&acc)[8]) {
        Raw v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = pack_bf16(acc[2 * e], acc[2 * e + 1]);
        return v;
    }
};

// Z[row] piece = sigma?(dinv[row] * acc)
template <bool BF16, int NV>
__device__ __forceinline__ void finish_row(char *z, int64_t row, int row_bytes, int sub, const float *dinv, int relu,
                                           const float (&acc)[NV]) {
    const float du = dinv ? dinv[row] : 1.0f;
    float out[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        out[q] = acc[q] * du;
        if (relu) out[q] = fmaxf(out[q], 0.0f);
    }
    __builtin_nontemporal_store(Piece<BF16>::pack(out), reinterpret_cast<typename Piece<BF16>::Raw *>(z + row * row_bytes + sub * 16));
}

template <int LPR, int SLICES>
__device__ __forceinline__ void zero_row(char *z, int64_t row) {
    for (int s = 0; s < LPR; ++s) __builtin_nontemporal_store(uintx4{0, 0, 0, 0}, reinterpret_cast<uintx4 *>(z + row * (LPR * SLICES * 16) + s * 16));
}

// LPR: lanes per feature row.  SCALE_V: multiply every gathered row by a per-entry factor: dinv of its
// column, or the entry's own value when the snapshot carries values (otherwise H already carries the factor).
// FAR: H or Z reaches beyond the 4 GB that a 32-bit offset from its first byte spans.  ONE: the range is a single sub-tile.
template <int LPR, int SLICES, bool BF16, bool SCALE_V, bool FAR, bool ONE>
__device__ __forceinline__ void spmm_stream(
    int range, int n, int nnz, int range_len, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const float *__restrict__ dinv, const char *__restrict__ h, char *__restrict__ z, int relu,
    RangeRec *__restrict__ recs, bool record, float *__restrict__ carry, const float *__restrict__ vals, bool gather_dinv, float rows_per_entry) {
    typedef typename Piece<BF16>::Raw Raw;
    constexpr int NV = Piece<BF16>::kVals;
    constexpr int F = LPR * NV;
    constexpr int G = kWave / LPR;          // lane groups per wavefront
    constexpr int kPer = per_group(LPR);
    constexpr int SUB = G * kPer;           // entries per sub-tile
    constexpr int CN = SUB / kWave;         // column indices fetched by one lane
    constexpr int kRowBytes = LPR * SLICES * 16;   // from a row to the next; h, z and carry are the slice's own, recs are the same for all (one of them records)
    constexpr int kStride = kPer + 4;       // words from a group's offsets to the next group's: 16-byte reads of the groups fall on different banks

    __shared__ __align__(16) uint32_t s_off[G * kStride];                  // where the rows of H that the entries name begin (FAR: their numbers)
    __shared__ __align__(16) float s_val[SCALE_V ? G * kStride : 4];       // the entries' factors
    __shared__ __align__(8) RowRef s_rows[SUB + 2];                        // the sub-tile's rows, those without entries left out
    __shared__ unsigned s_heads[G + 1];     // bit p of word g: a row begins at entry kPer g + p; the last word: their disjunction
    __shared__ __align__(16) float s_left[G][F];                           // a group's sum up to its first row start

    const int lane = threadIdx.x;
    const int sub = lane % LPR, g = lane / LPR;
    const uint32_t sub16 = sub * 16;
    const int e_begin = (int)((int64_t)range * range_len);
    // the host's count may be an upper bound (a snapshot whose size only the device knows): the last row pointer decides
    nnz = min(nnz, rowptr[n]);
    if (e_begin >= nnz) {                               // nothing stored here: a record that closes nothing and carries nothing
        if (lane == 0 && record) recs[range] = RangeRec{-1, 0, 0, 0};
        if (range == 0)
            for (int k = lane; k < n; k += kWave) zero_row<LPR, SLICES>(z, k);
        return;
    }
    const int e_end = (int)min((int64_t)e_begin + range_len, (int64_t)nnz);
    float *my_carry = carry + (int64_t)range * 2 * F;

    // column indices (and factors) of the coming sub-tile, consecutive ones per load
    int c_next[CN];
    float d_next[SCALE_V ? CN : 1] = {};
    if (SCALE_V && !vals)
#pragma unroll
        for (int i = 0; i < CN; ++i) d_next[i] = 1.0f;
    auto fetch_cols = [&](int e0) {
#pragma unroll
        for (int i = 0; i < CN; ++i) {
            const int idx = min(e0 + i * kWave + lane, e_end - 1);
            c_next[i] = __builtin_nontemporal_load(colidx + idx);   // a stream: the caches are for rows of H
            if (SCALE_V && vals) d_next[i] = vals[idx];
        }
    };
    // row pointers (and dinv) of the first 64 rows of the coming sub-tile; further rows are read on demand
    int m_v = 0, m_vn = 0;
    float m_du = 1.0f;
    auto fetch_rows = [&](int k0) {          // unconditional loads: the compiler then counts what is in flight exactly
        const int k = min(k0 + lane, n - 1);
        m_v = rowptr[k];
        m_vn = rowptr[k + 1];
        if (dinv) m_du = dinv[k];
    };
    auto row_ref = [&](int k, float du) { return RowRef{FAR ? (uint32_t)k : (uint32_t)k * kRowBytes, du}; };
    auto store_row = [&](const RowRef &r, const float (&acc)[NV]) {
        float out[NV];
        if (relu) {
            asm volatile("");                            // a branch of the whole wavefront, not a selection per value
#pragma unroll
            for (int q = 0; q < NV; ++q) out[q] = fmaxf(acc[q] * r.du, 0.0f);
        } else {
#pragma unroll
            for (int q = 0; q < NV; ++q) out[q] = acc[q] * r.du;
        }
        // written once, read by a later kernel
        __builtin_nontemporal_store(Piece<BF16>::pack(out), reinterpret_cast<Raw *>(FAR ? z + (int64_t)r.at * kRowBytes + sub16 : z + (size_t)(r.at + sub16)));
    };
    auto to_carry = [&](int side, const float (&acc)[NV]) {
#pragma unroll
        for (int q = 0; q < NV; ++q) my_carry[side * F + sub * NV + q] = acc[q];
    };

    fetch_cols(e_begin);
    // The row of e_begin: where it would be if rows were equally long, corrected by how far off that is, through the scalar
    // cache (a search by all lanes takes a cache line per lane from the units that the gathers need: 0.15 of a sub-tile's
    // time per round), then among the 64 rows around it.  k_cur: that row, or one up to 63 rows ahead of it.
    int k_cur = 0;
    if (e_begin > 0) {
        int k = min((int)((float)e_begin * rows_per_entry), n - 1);
        for (int round = 0; round < 3; ++round) {
            const float off = (float)(e_begin - as_constant(rowptr)[uniform(k)]) * rows_per_entry;
            k = max(0, min(k + (int)off, n - 1));
            if (fabsf(off) < (float)kWave) break;
        }
        k_cur = uniform(max(k - kWave / 4, 0));
    }
    fetch_rows(k_cur);
    if (!__ballot(m_v <= e_begin && m_vn > e_begin)) {
        k_cur = max(wave_find_row(rowptr, n, e_begin, lane), 0);
        if (range == 0)                      // rows without entries that the walk, which begins at k_cur, does not come to
            for (int k = lane; k < k_cur; k += kWave) zero_row<LPR, SLICES>(z, k);
        fetch_rows(k_cur);
    }

    // the row that is open at the end of a sub-tile goes on in the lanes of group 0
    float run[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) run[q] = 0.0f;
    bool running = false;       // such a row exists
    bool began_here = false;    // ... and it began inside this range
    RowRef run_ref{0, 1.0f};
    int open_row = -1;

    for (int e = e_begin; e < e_end;) {
        const int e_stop = min(e + SUB, e_end), cnt = e_stop - e;
        const bool final = ONE || e_stop == e_end;
        // ---- the sub-tile's columns go to LDS, and the first gathers out
        if (lane <= G) s_heads[lane] = 0u;
#pragma unroll
        for (int i = 0; i < CN; ++i) {
            const int p = i * kWave + lane, at = (p / kPer) * kStride + p % kPer;
            s_off[at] = FAR ? (uint32_t)c_next[i] : (uint32_t)c_next[i] * kRowBytes;
            if (SCALE_V) s_val[at] = gather_dinv ? d_next[i] * dinv[c_next[i]] : d_next[i];
        }
        wave_lds_sync();
        const uint32_t *my_off = &s_off[g * kStride];
        const float *my_val = &s_val[SCALE_V ? g * kStride : 0];
        auto gather = [&](uint32_t off) {
            if (FAR) return *reinterpret_cast<const Raw *>(h + (int64_t)off * kRowBytes + sub16);
            return *reinterpret_cast<const Raw *>(h + (size_t)(off + sub16));
        };
        Raw buf[kBatch];
        {
            const uintx4 o0 = *reinterpret_cast<const uintx4 *>(my_off), o1 = *reinterpret_cast<const uintx4 *>(my_off + 4);
#pragma unroll
            for (int k = 0; k < kBatch; ++k) buf[k] = gather(k < 4 ? o0[k % 4] : o1[k % 4]);
        }
        // ---- its rows
        int k_next = k_cur - 1, listed = 0;
        for (int k = k_cur + lane;;) {
            const bool row = k < n, has = m_vn > m_v;
            const bool list = row && has && m_vn > e && m_v < e_stop;
            const uint64_t mask = __ballot(list);
            if (list) {
                s_rows[min(listed + (int)__popcll(mask & ((1ull << lane) - 1)), SUB)] = row_ref(k, m_du);
                if (m_v >= e) {
                    const int p = m_v - e;
                    atomicOr(&s_heads[p / kPer], 1u << (p % kPer));
                    atomicOr(&s_heads[G], 1u << (p % kPer));
                }
            }
            listed += __popcll(mask);
            // no entries: zero output (those ahead of the first entry of all belong to the first range, see above for more than 64)
            if (row && !has && (m_v > e || e == 0) && m_v <= e_stop) zero_row<LPR, SLICES>(z, k);
            const uint64_t within = __ballot(row && m_v <= e_stop);
            k_next += __popcll(within);                  // ends as the row of entry e_stop
            if (~within) break;
            k += kWave;
            // nothing is stored behind: no look at these rows' pointers (2^20 rows of 128 bytes, the last 2^20 - 1000 without
            // entries: 10.0 -> 4.0 ms, the one wavefront's stores)
            if (e_stop == nnz && __builtin_amdgcn_readlane(m_vn, kWave - 1) == nnz) {
                for (; k < n; k += kWave) zero_row<LPR, SLICES>(z, k);
                break;
            }
            fetch_rows(k - lane);
            __builtin_amdgcn_s_waitcnt(kVmcntZero);      // here, on the rare path, and not ahead of the next prefetch
        }
        if (cnt < SUB && lane == 0) {                    // behind the last entry: what is gathered there belongs to no row
            atomicOr(&s_heads[cnt / kPer], 1u << (cnt % kPer));
            atomicOr(&s_heads[G], 1u << (cnt % kPer));
        }
        wave_lds_sync();
        if (!final) {                                    // fetched while this sub-tile is summed
            fetch_cols(e_stop);
            fetch_rows(k_next);
        }

        // ---- every lane group walks its entries
        const unsigned w = s_heads[g], any = __builtin_amdgcn_readfirstlane(s_heads[G]) & ~1u;
        const unsigned w_lane = lane < G ? s_heads[lane] : 0u;
        const uint64_t headed = __ballot(w_lane != 0u), at_once = __ballot((w_lane & 1u) != 0u);   // groups with a row start; with one at their first entry
        const bool starts = at_once & 1;                 // the sub-tile begins with a row
        const int before = wave_scan_add(__popc(w_lane), lane) - __popc(w_lane);
        const RowRef *next_ref = &s_rows[__shfl(before, g, kWave) + (int)(w & 1u) - (starts ? 1 : 0)];
        RowRef ref = *next_ref;
        if (running && starts && lane < LPR) {           // the row that was open ended with the last sub-tile
            if (began_here) store_row(run_ref, run); else to_carry(0, run);
        }
        const bool inherits = running && !starts && g == 0;
        uint64_t closed = __ballot((w & 1u) || (inherits && began_here));   // lanes whose sum holds its row from the row's first entry on
        const bool cut = !(closed & 1);                  // group 0 begins inside a row of an earlier range
        float acc[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) acc[q] = inherits ? run[q] : 0.0f;

        auto batch = [&](int b, auto more) {
            uintx4 o[2];
            floatx4 s[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (decltype(more)::value) o[i] = *reinterpret_cast<const uintx4 *>(my_off + (b + 1) * kBatch + i * 4);
                if (SCALE_V) s[i] = *reinterpret_cast<const floatx4 *>(my_val + b * kBatch + i * 4);
            }
            const unsigned wb = w >> (b * kBatch), anyb = any >> (b * kBatch);
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                if ((anyb >> k) & 1u) {                  // a row begins here in some group: those that end are put away
                    asm volatile("");                    // (two decisions: the first is the wavefront's)
                    const uint64_t begins = __ballot((wb >> k) & 1u);
                    if (__builtin_amdgcn_inverse_ballot_w64(begins & closed)) store_row(ref, acc);
                    if (begins & ~closed) {
                        if (__builtin_amdgcn_inverse_ballot_w64(begins & ~closed)) {
#pragma unroll
                            for (int q = 0; q < NV; ++q) s_left[g][sub * NV + q] = acc[q];
                        }
                    }
                    closed |= begins;
                    if (__builtin_amdgcn_inverse_ballot_w64(begins)) {
                        ref = *++next_ref;
#pragma unroll
                        for (int q = 0; q < NV; ++q) acc[q] = 0.0f;
                    }
                }
                Piece<BF16>::template add<SCALE_V>(acc, SCALE_V ? s[k / 4][k % 4] : 1.0f, buf[k]);
                if (decltype(more)::value) buf[k] = gather(o[k / 4][k % 4]);
            }
        };
#pragma unroll 1
        for (int b = 0; b + 1 < kPer / kBatch; ++b) batch(b, std::true_type{});
        batch(kPer / kBatch - 1, std::false_type{});

        // ---- rows cut between lane groups: the group where the row begins (group 0 for the one that is carried on) adds
        // the others' sums up to their first row start, in entry order
        if (g > 0 && w == 0u) {
#pragma unroll
            for (int q = 0; q < NV; ++q) s_left[g][sub * NV + q] = acc[q];
        }
        wave_lds_sync();
        const int from = headed ? 63 - __builtin_clzll(headed) : 0;      // the group whose row is open at the end
        const uint64_t behind = headed & ~((2ull << g) - 1);
        const int next = behind ? __builtin_ctzll(behind) : G;           // the next group with a row start
        const int last = behind && !((at_once >> next) & 1) ? next : next - 1;
        const bool whole = __builtin_amdgcn_inverse_ballot_w64(closed);
        if (g == 0 || w != 0u) {
            for (int gg = g + 1; gg <= last; ++gg)
#pragma unroll
                for (int q = 0; q < NV; ++q) acc[q] += s_left[gg][sub * NV + q];
            if (behind) {
                if (whole) store_row(ref, acc); else to_carry(0, acc);   // (not whole: group 0 with the row of an earlier range)
            } else if (final && cnt == SUB) {
                const int row = FAR ? ref.at : ref.at / kRowBytes;
                const bool ends = k_next > row || e_end == nnz;          // k_next: the row of the entry behind the range
                if (whole && ends) store_row(ref, acc);
                else to_carry(whole ? 1 : 0, acc);                       // goes on in the next range; or ends what earlier ranges began, or lies inside it
                if (whole && !ends) open_row = row;
            }
            if (g == 0 && cut && w != 0u) {                              // the row of an earlier range ended inside group 0
                float first[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) first[q] = s_left[0][sub * NV + q];
                to_carry(0, first);
            }
        }
        if (final) {
            open_row = __builtin_amdgcn_readlane(open_row, from * LPR);
            break;
        }
#pragma unroll
        for (int q = 0; q < NV; ++q) run[q] = __shfl(acc[q], from * LPR + sub, kWave);
        run_ref = RowRef{(uint32_t)__builtin_amdgcn_readlane((int)ref.at, from * LPR), __shfl(ref.du, from * LPR, kWave)};
        began_here = (closed >> (from * LPR)) & 1;
        running = true;
        k_cur = k_next;
        e = e_stop;
        wave_lds_sync();
    }
    if (lane == 0 && record) recs[range] = RangeRec{open_row, 0, 0, 0};
}

// Workgroups are dealt to the eight XCDs in turn, and each XCD has an L2 of its own, so what matters is which rows of H the
// wavefronts of one XCD gather at the same time.  A launch's work is a line of units, an item's slice of columns each (see
// slices_of), of `ranges` ranges, and every XCD takes an eighth of the line, or, where an XCD would get less than a unit,
// kXcds / units of them deal the ranges of a unit among themselves in chunks of kXcdChunk (so that each gets a share of
// every part of the matrix: parts differ in cost per entry when row lengths are clustered).  An XCD then has one frame of H (or one
// slice of it) at a time to keep in its L2.
struct Line { int first, units, ranges, per_xcd, sharing; };   // the first item of the launch; ranges of a unit; of an XCD; log2 of the XCDs that share a unit, or -1

// Four wavefronts per SIMD, but three where factors and several sub-tiles meet, which in bf16 and in rows of four lanes takes 133 - 158
// registers: four would spill up to 20 of them (R-MAT 2^23 x 32 bf16 with values 2280 -> 2440 us; 2^20 x 64 224 -> 236).
template <int LPR, int SLICES, bool BF16, bool SCALE_V, bool FAR, bool ONE>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(ONE || !SCALE_V ? 4 : 3, 8))) void spmm_stream_kernel(int n, int relu, Line line, Batch batch) {
    const int slot = blockIdx.x / kXcds, xcd = blockIdx.x % kXcds;
    int unit, range;
    if (line.sharing >= 0) {
        unit = xcd >> line.sharing;
        range = ((slot / kXcdChunk << line.sharing) + (xcd & ((1 << line.sharing) - 1))) * kXcdChunk + slot % kXcdChunk;
    } else {
        const int at = xcd * line.per_xcd + slot;
        unit = at / line.ranges;
        range = at - unit * line.ranges;
    }
    if (unit >= line.units) return;
    const Item &it = batch.item[line.first + unit / SLICES];
    if (range >= it.n_ranges) return;
    const int slice = unit % SLICES;
    constexpr int F = LPR * Piece<BF16>::kVals;                         // columns of a slice
    spmm_stream<LPR, SLICES, BF16, SCALE_V, FAR, ONE>(range, n, it.nnz, it.range_len, as_global(it.rowptr), as_global(it.colidx), as_global(it.dinv),
                                            as_global(it.h) + slice * LPR * 16, as_global(it.z) + slice * LPR * 16, relu,
                                            as_global(it.recs), slice == 0, as_global(it.carry) + (int64_t)slice * it.n_ranges * 2 * F,
                                            as_global(it.vals), it.gather_dinv != 0, it.rows_per_entry);
}

// Rows cut by range boundaries: the range where such a row begins owns it and adds the left carries of the following
// ranges up to the one that holds the row's end (known from the row pointers).  A row over more than kOwnPieces ranges is
// added up by the whole wavefront, its lane groups taking every G-th piece, so that a hub row is not one chain of dependent
// loads (R-MAT, 2^20 vertices, 16 M entries: 31 -> 5 us; 2^18 vertices: 25 -> 5 us).  The order of the sum depends on
// the row's extent and the range length alone.
constexpr int kOwnPieces = 4;

template <int LPR, int SLICES, bool BF16>
__global__ __launch_bounds__(256) void spmm_carry_kernel(int relu, Batch batch) {
    constexpr int NV = Piece<BF16>::kVals;
    constexpr int F = LPR * NV;
    constexpr int G = kWave / LPR;
    const Item &item = batch.item[blockIdx.y];
    const int slice = blockIdx.z;
    const float *__restrict__ carry = as_global(item.carry) + (int64_t)slice * item.n_ranges * 2 * F, *__restrict__ dinv = as_global(item.dinv);
    const RangeRec *__restrict__ recs = as_global(item.recs);
    const int32_t *__restrict__ rowptr = as_global(item.rowptr);
    char *__restrict__ z = as_global(item.z) + slice * LPR * 16;
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane % LPR, g = lane / LPR;
    const int first = (blockIdx.x * 256 + threadIdx.x) / kWave * G;     // the wavefront's records
    const int t = first + g;
    int row = -1, last = 0;
    if (t < item.n_ranges) {
        row = recs[t].open_row;
        if (row >= 0) last = min((rowptr[row + 1] - 1) / item.range_len, item.n_ranges - 1);
    }
    auto left = [&](int j, int q) { return carry[(int64_t)j * 2 * F + sub * NV + q]; };
    const bool own = row >= 0 && last - t <= kOwnPieces;
    if (own) {
        float acc[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) acc[q] = carry[((int64_t)t * 2 + 1) * F + sub * NV + q];
        for (int j = t + 1; j <= last; ++j)
#pragma unroll
            for (int q = 0; q < NV; ++q) acc[q] += left(j, q);
        finish_row<BF16, NV>(z, (int64_t)row, LPR * SLICES * 16, sub, dinv, relu, acc);
    }
    for (uint64_t todo = __ballot(row >= 0 && !own && sub == 0); todo; todo &= todo - 1) {
        const int src = __builtin_ctzll(todo);
        const int tt = first + src / LPR, rr = __shfl(row, src, kWave), ll = __shfl(last, src, kWave);
        float acc[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) acc[q] = 0.0f;
#pragma unroll 4
        for (int j = tt + 1 + g; j <= ll; j += G)
#pragma unroll
            for (int q = 0; q < NV; ++q) acc[q] += left(j, q);
#pragma unroll
        for (int d = LPR; d < kWave; d <<= 1)
#pragma unroll
            for (int q = 0; q < NV; ++q) acc[q] += __shfl_xor(acc[q], d, kWave);
        if (g == 0) {
#pragma unroll
            for (int q = 0; q < NV; ++q) acc[q] += carry[((int64_t)tt * 2 + 1) * F + sub * NV + q];
            finish_row<BF16, NV>(z, (int64_t)rr, LPR * SLICES * 16, sub, dinv, relu, acc);
        }
    }
}

struct Workspace {
    RangeRec *recs;
    float *carry;
};

// Entries per wavefront: a multiple of the sub-tile, at most kMaxRange, smaller when the input is small.
// max_ranges > 0: the caller has room for that many range records only; ranges are stretched to fit, up to
// kLongestRange (0 is returned if even that does not do).
int range_length(int64_t nnz, int sub_tile, int64_t max_ranges = 0) {
    int64_t len = (nnz + kTargetWaves - 1) / kTargetWaves;
    len = (len + sub_tile - 1) / sub_tile * sub_tile;
    if (len > kMaxRange) len = kMaxRange;
    if (max_ranges > 0 && (nnz + len - 1) / len > max_ranges) {
        len = (nnz + max_ranges - 1) / max_ranges;
        len = (len + sub_tile - 1) / sub_tile * sub_tile;
        if (len > kLongestRange) return 0;
    }
    return (int)len;
}

// Sized for the largest number of ranges any call with at most nnz entries can have (a smaller snapshot gets
// shorter ranges, never more than kTargetWaves + 1 of them), so a buffer queried for the largest snapshot of a
// block serves every snapshot of it, and both dtypes.
size_t workspace_layout(int64_t nnz, int32_t f, Workspace *ws, void *base, int64_t exact_ranges = 0) {
    // exact_ranges: the number of ranges of one particular call (a caller that knows the call and has little room)
    const int64_t ranges = exact_ranges > 0 ? exact_ranges
                                            : std::max<int64_t>(kTargetWaves + 1, (nnz + kMaxRange - 1) / kMaxRange) + 1;
    const size_t o_carry = round_up((size_t)ranges * sizeof(RangeRec), 256);
    const size_t total = o_carry + round_up((size_t)ranges * 2 * f * sizeof(float), 256);
    if (ws) {
        char *b = static_cast<char *>(base);
        ws->recs = reinterpret_cast<RangeRec *>(b);
        ws->carry = reinterpret_cast<float *>(b + o_carry);
    }
    return total;
}

// The aggregations of one launch pair; the line's units are as long as the longest, the others' wavefronts leave early.
template <int LPR, int SLICES, bool BF16>
int launch(int64_t n, int count, const Batch &b, bool scale_v, int relu, hipStream_t s) {
    constexpr int G = 256 / LPR;
    int ranges = 0;
    for (int k = 0; k < count; ++k) ranges = std::max(ranges, b.item[k].n_ranges);
    bool one = true;
    for (int k = 0; k < count; ++k) one = one && b.item[k].range_len == kWave / LPR * per_group(LPR);
    auto stream_kernel = [&](auto far, auto single) {
        return scale_v ? spmm_stream_kernel<LPR, SLICES, BF16, true, decltype(far)::value, decltype(single)::value>
                       : spmm_stream_kernel<LPR, SLICES, BF16, false, decltype(far)::value, decltype(single)::value>;
    };
    const auto kernel = n * (LPR * SLICES * 16) > (int64_t(1) << 32) ? stream_kernel(std::true_type{}, std::false_type{})
                        : one                                        ? stream_kernel(std::false_type{}, std::true_type{})
                                                                     : stream_kernel(std::false_type{}, std::false_type{});
    // a grid's threads are counted in 32 bits
    const int most = (int)std::max<int64_t>(1, ((int64_t(1) << 31) / kWave) / ((int64_t)ranges * SLICES + kXcds * kXcdChunk));
    for (int first = 0; first < count; first += most) {
        const int units = std::min(count - first, most) * SLICES;
        const int sharing = kXcds % units == 0 ? __builtin_ctz(kXcds / units) : -1, round = kXcdChunk << std::max(sharing, 0);
        const int per_xcd = sharing >= 0 ? (ranges + round - 1) / round * kXcdChunk : (int)(((int64_t)units * ranges + kXcds - 1) / kXcds);
        hipLaunchKernelGGL(kernel, dim3(kXcds * per_xcd), dim3(kWave), 0, s, (int)n, relu, Line{first, units, ranges, per_xcd, sharing}, b);
        DGNN_RETURN_IF_LAUNCH_FAILED();
    }
    hipLaunchKernelGGL((spmm_carry_kernel<LPR, SLICES, BF16>), dim3((ranges + G - 1) / G, count, SLICES), dim3(256), 0, s, relu, b);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}

// Into how many slices of columns an aggregation is cut, each with XCDs of its own: an L2 then holds that slice of H only, as if
// it were so much larger.  Every entry's bookkeeping is done once per slice, and below 128 bytes, the L2's line, nothing is saved
// (twice the time).  Slices of 128 bytes pay where H does not fit an L2 of 4 MB but a slice of it does for a good part.  us per
// aggregation of eight together, 17 entries per row, without / with slices of 128 bytes:
//                     64 columns fp32    128 columns bf16    128 columns fp32 (without: two slices of 256 bytes)
//   uniform   25 K      8.3 /  8.0         9.2 /  8.8          15.8 / 14.4
//             33 K     12.5 / 10.1        13.3 / 11.0          24.3 / 19.7
//             50 K     23.2 / 16.1        24.1 / 17.3          46.3 / 32.3
//            100 K     56.7 / 47.7        58.8 / 48.8           113 / 97
//            131 K     78.5 / 68.8        80.6 / 70.3           154 / 139
//   R-MAT    2^15       9.0 /  9.9        10.4 / 10.8          16.7 / 18.1
//            2^16      17.6 / 18.8        19.7 / 20.3          40.6 / 42.1
//            2^17      42.3 / 43.5        47.3 / 46.7          89.5 / 92.1
// (uniform 200 K equal, 1 M 664 / 690; R-MAT 2^20 361 / 373.)  On a power-law graph the rows that most entries name lie in the L2s anyway,
// and the slices cost 2 - 10 %; a uniform one gains up to 30 %.  The launch knows n and the entry count only, not how rows
// are named, so the line follows the larger of the two.  Rows of 512 bytes go in two slices of 256 everywhere else (uniform 32 K whole /
// two 45 / 36, R-MAT 2^20 1.10 / 0.91 ms).
int slices_of(int64_t n, int32_t f, dgnn_dtype dt) {
    const int row_bytes = f * (dt == DGNN_F32 ? 4 : 2);
    const bool narrow = row_bytes >= 256 && n * 128 >= (int64_t(3) << 20) && n * 128 <= (int64_t(16) << 20);
    return narrow ? row_bytes / 128 : row_bytes > 256 ? 2 : 1;
}

}  // namespace

extern "C" int dgnn_spmm_workspace(int64_t n, int64_t nnz, int32_t f, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (n <= 0 || nnz < 0 || !supported_width(f)) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz)) return DGNN_ERR_OVERFLOW;
    *bytes = workspace_layout(nnz, f, nullptr, nullptr);
    return DGNN_OK;
}

namespace {

// Entries per range of one call for this snapshot, width and storage type (max_ranges as in range_length).
int range_length_of_call(int64_t n, int64_t nnz, int32_t f, dgnn_dtype dt, int64_t max_ranges = 0) {
    const int lpr = (dt == DGNN_F32 ? f / 4 : f / 8) / slices_of(n, f, dt);
    return range_length(nnz, (kWave / lpr) * per_group(lpr), max_ranges);
}

int launch_width(int64_t n, int count, const Batch &b, bool scale_v, int32_t f, dgnn_dtype dt, int relu, hipStream_t s) {
    const bool bf = dt == DGNN_BF16;
    switch (slices_of(n, f, dt)) {
        case 4: return launch<8, 4, false>(n, count, b, scale_v, relu, s);                      // fp32, 128 columns
        case 2: return f == 128 && !bf ? launch<16, 2, false>(n, count, b, scale_v, relu, s)
                       : bf            ? launch<8, 2, true>(n, count, b, scale_v, relu, s) : launch<8, 2, false>(n, count, b, scale_v, relu, s);
        default: break;
    }
    switch (bf ? f / 8 : f / 4) {   // lanes per feature row, 16 bytes each
        case 2: return launch<2, 1, true>(n, count, b, scale_v, relu, s);
        case 4: return bf ? launch<4, 1, true>(n, count, b, scale_v, relu, s) : launch<4, 1, false>(n, count, b, scale_v, relu, s);
        case 8: return bf ? launch<8, 1, true>(n, count, b, scale_v, relu, s) : launch<8, 1, false>(n, count, b, scale_v, relu, s);
        case 16: return bf ? launch<16, 1, true>(n, count, b, scale_v, relu, s) : launch<16, 1, false>(n, count, b, scale_v, relu, s);
        default: return DGNN_ERR_SHAPE;
    }
}

int spmm(int64_t n, int64_t nnz, const int32_t *rowptr, const int32_t *colidx, const float *dinv, const float *vals,
         const void *h, int32_t f, void *z, dgnn_dtype dt, uint32_t flags, uint32_t allowed, void *ws, size_t ws_bytes,
         void *stream, int64_t max_ranges = 0) {
    if (!rowptr || !colidx || !h || !z || !ws) return DGNN_ERR_NULL;
    if (n <= 0 || nnz <= 0 || !supported_width(f) || (flags & ~allowed)) return DGNN_ERR_SHAPE;
    if (dt != DGNN_F32 && dt != DGNN_BF16) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz)) return DGNN_ERR_OVERFLOW;
    if (!aligned16(h) || !aligned16(z) || !aligned16(ws)) return DGNN_ERR_ALIGN;
    if (h == z) return DGNN_ERR_ALIAS;
    // max_ranges > 0: the records of exactly this call, laid out for its own number of ranges
    const int range_len = range_length_of_call(n, nnz, f, dt, max_ranges);
    if (range_len <= 0) return DGNN_ERR_CAPACITY;
    const int64_t ranges = (nnz + range_len - 1) / range_len;
    Workspace w;
    if (ws_bytes < workspace_layout(nnz, f, &w, ws, max_ranges > 0 ? ranges : 0)) return DGNN_ERR_CAPACITY;
    const bool scale_v = vals != nullptr || (dinv != nullptr && !(flags & DGNN_H_PRESCALED));
    Batch b;
    b.item[0] = Item{rowptr, colidx, dinv, vals, static_cast<const char *>(h), static_cast<char *>(z), w.recs, w.carry, (int32_t)nnz,
                     range_len, (int32_t)ranges, dinv && !(flags & DGNN_H_PRESCALED) ? 1 : 0, (float)n / (float)nnz};
    return launch_width(n, 1, b, scale_v, f, dt, (flags & DGNN_RELU) ? 1 : 0, (hipStream_t)stream);
}

}  // namespace

extern "C" int dgnn_spmm(int64_t n, int64_t nnz, const int32_t *rowptr, const int32_t *colidx, const float *dinv,
                         const void *h, int32_t f, void *z, dgnn_dtype dt, uint32_t flags,
                         void *ws, size_t ws_bytes, void *stream) {
    return spmm(n, nnz, rowptr, colidx, dinv, nullptr, h, f, z, dt, flags, DGNN_RELU | DGNN_H_PRESCALED, ws, ws_bytes, stream);
}

// ---- the aggregations of several timesteps in one launch pair: on small snapshots one of them leaves most of the chip
// idle, and every launch costs as long as the aggregation itself
extern "C" int dgnn_spmm_batch_workspace(int32_t count, int64_t nnz, int32_t f, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (count <= 0 || nnz < 0 || !supported_width(f)) return DGNN_ERR_SHAPE;
    if (!fits_index(nnz)) return DGNN_ERR_OVERFLOW;
    // the shortest range any storage type uses at this width is one sub-tile; no call has more ranges than this
    const int lanes = std::min(f / 4, 16);                        // per row, at most: fp32 rows of 128 columns are always cut (see slices_of)
    const int64_t shortest = kWave / lanes * per_group(lanes);    // (slices make sub-tiles longer)
    const int64_t ranges = std::min<int64_t>((nnz + shortest - 1) / shortest, std::max<int64_t>(kTargetWaves + 1, (nnz + kMaxRange - 1) / kMaxRange));
    *bytes = (size_t)count * workspace_layout(nnz, f, nullptr, nullptr, ranges + 1);
    return DGNN_OK;
}

extern "C" int dgnn_spmm_batch(int64_t n, int32_t count, const dgnn_spmm_item *items, int32_t f, dgnn_dtype dt, uint32_t flags,
                               void *ws, size_t ws_bytes, void *stream) {
    if (!items || !ws) return DGNN_ERR_NULL;
    if (n <= 0 || count <= 0 || !supported_width(f) || (flags & ~(DGNN_RELU | DGNN_H_PRESCALED))) return DGNN_ERR_SHAPE;
    if (dt != DGNN_F32 && dt != DGNN_BF16) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1)) return DGNN_ERR_OVERFLOW;
    if (!aligned16(ws)) return DGNN_ERR_ALIGN;
    const bool weighted = items[0].val != nullptr, normalised = items[0].dinv != nullptr;
    size_t needed = 0;
    auto ranges_of = [&](const dgnn_spmm_item &it, int &range_len) {
        range_len = range_length_of_call(n, it.nnz, f, dt);
        return (it.nnz + range_len - 1) / range_len;
    };
    int range_len;
    for (int k = 0; k < count; ++k) {
        const dgnn_spmm_item &it = items[k];
        if (!it.rowptr || !it.colidx || !it.h || !it.z) return DGNN_ERR_NULL;
        if (it.nnz <= 0 || (it.val != nullptr) != weighted || (it.dinv != nullptr) != normalised) return DGNN_ERR_SHAPE;
        if (weighted && !it.dinv && (flags & DGNN_H_PRESCALED)) return DGNN_ERR_SHAPE;
        if (!fits_index(it.nnz)) return DGNN_ERR_OVERFLOW;
        if (!aligned16(it.h) || !aligned16(it.z)) return DGNN_ERR_ALIGN;
        if (it.h == it.z) return DGNN_ERR_ALIAS;
        needed += workspace_layout(it.nnz, f, nullptr, nullptr, ranges_of(it, range_len));
    }
    if (ws_bytes < needed) return DGNN_ERR_CAPACITY;
    // whether a per-entry factor is gathered is the launch's choice, not the item's
    const bool scale_v = weighted || (normalised && !(flags & DGNN_H_PRESCALED));
    char *base = static_cast<char *>(ws);
    for (int done = 0; done < count; done += kMaxBatch) {
        const int m = std::min(count - done, kMaxBatch);
        Batch b;
        for (int k = 0; k < m; ++k) {
            const dgnn_spmm_item &it = items[done + k];
            const int64_t ranges = ranges_of(it, range_len);
            Workspace w;
            base += workspace_layout(it.nnz, f, &w, base, ranges);
            b.item[k] = Item{it.rowptr, it.colidx, it.dinv, it.val, static_cast<const char *>(it.h), static_cast<char *>(it.z), w.recs, w.carry,
                             (int32_t)it.nnz, range_len, (int32_t)ranges, it.dinv && !(flags & DGNN_H_PRESCALED) ? 1 : 0, (float)n / (float)it.nnz};
        }
        const int rc = launch_width(n, m, b, scale_v, f, dt, (flags & DGNN_RELU) ? 1 : 0, (hipStream_t)stream);
        if (rc != DGNN_OK) return rc;
    }
    return DGNN_OK;
}

// ---- the same aggregation for callers that cannot allocate: its carry records live in a file-scope device array ----
namespace {

constexpr size_t kStaticScratchBytes = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void *g_scratch_ptr[kMaxDevices];   // per device: the address of that device's copy of `scratch`, asked for once

// The device address of the current device's `scratch` (the array's name is only a host-side handle).
int static_scratch(void **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return DGNN_ERR_HIP;
    }
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return DGNN_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DGNN_OK;
}

}  // namespace

extern "C" int dgnn_spmm_static_limit(size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    *bytes = kStaticScratchBytes;
    return DGNN_OK;
}

extern "C" int dgnn_spmm_static(int64_t n, int64_t nnz, const int32_t *rowptr, const int32_t *colidx, const float *dinv,
                                const void *h, int32_t f, void *z, dgnn_dtype dt, uint32_t flags, void *stream) {
    // argument errors first, so that they are reported without touching the device
    if (!rowptr || !colidx || !h || !z) return DGNN_ERR_NULL;
    if (n <= 0 || nnz <= 0 || !supported_width(f) || (flags & ~(DGNN_RELU | DGNN_H_PRESCALED))) return DGNN_ERR_SHAPE;
    if (dt != DGNN_F32 && dt != DGNN_BF16) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz)) return DGNN_ERR_OVERFLOW;
    // as many ranges as the array has room for records of: ranges grow longer where the usual ones would be too many
    const int64_t max_ranges = (int64_t)((kStaticScratchBytes - 512) / (sizeof(RangeRec) + 2 * (size_t)f * sizeof(float)));
    if (range_length_of_call(n, nnz, f, dt, max_ranges) <= 0) return DGNN_ERR_CAPACITY;
    void *ptr = nullptr;
    const int rc = static_scratch(&ptr);
    if (rc != DGNN_OK) return rc;
    // every range writes its record and the carries its flags announce before the second kernel reads them, so nothing
    // in the array has to start at zero; what the previous call left there is never read
    return spmm(n, nnz, rowptr, colidx, dinv, nullptr, h, f, z, dt, flags, DGNN_RELU | DGNN_H_PRESCALED, ptr,
                kStaticScratchBytes, stream, max_ranges);
}

extern "C" int dgnn_spmm_weighted(int64_t n, int64_t nnz, const int32_t *rowptr, const int32_t *colidx, const float *val,
                                  const float *dinv, const void *h, int32_t f, void *z, dgnn_dtype dt, uint32_t flags,
                                  void *ws, size_t ws_bytes, void *stream) {
    if (!val) return DGNN_ERR_NULL;
    // with a normalisation the right-hand factor must already be in the rows of h: the kernel gathers one
    // per-entry factor (the value), not two
    if (dinv && !(flags & DGNN_H_PRESCALED)) return DGNN_ERR_SHAPE;
    if (!dinv && (flags & DGNN_H_PRESCALED)) return DGNN_ERR_SHAPE;
    return spmm(n, nnz, rowptr, colidx, dinv, val, h, f, z, dt, flags, DGNN_RELU | DGNN_H_PRESCALED, ws, ws_bytes, stream);
}

namespace {

// ---- dinv[u] = (sum of the values of row u)^(-1/2): the weighted counterpart of 1 + deg_u -------------------
// Split by ENTRIES like the aggregation, so that hub rows of a power-law graph cost what their entries cost:
// a wavefront owns kSumRange consecutive entries, copies their values to LDS with coalesced loads, and then
// every lane adds up whole rows out of LDS (rows that hold more than kCoop of the range's entries are summed
// by the 64 lanes together).  A row cut by the range's ends leaves a piece in the workspace; a second small
// kernel adds a cut row's pieces in entry order.  Every sum has an order fixed by the row structure alone:
// results repeat bit for bit.
constexpr int kSumRange = 2048;
constexpr int kCoop = 64;

// p_cont: piece of the row that began in an earlier range; p_own/owner: first piece of the row that begins in
// this range and runs past its end (owner = -1: there is none)
struct SumRec { float p_cont, p_own; int32_t owner, pad; };

// Sums of eight rows at once: v[q] is this lane's share of row q.  Three exchange steps halve what a lane keeps
// (the lane's bit 0 chooses the half of q, bit 1 the quarter, bit 2 the row), three more add up over the other
// lane bits: eleven cross-lane moves instead of forty-eight.  Returns, in lane l, the sum of row l % 8.
__device__ __forceinline__ float wave_sum8(const float (&v)[8], int lane) {
    float w4[4], w2[2];
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) w4[q] = (b0 ? v[q + 4] : v[q]) + __shfl_xor(b0 ? v[q] : v[q + 4], 1, kWave);
#pragma unroll
    for (int q = 0; q < 2; ++q) w2[q] = (b1 ? w4[q + 2] : w4[q]) + __shfl_xor(b1 ? w4[q] : w4[q + 2], 2, kWave);
    float r = (b2 ? w2[1] : w2[0]) + __shfl_xor(b2 ? w2[0] : w2[1], 4, kWave);
    r += __shfl_xor(r, 8, kWave);
    r += __shfl_xor(r, 16, kWave);
    r += __shfl_xor(r, 32, kWave);
    // this lane now holds row 4 * bit0 + 2 * bit1 + bit2; row q is wanted in the lanes with l % 8 == q
    const int q = lane & 7;
    return __shfl(r, ((q >> 2) & 1) | (q & 2) | ((q & 1) << 2), kWave);
}

// A vertex whose row sum is not positive (no entries at all, or weights that cancel) has no normalisation; it gets
// the factor 0, so it neither sends nor receives anything, instead of an infinity that would turn into NaN.
__device__ __forceinline__ float inv_sqrt_or_zero(float s) { return s > 0.0f ? 1.0f / sqrtf(s) : 0.0f; }

__global__ __launch_bounds__(kWave) void weighted_rowsum_kernel(int n, int nnz, const int32_t *__restrict__ rowptr,
                                                               const float *__restrict__ val, SumRec *__restrict__ recs,
                                                               float *__restrict__ dinv) {
    __shared__ float s_val[kSumRange];
    const int lane = threadIdx.x, range = blockIdx.x;
    nnz = min(nnz, rowptr[n]);                          // the host's count may be an upper bound: the last row pointer decides
    const int e0 = (int)min((int64_t)range * kSumRange, (int64_t)nnz), e1 = (int)min((int64_t)e0 + kSumRange, (int64_t)nnz);
    if (e0 >= nnz && range > 0) {                       // nothing stored here
        if (lane == 0) recs[range] = SumRec{0.0f, 0.0f, -1, 0};
        return;
    }
    const bool last = e1 == nnz;
    // the values of the range, 64 consecutive ones per load
#pragma unroll 16
    for (int i = lane; i < kSumRange; i += kWave) s_val[i] = val[max(min(e0 + i, nnz - 1), 0)];   // unconditional: loads stay in flight together
    // rows of the range: the one cut by its begin (if any), then every row that begins in [e0, e1), empty ones
    // included; the last range also takes the empty rows behind the last entry
    const int k_lo = wave_find_row(rowptr, n, e0 - 1, lane) + 1;          // first row that begins at e0 or later
    const int k_first = rowptr[k_lo] > e0 ? k_lo - 1 : k_lo;              // rowptr[n] = nnz > e0
    wave_lds_sync();
    float p_cont = 0.0f, p_own = 0.0f;
    int owner = -1;
    bool more = true;
    for (int base = k_first; more; base += kWave) {
        const int r = base + lane;
        const int rb_raw = rowptr[min(r, n)];
        const bool valid = r < n && (last || rb_raw < e1);     // the range's rows end where a row begins at e1 or later
        more = __ballot(valid) == ~0ull;
        const int rb = valid ? rb_raw : e1, re = valid ? rowptr[r + 1] : e1;
        const int b = max(rb, e0) - e0, e = min(re, e1) - e0;
        const bool coop = e - b > kCoop;
        float sum = 0.0f;
        if (!coop) {                                                       // four entries a round, reads past the row's end masked
            float s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
            for (int i = b; i < e; i += 4) {
                const float x0 = s_val[i], x1 = s_val[min(i + 1, kSumRange - 1)], x2 = s_val[min(i + 2, kSumRange - 1)],
                            x3 = s_val[min(i + 3, kSumRange - 1)];
                sum += x0;
                s1 += i + 1 < e ? x1 : 0.0f;
                s2 += i + 2 < e ? x2 : 0.0f;
                s3 += i + 3 < e ? x3 : 0.0f;
            }
            sum = (sum + s1) + (s2 + s3);
        }
        // longer rows: all lanes together, eight rows per round so that one set of cross-lane moves serves eight sums
        const uint64_t coop_mask = __ballot(coop);
        const int rank = __popcll(coop_mask & ((1ull << lane) - 1));
        int group = 0;
        for (uint64_t todo = coop_mask; todo; ++group) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                float a0 = 0.0f, a1 = 0.0f;
                if (todo) {
                    const int src = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    const int bb = __builtin_amdgcn_readlane(b, src), ee = __builtin_amdgcn_readlane(e, src);
                    int i = bb + lane;
                    for (; i + kWave < ee; i += 2 * kWave) { a0 += s_val[i]; a1 += s_val[i + kWave]; }
                    if (i < ee) a0 += s_val[i];
                }
                v[q] = a0 + a1;
            }
            const float t = __shfl(wave_sum8(v, lane), rank & 7, kWave);
            if (coop && (rank >> 3) == group) sum = t;
        }
        const bool open_l = rb < e0, open_r = re > e1;
        if (valid && !open_l && !open_r) dinv[r] = inv_sqrt_or_zero(sum);
        const uint64_t m_cont = __ballot(valid && open_l), m_own = __ballot(valid && !open_l && open_r);
        if (m_cont) p_cont = __shfl(sum, __builtin_ctzll(m_cont), kWave);
        if (m_own) { const int src = __builtin_ctzll(m_own); p_own = __shfl(sum, src, kWave); owner = base + src; }
    }
    if (lane == 0) recs[range] = SumRec{p_cont, p_own, owner, 0};
}

// a row that begins in range w and ends in a later one: its pieces in entry order
__global__ __launch_bounds__(256) void weighted_rowsum_fix_kernel(int n_ranges, const int32_t *__restrict__ rowptr,
                                                                  const SumRec *__restrict__ recs, float *__restrict__ dinv) {
    const int w = blockIdx.x * 256 + threadIdx.x;
    if (w >= n_ranges) return;
    const SumRec rec = recs[w];
    if (rec.owner < 0) return;
    const int end = rowptr[rec.owner + 1];
    float acc = rec.p_own;
    for (int r = w + 1; (int64_t)r * kSumRange < end; ++r) acc += recs[r].p_cont;
    dinv[rec.owner] = inv_sqrt_or_zero(acc);
}

size_t weighted_dinv_workspace(int64_t nnz) {
    return round_up(sizeof(SumRec) * (size_t)((nnz + kSumRange - 1) / kSumRange), (size_t)256) + 256;
}

}  // namespace

extern "C" int dgnn_csr_weighted_dinv_workspace(int64_t nnz, size_t *bytes) {
    if (!bytes) return DGNN_ERR_NULL;
    if (nnz < 0) return DGNN_ERR_SHAPE;
    if (!fits_index(nnz)) return DGNN_ERR_OVERFLOW;
    *bytes = weighted_dinv_workspace(nnz);
    return DGNN_OK;
}

extern "C" int dgnn_csr_weighted_dinv(int64_t n, int64_t nnz, const int32_t *rowptr, const float *val, float *dinv,
                                      void *ws, size_t ws_bytes, void *stream) {
    if (!rowptr || !val || !dinv || !ws) return DGNN_ERR_NULL;
    if (n <= 0 || nnz <= 0) return DGNN_ERR_SHAPE;
    if (!fits_index(n + 1) || !fits_index(nnz)) return DGNN_ERR_OVERFLOW;
    if (!aligned16(ws)) return DGNN_ERR_ALIGN;
    if (ws_bytes < weighted_dinv_workspace(nnz)) return DGNN_ERR_CAPACITY;
    hipStream_t s = (hipStream_t)stream;
    const int ranges = (int)((nnz + kSumRange - 1) / kSumRange);
    hipLaunchKernelGGL(weighted_rowsum_kernel, dim3((unsigned)ranges), dim3(kWave), 0, s, (int)n, (int)nnz, rowptr, val,
                       (SumRec *)ws, dinv);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    hipLaunchKernelGGL(weighted_rowsum_fix_kernel, dim3((unsigned)((ranges + 255) / 256)), dim3(256), 0, s, ranges, rowptr,
                       (const SumRec *)ws, dinv);
    DGNN_RETURN_IF_LAUNCH_FAILED();
    return DGNN_OK;
}
