// libcsr5: CSR -> CSR5 conversion and CSR5 SpMV for gfx950 (MI355X).
//
// Follows Liu & Vinter, "CSR5: An Efficient Storage Format for Cross-Platform
// Sparse Matrix-Vector Multiplication" (ICS'15): format in Section 3, SpMV in
// Section 4.  omega = 64 = one wavefront per tile, one lane per tile column.
//
// What is different from the paper's own GPU design, and why, is said at each
// kernel.  The C ABI is declared in include/csr5.h.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <mutex>
#include <new>
#include <type_traits>

#include "csr5.h"
#include "far_lists.h"
#include "row_share.h"

namespace {

constexpr int OMEGA = CSR5_OMEGA;
constexpr int SBITS = 6;  // ceil(log2 omega)
constexpr uint32_t BAD_BITS = CSR5_STATUS_BAD_ROW_PTR | CSR5_STATUS_BAD_COL_IDX;
// Internal status bit (not reported): some COMPLETE tile is marked, so the
// empty_offset layout has to be scanned.  Set by the descriptor step of k_transpose only; the scan
// kernels decide on it, and nothing in their own launches changes it.
constexpr uint32_t STATUS_SCAN_NEEDED = 1u << 16;
// Internal status bit: some tile (the incomplete one included) starts further
// into a row than the look-behind can make up for, so the SpMV sends its
// cross-tile sums through the auxiliary array (see k_spmv and k_prepare).
constexpr uint32_t STATUS_NEEDS_CARRY = 1u << 17;
// Internal status bit: some first tile of a workgroup (or the incomplete tile)
// starts more than LOOK entries into a row: the look-behind of this matrix reads
// the far part of the records too (see below).
constexpr uint32_t STATUS_FAR_HEADS = 1u << 18;
// Internal status bit: at least one in ORDER_MIN_SHARE complete tiles lies inside
// a single row (the tile order by columns may pay, see order_place).
constexpr uint32_t STATUS_LONG_ROWS = 1u << 19;
constexpr int ORDER_MIN_SHARE = 2;
constexpr int ORDER_BUCKETS = 1024;      // of its sort, twice
// A tile whose first segment continues a row of the previous tile completes
// that row itself when it can get at the row's head.  The tiles of one
// workgroup of the tile kernel are neighbours and hand the finished head over
// through LDS (any head that began inside the previous tile).  The first tile of
// a workgroup sums the head itself, from a copy of the last LOOK_MAX entries of
// the tile before it that the conversion keeps in CSR order next to the format
// (in the transposed tile they are spread over sigma cache lines each for val
// and col_idx; re-reading them there cost 16 % more memory traffic).  The last
// LOOK = 32 of them are three cache lines, read without first asking how long
// the head is (a dependent load at that point costs more than the lines); the
// LOOK_FAR = 128 before them are read only by a tile whose head is longer than
// LOOK.  One record per workgroup of tiles (tile_group_waves), none for
// sigma < LOOK_MIN_SIGMA, where the matrices are small, nor for
// sigma > LOOK_MAX_SIGMA, where the tile kernel has no registers to spare (those
// matrices always take the auxiliary-array path).
constexpr int LOOK = 32;
constexpr int LOOK_FAR = 128;
constexpr int LOOK_MAX = LOOK + LOOK_FAR;
// Heads longer than LOOK are re-read only in matrices of at most this many
// nonzeros; larger ones take the auxiliary array and its second kernel instead.
// The far part costs the tile kernel 5-8 % on matrices with 64- and 128-entry
// rows, the second kernel about 3 us and a launch: measured at 8 to 60 M
// nonzeros, re-reading wins up to 24 M (5-9 % of the SpMV), is level at 32 M and
// loses beyond (3-5 %).
constexpr int64_t LOOK_FAR_MAX_NNZ = 28 * 1000 * 1000;
// The three instantiations of the tile kernel: cross-tile sums through the
// auxiliary array and a second kernel; by look-behind; through the auxiliary array
// inside the one kernel (see "One-launch form of the auxiliary-array path" below).
constexpr int MODE_CARRY = 0, MODE_LOOK = 1, MODE_ONE = 2;
// The one-launch form saves the second kernel (3 us and a launch) and pays for
// one or two atomics with a return value per group of tiles (0.2-1 ns of kernel
// time each, whenever they are sent).  Measured against the
// two-kernel form: matrices of a few thousand tiles gain 7-20 % whatever their
// rows look like (a dense 2000 x 2000 matrix 13.1 -> 10.7 us); with rows of 701
// or 2000 entries throughout the gain is 2-7 % at 6 M nonzeros and level, within
// 2 %, at 10-21 M (it was gone at 6 M and a loss of 4-13 % at 8-21 M when the line
// was drawn, before the tile's loads went through buffer descriptors); matrices
// whose rows are short on average and that take this path for a few long rows still
// gain at 17 M (power-law: 2.3 %) and are level at 30 M.  Hence: up to ONE_LAUNCH_ANY_TILES tiles always, up to
// ONE_LAUNCH_MAX_TILES when the average row is shorter than ONE_LAUNCH_SHORT_ROWS.
constexpr int ONE_LAUNCH_ANY_TILES = 6144;
constexpr int ONE_LAUNCH_MAX_TILES = 32768;
constexpr int ONE_LAUNCH_SHORT_ROWS = 64;
constexpr int LOOK_MIN_SIGMA = 8, LOOK_MAX_SIGMA = 32;
constexpr bool look_sigma(int sigma) { return sigma >= LOOK_MIN_SIGMA && sigma <= LOOK_MAX_SIGMA; }
constexpr bool one_launch_fits(int sigma, int64_t tiles) { return look_sigma(sigma) && tiles <= ONE_LAUNCH_MAX_TILES; }
// Tiles (= wavefronts) per workgroup of the tile kernel and of the transposition,
// chosen so the LDS buffer stays under 40 KB.
constexpr int tile_group_waves(int sigma) { return sigma <= 16 ? 4 : (sigma <= 32 ? 2 : 1); }
// One record per group of tiles, holding the last LOOK_MAX entries, in CSR
// order, of the group's last tile (of the last complete tile, for the last
// group).  Near part first: LOOK values (8 bytes each, 4 used in single
// precision) followed by LOOK column indices, contiguous, so that a tile fetches
// it with one run of three cache lines; then the far part, LOOK_FAR values and
// LOOK_FAR column indices (entry j of the far part is entry T - LOOK_MAX + j of
// the tile, entry i of the near part entry T - LOOK + i).  Record of tile t:
// number t / tile_group_waves.  Strides of the two views of the record array
// (last_val points at a record's first byte, last_col at its near indices):
// A matrix too large for far heads (LOOK_FAR_MAX_NNZ) keeps the near part only.
constexpr int NEAR_REC_BYTES = LOOK * 8 + LOOK * 4;
constexpr int LAST_REC_BYTES = LOOK_MAX * 8 + LOOK_MAX * 4;
constexpr int record_bytes(int64_t nnz) { return nnz <= LOOK_FAR_MAX_NNZ ? LAST_REC_BYTES : NEAR_REC_BYTES; }
// where a record's far part begins, counted from last_val / last_col of the record
template <typename VT> constexpr int far_val_at() { return (LOOK * 8 + LOOK * 4) / int(sizeof(VT)); }
constexpr int FAR_COL_AT = (LOOK * 8 + LOOK * 4 + LOOK_FAR * 8 - LOOK * 8) / 4;
constexpr uint32_t STATUS_PUBLIC = 0xffu;
// Where sample_window adds up, in words from the status word: in another line than that, at which
// every workgroup of the transposition may queue up.
constexpr int WINDOW_ANSWER_AT = 32, FAR_ANSWER_AT = 40;
constexpr int NUM_XCD = 8;  // MI355X: 8 accelerator dies, each with its own L2

// sigma rule constants <r, s, t, u> for MI355X (Section 3.2 leaves them to the
// hardware; measured with calibrate.py, see csr5_sigma_auto).  On this GPU the
// best sigma does not depend on nnz/row at all for matrices that fill the chip
// (16 wins by 2-3 % from 1 to 256 nonzeros per row), so r = s = u.
constexpr int RULE_R = 16, RULE_S = 16, RULE_T = 256, RULE_U = 16;
// What does matter is the number of tiles: the chip holds 256 CUs x 16
// wavefronts of this kernel, and below about three rounds of them the ramp-up and
// the last partial round dominate; such a matrix gets the smaller tile.  Placed
// with matrices of 8 and of 27 entries per row at 8 to 40 M nonzeros: at sigma 16
// the 27-per-row ones win from 12 M nonzeros on (7 % at 14 M), the 8-per-row
// ones are within 2 % either way between 12 M and 20 M.
constexpr int64_t RULE_MIN_TILES = 3 * 256 * 16;
constexpr int RULE_SIGMA_SMALL = 8;
constexpr bool rule_sigma(int sigma) { return sigma == RULE_SIGMA_SMALL || sigma == RULE_R; }

// Index width of row_ptr, tile_ptr and empty_offset_ptr.  int32 is the layout the
// paper describes first (tile_ptr: 31-bit row index, top bit = "tile holds an
// empty row"); int64 is its 64-bit variant (Section 3.3: 63-bit index plus the
// flag bit) for matrices of 2^31 nonzeros and more, which this GPU's memory holds
// many times over.  Row and column indices stay below 2^31 in both.
template <typename IT> struct Index;
template <> struct Index<int32_t> {
    using tp_t = uint32_t;
    static constexpr tp_t DIRTY = 0x80000000u, ROWMASK = 0x7fffffffu;
};
template <> struct Index<int64_t> {
    using tp_t = uint64_t;
    static constexpr tp_t DIRTY = 0x8000000000000000ull, ROWMASK = 0x7fffffffffffffffull;
};

inline int ceil_log2_host(int64_t v) {
    int b = 0;
    while ((int64_t(1) << b) < v) b++;
    return b;
}

constexpr int MEET_STRIDE_WORDS = 1;

struct Geom {
    int32_t sigma, T, W, ybits;
    int32_t p, pc;
};

inline Geom make_geom(int64_t nnz, int sigma) {
    Geom g;
    g.sigma = sigma;
    g.T = OMEGA * sigma;
    g.ybits = ceil_log2_host(int64_t(OMEGA) * sigma);
    g.W = (sigma + SBITS + g.ybits + 31) / 32;
    g.p = int32_t((nnz + g.T - 1) / g.T);
    g.pc = int32_t(nnz / g.T);
    return g;
}

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }
// one slot of the cross-tile sums of an SpMV: carry, then (one-launch form) the meeting words and the counters
// (meeting words and counters: one per group of tiles, the incomplete tile being a group of its own)
inline size_t tile_groups(const Geom& g, int waves) { return (size_t(g.pc) + waves - 1) / waves + 1; }
inline size_t slot_off_meet(const Geom& g) { return align256((size_t(g.p) + 1) * 8); }
inline size_t slot_off_arrived(const Geom& g, int waves) { return slot_off_meet(g) + align256(tile_groups(g, waves) * 8 * MEET_STRIDE_WORDS); }
inline size_t slot_bytes_one(const Geom& g, int waves) { return slot_off_arrived(g, waves) + align256(tile_groups(g, waves) * 4); }

// ----------------------------------------------------------------------------
// device helpers
// ----------------------------------------------------------------------------

// Number of entries of a[0..len) that are <= key ("upper bound").  This is the
// binary search of Algorithms 4 and 7: with empty rows several row_ptr entries
// are equal, and count-1 is then the non-empty row that owns nonzero `key`.
template <typename IT>
__device__ __forceinline__ int count_le(const IT* __restrict__ a, int len, int64_t key) {
    int lo = 0, hi = len;
    while (lo < hi) {
        int mid = lo + ((hi - lo) >> 1);
        if (int64_t(a[mid]) <= key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (OMEGA - 1); }

// Group of tiles (= workgroup of the tile kernel) that holds a nonzero: tile t of
// the complete tiles belongs to group t / waves, the incomplete tile is a group
// of its own behind them.
__device__ __forceinline__ int tile_group_of(int64_t entry, int T, int pc, int waves) {
    const int64_t t = entry / T;
    return t < int64_t(pc) ? int(t / waves) : (pc + waves - 1) / waves;
}
// "nobody has been here yet" in the meeting words of the one-launch SpMV (a NaN pattern no sum is stored as)
constexpr uint64_t MEET_EMPTY = 0xfff8c5125eaf0001ull;
// Distance, in 8-byte words, between the meeting words of neighbouring groups.
constexpr int MEET_STRIDE = MEET_STRIDE_WORDS;
__device__ __forceinline__ uint64_t* meet_at(uint64_t* meet, uint32_t g) { return meet + size_t(g) * MEET_STRIDE; }

// Sets a bit of the status word.  Hundreds of thousands of threads may want the
// same bit, and atomics on one address are served one after the other, so look
// first: after the first few, everybody finds it set.
__device__ __forceinline__ void raise_status(uint32_t* status, uint32_t bit) {
    if ((__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit) != bit) atomicOr(status, bit);
}

// Native global floating-point atomic add (fp64 or fp32), no return value.
template <typename VT>
__device__ __forceinline__ void atomic_add_fp(VT* addr, VT v) {
    __hip_atomic_fetch_add(addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Which tiles a workgroup takes.  Workgroups are dealt round-robin to the 8
// XCDs (workgroup w runs on XCD w mod 8), each with its own L2.  Three orders,
// chosen per matrix at launch (measured on stencil, power-law and banded random
// matrices from 3 M to 2.2 G nonzeros; the crossovers sat at the same places in
// all families):
//  * contiguous (chunk = 0): XCD k gets the k-th eighth of the tiles, so
//    neighbouring tiles, which gather neighbouring parts of x, share one L2.
//    Wins by 1-14 % while x is at most about 9 MiB, i.e. while the part of x one
//    XCD works on stays in its L2 next to the streamed tiles; beyond that it
//    loses 2-9 %: eight distant streams cost more than a shared sweep.
//  * plain (chunk = 1): workgroup w takes tiles 4w..4w+3; all XCDs sweep the same
//    region, and expensive stretches (a long row's tiles) are spread evenly.
//    But neighbouring tiles then sit on different XCDs, and when a tile holds
//    fewer rows than a cache line of y (16), every line of y is written piecewise
//    from several L2s: 8 % slower on a matrix with 350 nonzeros per row.
//  * chunked (chunk = 16): runs of 16 workgroups go to the XCDs in turn; as good
//    as plain on regular matrices and without its piecewise writes.  Also the
//    choice when x is so small (below 2.5 MB) that it stays in every L2 anyway:
//    1-4 % faster than contiguous there.
constexpr size_t XCD_CONTIGUOUS_MIN_X_BYTES = 2500u * 1000u;
constexpr size_t XCD_CONTIGUOUS_MAX_X_BYTES = 10u * 1000u * 1000u;
constexpr uint32_t XCD_CHUNK = 16;
constexpr int Y_LINE_ROWS = 16;            // 128-byte line / 8-byte value

__device__ __forceinline__ uint32_t xcd_order(uint32_t w, uint32_t nb, uint32_t chunk) {
    const uint32_t xcd = w % NUM_XCD, k = w / NUM_XCD;
    if (chunk == 0) {
        const uint32_t per = nb / NUM_XCD, rem = nb % NUM_XCD;
        return xcd * per + (xcd < rem ? xcd : rem) + k;
    }
    // a permutation of [0, full); the ragged rest keeps the plain order
    const uint32_t full = (nb / (NUM_XCD * chunk)) * (NUM_XCD * chunk);
    if (w >= full) return w;
    return (k / chunk) * (NUM_XCD * chunk) + xcd * chunk + (k % chunk);
}

// Place in the list of order_place that workgroup w of nb takes (nb and the first
// `ends` places, in workgroups, are multiples of NUM_XCD).  The list's first part
// is dealt out evenly among its second: the one waits for lines from memory, the
// other for the L2.  First part: plain; second part: XCD k takes the k-th eighth.
__device__ __forceinline__ uint32_t order_place(uint32_t w, uint32_t nb, uint32_t ends) {
    const uint32_t xcd = w % NUM_XCD, o = w / NUM_XCD, no = nb / NUM_XCD, ne = ends / NUM_XCD;
    const uint32_t before = uint32_t(uint64_t(o) * ne / no), after = uint32_t(uint64_t(o + 1) * ne / no);
    if (after > before) return before * NUM_XCD + xcd;
    return ends + xcd * (no - ne) + (o - before);
}

// ----------------------------------------------------------------------------
// Conversion step 2a: tile_ptr (Algorithm 4, first loop), and everything else that
// only row_ptr is needed for.
// The first `nb_tiles` workgroups (at most PREP_TILE_WG): one thread per tile
// boundary searches its row, notes how many entries of the tile's first row lie
// before it (tile_head, an auxiliary array of the SpMV) and, where the one-launch
// SpMV may run, which groups of tiles that row touches.  The others (at most
// PREP_ROW_WG) check row_ptr and look for empty rows in the incomplete tile.  All
// of them put the words of the one-launch SpMV at rest.
// What they find goes into a word per workgroup, not to the status word: this
// launch clears that word, and many workgroups aiming at one word queue up.  The
// transposition that follows collects them.
// Bound by the latency of the search, a chain of dependent loads: seven probes a
// round, 7 rounds at 1 M rows instead of 20 (count_le_wide).  With more tiles than
// SEARCH_WIDE_MAX_TILES the lines touched count and the binary search is better.
// (The flags of the rows' first nonzeros, one atomic OR per descriptor word into
// words cleared here, were a launch of their own between this one and the
// transposition, which now forms them where it forms the descriptors: 100^3 stencil
// 18.0 -> 8.8 us for what is left of the two launches, the transposition the same;
// 1.5 M rows of which a third are empty 47 -> 9.3 us, the transposition 133 -> 140.)
// ----------------------------------------------------------------------------
constexpr int PREP_TILE_WG = 256, PREP_ROW_WG = 1024, PREP_THREADS = 256, PREP_UNROLL = 4;
constexpr int SEARCH_WIDE_MAX_TILES = 1 << 17;
// the words of the row part
constexpr uint32_t ROWS_BAD = 1u, ROWS_FIRST_EMPTY = 2u, ROWS_TAIL_EMPTY = 4u;
// the words of the tile part: two bits, and above them how many tiles lie inside one row
constexpr uint32_t TILES_FAR = 1u, TILES_FAR_HEADS = 2u;
constexpr int TILES_INSIDE_SHIFT = 2;

// count_le with seven probes of eight parts a round, in flight together.
template <typename IT>
__device__ __forceinline__ int count_le_wide(const IT* __restrict__ a, int len, int64_t key) {
    int lo = 0;
    while (len > 8) {
        const int step = len >> 3;
        int found = 0;
#pragma unroll
        for (int i = 1; i < 8; i++) found += int(int64_t(a[lo + i * step - 1]) <= key);
        lo += found * step;
        len = found == 7 ? len - 7 * step : step - 1;
    }
    int found = 0;
#pragma unroll
    for (int i = 0; i < 8; i++)
        if (i < len) found += int(int64_t(a[lo + i]) <= key);
    return lo + found;
}

template <typename IT>
__global__ void __launch_bounds__(PREP_THREADS)
k_prepare(int m, IT nnz, const IT* __restrict__ row_ptr, int T, int p, int pc, int group, int record_reach, uint32_t nb_tiles,
          typename Index<IT>::tp_t* __restrict__ tile_ptr, uint32_t* __restrict__ tile_head, uint32_t* __restrict__ words,
          uint32_t* __restrict__ arrived, uint64_t* __restrict__ meet, size_t slot_bytes, int slots,
          uint2* __restrict__ span, uint32_t* __restrict__ status, uint32_t* __restrict__ order_total) {
    using tp_t = typename Index<IT>::tp_t;
    const size_t gid = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    // the one-launch SpMV finds its counters at zero and its meeting places empty, and leaves them so
    const size_t groups = (size_t(pc) + group - 1) / group + 1;         // one word of each per group of tiles
    for (int slot = 0; slot < slots; slot++) {
        const size_t stride = size_t(gridDim.x) * blockDim.x;
        for (size_t t = gid; t < groups; t += stride) arrived[slot * (slot_bytes / 4) + t] = 0u;
        for (size_t w = gid; w < groups * MEET_STRIDE; w += stride) meet[slot * (slot_bytes / 8) + w] = MEET_EMPTY;
    }
    if (gid <= WINDOW_ANSWER_AT + 2) status[gid] = 0u;        // and the plan of the tile order, the answers of sample_columns and sample_window
    if (order_total)
        for (size_t b = gid; b < 2 * ORDER_BUCKETS; b += size_t(gridDim.x) * blockDim.x) order_total[b] = 0u;
    uint32_t found = 0;
    if (blockIdx.x >= nb_tiles) {         // ---- rows
        const int64_t stride = int64_t(gridDim.x - nb_tiles) * PREP_THREADS;
        for (int64_t r0 = int64_t(blockIdx.x - nb_tiles) * PREP_THREADS + threadIdx.x; r0 < m; r0 += stride * PREP_UNROLL) {
            IT a[PREP_UNROLL], b[PREP_UNROLL];
#pragma unroll
            for (int q = 0; q < PREP_UNROLL; q++) {
                const int64_t r = r0 + q * stride < m ? r0 + q * stride : r0;
                a[q] = row_ptr[r];
                b[q] = row_ptr[r + 1];
            }
#pragma unroll
            for (int q = 0; q < PREP_UNROLL; q++) {
                const int64_t r = r0 + q * stride < m ? r0 + q * stride : r0;
                const bool bad = a[q] < 0 || b[q] < a[q] || b[q] > nnz || (r == 0 && a[q] != 0) || (r == m - 1 && b[q] != nnz);
                const bool empty = !bad && a[q] == b[q];
                found |= (bad ? ROWS_BAD : 0u) | (empty && r == 0 ? ROWS_FIRST_EMPTY : 0u) |
                         (empty && p > pc && int64_t(a[q]) > int64_t(pc) * T ? ROWS_TAIL_EMPTY : 0u);
            }
        }
        found = (__syncthreads_or(found & ROWS_BAD) ? ROWS_BAD : 0u) | (__syncthreads_or(found & ROWS_FIRST_EMPTY) ? ROWS_FIRST_EMPTY : 0u) |
                (__syncthreads_or(found & ROWS_TAIL_EMPTY) ? ROWS_TAIL_EMPTY : 0u);
        if (threadIdx.x == 0) words[PREP_TILE_WG + blockIdx.x - nb_tiles] = found;
        return;
    }
    // ---- tile boundaries
    __shared__ uint32_t inside_rows;
    if (threadIdx.x == 0) inside_rows = 0;
    __syncthreads();
    uint32_t inside = 0;
    const size_t stride = size_t(nb_tiles) * PREP_THREADS;
    for (size_t t = gid; t <= size_t(p); t += stride) {
        const int64_t bnd = int64_t(t) * T;
        const int row = (p <= SEARCH_WIDE_MAX_TILES ? count_le_wide(row_ptr, m + 1, bnd) : count_le(row_ptr, m + 1, bnd)) - 1;
        tile_ptr[t] = tp_t(row) & Index<IT>::ROWMASK;
        // how far into its first row the tile starts (0: the row starts with the
        // tile), saturated at 32 bits: what the SpMV needs to know about the
        // boundary, so that it does not have to look into row_ptr itself
        int64_t head = 0, rs = 0, re = 0;
        if (row >= 0 && row < m) {
            rs = int64_t(row_ptr[row]);
            re = int64_t(row_ptr[row + 1]);
            if (t < size_t(p)) head = bnd - rs;
        }
        tile_head[t] = uint32_t(head < 0 ? 0 : (head > int64_t(0xffffffffu) ? int64_t(0xffffffffu) : head));
        inside += uint32_t(t < size_t(pc) && re >= bnd + T);
        // for the one-launch SpMV: the groups of tiles that row touches (first, how many)
        if (slots > 0) {
            uint2 sp = {0u, 1u};
            if (re > rs && rs >= 0) {
                const int g0 = tile_group_of(rs, T, pc, group), g1 = tile_group_of(re - 1, T, pc, group);
                if (g1 >= g0) sp = uint2{uint32_t(g0), uint32_t(g1 - g0 + 1)};
            }
            span[t] = sp;
        }
        // Can the tile kernel complete that row on its own?  The first tile of a
        // workgroup (and the workgroup of the incomplete tile) re-reads the head
        // from the previous tile's record: at most record_reach entries (LOOK_MAX,
        // or LOOK in a large matrix, see LOOK_FAR_MAX_NNZ).  The other
        // tiles are handed their neighbour's last segment, which is the whole
        // head if the row began inside (or with) that neighbour: at most T entries.
        const bool from_record = (t % size_t(group)) == 0 || t >= size_t(pc);
        if (head > (from_record ? int64_t(record_reach) : int64_t(T))) found |= TILES_FAR;
        if (from_record && head > int64_t(LOOK)) found |= TILES_FAR_HEADS;
    }
    if (inside) atomicAdd(&inside_rows, inside);
    found = (__syncthreads_or(found & TILES_FAR) ? TILES_FAR : 0u) | (__syncthreads_or(found & TILES_FAR_HEADS) ? TILES_FAR_HEADS : 0u);
    if (threadIdx.x == 0) words[blockIdx.x] = found | (inside_rows << TILES_INSIDE_SHIFT);
}

// What the workgroups of k_prepare found goes to the status word (and the mark of
// the incomplete tile, which has no wavefront of its own, to tile_ptr[pc]).  One
// workgroup; every thread of it must call this.
template <typename IT>
__device__ __forceinline__ void collect_words(const uint32_t* __restrict__ words, int nb_tiles, int nb_rows, int pc,
                                              typename Index<IT>::tp_t* tile_ptr, uint32_t* status) {
    __shared__ uint32_t inside_rows;
    if (threadIdx.x == 0) inside_rows = 0;
    __syncthreads();
    uint32_t tiles = 0, rows = 0, inside = 0;
    for (int w = threadIdx.x; w < nb_tiles; w += blockDim.x) {
        const uint32_t word = words[w];
        tiles |= word;
        inside += word >> TILES_INSIDE_SHIFT;
    }
    for (int w = threadIdx.x; w < nb_rows; w += blockDim.x) rows |= words[PREP_TILE_WG + w];
    if (inside) atomicAdd(&inside_rows, inside);
    const int far = __syncthreads_or(tiles & TILES_FAR), far_heads = __syncthreads_or(tiles & TILES_FAR_HEADS);
    const int bad = __syncthreads_or(rows & ROWS_BAD), first = __syncthreads_or(rows & ROWS_FIRST_EMPTY);
    const int tail = __syncthreads_or(rows & ROWS_TAIL_EMPTY);
    if (threadIdx.x == 0) {
        const bool long_rows = pc > 0 && inside_rows >= uint32_t(pc / ORDER_MIN_SHARE + 1);
        const uint32_t raise = (far ? STATUS_NEEDS_CARRY : 0u) | (far_heads ? STATUS_FAR_HEADS : 0u) | (long_rows ? STATUS_LONG_ROWS : 0u) |
                               (bad ? CSR5_STATUS_BAD_ROW_PTR : 0u) | (first ? CSR5_STATUS_HAS_EMPTY_ROWS : 0u);
        if (raise) atomicOr(status, raise);
        if (tail) tile_ptr[pc] |= Index<IT>::DIRTY;
    }
}

// ----------------------------------------------------------------------------
// empty_offset layout: exclusive prefix sum of the per-tile segment counts
// (non-zero only for tiles with an empty row); the array has p_c + 1 entries.
// Nothing to scan when no tile is marked (status bit from the descriptor step of k_transpose).  Up to
// SCAN_SINGLE tiles one workgroup walks the array chunk by chunk; beyond that
// every chunk gets a workgroup (local scan + chunk total) and a second launch
// adds to every chunk the sum of the totals before it.
// ----------------------------------------------------------------------------
constexpr uint32_t CARRY_SLOTS = 4;            // carry arrays per handle = SpMVs of one handle that may overlap
constexpr int SCAN_THREADS = 1024, SCAN_ITEMS = 8, SCAN_CHUNK = SCAN_THREADS * SCAN_ITEMS;
constexpr int SCAN_SINGLE = 4 * SCAN_CHUNK;

// Exclusive scan of a[base .. base + SCAN_CHUNK) (entries at or beyond len count
// as 0) by one workgroup of SCAN_THREADS threads, in place, plus `carry`;
// returns the chunk's total to every thread.
template <typename IT>
__device__ IT scan_chunk(IT* __restrict__ a, int64_t base, int64_t len, IT carry) {
    __shared__ IT wave_sum[SCAN_THREADS / OMEGA];
    __shared__ IT chunk_total;
    const int lane = lane_id(), wave = threadIdx.x / OMEGA;
    const int64_t idx0 = base + int64_t(threadIdx.x) * SCAN_ITEMS;
    IT local[SCAN_ITEMS];
    IT s = 0;
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS; q++) {
        IT v = (idx0 + q < len) ? a[idx0 + q] : IT(0);
        local[q] = s;
        s += v;
    }
    IT incl = s;
#pragma unroll
    for (int d = 1; d < OMEGA; d <<= 1) {
        IT up = __shfl_up(incl, d, OMEGA);
        if (lane >= d) incl += up;
    }
    if (lane == OMEGA - 1) wave_sum[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        IT v = (lane < SCAN_THREADS / OMEGA) ? wave_sum[lane] : IT(0);
        IT ws = v;
#pragma unroll
        for (int d = 1; d < SCAN_THREADS / OMEGA; d <<= 1) {
            IT up = __shfl_up(ws, d, OMEGA);
            if (lane >= d) ws += up;
        }
        if (lane < SCAN_THREADS / OMEGA) wave_sum[lane] = ws - v;  // exclusive
        if (lane == SCAN_THREADS / OMEGA - 1) chunk_total = ws;
    }
    __syncthreads();
    const IT excl = carry + wave_sum[wave] + incl - s;
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS; q++)
        if (idx0 + q < len) a[idx0 + q] = excl + local[q];
    const IT total = chunk_total;
    __syncthreads();                                    // the shared words are reused by the next call
    return total;
}

// The last words of the scan: the total number of entries, and the status bits
// for a marked incomplete tile (it has no descriptor, so the descriptor step never sees
// it).  One thread.
template <typename IT>
__device__ __forceinline__ void scan_epilogue(int pc, int p, IT total, IT* __restrict__ eop,
                                              const typename Index<IT>::tp_t* __restrict__ tile_ptr,
                                              uint32_t* __restrict__ status) {
    eop[pc] = total;
    if (p > pc && (tile_ptr[pc] & Index<IT>::DIRTY))
        atomicOr(status, CSR5_STATUS_HAS_DIRTY | CSR5_STATUS_HAS_EMPTY_ROWS);
}

// ----------------------------------------------------------------------------
// Order in which the tile kernel takes the tiles of a matrix with long rows and a
// large x.  A tile inside one row gathers from a narrow stretch of x (the row's
// columns ascend), but the tiles in flight at a time, neighbours in the matrix,
// belong to all parts of a few rows: together they touch all of x, and an x larger
// than an XCD's L2 is fetched again for every few rows, a 128-byte line per
// gather.  Taken by first column instead, with the k-th eighth of the list going
// to XCD k, the tiles in flight on an XCD share about (1/64 of x + a tile's
// stretch), which its L2 holds: 1500 rows of 20 000 entries among 1.5 M short
// ones, x of 32 MB, 600 -> 227 us (10 -> 26 % of the HBM peak on the bytes the
// product cannot do without); x of 8 MB, 1000 such rows, 233 -> 134 us; x of
// 4.8 MB, 200 of them, 40.3 -> 35.2 us.
// Where the line lies (measured with such matrices and with power-law ones):
// ORDER_MIN_X_BYTES is the L2 of one XCD, which holds any smaller x whole;
// ORDER_MIN_SHARE: with half of the tiles inside one row and more the order wins,
// with a third (power-law, whose long rows all gather from the same low columns)
// it loses 15-20 %; below ORDER_MIN_TILES the chip takes all tiles at once.
// ORDER_MAX_CROWD of ORDER_CROWD_PARTS: not where more of the tiles inside one row
// begin in an eighth of the columns (in the 128 fullest of the 1024 buckets). There
// the rows' dense stretches are short, in every L2 anyhow, and what gathers from far
// apart ends up on one or two XCDs.  Rows whose columns thin out like a power law,
// by number -> by column: a share of 0.83 252 -> 272 us, 0.87 170 -> 191 (single
// precision 111 -> 158), 0.99 70 -> 91; but 0.74 240 -> 147, 0.70 31.3 -> 31.9 and
// 315 -> 199, 0.57 375 -> 189, 0.23 (uniform) 490 -> 189 (given up: 0.82 193 -> 150,
// 0.76 281 -> 270).  The same rows with their columns in random order, a share of
// 0.2: 347 -> 196, 460 -> 302, 123 -> 108, single precision 227 -> 163.
// The list: the tiles that hold row ends, in (nearly) their own order, then, from
// a multiple of `align` on, the tiles inside one row by first column: a counting
// sort over 2 * ORDER_BUCKETS keys, a slice of the tiles per workgroup.  The slices
// are counted next to the scan of empty_offset_ptr (order_count; the bucket's total
// so far is the slice's place in it) and dealt out in the launch that follows
// (order_place, which first adds the totals up); within a bucket any order will do.
// Blocking conversions of 33 000 and 488 000 tiles take 185 and 2242 us (216 and 3066
// with one workgroup for all tiles, 178 and 2220 before there was an order): 0.2 us
// of the scan's launch, 3 to 4.5 of the next.
// plan[0]: where the second part begins, plan[1]: entries in all (those between the
// parts hold no tile: 0xffffffff); both 0: no order.  first_col: from the
// transposition.
// ----------------------------------------------------------------------------
constexpr size_t ORDER_MIN_X_BYTES = 4u << 20;
constexpr int ORDER_MIN_TILES = 2048;
constexpr int ORDER_CROWD_PARTS = 4, ORDER_MAX_CROWD = 3, ORDER_CROWDED = ORDER_BUCKETS / 8;
constexpr int ORDER_SLICE = 1024, ORDER_MAX_SLICES = 256;
constexpr int PLACE_THREADS = 256, PLACE_BUCKETS = 2 * ORDER_BUCKETS / PLACE_THREADS;

struct OrderJob {
    int32_t n, align;
    int32_t slices;                  // 0: nothing to do
    const int32_t* first_col;
    uint32_t *total, *base;          // per bucket; per slice and bucket
    uint32_t *order, *plan;
};

// Whether this matrix gets the order, as far as its row lengths say (plan was cleared with the status word).
__device__ __forceinline__ bool order_wanted(const uint32_t* __restrict__ status) {
    constexpr uint32_t both = STATUS_LONG_ROWS | STATUS_NEEDS_CARRY;
    return (*status & both) == both;
}

// f(tile, bucket) for the tiles of slice k, by all threads of the workgroup.
template <typename IT, typename F>
__device__ __forceinline__ void order_slice(int pc, const OrderJob& job, int k, const typename Index<IT>::tp_t* __restrict__ tile_ptr, F f) {
    constexpr auto ROWMASK = Index<IT>::ROWMASK;
    const float per_col = float(ORDER_BUCKETS) / float(job.n), per_tile = float(ORDER_BUCKETS) / float(pc);
    const int first = int(int64_t(pc) * k / job.slices), end = int(int64_t(pc) * (k + 1) / job.slices);
#pragma unroll 4
    for (int t = first + int(threadIdx.x); t < end; t += int(blockDim.x)) {
        const int32_t c = job.first_col[t];
        const bool inside = (tile_ptr[t] & ROWMASK) == (tile_ptr[t + 1] & ROWMASK);
        const int b = int(inside ? float(c < 0 ? 0 : c) * per_col : float(t) * per_tile);      // (a column out of range: rejected input)
        f(t, (inside ? ORDER_BUCKETS : 0) + (b < ORDER_BUCKETS ? b : ORDER_BUCKETS - 1));
    }
}

template <typename IT>
__device__ void order_count(int pc, const OrderJob& job, int k, const typename Index<IT>::tp_t* __restrict__ tile_ptr,
                            const uint32_t* __restrict__ status) {
    if (!order_wanted(status)) return;
    __shared__ uint32_t count[2 * ORDER_BUCKETS];
    for (int b = threadIdx.x; b < 2 * ORDER_BUCKETS; b += blockDim.x) count[b] = 0;
    __syncthreads();
    order_slice<IT>(pc, job, k, tile_ptr, [&](int, int b) { atomicAdd(&count[b], 1u); });
    __syncthreads();
    uint32_t* const base = job.base + size_t(k) * (2 * ORDER_BUCKETS);
    for (int b = threadIdx.x; b < 2 * ORDER_BUCKETS; b += blockDim.x)
        base[b] = count[b] ? atomicAdd(&job.total[b], count[b]) : 0u;
}

// Whether the fullest eighth of the buckets of tiles inside one row holds more than
// ORDER_MAX_CROWD of ORDER_CROWD_PARTS of them all (`inside`).  One wavefront, without
// barriers: its bisection is the longest chain of the workgroup that does it.
__device__ bool crowded(const uint32_t* __restrict__ total, uint32_t inside) {
    constexpr int PER_LANE = ORDER_BUCKETS / OMEGA;
    const int lane = lane_id();
    uint32_t mine[PER_LANE];
#pragma unroll
    for (int q = 0; q < PER_LANE; q++) mine[q] = total[ORDER_BUCKETS + q * OMEGA + lane];
    const auto fuller = [&](uint32_t c) {
        int n = 0;
#pragma unroll
        for (int q = 0; q < PER_LANE; q++) n += __popcll(__ballot(mine[q] > c));
        return n;
    };
    uint32_t lo = 0, hi = inside / ORDER_CROWDED;      // the smallest count that at most ORDER_CROWDED buckets exceed
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (fuller(mid) > ORDER_CROWDED) lo = mid + 1; else hi = mid;
    }
    uint32_t fullest = 0;
#pragma unroll
    for (int q = 0; q < PER_LANE; q++) fullest += mine[q] > lo ? mine[q] : 0u;
#pragma unroll
    for (int d = OMEGA / 2; d >= 1; d >>= 1) fullest += __shfl_xor(fullest, d, OMEGA);
    fullest += uint32_t(ORDER_CROWDED - fuller(lo)) * lo;
    return uint64_t(fullest) * ORDER_CROWD_PARTS > uint64_t(inside) * ORDER_MAX_CROWD;
}

template <typename IT>
__device__ void order_place(int pc, const OrderJob& job, int k, const typename Index<IT>::tp_t* __restrict__ tile_ptr,
                            const uint32_t* __restrict__ status) {
    if (!order_wanted(status)) return;
    __shared__ uint32_t at[2 * ORDER_BUCKETS];
    __shared__ uint32_t wave_total[PLACE_THREADS / OMEGA];
    // exclusive scan of the buckets' totals, PLACE_BUCKETS neighbours per thread
    const int lane = lane_id(), wave = threadIdx.x / OMEGA;
    uint32_t mine[PLACE_BUCKETS], sum = 0;
#pragma unroll
    for (int q = 0; q < PLACE_BUCKETS; q++) {
        mine[q] = job.total[threadIdx.x * PLACE_BUCKETS + q];
        sum += mine[q];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < OMEGA; d <<= 1) {
        const uint32_t up = __shfl_up(incl, d, OMEGA);
        if (lane >= d) incl += up;
    }
    if (lane == OMEGA - 1) wave_total[wave] = incl;
    __syncthreads();
    uint32_t before = incl - sum, ends = 0;              // ends: tiles that hold row ends, the first half of the buckets
    for (int w = 0; w < PLACE_THREADS / OMEGA; w++) {
        if (w < wave) before += wave_total[w];
        if (w < PLACE_THREADS / OMEGA / 2) ends += wave_total[w];
    }
    const uint32_t align = uint32_t(job.align), second = (ends + align - 1) / align * align;
    if (threadIdx.x >= PLACE_THREADS / 2) before += second - ends;
    const uint32_t* const base = job.base + size_t(k) * (2 * ORDER_BUCKETS);
#pragma unroll
    for (int q = 0; q < PLACE_BUCKETS; q++) {
        const int b = threadIdx.x * PLACE_BUCKETS + q;
        at[b] = before + base[b];
        before += mine[q];
    }
    __syncthreads();
    order_slice<IT>(pc, job, k, tile_ptr, [&](int t, int b) { job.order[atomicAdd(&at[b], 1u)] = uint32_t(t); });
    if (k == 0) {
        for (uint32_t q = ends + threadIdx.x; q < second; q += PLACE_THREADS) job.order[q] = 0xffffffffu;
        if (wave == 0 && !crowded(job.total, uint32_t(pc) - ends) && lane == 0) {
            job.plan[0] = second;
            job.plan[1] = uint32_t(pc) + second - ends;
        }
    }
}

// How many of SAMPLES pairs of neighbouring entries lie in different lines of x, 0 if the
// columns are none for k_spmv_staged: what the host needs beside sizes to decide for it
// (staged_min_entries).  A sample of SAMPLE_TILES tiles (in CSR5 order already), two neighbours of
// each of a tile's 64 columns, by one workgroup of SCAN_THREADS threads beside the scan.
// Different lines: each entry is a line from the L2 (random columns 0.95-1.0; stencils 0.36,
// power-law rows 0.35, rows with a sixth of all columns 0.37, dense 0).  Not for it are
//  * fewer than half in different lines (rows of 2000 out of 12 000 columns, 20 M entries 58.5 -> 65.7).
//  * tiles whose entries do not spread over half of x or SAMPLE_WIDE_BYTES: the entries that
//    a CU has at a time share what its L1 holds, and every part of x would be read for
//    nothing (random columns, and bands of 160 KB: all tiles spread; stencils none,
//    power-law rows one in six; a band with a few entries elsewhere does, see window_rather).
//  * columns that all together fall on far fewer lines than random ones would (1.0; normally
//    distributed 0.7): a few columns have most entries, and the L1 holds those (power-law
//    columns in random order, x of 480 KB: 0.35 and 14.1 us, here 16.8).
constexpr int SAMPLE_TILES = 64, SAMPLES = SAMPLE_TILES * OMEGA, SAMPLE_MAX_LINES = 32768;
constexpr int SAMPLE_WIDE_BYTES = 128 << 10, SAMPLE_WIDE_PERCENT = 90, SAMPLE_LINES_PERCENT = 60, SAMPLE_MIN_PERCENT = 50;

struct SampleJob {
    const int32_t* col_idx;          // NULL: nothing to do
    int32_t n, sigma, value_bytes;   // at most SAMPLE_MAX_LINES lines of x
    uint32_t* changes;               // the answer; cleared with the status word
};

__device__ void sample_columns(int pc, const SampleJob& job) {
    __shared__ uint32_t seen[SAMPLE_MAX_LINES / 4];       // a byte per line of x, which many may set at a time
    __shared__ uint32_t changes, wide, lines;
    const int lane = lane_id(), wave = threadIdx.x / OMEGA;
    const uint32_t per_line = 128u / uint32_t(job.value_bytes), last = uint32_t(job.n - 1), words = last / per_line / 4 + 1;
    const uint32_t spread = last / 2 < SAMPLE_WIDE_BYTES / uint32_t(job.value_bytes) ? last / 2 : SAMPLE_WIDE_BYTES / uint32_t(job.value_bytes);
    // everything is asked for at once: one round trip
    constexpr int PER_WAVE = SAMPLE_TILES / (SCAN_THREADS / OMEGA);
    uint32_t at[PER_WAVE], next[PER_WAVE];
#pragma unroll
    for (int u = 0; u < PER_WAVE; u++) {
        const int q = wave * PER_WAVE + u;
        // rows of one length repeat in step with the columns: another place in them for every 16 lanes, and from tile to tile
        // (every lane its own would be 16 lines a load, 9 us in all)
        const int j = (q + lane / 16 * job.sigma / 4) % (job.sigma - 1);
        const int32_t* const pair = job.col_idx + int64_t(pc) * q / SAMPLE_TILES * (job.sigma * OMEGA) + j * OMEGA + lane;
        at[u] = uint32_t(pair[0]);
        next[u] = uint32_t(pair[OMEGA]);
    }
    for (uint32_t w = threadIdx.x; w < words; w += SCAN_THREADS) seen[w] = 0;
    if (threadIdx.x == 0) changes = wide = lines = 0;
    __syncthreads();
    uint32_t my_changes = 0, my_wide = 0;                 // of the wavefront's tiles
#pragma unroll
    for (int u = 0; u < PER_WAVE; u++) {
        const uint32_t a = at[u] < last ? at[u] : last, b = next[u] < last ? next[u] : last;      // (out of range: rejected input)
        const uint32_t line = a / per_line, next_line = b / per_line;
        reinterpret_cast<uint8_t*>(seen)[line] = 1;
        reinterpret_cast<uint8_t*>(seen)[next_line] = 1;
        my_changes += uint32_t(__popcll(__ballot(line != next_line)));
        // `spread` columns between the outermost two: bounded from below by what lies furthest on either side of lane 0's
        const uint32_t from = __builtin_amdgcn_readfirstlane(a), up = a > from ? a - from : 0u, down = a < from ? from - a : 0u;
        my_wide += __ballot(up > spread || down > spread) != 0 || (__ballot(up > spread / 2) != 0 && __ballot(down > spread / 2) != 0) ? 1u : 0u;
    }
    if (lane == 0) {
        atomicAdd(&changes, my_changes);
        atomicAdd(&wide, my_wide);
    }
    __syncthreads();
    uint32_t mine = 0;
    for (uint32_t w = threadIdx.x; w < words; w += SCAN_THREADS) mine += uint32_t(__popc(seen[w]));
    if (mine) atomicAdd(&lines, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        const float all = float(last / per_line + 1), random = all * (1.0f - expf(-float(2 * SAMPLES) / all));
        if (changes * 100 >= uint32_t(SAMPLES * SAMPLE_MIN_PERCENT) && wide * 100 >= uint32_t(SAMPLE_TILES * SAMPLE_WIDE_PERCENT) &&
            float(lines) * 100.0f >= random * float(SAMPLE_LINES_PERCENT)) *job.changes = changes;
    }
}

// Orders LDS traffic between the lanes of ONE wavefront: LDS instructions of a
// wavefront execute in order, so what is needed is that the compiler keeps the
// stores before and the loads after this point.
__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The part of x that a workgroup of k_spmv_staged's window form keeps in LDS: around the place
// where the diagonal passes through its rows (r0 to r1), in bytes.  slope: columns per row.
// As much as lets two workgroups share a CU (in single precision 52 KB and three workgroups
// gain 3 % on rows with a window of 40 KB and lose 22 % on one of 80 KB).
constexpr int WINDOW_BYTES = 78 * 1024;
__device__ __forceinline__ int window_first(uint32_t r0, uint32_t r1, float slope, int x_bytes, int value_bytes) {
    const int first = int(float(r0 + (r1 - r0) / 2) * slope) * value_bytes - WINDOW_BYTES / 2;
    const int most = x_bytes > WINDOW_BYTES ? x_bytes - WINDOW_BYTES : 0;
    return (first < 0 ? 0 : (first < most ? first : most)) & ~127;
}

// A sample for the window form, taken by the transposition: two neighbours in each of the 64 columns of
// one tile in 1 << shift, 64 to 127 tiles in all (another place among its workgroup's tiles for each).
// What the host needs beside sizes (window_pays) is how many of the entries lie in their
// workgroup's window, and in how many lines of it, tile by tile; and for k_far_gather how many lie further
// from it than an L2 reaches, and in how many of the tiles these spread over more than that; and for
// gather_pairs how many of the second ones lie next to the first, and how many a line and more away.
constexpr int FAR_REACH_BYTES = 2 << 20;
struct WindowJob {
    uint32_t* answer;                // entries << 16 | lines, further entries << 16 | tiles, next << 16 | away; cleared with the status word.  NULL: nothing to do
    int32_t shift, tiles;            // tiles of a workgroup, a power of two
    float slope;
};
inline int window_shift(int pc) {                         // of at least SAMPLE_TILES tiles
    int shift = 0;
    while (pc >> (shift + 1) >= SAMPLE_TILES) shift++;
    return shift;
}
constexpr bool window_sampled(const WindowJob& job, int tile) {
    return (tile & ((1 << job.shift) - 1)) == ((tile >> job.shift) & (job.tiles - 1));
}
inline uint32_t window_samples(const WindowJob& job, int pc) {      // entries in it
    const int strides = pc >> job.shift, last = strides << job.shift | (strides & (job.tiles - 1));
    return uint32_t(strides + (last < pc ? 1 : 0)) * (2 * OMEGA);
}

// One tile of it, by its wavefront.  c: columns of a tile column in the order of CSR; who: LDS of the
// wavefront, a word per line of the window; r0, r1: the rows that the workgroup's tiles begin and end in.
// The few wavefronts that come here are among the last where the matrix has one round of them: nothing is
// waited for but two LDS accesses.  (Beside the scan, by one workgroup of its own, 2-6 us of every conversion of
// the size: 60^3 stencil there and back with one product 101.9 -> 98.8, power-law of 2 M rows 237.0 -> 234.0,
// mixed of 12.6 M entries 212.4 -> 206.7.)
constexpr int WINDOW_LINES = WINDOW_BYTES / 128;
template <int SIGMA>
__device__ void sample_window(const WindowJob& job, int tile, const int32_t* c, uint32_t* who, uint32_t r0, uint32_t r1, int n, int value_bytes) {
    const int lane = lane_id();
    // rows of one length repeat in step with the columns: another place in them for every 16 lanes, and from tile to tile
    const int at = ((tile >> job.shift) + lane / 16 * (SIGMA / 4)) % (SIGMA - 1);
    int32_t first = 0, second = 0;
#pragma unroll
    for (int j = 0; j < SIGMA - 1; j++) {
        if (j == at) {
            first = c[j];
            second = c[j + 1];
        }
    }
    const uint32_t window = uint32_t(window_first(r0, r1, job.slope, n * value_bytes, value_bytes));
    const uint32_t last = uint32_t(n - 1);                 // (out of range: rejected input)
    const uint32_t a = (uint32_t(first) < last ? uint32_t(first) : last) * uint32_t(value_bytes) - window;
    const uint32_t b = (uint32_t(second) < last ? uint32_t(second) : last) * uint32_t(value_bytes) - window;
    const bool a_near = a < uint32_t(WINDOW_BYTES), b_near = b < uint32_t(WINDOW_BYTES);
    wave_sync_lds();
    if (a_near) who[a / 128] = uint32_t(lane);            // of the entries in a line one stays
    if (b_near) who[b / 128] = uint32_t(OMEGA + lane);
    wave_sync_lds();
    const uint32_t near = uint32_t(__popcll(__ballot(a_near)) + __popcll(__ballot(b_near)));
    const uint32_t lines = uint32_t(__popcll(__ballot(a_near && who[a / 128] == uint32_t(lane))) +
                                    __popcll(__ballot(b_near && who[b / 128] == uint32_t(OMEGA + lane))));
    wave_sync_lds();
    const bool a_far = a + FAR_REACH_BYTES >= uint32_t(2 * FAR_REACH_BYTES), b_far = b + FAR_REACH_BYTES >= uint32_t(2 * FAR_REACH_BYTES);
    const uint64_t far_lanes = __ballot(a_far);
    const uint32_t far = uint32_t(__popcll(far_lanes) + __popcll(__ballot(b_far)));
    const uint32_t one = __builtin_amdgcn_readlane(a, far_lanes ? __builtin_ctzll(far_lanes) : 0);
    const bool spread = far_lanes && __ballot(a_far && a - one + 2 * FAR_REACH_BYTES >= uint32_t(4 * FAR_REACH_BYTES)) != 0;
    const uint32_t next = uint32_t(__popcll(__ballot(first + 1 == second)));
    const uint32_t away = uint32_t(__popcll(__ballot(uint32_t(second - first + 32) >= 64u)));
    if (lane == 0) {
        atomicAdd(job.answer, near << 16 | lines);
        atomicAdd(job.answer + 2, next << 16 | away);
        if (far) atomicAdd(job.answer + 1, far << 16 | (spread ? 1u : 0u));
    }
}

template <typename IT>
__global__ void __launch_bounds__(SCAN_THREADS)
k_scan_eop(int pc, int p, IT* __restrict__ eop, const typename Index<IT>::tp_t* __restrict__ tile_ptr,
           uint32_t* __restrict__ status, const OrderJob job, const SampleJob sample) {
    if (sample.col_idx && blockIdx.x == gridDim.x - 1) return sample_columns(pc, sample);
    if (blockIdx.x > 0) return order_count<IT>(pc, job, int(blockIdx.x) - 1, tile_ptr, status);
    IT total = 0;
    if (*status & STATUS_SCAN_NEEDED)
        for (int64_t base = 0; base < pc; base += SCAN_CHUNK) total += scan_chunk(eop, base, int64_t(pc), total);
    if (threadIdx.x == 0) scan_epilogue(pc, p, total, eop, tile_ptr, status);
}

// more than SCAN_SINGLE tiles, step 1: workgroup b scans chunk b on its own
template <typename IT>
__global__ void __launch_bounds__(SCAN_THREADS)
k_scan_chunks(int pc, IT* __restrict__ eop, IT* __restrict__ chunk_sum, const typename Index<IT>::tp_t* __restrict__ tile_ptr,
              const uint32_t* __restrict__ status, const OrderJob job) {
    const int chunk = int(blockIdx.x) - job.slices;
    if (chunk < 0) return order_count<IT>(pc, job, int(blockIdx.x), tile_ptr, status);
    if (!(*status & STATUS_SCAN_NEEDED)) return;
    const IT total = scan_chunk(eop, int64_t(chunk) * SCAN_CHUNK, int64_t(pc), IT(0));
    if (threadIdx.x == 0) chunk_sum[chunk] = total;
}

// step 2: workgroup b sums the totals of the chunks before its own (at most
// SCAN_CHUNK of them) and adds that to its chunk; the last one finishes the array
template <typename IT>
__global__ void __launch_bounds__(SCAN_THREADS)
k_scan_finish(int pc, int p, IT* __restrict__ eop, const IT* __restrict__ chunk_sum,
              const typename Index<IT>::tp_t* __restrict__ tile_ptr, uint32_t* __restrict__ status) {
    const int b = blockIdx.x, last = int(gridDim.x) - 1;
    if (!(*status & STATUS_SCAN_NEEDED)) {
        if (b == last && threadIdx.x == 0) scan_epilogue(pc, p, IT(0), eop, tile_ptr, status);
        return;
    }
    __shared__ IT wave_part[SCAN_THREADS / OMEGA];
    __shared__ IT before;
    const int lane = lane_id(), wave = threadIdx.x / OMEGA;
    IT part = 0;
    for (int c = threadIdx.x; c < b; c += SCAN_THREADS) part += chunk_sum[c];
#pragma unroll
    for (int d = OMEGA / 2; d >= 1; d >>= 1) part += __shfl_down(part, d, OMEGA);
    if (lane == 0) wave_part[wave] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        IT sum = 0;
        for (int k = 0; k < SCAN_THREADS / OMEGA; k++) sum += wave_part[k];
        before = sum;
    }
    __syncthreads();
    const IT offset = before;
    if (offset != 0) {
        const int64_t i0 = int64_t(b) * SCAN_CHUNK + int64_t(threadIdx.x) * SCAN_ITEMS;
#pragma unroll
        for (int q = 0; q < SCAN_ITEMS; q++)
            if (i0 + q < pc) eop[i0 + q] += offset;
    }
    if (b == last && threadIdx.x == 0) scan_epilogue(pc, p, IT(offset + chunk_sum[b]), eop, tile_ptr, status);
}

// ----------------------------------------------------------------------------
// empty_offset values (Algorithm 7), one thread per matrix row instead of one
// sequential walk per tile: a non-empty row whose first nonzero lies in a
// marked complete tile is segment number  y_offset[column] + (flags below it in
// the column)  of that tile, and its entry is  row - tile_ptr.  Segment 0 of a
// marked tile may start with the forced flag (a row continued from the previous
// tile, which is then the tile's first row): its entry is 0 and is written by
// the extra p_c threads at the end of the grid.  The first workgroups lay out the
// tile order where there is one.
// ----------------------------------------------------------------------------
template <typename IT>
__global__ void __launch_bounds__(PLACE_THREADS)
k_empty_offset(int m, const IT* __restrict__ row_ptr, int sigma, int T, int W, int pc,
               const typename Index<IT>::tp_t* __restrict__ tile_ptr, const uint32_t* __restrict__ desc,
               const IT* __restrict__ eop, int32_t* __restrict__ eo,
               const uint32_t* __restrict__ status, const OrderJob job) {
    using tp_t = typename Index<IT>::tp_t;
    constexpr tp_t DIRTY = Index<IT>::DIRTY, ROWMASK = Index<IT>::ROWMASK;
    if (int(blockIdx.x) < job.slices) return order_place<IT>(pc, job, int(blockIdx.x), tile_ptr, status);
    uint32_t st = *status;
    if (!(st & CSR5_STATUS_HAS_DIRTY) || (st & BAD_BITS)) return;
    int64_t g = int64_t(int(blockIdx.x) - job.slices) * blockDim.x + threadIdx.x;
    if (g >= int64_t(m)) {
        int64_t t = g - m;
        if (t < pc && (tile_ptr[t] & DIRTY)) eo[eop[t]] = 0;
        return;
    }
    int r = int(g);
    IT a = row_ptr[r], b = row_ptr[r + 1];
    if (a == b || int64_t(a) >= int64_t(pc) * T) return;
    int tile = int(a / T);
    tp_t tp = tile_ptr[tile];
    if (!(tp & DIRTY)) return;
    int w = int(a - IT(tile) * T);
    int i = w / sigma;
    int j = w - i * sigma;
    size_t base = size_t(tile) * W * OMEGA + i;
    uint64_t lo = desc[base];
    if (W > 1) lo |= uint64_t(desc[base + OMEGA]) << 32;
    uint64_t hi = (W > 2) ? desc[base + 2 * OMEGA] : 0u;
    int ysh = sigma + SBITS;
    uint64_t yo = lo >> ysh;
    if (W > 2) yo |= hi << (64 - ysh);
    // y_offset occupies every bit above seg_offset (unused high bits are zero)
    uint64_t below = lo & ((uint64_t(1) << j) - 1);
    int seg = int(yo) + __popcll(below);
    eo[eop[tile] + seg] = int32_t(int64_t(r) - int64_t(tp & ROWMASK));
}

// ----------------------------------------------------------------------------
// Conversion step 4 (Section 3.1): in-place transposition of col_idx and val
// inside every complete tile, one wavefront per tile.  The tile is read in CSR
// order (lane-contiguous), parked in LDS, and written back column-major
// (lane-contiguous again), so both HBM directions are fully coalesced and each
// lane happens to write exactly the addresses it read.  LDS rows are padded to
// an odd pitch to avoid bank conflicts on the strided LDS read.  BACK = the
// inverse permutation (CSR5 -> CSR, Section 3.6).  The last block also checks
// the column indices of the incomplete tile.  The forward pass also keeps, per
// workgroup, a copy of its last tile's last LOOK entries in CSR order when asked to,
// and forms the tile's descriptors (steps 2b, 3a, 3b) from the rows that begin in
// it: rows tile_ptr[t] + 1 .. tile_ptr[t + 1], 64 at a time, which are asked for
// behind the tile's entries.  A row with nonzeros sets the bit_flag of its first
// (Section 3.4; the scatter of Algorithm 3 step 1) in LDS, one without marks the
// tile (Algorithm 4, second loop: the rows of the inclusive range that begin after
// the tile does).  A range of more than FLAG_ROWS_MAX rows is nearly all empty
// rows, perhaps millions: there every lane searches for the row starts in its
// column instead.
// ----------------------------------------------------------------------------
template <int SIGMA>
struct TransposeShape {
    static constexpr int WAVES = tile_group_waves(SIGMA);
    static constexpr int PITCH = SIGMA | 1;
};

constexpr int FLAG_ROWS_MAX = 4096;
// Rows beyond a tile's first 64 are asked for this many wavefronts of them at a time:
// one at a time made the conversion of very short rows in tall tiles slower than one
// thread per row was (6 M rows of one entry, height 48: 82.6 us by a thread per row,
// 105.5, now 84.6; height 32 83.7, 92.0, 83.7; height 16 82.0, 74.5, 66.2; 8 M rows of 0
// to 2 entries, height 16: 616, 113.3, 102.5); 2 at a time leave 3-7 % of that, 8 add
// nothing.
constexpr int FLAG_ROWS_AHEAD = 4;

// A tile's arrays through buffer descriptors: the address of a load is the
// descriptor, a lane offset that all loads of the tile share and a constant, so the
// loads of a tile leave back to back with a quarter of the address arithmetic; any
// dword-aligned base will do for 16-byte loads (a col_idx that is a view at an odd
// offset took four loads each); nothing outside the tile is read.  Measured on the
// tile kernel (plain 64-bit addresses before): 100 000 rows of 100 random columns
// 65.4 -> 58.4 us, 30 000 rows of 201 38.2 -> 36.3, dense rows with the tile order
// 226 -> 200, 60 000 short rows 11.8 -> 10.9, 100^3 stencil 61.6 -> 61.0, rows of 700
// in single precision 95.4 -> 91.3 (one instantiation reads plainly, see k_spmv).
// Non-temporal, as a rule: without it the streams stay in the 256 MB memory-side cache
// as far as they fit, and one matrix multiplied again and again gains (90^3 stencil
// 43.2 -> 37.7 us, 100^3 with half of its tiles 61.0 -> 51.5), but matrices used in
// turn lose (44.8 -> 52.1, 61.2 -> 67.5): not known here which it is.
// KEEP: plain, where the next use of the entries is known to be near.  See keep_near.
constexpr int POLICY_STREAM = 2, POLICY_KEEP = 0;         // nt; none
template <typename P>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_buffer(P* first, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<typename std::remove_const<P>::type*>(first), 0, bytes, 0x00020000);
}
template <typename P, bool KEEP>
__device__ __forceinline__ P stream_from(__amdgpu_buffer_rsrc_t r, int offset) {
    constexpr int POLICY = KEEP ? POLICY_KEEP : POLICY_STREAM;
    if constexpr (sizeof(P) == 16) return __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b128(r, offset, 0, POLICY));
    else if constexpr (sizeof(P) == 8) return __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b64(r, offset, 0, POLICY));
    else if constexpr (sizeof(P) == 2) return __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b16(r, offset, 0, POLICY));
    else return __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b32(r, offset, 0, POLICY));
}
template <bool KEEP, typename P>
__device__ __forceinline__ P stream_from(const P* a) {
    if constexpr (KEEP) return *a;
    else return __builtin_nontemporal_load(a);
}
template <bool KEEP, typename P>
__device__ __forceinline__ void stream_to(P* a, P v) {
    if constexpr (KEEP) *a = v;
    else __builtin_nontemporal_store(v, a);
}

// What the forward pass needs of the conversion beside the entries themselves.
struct DescJob {
    int32_t m, wide;                    // wide: 64-bit row_ptr, tile_ptr and eop
    const void* row_ptr;
    void* tile_ptr;
    uint32_t* desc;
    void* eop;
    const uint32_t* words;              // of k_prepare
    int32_t nb_tiles, nb_rows;
    int32_t* first_col;                 // every tile's first column, for the tile order, or NULL
    WindowJob window;
};

template <int SIGMA, bool BACK, bool KEEP, typename VT>
__global__ void __launch_bounds__(TransposeShape<SIGMA>::WAVES * OMEGA)
k_transpose(int pc, int n, int64_t nnz, int32_t* __restrict__ col_idx, VT* __restrict__ val,
            uint32_t* __restrict__ status, int32_t* __restrict__ last_col, VT* __restrict__ last_val, int rec_bytes, const DescJob job) {
    constexpr int T = OMEGA * SIGMA;
    constexpr int YBITS = 32 - __builtin_clz(uint32_t(T - 1));        // ceil(log2(64*sigma))
    constexpr int W = (SIGMA + SBITS + YBITS + 31) / 32;
    constexpr int PITCH = TransposeShape<SIGMA>::PITCH;
    constexpr int WAVES = TransposeShape<SIGMA>::WAVES;
    __shared__ double lds[WAVES][OMEGA * PITCH];
    const int wave = threadIdx.x / OMEGA, lane = lane_id();
    const int tile = blockIdx.x * WAVES + wave;
    const bool active = tile < pc;                 // uniform per wavefront
    const size_t base = size_t(active ? tile : 0) * T;
    VT* buf = reinterpret_cast<VT*>(lds[wave]);
    int32_t* ibuf = reinterpret_cast<int32_t*>(lds[wave]);
    bool bad = false;
    // The copy of the tile's last entries is for the SpMV's look-behind, which a
    // matrix with a tile far into a row never uses (the words of k_prepare say so).
    // Only a group's last tile is looked at from outside its workgroup; the last
    // complete tile also by the workgroup of the incomplete one.
    bool keep_last = !BACK && last_val && last_col && active && (wave == WAVES - 1 || tile == pc - 1);
    bool keep_far = false;
    if constexpr (!BACK) {
        if (keep_last) {
            uint32_t found = 0;
            for (int w = lane; w < job.nb_tiles; w += OMEGA) found |= job.words[w];
            keep_last = !__any(found & TILES_FAR);
            keep_far = keep_last && rec_bytes == LAST_REC_BYTES && __any(found & TILES_FAR_HEADS);   // nobody reads the far part otherwise
        }
    }
    const size_t rec = size_t(tile) / WAVES;

    // ---- the row the tile starts in and the next tile's (either may carry its mark
    // by now: masked).  Clamped: a row_ptr that is not monotone gives anything.
    const auto row_at = [&](int r) -> int64_t {
        return job.wide ? static_cast<const int64_t*>(job.row_ptr)[r] : int64_t(static_cast<const int32_t*>(job.row_ptr)[r]);
    };
    const auto tile_row = [&](int t) -> int {
        const uint64_t v = job.wide ? static_cast<const uint64_t*>(job.tile_ptr)[t] & Index<int64_t>::ROWMASK
                                    : uint64_t(static_cast<const uint32_t*>(job.tile_ptr)[t] & Index<int32_t>::ROWMASK);
        return v < uint64_t(job.m) ? int(v) : job.m;
    };
    int row0 = 0, row1 = 0;              // rows row0 + 1 .. row1 begin in the tile, or are empty rows of its range
    if constexpr (!BACK) {
        if (active) {
            row0 = tile_row(tile);
            row1 = tile_row(tile + 1);
        }
    }
    bool sampled = false;                // uniform per wavefront
    int group0 = 0, group1 = 0;          // rows, see sample_window
    if constexpr (!BACK && rule_sigma(SIGMA)) {
        sampled = active && job.window.answer && window_sampled(job.window, tile);
        if (sampled) {
            const int t0 = tile & -job.window.tiles;
            group0 = tile_row(t0);
            group1 = tile_row(t0 + job.window.tiles < pc ? t0 + job.window.tiles : pc);
        }
    }

    // ---- val: HBM -> registers -> LDS -> registers -> HBM
    VT v[SIGMA];
    int64_t begins = 0, ends = 0;        // of row row0 + 1 + lane
    if (active) {
#pragma unroll
        for (int k = 0; k < SIGMA; k++) v[k] = stream_from<KEEP>(&val[base + k * OMEGA + lane]);
        if constexpr (!BACK) {
            if (row1 >= job.m) row1 = job.m - 1;
            if (lane < row1 - row0) {
                begins = row_at(row0 + 1 + lane);
                ends = row_at(row0 + 2 + lane);
            }
        }
        // the tile's last LOOK_MAX entries, still in CSR order (entry k*64 + lane of
        // the tile is v[k] here), for the SpMV's look-behind: near part, far part
        if constexpr (!BACK && look_sigma(SIGMA)) {
            if (keep_last) {
                VT* const near_v = last_val + rec * size_t(rec_bytes / int(sizeof(VT)));
                VT* const far_v = near_v + far_val_at<VT>();
                if (lane >= OMEGA - LOOK) near_v[lane - (OMEGA - LOOK)] = v[SIGMA - 1];
                if (keep_far) {
                    if (lane >= OMEGA - LOOK) far_v[lane - (OMEGA - LOOK)] = v[SIGMA - 3];
                    else far_v[LOOK_FAR - LOOK + lane] = v[SIGMA - 1];
                    far_v[LOOK + lane] = v[SIGMA - 2];
                }
            }
        }
        if (!BACK) {
#pragma unroll
            for (int k = 0; k < SIGMA; k++) {
                int e = k * OMEGA + lane;          // CSR offset inside the tile
                buf[(e / SIGMA) * PITCH + (e % SIGMA)] = v[k];
            }
        } else {
#pragma unroll
            for (int j = 0; j < SIGMA; j++) buf[lane * PITCH + j] = v[j];
        }
    }
    wave_sync_lds();    // every wavefront works in its own LDS slice
    if (active) {
        if (!BACK) {
#pragma unroll
            for (int j = 0; j < SIGMA; j++) v[j] = buf[lane * PITCH + j];
        } else {
#pragma unroll
            for (int k = 0; k < SIGMA; k++) {
                int e = k * OMEGA + lane;
                v[k] = buf[(e / SIGMA) * PITCH + (e % SIGMA)];
            }
        }
#pragma unroll
        for (int k = 0; k < SIGMA; k++) stream_to<KEEP>(&val[base + k * OMEGA + lane], v[k]);
    }
    wave_sync_lds();    // every wavefront works in its own LDS slice
    // ---- col_idx, same path through the same LDS buffer
    int32_t c[SIGMA];
    if (active) {
#pragma unroll
        for (int k = 0; k < SIGMA; k++) {
            c[k] = stream_from<KEEP>(&col_idx[base + k * OMEGA + lane]);
            bad |= (c[k] < 0) | (c[k] >= n);
        }
        if constexpr (!BACK && look_sigma(SIGMA)) {
            if (job.first_col && lane == 0) job.first_col[tile] = c[0];
            if (keep_last) {
                int32_t* const near_c = last_col + rec * size_t(rec_bytes / 4);
                int32_t* const far_c = near_c + FAR_COL_AT;
                if (lane >= OMEGA - LOOK) near_c[lane - (OMEGA - LOOK)] = c[SIGMA - 1];
                if (keep_far) {
                    if (lane >= OMEGA - LOOK) far_c[lane - (OMEGA - LOOK)] = c[SIGMA - 3];
                    else far_c[LOOK_FAR - LOOK + lane] = c[SIGMA - 1];
                    far_c[LOOK + lane] = c[SIGMA - 2];
                }
            }
        }
        if (!BACK) {
#pragma unroll
            for (int k = 0; k < SIGMA; k++) {
                int e = k * OMEGA + lane;
                ibuf[(e / SIGMA) * PITCH + (e % SIGMA)] = c[k];
            }
        } else {
#pragma unroll
            for (int j = 0; j < SIGMA; j++) ibuf[lane * PITCH + j] = c[j];
        }
    }
    wave_sync_lds();    // every wavefront works in its own LDS slice
    if (active) {
        if (!BACK) {
#pragma unroll
            for (int j = 0; j < SIGMA; j++) c[j] = ibuf[lane * PITCH + j];
        } else {
#pragma unroll
            for (int k = 0; k < SIGMA; k++) {
                int e = k * OMEGA + lane;
                c[k] = ibuf[(e / SIGMA) * PITCH + (e % SIGMA)];
            }
        }
#pragma unroll
        for (int k = 0; k < SIGMA; k++) stream_to<KEEP>(&col_idx[base + k * OMEGA + lane], c[k]);
        if constexpr (!BACK && rule_sigma(SIGMA)) {
            static_assert(WINDOW_LINES * 4 <= int(sizeof(lds[0])), "in the wavefront's slice");
            if (sampled) sample_window<SIGMA>(job.window, tile, c, reinterpret_cast<uint32_t*>(lds[wave]), uint32_t(group0), uint32_t(group1), n, int(sizeof(VT)));
        }
    }
    if (!BACK && blockIdx.x == gridDim.x - 1) {
        for (size_t e = size_t(pc) * T + threadIdx.x; e < size_t(nnz); e += blockDim.x) {
            int32_t ce = col_idx[e];
            bad |= (ce < 0) | (ce >= n);
        }
    }
    if (!BACK && bad) raise_status(status, CSR5_STATUS_BAD_COL_IDX);

    // ---- conversion steps 2b, 3a and 3b, lane = tile column: the rows' flags, forced
    // first flag, y_offset = exclusive scan of the columns' flag counts, seg_offset =
    // run of flag-less columns to the right (Algorithm 5; the scan and the run length
    // are wavefront operations here), packing (Section 3.5), and the tile's segment
    // count for the empty_offset layout.
    if constexpr (!BACK) {
        bool marked = false;
        if (job.desc) {                                    // uniform over the grid
            if (active) {
                using word_t = typename std::conditional<(SIGMA > 32), unsigned long long, uint32_t>::type;
                word_t* const fl = reinterpret_cast<word_t*>(lds[wave]);      // one word per column; the entries have left
                wave_sync_lds();
                fl[lane] = 0;
                wave_sync_lds();
                const int64_t lo_e = int64_t(base);
                const auto flag_at = [&](int64_t e) {
                    const int w = int(e - lo_e), i = w / SIGMA;
                    atomicOr(&fl[i], word_t(1) << (w - i * SIGMA));
                };
                if (row1 - row0 <= FLAG_ROWS_MAX) {        // uniform
                    bool empty = false;
                    const int rows = row1 - row0;
                    const auto take = [&](int64_t from, int64_t to) {        // a row, row0 + 1 + k for the lane's k
                        if (from == to) empty = true;
                        else if (from >= lo_e && from < lo_e + T) flag_at(from);
                    };
                    if (lane < rows) take(begins, ends);
                    for (int k = OMEGA + lane; k - lane < rows; k += FLAG_ROWS_AHEAD * OMEGA) {
                        int64_t from[FLAG_ROWS_AHEAD], to[FLAG_ROWS_AHEAD];
                        const auto ask = [&](const auto* __restrict__ row_ptr) {
#pragma unroll
                            for (int q = 0; q < FLAG_ROWS_AHEAD; q++) {
                                const int r = row0 + 1 + (k + q * OMEGA < rows ? k + q * OMEGA : rows - 1);
                                from[q] = row_ptr[r];
                                to[q] = row_ptr[r + 1];
                            }
                        };
                        if (job.wide) ask(static_cast<const int64_t*>(job.row_ptr));
                        else ask(static_cast<const int32_t*>(job.row_ptr));
#pragma unroll
                        for (int q = 0; q < FLAG_ROWS_AHEAD; q++)
                            if (k + q * OMEGA < rows) take(from[q], to[q]);
                    }
                    marked = __any(empty);
                } else {
                    marked = true;
                    int64_t e = lo_e + lane * SIGMA;       // every start in [e, end) is this lane's
                    const int64_t end = e + SIGMA;
                    const auto next_start = [&](int64_t key) -> int64_t {      // the first row start above key
                        int lo = row0, hi = row1 + 1;
                        while (lo < hi) {
                            const int mid = lo + ((hi - lo) >> 1);
                            if (row_at(mid) <= key) lo = mid + 1; else hi = mid;
                        }
                        return row_at(lo);
                    };
                    for (e = next_start(e - 1); e < end && e >= lo_e;) {
                        flag_at(e);
                        const int64_t next = next_start(e);
                        if (next <= e) break;              // not monotone: rejected input
                        e = next;
                    }
                }
                wave_sync_lds();
                uint64_t flags = fl[lane];
                if (lane == 0) flags |= 1u;
                const int cnt = __popcll(flags);
                int incl = cnt;
#pragma unroll
                for (int d = 1; d < OMEGA; d <<= 1) {
                    const int up = __shfl_up(incl, d, OMEGA);
                    if (lane >= d) incl += up;
                }
                const uint32_t yo = uint32_t(incl - cnt);
                const int total = __shfl(incl, OMEGA - 1, OMEGA);
                const uint64_t heads = __ballot(cnt > 0);
                const uint64_t right = (lane == OMEGA - 1) ? 0ull : (heads >> (lane + 1));
                uint32_t so = 0;
                if (cnt > 0) so = right ? uint32_t(__builtin_ctzll(right)) : uint32_t(OMEGA - 1 - lane);
                // little-endian bit field: flags | seg_offset << sigma | y_offset << (sigma+6)
                constexpr int YSH = SIGMA + SBITS;  // <= 54
                const uint64_t lo = flags | (uint64_t(so) << SIGMA) | (uint64_t(yo) << YSH);
                const uint64_t hi = (YSH + YBITS > 64) ? (uint64_t(yo) >> (64 - YSH)) : 0ull;
                uint32_t* const desc = job.desc + size_t(tile) * W * OMEGA + lane;
                desc[0] = uint32_t(lo);
                if (W > 1) desc[OMEGA] = uint32_t(lo >> 32);
                if (W > 2) desc[2 * OMEGA] = uint32_t(hi);
                if (lane == 0) {
                    if (job.wide) static_cast<int64_t*>(job.eop)[tile] = marked ? total : 0;
                    else static_cast<int32_t*>(job.eop)[tile] = marked ? total : 0;
                    if (marked) {                          // (a neighbour that reads the word masks the bit)
                        if (job.wide) static_cast<uint64_t*>(job.tile_ptr)[tile] |= Index<int64_t>::DIRTY;
                        else static_cast<uint32_t*>(job.tile_ptr)[tile] |= Index<int32_t>::DIRTY;
                    }
                }
            }
            // "some tile is marked" (and hence "some row is empty"): once per workgroup, not
            // once per tile -- everything that aims at the one status word queues up
            __shared__ int wg_met_marked;
            if (threadIdx.x == 0) wg_met_marked = 0;
            __syncthreads();
            if (active && marked && lane == 0) wg_met_marked = 1;
            __syncthreads();
            if (threadIdx.x == 0 && wg_met_marked)
                raise_status(status, CSR5_STATUS_HAS_DIRTY | CSR5_STATUS_HAS_EMPTY_ROWS | STATUS_SCAN_NEEDED);
        }
        if (blockIdx.x == 0) {
            if (job.wide) collect_words<int64_t>(job.words, job.nb_tiles, job.nb_rows, pc, static_cast<uint64_t*>(job.tile_ptr), status);
            else collect_words<int32_t>(job.words, job.nb_tiles, job.nb_rows, pc, static_cast<uint32_t*>(job.tile_ptr), status);
        }
    }
}

// ----------------------------------------------------------------------------
// CSR5 SpMV (Algorithm 8), one wavefront per complete tile, lane i = column i.
//
// Lane i streams its sigma (val, col_idx) pairs -- at each step j the 64 lanes
// read 64 consecutive entries -- gathers x, and walks its bit_flag word: a set
// flag closes the running sum either as the column's "red" head (belongs to a
// segment opened by an earlier column) or as a "green" complete segment that is
// stored straight to y[tile_ptr + y_offset + k].  What follows the last flag is
// the "blue" tail.
//
// In-tile segmented sum (the step of Algorithm 8 that calls Algorithm 6).
// Algorithm 6 computes it as a difference of two prefix sums over the whole
// tile, which loses the accuracy of a small row sitting after large ones.  Here: red partials are shifted one
// lane down (tmp[i] = red[i+1], the printed tmp[i-1] <- sum) and summed by a
// segmented suffix scan across the wavefront (sum_to_next_head), the segments being
// delimited by the ballot of "column has a flag".  The range it sums for a head
// column i is exactly tmp[i .. i+seg_offset[i]], the value Algorithm 6 defines;
// seg_offset itself is not read (the ballot carries the same information).
//
// Cross-tile (Section 4 offers atomic adds or a global auxiliary array; device
// wide fp64 atomics are resolved on the memory side of the eight L2s on this
// chip and, at two per tile, measured slower than everything else in the kernel
// together).  Only segment 0 of a tile can continue a row that an earlier tile
// opened (it does iff the tile's first nonzero is not its row's first:
// row_ptr[tile_ptr] != tile*T).  Two ways, chosen per MATRIX during conversion
// (status word), so that both tiles at a boundary decide alike without talking
// to each other:
//  * every tile can get at the head of its first row: it adds the head to its
//    segment 0 and stores the finished row; the previous tile does not store its
//    last segment.  That segment IS the head when the row began inside the
//    previous tile, and inside a workgroup (four neighbouring tiles up to
//    sigma = 16, two up to 32) it is handed over through LDS behind one barrier.
//    The workgroup's first tile sums the head itself, from a CSR-order copy of the
//    last LOOK_MAX = 160 entries of the previous workgroup's last tile (one extra
//    gather for heads up to 32 entries, three beyond).  So the condition is: no
//    first tile of a workgroup starts more than 160 entries into a row, and no
//    other tile more than a tile's length.  Such a matrix needs no second kernel.
//  * otherwise: the auxiliary array.  Segment 0 goes to carry[tile]; the tile that
//    holds the row's first nonzero stores the row's base value, and k_spmv_fixup
//    adds the carries afterwards.  Or, for matrices where that is faster (the
//    host decides, see ONE_LAUNCH_ANY_TILES), inside this kernel: the tiles of a
//    workgroup settle their common rows through LDS, workgroups meet per row at a
//    word of the auxiliary memory, and whoever comes last stores the row (see
//    "One-launch form of the auxiliary-array path" above spmv_tail).
// The third template argument (MODE) is the way: MODE_LOOK, MODE_CARRY, MODE_ONE.
// y needs no zero-fill.  Rows that receive carries from more than one wavefront
// of k_spmv_fixup, and rows cut by 64-entry chunks of the incomplete tile, are
// summed with atomic adds, in whatever order they arrive: their last bits can
// differ from run to run.  Everything else is summed in a fixed order.
//
// Workgroup 0 handles the entries after the last complete tile when there are
// any (early, so that its dependent searches hide behind the tiles); workgroups
// after the tiles write the zeros of rows without nonzeros when the matrix has
// such rows.
// ----------------------------------------------------------------------------
template <int SIGMA>
struct FlagWord {
    using type = typename std::conditional<(SIGMA > 32), uint64_t, uint32_t>::type;
};

// A value from another lane of the 16 that form a row, without LDS: the wavefront's
// scans are chains of dependent steps, and a step through LDS (ds_bpermute, what
// __shfl is) takes many times what one of these does.  DPP_SHIFT_DOWN + d: from
// lane + d, 0 behind the row's end; DPP_ROTATE + d: from lane - d around the row.
// The tile kernel with its scan and sum made of them instead of six shuffles each
// (two LDS operations per shuffle of a double): 2000 short rows 4.29 -> 3.98 us,
// 40^3 stencil 6.82 -> 6.38, 100^3 stencil 60.9 -> 59.6, single precision 45.3 ->
// 44.2, 20 000 rows with dense ones 7.2 -> 6.85; matrices bound by their gathers
// 0-1 %.
constexpr int DPP_SHIFT_DOWN = 0x100, DPP_ROTATE = 0x120;
template <int CTRL>
__device__ __forceinline__ float from_row(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double from_row(double v) {
    const int2 w = __builtin_bit_cast(int2, v);
    const int2 r = {__builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xf, 0xf, true), __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xf, 0xf, true)};
    return __builtin_bit_cast(double, r);
}
__device__ __forceinline__ float from_lane(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double from_lane(double v, int l) {
    const int2 w = __builtin_bit_cast(int2, v);
    const int2 r = {__builtin_amdgcn_readlane(w.x, l), __builtin_amdgcn_readlane(w.y, l)};
    return __builtin_bit_cast(double, r);
}

// Sum over the 64 lanes (all of them active); every lane gets the total.
template <typename VT>
__device__ __forceinline__ VT wave_sum(VT v) {
    v += from_row<DPP_ROTATE + 8>(v);
    v += from_row<DPP_ROTATE + 4>(v);
    v += from_row<DPP_ROTATE + 2>(v);
    v += from_row<DPP_ROTATE + 1>(v);
    return (from_lane(v, 0) + from_lane(v, 16)) + (from_lane(v, 32) + from_lane(v, 48));
}

// For every lane the sum of v over the lanes lane .. end, `end` being the last lane
// before the next one whose bit is set in `heads` (63: none).  Rows of 16 first,
// then the sums of the rows behind: (own + second) + (third + fourth), as deep as a
// tree over 64 lanes.  (One after the other from the last row forward they were
// 2 % further off 64-bit sums where a sum spans the wavefront; like this they are
// as far off as the tree, within 0.7 % at any density of heads.)  All lanes active.
template <typename VT>
__device__ __forceinline__ VT sum_to_next_head(VT v, uint64_t heads, int lane, int end) {
    VT w = from_row<DPP_SHIFT_DOWN + 1>(v);
    if (lane + 1 <= end) v += w;
    w = from_row<DPP_SHIFT_DOWN + 2>(v);
    if (lane + 2 <= end) v += w;
    w = from_row<DPP_SHIFT_DOWN + 4>(v);
    if (lane + 4 <= end) v += w;
    w = from_row<DPP_SHIFT_DOWN + 8>(v);
    if (lane + 8 <= end) v += w;
    const VT from48 = from_lane(v, 48), from16 = from_lane(v, 16);
    VT from32 = from_lane(v, 32);
    if (((heads >> 33) & 0xffffu) == 0) from32 += from48;              // lane 32's sum goes on past lane 47
    if (lane < 16 && end >= 16) v += from16;
    if (lane < 32 && end >= 32) v += from32;
    else if (lane >= 32 && lane < 48 && end >= 48) v += from48;
    return v;
}

// The last `count` (<= LOOK_MAX) entries of a complete tile, read from the
// CSR-order record of its last entries (near part: the last LOOK; far part: the
// LOOK_FAR before them): every lane multiplies up to three of them by their x
// and the wavefront sums the products.  This is how the incomplete tile's
// workgroup completes a row that began shortly before it, instead of handing its
// part to a second kernel (the first tile of a workgroup does the same inside
// k_spmv).  last_col, last_val: the record's two views.
template <typename VT>
__device__ __forceinline__ VT look_behind(const int32_t* __restrict__ last_col, const VT* __restrict__ last_val,
                                          const VT* __restrict__ x, int count, int lane) {
    VT prod = VT(0);
    const int near_n = count < LOOK ? count : LOOK;
    if (lane >= LOOK - near_n && lane < LOOK) prod = last_val[lane] * x[last_col[lane]];
    if (count > LOOK) {                                   // uniform
        const int32_t* const far_c = last_col + FAR_COL_AT;
        const VT* const far_v = last_val + far_val_at<VT>();
        const int first = LOOK_FAR - (count - LOOK);      // far entries first .. LOOK_FAR - 1 belong to the head
#pragma unroll
        for (int j = lane; j < LOOK_FAR; j += OMEGA)
            if (j >= first) prod = fma(far_v[j], x[far_c[j]], prod);
    }
    return wave_sum(prod);
}

// ----------------------------------------------------------------------------
// One-launch form of the auxiliary-array path (Section 4: the sums of a row that
// spans tiles meet in a global auxiliary array).  The tiles of a workgroup are
// neighbours and settle the rows that cross between them through LDS.  A row that
// crosses workgroups is settled through memory without anybody waiting.  Groups:
// tile t of the complete tiles belongs to group t / waves, the incomplete tile is
// a group of its own behind them; span[t] (conversion) says for the row that holds
// tile t's first entry in which group it starts and how many groups it touches.
//  * Two groups (nearly all such rows): each swaps its part into meet[first group]
//    with one atomic exchange.  Whoever gets EMPTY back was first and is done;
//    whoever gets the other's part back adds the two, stores the row and puts
//    EMPTY back.  One memory round trip, and the value travels inside the atomic,
//    so nothing has to be ordered.
//  * More groups: the first group leaves its part in meet[first group], every
//    later group its part in carry[group]; each then counts itself in at
//    arrived[first group], and whoever finds that all the others have been there
//    adds the parts up, in group order, stores the row and resets the two words.
//    A part must have reached memory before its group is counted, and is read by
//    a wavefront of another XCD, whose L2 knows nothing of it: parts and counters
//    are written and read with device-scope atomic accesses (which pass the L2s),
//    and the wait between "part written" and "counted" is the plain wait for the
//    wavefront's outstanding memory operations.  (A release fence would also
//    write back every dirty line of the L2, the rows of y included: measured once
//    per tile, it made the kernel eleven times slower.)
// Either way the parts are added in group order: the result does not depend on
// who came last.
// ----------------------------------------------------------------------------
// A part as the 64-bit word of meet[]: a double's bits (with the one NaN pattern
// that means EMPTY replaced by another NaN), a float's bits under a tag.
__device__ __forceinline__ uint64_t meet_word(double v) {
    const uint64_t b = uint64_t(__double_as_longlong(v));
    return b == MEET_EMPTY ? 0x7ff8000000000000ull : b;
}
__device__ __forceinline__ uint64_t meet_word(float v) { return (1ull << 32) | uint64_t(__float_as_uint(v)); }
template <typename VT> __device__ __forceinline__ VT meet_value(uint64_t w);
template <> __device__ __forceinline__ double meet_value<double>(uint64_t w) { return __longlong_as_double(static_cast<long long>(w)); }
template <> __device__ __forceinline__ float meet_value<float>(uint64_t w) { return __uint_as_float(uint32_t(w)); }

__device__ __forceinline__ uint64_t swap_in(uint64_t* slot, uint64_t w) {
    return __hip_atomic_exchange(slot, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ void publish(T* slot, T v) {
    __hip_atomic_store(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// lane 0 of a wavefront, after publish() and wait_for_memory(): count this group
// in at `counter`; returns how many were there before
__device__ __forceinline__ uint32_t count_in(uint32_t* counter) {
    return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Barrier of the workgroup that orders LDS only: the wavefronts exchange their
// sums through LDS, and a wavefront's atomics to memory may still be on their way.
__device__ __forceinline__ void meet_at_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void wait_for_memory() {
    __builtin_amdgcn_s_waitcnt(0);          // every counter at zero: loads, stores and LDS of this wavefront are done
    asm volatile("" ::: "memory");
}

// The whole wavefront: row R spans groups g0..g1 (three or more) and all of them have published.
template <typename VT>
__device__ __forceinline__ void assemble_row(const VT* piece_in, uint64_t* meet, uint32_t* arrived,
                                             int g0, int g1, VT* __restrict__ y, uint32_t R, int m, int lane) {
    VT sum = VT(0);
    for (int g = g0 + 1 + lane; g <= g1; g += OMEGA)
        sum += __hip_atomic_load(piece_in + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sum = wave_sum(sum);
    if (lane == 0) {
        sum = meet_value<VT>(__hip_atomic_load(meet_at(meet, g0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) + sum;
        if (R < uint32_t(m)) y[R] = sum;
        publish(meet_at(meet, g0), MEET_EMPTY);
        publish(arrived + g0, 0u);
    }
}

constexpr int TAIL_MAX_CHUNKS = (CSR5_SIGMA_MAX * OMEGA) / OMEGA + 1;   // 64-entry chunks in < one tile

// Entries after the last complete tile (Section 4, last paragraph: a CSR-vector
// style pass).  64 consecutive entries per wavefront step; the row of each entry
// comes from a binary search (so runs of empty rows cost nothing); a shuffle
// scan sums runs of equal row.  A row that lies inside one 64-entry chunk is
// stored directly.  A row cut by a chunk boundary is accumulated in LDS, in the
// slot of the chunk it starts in (at most one row starts in a chunk and leaves
// it), and stored at the end.  The part of a row that began in the complete
// tiles is treated like a tile's segment 0: completed here when the row began at
// most LOOK entries earlier, handed to carry[pc] otherwise.
template <typename VT, typename IT>
__device__ void spmv_tail(int m, IT nnz, IT first, uint32_t row_first,
                          const IT* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                          const VT* __restrict__ val, const VT* __restrict__ x,
                          VT* __restrict__ y, VT* __restrict__ carry_slot,
                          VT* piece_in, uint64_t* meet, uint32_t* arrived, uint2 row_span,
                          const int32_t* __restrict__ last_col, const VT* __restrict__ last_val) {
    __shared__ VT acc[TAIL_MAX_CHUNKS];
    __shared__ int acc_row[TAIL_MAX_CHUNKS];
    __shared__ VT acc_first;
    const int lane = lane_id();
    const int wave = threadIdx.x / OMEGA, nwaves = blockDim.x / OMEGA;
    for (int q = threadIdx.x; q < TAIL_MAX_CHUNKS; q += blockDim.x) { acc[q] = VT(0); acc_row[q] = -1; }
    if (threadIdx.x == 0) acc_first = VT(0);
    __syncthreads();
    int row_lo = row_first > uint32_t(m) ? m : int(row_first);
    const int span = int(nnz - first);                   // < one tile
    const int nchunks = (span + OMEGA - 1) / OMEGA;
    for (int q = wave; q < nchunks && q < TAIL_MAX_CHUNKS; q += nwaves) {
        // 64-bit: with 32-bit indices and nnz within 64 of 2^31 these would overflow
        const int64_t chunk_lo = int64_t(first) + q * OMEGA;
        const int64_t e = chunk_lo + lane;
        const bool live = e < nnz;
        int row = -2 - lane;                         // distinct keys for dead lanes
        VT prod = VT(0);
        if (live) {
            row = row_lo + count_le(row_ptr + row_lo, m + 1 - row_lo, e) - 1;
            prod = val[e] * x[col_idx[e]];
        }
#pragma unroll
        for (int d = 1; d < OMEGA; d <<= 1) {
            VT up = __shfl_up(prod, d, OMEGA);
            int rup = __shfl_up(row, d, OMEGA);
            if (lane >= d && rup == row) prod += up;
        }
        int rnext = __shfl_down(row, 1, OMEGA);
        bool run_end = live && ((lane == OMEGA - 1) || (rnext != row));
        if (run_end && row >= 0 && row < m) {
            IT rs = row_ptr[row], re = row_ptr[row + 1];
            if (rs >= chunk_lo && re <= chunk_lo + OMEGA) {
                y[row] = prod;                       // the whole row lies in this chunk
            } else if (rs < first) {
                atomicAdd(&acc_first, prod);         // continues a row of the complete tiles
            } else {
                int q1 = int((rs - first) / OMEGA);  // chunk the row starts in
                if (q1 >= 0 && q1 < TAIL_MAX_CHUNKS) {
                    atomicAdd(&acc[q1], prod);
                    acc_row[q1] = row;
                }
            }
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < TAIL_MAX_CHUNKS; q += blockDim.x)
        if (acc_row[q] >= 0) y[acc_row[q]] = acc[q];
    if (threadIdx.x < OMEGA && piece_in) {               // first wavefront, one-launch form: this is the last group of its first row
        if (row_lo < m && first > 0 && row_ptr[row_lo] < first) {
            const int g0 = int(row_span.x), g1 = g0 + int(row_span.y) - 1;
            if (row_span.y == 2u) {
                uint64_t other = MEET_EMPTY;
                if (lane == 0) other = swap_in(meet_at(meet, g0), meet_word(acc_first));
                if (lane == 0 && other != MEET_EMPTY) {
                    y[row_lo] = meet_value<VT>(other) + acc_first;
                    publish(meet_at(meet, g0), MEET_EMPTY);
                }
            } else {
                uint32_t before = 0;
                if (lane == 0) {
                    publish(piece_in + g1, acc_first);
                    wait_for_memory();
                    before = count_in(arrived + g0);
                }
                if (__shfl(before, 0, OMEGA) == uint32_t(g1 - g0))
                    assemble_row<VT>(piece_in, meet, arrived, g0, g1, y, uint32_t(row_lo), m, lane);
            }
        }
    } else if (threadIdx.x < OMEGA) {                    // first wavefront
        VT carried = acc_first;
        if (last_col && row_lo < m && first > 0) {       // last_col: entries of the last complete tile, or null
            const IT rs = row_ptr[row_lo];
            if (rs < first && first - rs <= IT(LOOK_MAX)) {  // the first row began shortly before: finish it here
                const VT head = look_behind<VT>(last_col, last_val, x, int(first - rs), lane);
                if (lane == 0) y[row_lo] = head + acc_first;
                carried = VT(0);
            }
        }
        if (lane == 0) *carry_slot = carried;
    }
}

// The per-column walk and the in-tile segmented sum of a tile (flags, yo: the lane's
// column; v, xv: its entries and their x).  Every segment's sum goes to yb[its number];
// returns the number of segments.
template <int SIGMA, typename VT>
__device__ __forceinline__ uint32_t walk_columns(typename FlagWord<SIGMA>::type flags, uint32_t yo, const VT* v, const VT* xv, VT* yb, int lane) {
    constexpr int T = OMEGA * SIGMA;
    VT sum = VT(0), red = VT(0);
    bool seen = false;
    uint32_t seg = yo;
#pragma unroll
    for (int j = 0; j < SIGMA; j++) {
        if ((flags >> j) & 1) {
            if (seen) {                                   // a green segment ends
                if (seg < uint32_t(T)) yb[seg] = sum;
                seg++;
            } else {                                      // the red head ends (empty when j == 0)
                red = sum;
                seen = true;
            }
            sum = VT(0);
        }
        sum = fma(v[j], xv[j], sum);
    }
    VT blue = sum;
    if (!seen) { red = sum; blue = VT(0); }                 // whole column is red

    // ---- in-tile segmented sum of the red partials
    uint64_t heads = __ballot(seen);                      // bit 0 is always set
    VT tmp = from_row<DPP_SHIFT_DOWN + 1>(red);          // the next lane's; 0 for the last
    {
        const VT from16 = from_lane(red, 16), from32 = from_lane(red, 32), from48 = from_lane(red, 48);
        if (lane == 15) tmp = from16;
        if (lane == 31) tmp = from32;
        if (lane == 47) tmp = from48;
    }
    uint64_t right = (lane == OMEGA - 1) ? 0ull : (heads >> (lane + 1));
    int end = right ? (lane + __builtin_ctzll(right)) : (OMEGA - 1);   // last lane of my segment
    tmp = sum_to_next_head(tmp, heads, lane, end);
    if (seen && seg < uint32_t(T)) yb[seg] = blue + tmp;
    // number of segments of the tile = flags before the last column + its own
    return __builtin_amdgcn_readlane(seen ? seg + 1 : seg, OMEGA - 1);
}

// Gathers in single precision, two entries at a time.  What a gather costs in the L1 goes by the lanes that
// ask, unless they ask for one stretch of a line: next to a stream of 8 bytes an entry that is the bound (100^3
// stencil: L1 busy 29 us with 43 accesses per 64 entries, of 45).  So where the entry of an odd lane has
// the column next to that of the lane before it, that one loads 8 bytes and the odd lane asks for nothing.
// Single precision, whole SpMV, before -> after: 27-point stencil 100^3 45.0 -> 40.4 us, 140^3 124 -> 114;
// blocks of 3 columns (9 a row) 49.1 -> 40.6, of 4 (7) 45.5 -> 38.6, of 6 (5) 42.4 -> 39.4; 9-point stencil
// 40.0 -> 38.4, 5-point 42.1 -> 40.2.  Not for entries one by one (24 diagonals 46.7 -> 51.4, 20 random
// columns a row 98 -> 104) and not where a gather is one stretch already (tridiagonal 37.1 -> 38.9, five
// diagonals 37.4 -> 40.0): the host decides, see pairs_pay.
// Tried: three and four entries at a time (44.3, 45.4 on the 100^3 stencil: more registers, and 12 and 16
// bytes a lane to bring back); pairs at any place, not only from even lanes: the same; in double precision
// (16 bytes) 60.3 -> 71.7; either way in one kernel, decided per tile: 44.0 (98 registers instead of 79).
constexpr int PAIR_NOWHERE = 0x7ffffff0;                          // outside of any x
constexpr int DPP_QUAD_EVEN = 0xa0;                               // lanes 0, 0, 2, 2 of every four
template <int COUNT>
__device__ __forceinline__ void gather_pairs(const float* x, int x_bytes, const int32_t* c, float* xv) {
    typedef float pair_t __attribute__((ext_vector_type(2)));
    const auto xbuf = tile_buffer(x, x_bytes);
    pair_t got[COUNT];
    bool second[COUNT];
#pragma unroll
    for (int k = 0; k < COUNT; k++) {
        // (in this form: the difference of the two came out with its sign changed)
        second[k] = __builtin_amdgcn_update_dpp(0, c[k], DPP_QUAD_EVEN, 0xf, 0xf, true) + 1 == c[k];
        got[k] = __builtin_bit_cast(pair_t, __builtin_amdgcn_raw_buffer_load_b64(xbuf, second[k] ? PAIR_NOWHERE : c[k] * 4, 0, 0));
    }
#pragma unroll
    for (int k = 0; k < COUNT; k++) {
        const float from_even = from_row<DPP_QUAD_EVEN>(float(got[k].y));
        xv[k] = second[k] ? from_even : float(got[k].x);
    }
}

template <int SIGMA, typename VT, typename IT, int MODE, bool KEEP, bool PAIRS = false>
__global__ void __launch_bounds__(TransposeShape<SIGMA>::WAVES * OMEGA)
k_spmv(int m, int x_bytes, IT nnz, int pc, int p, uint32_t nb_tiles, uint32_t has_tail, uint32_t xcd_chunk, uint32_t far_mode,
       int rec_bytes, const IT* __restrict__ row_ptr, const typename Index<IT>::tp_t* __restrict__ tile_ptr,
       const uint32_t* __restrict__ tile_desc, const IT* __restrict__ eop,
       const int32_t* __restrict__ eo, const int32_t* __restrict__ col_idx,
       const VT* __restrict__ val, const VT* __restrict__ x, VT* __restrict__ y,
       VT* __restrict__ carry, uint64_t* __restrict__ meet, uint32_t* __restrict__ arrived,
       const uint2* __restrict__ span, const uint32_t* __restrict__ status, const uint32_t* __restrict__ tile_head,
       const int32_t* __restrict__ last_col, const VT* __restrict__ last_val,
       const uint32_t* __restrict__ order, uint32_t order_second, uint32_t order_len) {
    constexpr bool CAN_LOOK = MODE == MODE_LOOK;
    constexpr bool ONE = MODE == MODE_ONE;
    constexpr bool MEET = CAN_LOOK || ONE;      // the wavefronts of a workgroup meet at one barrier
    constexpr int T = OMEGA * SIGMA;
    constexpr int YBITS = 32 - __builtin_clz(uint32_t(T - 1));        // ceil(log2(64*sigma))
    constexpr int W = (SIGMA + SBITS + YBITS + 31) / 32;
    constexpr int YSH = SIGMA + SBITS;
    constexpr int WAVES = TransposeShape<SIGMA>::WAVES;
    constexpr int PITCH = TransposeShape<SIGMA>::PITCH;
    using flag_t = typename FlagWord<SIGMA>::type;
    using tp_t = typename Index<IT>::tp_t;
    // one slot per tile entry: a column index on the way in, an x value on the way back,
    // a segment sum at the end (so single precision needs half the space)
    __shared__ VT lds[WAVES][OMEGA * PITCH];
    __shared__ VT last_sum[WAVES];    // look-behind inside a workgroup: every tile's last segment, for the next tile

    const uint32_t st = *status;      // consulted below, after the streaming loads are in flight
    // Rows that cross a tile boundary are completed by look-behind in the whole
    // matrix or nowhere: both tiles at a boundary must decide alike.
    // CAN_LOOK = false is the instantiation for matrices the host knows to need
    // the carry array: the same kernel without the look-behind's loads.
    const bool look = CAN_LOOK && last_col != nullptr && !(st & STATUS_NEEDS_CARRY);

    if (blockIdx.x < has_tail) {      // workgroup 0: incomplete last tile
        if (st & BAD_BITS) return;
        const tp_t first_row = tile_ptr[pc] & Index<IT>::ROWMASK;
        spmv_tail<VT, IT>(m, nnz, IT(pc) * T, first_row > tp_t(m) ? uint32_t(m) : uint32_t(first_row),
                          row_ptr, col_idx, val, x, y, carry + pc,
                          ONE ? carry : nullptr, meet, arrived, ONE ? span[pc] : uint2{0u, 1u},
                          (look && pc > 0) ? last_col + size_t((pc - 1) / WAVES) * size_t(rec_bytes / 4) : nullptr,
                          (look && pc > 0) ? last_val + size_t((pc - 1) / WAVES) * size_t(rec_bytes / int(sizeof(VT))) : nullptr);
        return;
    }
    if (blockIdx.x >= has_tail + nb_tiles) {   // workgroups after the tiles: the zeros of rows without nonzeros
        if ((st & BAD_BITS) || !(st & CSR5_STATUS_HAS_EMPTY_ROWS)) return;
        const uint32_t b = blockIdx.x - has_tail - nb_tiles, nb = gridDim.x - has_tail - nb_tiles;
        const int64_t stride = int64_t(nb) * blockDim.x;
        for (int64_t r = int64_t(b) * blockDim.x + threadIdx.x; r < int64_t(m); r += stride)
            if (row_ptr[r] == row_ptr[r + 1]) y[r] = VT(0);
        return;
    }
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / OMEGA);
    int tile;
    if (MODE == MODE_CARRY && order) {      // the list of order_place
        const uint32_t k = order_place(blockIdx.x - has_tail, nb_tiles, order_second / WAVES) * WAVES + wave;
        const uint32_t t = k < order_len ? order[k] : 0xffffffffu;
        tile = t < uint32_t(pc) ? int(t) : pc;
    } else {
        tile = int(xcd_order(blockIdx.x - has_tail, nb_tiles, xcd_chunk)) * WAVES + wave;
    }
    // (every wavefront of a tile workgroup passes exactly one barrier, see below)
    if (tile >= pc) {
        if constexpr (MEET) __syncthreads();
        return;
    }

    // How far into its first row the tile starts, and the next tile into its own
    // (tile_head: entries of a tile's first row that lie before the tile; p + 1
    // entries, 0 at p).  The same for every lane: scalar loads.
    const uint32_t head_len = tile_head[tile];
    const uint32_t next_head = tile_head[tile + 1];
    // One-launch form of the auxiliary-array path: the rows that cross this tile's
    // two boundaries (first group, number of groups), and the row of the second.
    uint2 span_in = {0u, 1u}, span_out = {0u, 1u};
    uint32_t out_row = 0;
    if constexpr (ONE) {
        span_in = span[tile];
        span_out = span[tile + 1];
        const typename Index<IT>::tp_t next_wide = tile_ptr[tile + 1] & Index<IT>::ROWMASK;
        out_row = next_wide < typename Index<IT>::tp_t(m) ? uint32_t(next_wide) : 0u;
    }

    // ---- look-behind, first part: the previous tile's last LOOK entries, whether
    // or not this tile turns out to need them (asking first would put a dependent
    // load in front of these, and everything the wavefront loads later waits for
    // them in turn).  Lanes LOOK.. repeat the addresses of lanes 0..LOOK-1.
    // Only the first tile of a workgroup needs them: the others get the finished
    // sum of their row's head from the wavefront next door (last_sum).  A head
    // longer than LOOK also takes the far part of the record, two entries per lane.
    VT head_v = VT(0), head_x = VT(0), far_v0 = VT(0), far_v1 = VT(0), far_prod = VT(0);
    int32_t head_c = 0, far_c0 = 0, far_c1 = 0;
    // far_mode, from the host: 0 = this matrix has no such head (nobody waits for
    // head_len then), 1 = it has, or the host does not know yet.  (Taking the far
    // part without asking whenever the matrix has such heads was slower than
    // asking: 114 against 110 us on a 53 M-nonzero matrix of 128-entry rows.)
    const bool far_head = CAN_LOOK && look && wave == 0 && far_mode != 0u && head_len > uint32_t(LOOK) &&
                          rec_bytes == LAST_REC_BYTES;      // uniform (the last test cannot fail: such a matrix has no long head in look mode)
    if constexpr (CAN_LOOK) {
        if (wave == 0) {
            const size_t rec = size_t(tile > 0 ? tile - 1 : 0) / WAVES;      // the group before this one
            const int32_t* const near_c = last_col + rec * size_t(rec_bytes / 4);
            const VT* const near_v = last_val + rec * size_t(rec_bytes / int(sizeof(VT)));
            head_c = near_c[lane & (LOOK - 1)];
            head_v = near_v[lane & (LOOK - 1)];
        }
    }

    // ---- stream the tile.  val: at step j the 64 lanes read 64 consecutive
    // doubles, lane i keeping entry (column i, step j).  col_idx is not needed by
    // its owner lane at all (see the gather below), so it is read with 16-byte
    // loads in plain memory order: 4 steps of the tile per instruction.
    const size_t tile_base = size_t(tile) * T;
    constexpr int NC4 = (SIGMA + 3) / 4;                  // 16-byte col loads per lane (past the tile's end: 0)
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    i32x4 c4[NC4];
    VT v[SIGMA];
    const uint32_t* dp = tile_desc + size_t(tile) * W * OMEGA;
    uint32_t dw[W];
    // Through buffer descriptors (tile_buffer), with one exception that measurement
    // makes, not a cause that was found: in single precision with the look-behind at the
    // automatic height, plain loads are faster by 2-8 % where x is at home in the L2s
    // (20 M nonzeros in rows of 17 random columns, x of 80 and 600 KB: 78.6 -> 72.6 and
    // 96.8 -> 93.0 us; rows of 130, x of 80 KB: 82.9 -> 78.2; 100^3 stencil 43.9 -> 43.2;
    // x of 8 MB level).  At the other heights from 8 to 32 the descriptors are level or up
    // to 14 % faster (14: 3 % slower), and 1-5 % faster without the look-behind.
    if constexpr (sizeof(VT) == 4 && CAN_LOOK && SIGMA == RULE_R) {
        static_assert(RULE_R % 4 == 0, "NC4 loads per lane are the tile");
        if ((reinterpret_cast<uintptr_t>(col_idx) & 15) == 0) {
            const i32x4* const col4 = reinterpret_cast<const i32x4*>(col_idx + tile_base);
#pragma unroll
            for (int q = 0; q < NC4; q++) c4[q] = stream_from<KEEP>(&col4[q * OMEGA + lane]);
        } else {      // a view at an odd offset
            const auto cols = tile_buffer(col_idx + tile_base, T * 4);
#pragma unroll
            for (int q = 0; q < NC4; q++) c4[q] = stream_from<i32x4, KEEP>(cols, (q * OMEGA + lane) * 16);
        }
#pragma unroll
        for (int j = 0; j < SIGMA; j++) v[j] = stream_from<KEEP>(&val[tile_base + j * OMEGA + lane]);
#pragma unroll
        for (int w = 0; w < W; w++) dw[w] = stream_from<KEEP>(&dp[w * OMEGA + lane]);
    } else {
        const auto cols = tile_buffer(col_idx + tile_base, T * 4);
        const auto vals = tile_buffer(val + tile_base, T * int(sizeof(VT)));
        const auto descs = tile_buffer(dp, W * OMEGA * 4);
#pragma unroll
        for (int q = 0; q < NC4; q++) c4[q] = stream_from<i32x4, KEEP>(cols, (q * OMEGA + lane) * 16);
#pragma unroll
        for (int j = 0; j < SIGMA; j++) v[j] = stream_from<VT, KEEP>(vals, (j * OMEGA + lane) * int(sizeof(VT)));
#pragma unroll
        for (int w = 0; w < W; w++) dw[w] = stream_from<uint32_t, KEEP>(descs, (w * OMEGA + lane) * 4);
    }

    // ---- descriptor
    const tp_t tp = tile_ptr[tile];
    const bool dirty = (tp & Index<IT>::DIRTY) != 0;
    const tp_t row0_wide = tp & Index<IT>::ROWMASK;
    const uint32_t row0 = uint32_t(row0_wide);
    uint64_t lo = dw[0], hi = 0;
    if constexpr (W > 1) lo |= uint64_t(dw[1]) << 32;
    if constexpr (W > 2) hi = dw[2];
    constexpr int FLAG_BITS = 8 * int(sizeof(flag_t));
    constexpr flag_t FLAG_MASK = (SIGMA == FLAG_BITS) ? ~flag_t(0) : flag_t((flag_t(1) << (SIGMA % FLAG_BITS)) - 1);
    const flag_t flags = flag_t(lo) & FLAG_MASK;
    uint32_t yo = uint32_t(lo >> YSH);
    if (W > 2) yo |= uint32_t(hi << (64 - YSH));
    // empty_offset slice of a tile that holds empty rows (Algorithm 8, where y_offset is replaced by empty_offset[y_offset])
    const int32_t* eo_t = nullptr;
    uint32_t nseg_t = 0;
    if (dirty) {
        IT e0 = eop[tile], e1 = eop[tile + 1];
        eo_t = eo + e0;
        nseg_t = uint32_t(e1 - e0);
    }
    // look-behind, the far part of the record.  Asked for only here, behind the
    // tile's own loads: the decision needs head_len, and a wait for it further up
    // would hold back the stream of every tile, also of those that never take it.
    if constexpr (CAN_LOOK) {
        if (far_head) {
            const size_t rec = size_t(tile - 1) / WAVES;                  // tile > 0: it has a head
            const int32_t* const far_c = last_col + rec * size_t(rec_bytes / 4) + FAR_COL_AT;
            const VT* const far_v = last_val + rec * size_t(rec_bytes / int(sizeof(VT))) + far_val_at<VT>();
            far_c0 = far_c[lane];
            far_c1 = far_c[OMEGA + lane];
            far_v0 = far_v[lane];
            far_v1 = far_v[OMEGA + lane];
        }
    }
    if ((st & BAD_BITS) || row0_wide >= tp_t(m)) {        // rejected input: gather and store nothing
        if constexpr (MEET) __syncthreads();
        return;
    }
    // Does segment 0 continue a row that an earlier tile opened?  Then either this
    // tile gets hold of the row's head (see `look`) and stores the finished row,
    // or its part goes through the carry array.
    // The mirror image: when the next tile (or the incomplete tile's workgroup)
    // completes this tile's last row, this tile must not store its part of it.
    const bool cont0 = head_len != 0;
    const bool skip_last = look && next_head != 0;
    const bool fetch_head = look && cont0 && wave == 0;   // uniform; the head is then at most LOOK_MAX entries long
    // the last min(head_len, LOOK) of the near LOOK entries belong to the head
    const bool head_lane = fetch_head && lane < LOOK && lane >= LOOK - int(head_len < uint32_t(LOOK) ? head_len : uint32_t(LOOK));

    // ---- gather x.  Lane i owns the CSR entries i*sigma .. i*sigma+sigma-1 of the
    // tile, so at a fixed step the 64 lanes would gather from 64 unrelated
    // places.  Consecutive CSR entries, however, have increasing and often
    // adjacent columns.  So the column indices are laid out in LDS in CSR order
    // (entry (i, j) at i*PITCH + j, rows padded to an odd pitch), read back so
    // that lane L holds CSR entries k*64+L (64 consecutive entries per gather
    // instruction: few distinct cache lines), x is gathered in that order, and
    // the values return through the same LDS buffer to the owner lanes.
    VT* const xb = reinterpret_cast<VT*>(lds[wave]);
    int32_t* const cb = reinterpret_cast<int32_t*>(lds[wave]);
    VT xv[SIGMA];
    {
#pragma unroll
        for (int q = 0; q < NC4; q++) {
            const int m0 = (q * OMEGA + lane) * 4;        // memory offset inside the tile = j*64 + i
            const int j = m0 / OMEGA, i0 = m0 % OMEGA;
            if (SIGMA % 4 == 0 || m0 < T) {
                cb[(i0 + 0) * PITCH + j] = c4[q].x;
                cb[(i0 + 1) * PITCH + j] = c4[q].y;
                cb[(i0 + 2) * PITCH + j] = c4[q].z;
                cb[(i0 + 3) * PITCH + j] = c4[q].w;
            }
        }
        wave_sync_lds();
        int32_t c[SIGMA];
#pragma unroll
        for (int k = 0; k < SIGMA; k++) {
            const int e = k * OMEGA + lane;
            c[k] = cb[(e / SIGMA) * PITCH + (e % SIGMA)];
        }
        wave_sync_lds();
        // All gathers of the tile are in flight together up to sigma = 32.  Beyond
        // that they go in groups of 16 (8 from sigma = 47 on): each gather holds four registers (address and
        // result) next to the tile's 2*sigma value registers, and with all of them
        // at once the kernel ran out of the 256 a wavefront can have (sigma >= 42:
        // spills into accumulator registers, one wavefront per SIMD).
        constexpr int GROUP = SIGMA > 46 ? 8 : (SIGMA > 32 ? 16 : SIGMA);
        // (without the look-behind the record holds nothing: the conversion did not fill it)
        VT far_x0 = VT(0), far_x1 = VT(0);
        if constexpr (CAN_LOOK) {
            if (wave == 0) {
                head_x = x[look ? head_c : 0];
                if (far_head) {
                    far_x0 = x[far_c0];
                    far_x1 = x[far_c1];
                }
            }
        }
        if constexpr (PAIRS) {
            static_assert(sizeof(VT) == 4 && GROUP == SIGMA, "all at once");
            gather_pairs<SIGMA>(x, x_bytes, c, xv);
        }
#pragma unroll
        for (int k0 = 0; k0 < SIGMA; k0 += GROUP) {
            if constexpr (!PAIRS) {
#pragma unroll
                for (int k = k0; k < k0 + GROUP && k < SIGMA; k++) xv[k] = x[c[k]];
            }
#pragma unroll
            for (int k = k0; k < k0 + GROUP && k < SIGMA; k++) {
                const int e = k * OMEGA + lane;
                xb[(e / SIGMA) * PITCH + (e % SIGMA)] = xv[k];
            }
            wave_sync_lds();
        }
#pragma unroll
        for (int j = 0; j < SIGMA; j++) xv[j] = xb[lane * PITCH + j];
        wave_sync_lds();
        if constexpr (CAN_LOOK) {
            if (far_head) {     // far entries first .. LOOK_FAR - 1 belong to the head (none when it is short); lane holds entries lane and lane + 64
                const int first = LOOK_FAR + LOOK - int(head_len);
                if (lane >= first) far_prod = far_v0 * far_x0;
                if (lane + OMEGA >= first) far_prod = fma(far_v1, far_x1, far_prod);
            }
        }
    }

    // ---- finished segment sums go to LDS (the buffer is free again), slot = segment
    // number inside the tile, and are written to y afterwards, 64 consecutive segments
    // per store instruction.
    VT* const yb = xb;                                // T <= 64*PITCH slots
    uint32_t nseg = walk_columns<SIGMA, VT>(flags, yo, v, xv, yb, lane);
    if (nseg > uint32_t(T)) nseg = T;
    if (dirty && nseg > nseg_t) nseg = nseg_t;            // cannot happen for a consistent format
    wave_sync_lds();

    // The head of the tile's first row.  Tiles of one workgroup are neighbours: a
    // tile's last segment, which the tile itself does not store when the row goes
    // on (skip_last), is the head its successor needs, finished (in look-behind
    // mode a row begins at most LOOK entries before a tile, so inside the previous
    // one).  It crosses through LDS; the workgroup's first tile has no neighbour
    // here and sums its head from the previous tile's record.
    VT head = VT(0);
    if constexpr (CAN_LOOK) {
        if (lane == 0) last_sum[wave] = nseg ? yb[nseg - 1] : VT(0);     // (nseg >= 1: a tile's first flag is forced)
        __syncthreads();
        if (wave == 0) head = wave_sum(head_lane ? fma(head_v, head_x, far_prod) : far_prod);
        else if (look && cont0) head = last_sum[wave - 1];
    }

    // One-launch form.  What the tiles before this one, inside the workgroup, hold
    // of its first row comes through LDS: a tile that lies wholly inside the row
    // passes on what it got plus its own sum, the tile the row starts in its last
    // segment.  `outside`: the row began before the workgroup.
    bool store_first = true, drop_last = false, pub_in = false, pub_out = false, pub_out_first = false;
    uint32_t before_in = 0, before_out = 0;
    uint64_t other_in = MEET_EMPTY, other_out = MEET_EMPTY;
    VT part_in = VT(0), part_out = VT(0);
    const int group = tile / WAVES;
    if constexpr (ONE) {
        __shared__ VT first_sum[WAVES];
        __shared__ int inside_row[WAVES];
        const bool goes_on = next_head != 0;                       // the last segment's row continues in the next tile
        const bool last_of_group = wave == WAVES - 1 || tile + 1 >= pc;
        const bool leaves = nseg == 1 && goes_on;                  // the tile's only segment goes on
        // Parts that do not depend on the neighbours set out before the barrier: the
        // last segment of the group's last tile, and the first tile's first segment
        // when its row ends there.
        const bool early_out = nseg > 1 && goes_on && last_of_group;
        const bool early_in = wave == 0 && cont0 && !leaves;
        if (lane == 0) {
            first_sum[wave] = nseg ? yb[0] : VT(0);
            last_sum[wave] = nseg ? yb[nseg - 1] : VT(0);
            inside_row[wave] = (nseg == 1 && cont0) ? 1 : 0;
            if (early_in) {
                part_in = first_sum[wave];
                if (span_in.y == 2u) other_in = swap_in(meet_at(meet, span_in.x), meet_word(part_in));
                else publish(carry + group, part_in);
            }
            if (early_out) {
                part_out = last_sum[wave];
                if (span_out.y == 2u) other_out = swap_in(meet_at(meet, group), meet_word(part_out));
                else publish(meet_at(meet, group), meet_word(part_out));
            }
        }
        meet_at_barrier();
        bool outside = false;
        if (cont0) {
            outside = true;
            for (int v = wave - 1; v >= 0; v--) {
                if (inside_row[v]) {
                    head += first_sum[v];
                } else {
                    head += last_sum[v];
                    outside = false;
                    break;
                }
            }
        }
        store_first = !leaves && !(cont0 && outside);
        drop_last = goes_on;
        // the group's part of a row that came in from outside: published where the row ends, or by the group's last tile
        pub_in = cont0 && outside && (!leaves || last_of_group);
        // the group's part of a row that began inside it and leaves it
        pub_out_first = leaves && last_of_group && !(cont0 && outside);
        pub_out = pub_out_first || early_out;
        if (lane == 0 && (pub_in || pub_out)) {
            const bool late_in = pub_in && !early_in, late_out = pub_out_first;
            if (late_in || late_out) {
                const VT whole = first_sum[wave] + head;
                if (late_in) part_in = whole;
                if (late_out) part_out = whole;
            }
            const bool count_in_row = pub_in && span_in.y != 2u, count_out_row = pub_out && span_out.y != 2u;
            if (late_in && !count_in_row) other_in = swap_in(meet_at(meet, span_in.x), meet_word(part_in));
            if (late_out && !count_out_row) other_out = swap_in(meet_at(meet, group), meet_word(part_out));
            if (count_in_row || count_out_row) {
                if (late_in && count_in_row) publish(carry + group, part_in);
                if (late_out && count_out_row) publish(meet_at(meet, group), meet_word(part_out));
                wait_for_memory();
                if (count_in_row) before_in = count_in(arrived + span_in.x);
                if (count_out_row) before_out = count_in(arrived + group);
            }
        }
    }

    // ---- write the tile's rows.  Segment s is row tile_ptr + s, or
    // tile_ptr + empty_offset[s] when the tile holds empty rows.  In the
    // two-kernel form segment 0 goes to the carry array when it continues an
    // earlier tile's row.
    for (uint32_t s0 = 0; s0 < nseg; s0 += OMEGA) {
        const uint32_t sg = s0 + lane;
        if (sg < nseg) {
            VT value = yb[sg];
            const uint32_t row = row0 + (dirty ? uint32_t(eo_t[sg]) : sg);
            bool mine;
            if constexpr (ONE) {
                if (sg == 0) value += head;
                mine = sg == 0 ? store_first : !(drop_last && sg == nseg - 1);
            } else {
                if (sg == 0) {
                    carry[tile] = (cont0 && !look) ? value : VT(0);
                    value += head;                         // 0 unless this tile completes the row
                }
                mine = (sg != 0 || !cont0 || look) && !(skip_last && sg == nseg - 1);
            }
            if (mine && row < uint32_t(m)) y[row] = value;
        }
    }
    if constexpr (ONE) {
        // (the answers come back while the rows above are stored)
        const uint32_t row_out = pub_out_first ? row0 : out_row;
        if (pub_in && span_in.y == 2u) {               // two groups: the second to come stores the row
            if (lane == 0 && other_in != MEET_EMPTY) {
                if (row0 < uint32_t(m)) y[row0] = meet_value<VT>(other_in) + part_in;
                publish(meet_at(meet, span_in.x), MEET_EMPTY);
            }
        } else if (pub_in && __shfl(before_in, 0, OMEGA) == span_in.y - 1u) {
            assemble_row<VT>(carry, meet, arrived, int(span_in.x), int(span_in.x + span_in.y) - 1, y, row0, m, lane);
        }
        if (pub_out && span_out.y == 2u) {
            if (lane == 0 && other_out != MEET_EMPTY) {
                if (row_out < uint32_t(m)) y[row_out] = part_out + meet_value<VT>(other_out);
                publish(meet_at(meet, group), MEET_EMPTY);
            }
        } else if (pub_out && __shfl(before_out, 0, OMEGA) == span_out.y - 1u) {
            assemble_row<VT>(carry, meet, arrived, group, group + int(span_out.y) - 1, y, row_out, m, lane);
        }
    }
}

// ----------------------------------------------------------------------------
// SpMV with x through LDS, for matrices whose columns are spread over an x that an L2
// holds and an L1 does not.  k_spmv gathers from the L1, and every entry there is a
// 128-byte line from the L2: 225 G/s on the whole chip whatever the kernel does (6 M
// entries in rows of 201, x of 480 KB: 27 of 36.7 us).  Here one workgroup per CU
// takes WAVES * K tiles at a time, keeps their columns in registers, and has x come by in parts
// through two buffers in LDS, straight from memory to LDS, one on its way while the
// other is read; in each part every entry whose column lies in it picks its x (which
// lanes read is the execution mask, so a step is a subtraction, a comparison and the
// read).  x is read once per workgroup, in whole lines, instead of a line per entry.
// Bound by the LDS reads, one per entry and part, and by the stream in front of them:
// 1.0-1.25 us per part of 79 KB, and 18.5 us for everything else on that matrix.
// Whole SpMV, before -> after: that matrix 36.7 -> 23.8 us, single precision 34.5 ->
// 16.5; 6 M entries in rows of 100, x of 160 KB 34.6 -> 18.9, of 800 KB 37.7 -> 28.5;
// 12.4 M, x of 320 KB 68.8 -> 40.5; in rows of 500 (height 16), 6 M, x of 480 KB 34.9 ->
// 23.3, 20 M in single precision 92 -> 49.
// Where it is taken: staged_tiles, sample_columns.
// Tried: x through registers instead of straight to LDS, one buffer of 156 KB: 31.4; 12
// or 8 wavefronts with more tiles each, height 8: 27.4, 31.0 (at height 16 in double precision 12
// with two tiles, 23.3, against 16 with two 30.1: spills; 16 with one 31.8: two rounds);
// the first two parts asked for up front: 26.2; another tile's values in the second part:
// the same.
//
// Columns of a tile stay with their owner lane (no reordering: LDS does not care), so
// the sums are those of k_spmv: walk_columns for each tile, then the rows that cross
// tiles inside the workgroup in one step over the tiles (lane = tile).  A row that
// crosses workgroups is settled like in the one-launch form (see there), its groups
// being the workgroups here.  One launch; rows without nonzeros are zeroed on the way,
// a share per workgroup.
// ----------------------------------------------------------------------------
constexpr int LDS_BYTES = 160 * 1024;       // of a CU
constexpr int STAGE_BYTES = 79 * 1024;     // twice, and the tail's few hundred bytes: of 160 KB
constexpr int WAIT_LDS = 0xc07f, WAIT_LOADS = 0x0f70;       // s_waitcnt: lgkmcnt(0); vmcnt(0)

// 16 or 4 bytes per lane from a buffer to consecutive bytes of LDS (counted as a load of the wavefront)
__device__ __forceinline__ void to_lds_16(__amdgpu_buffer_rsrc_t r, char* lds, int offset) {
#ifdef __HIP_DEVICE_COMPILE__
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, offset, 0, 0, 0);
#endif
}
__device__ __forceinline__ void to_lds_4(__amdgpu_buffer_rsrc_t r, char* lds, int offset) {
#ifdef __HIP_DEVICE_COMPILE__
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 4, offset, 0, 0, 0);
#endif
}

// ----------------------------------------------------------------------------
// Entries whose x no cache near them holds: columns anywhere in an x larger than the L2s.
//
// A gather from such an x is a 128-byte line from memory for one value, 55 G/s on the whole chip
// (rows of 30 random columns out of 4 M: 80 M entries 1350 us, 8 times their stream).  So these
// entries' values of x are brought to them in two steps, both in whole lines:
//  1. k_far_gather: x in blocks of FAR_BLOCK_BYTES through LDS, one per workgroup; from each it
//     picks the values that the matrix asks of it, in a list of 2-byte columns, and writes them
//     to a buffer one after the other.  x is read once.
//  2. k_spmv_staged (FORM_FAR): a workgroup of FAR_ENTRIES entries fetches its own from the
//     buffer.  The list of a block is in the order of the workgroups, so what one of them takes
//     from a block lies together (7 entries and more on the matrices this is for), and the rest of the line is
//     its neighbours', which run on the same XCD.  They go to LDS, to the entry's place among the
//     workgroup's (which of the two, 4 and 2 bytes, is a list as well), when the entries near
//     the diagonal have taken theirs from the window there; from LDS every lane picks its own.
// Where few entries are near the diagonal all of them go that way, and the tile kernel reads no columns
// (FORM_ALL).  22 to 40 bytes an entry instead of 128 and more.  Whole SpMV, before -> after:
// mixed (four fifths of the rows within +-5000 columns, the others anywhere) 136 M entries 1187 -> 688
// us, single precision 1020 -> 464, 51 M 405 -> 247; rows of 0-20 columns out of 4 M
// 682 -> 258, 554 -> 167.  Of the 688, 147 are the first kernel (0.66 GB, 4.5 TB/s: stores), 540
// the second: 175 for the lists and the buffer, 70 for the stores of y, 45 for the window.
// The buffer is a handle's, of FAR_BUFFER_BYTES at most; the handle's products take turns (launch_far), and a captured
// one, which may be replayed beside any other, goes without (68 M entries 335.3 us, with the event between products 338.1).  A matrix
// with more such entries goes through it in chunks of workgroups (136 M entries in 1, 2, 4, 8 chunks 717,
// 709, 717, 789; 34 M in 1, 2, 4 187, 196, 219: a drained chip between any two kernels).
// Tried: the buffer read past the caches (nt) 709 -> 808; written so 709 -> 712, single precision 472 ->
// 490; 4, 8, 9, 11, 12 and 14 entries per thread asked for ahead of the window instead of 10: 722, 708, 700, 691,
// 696, 739; without a window 10 and 13 instead of 16: rows of 0-20 268 -> 279, 291; blocks of 64 KB 708 -> 720.
//
// The lists are the conversion's (far_make): where it blocks, allocates for itself and the columns
// pay for it.  A block's entries are counted per workgroup (k_far_count), the counts scanned in
// the order chunk, block, workgroup (k_far_segments, k_far_bases, k_far_starts), and every workgroup
// sorts its entries by block in LDS and writes them to their places (k_far_place).  The order of
// a workgroup's entries in a block is any; the sums do not depend on it.
// ----------------------------------------------------------------------------
constexpr int FAR_THREADS = 512, FAR_PLACE_BITS = 13, FAR_AHEAD = 10, FAR_AHEAD_ALL = 16;
template <typename VT> constexpr int far_block_shift() { return sizeof(VT) == 8 ? 14 : 15; }

struct FarShape {
    int pc, n, groups, blocks, segments;              // workgroups, blocks of x, FAR_SEGMENTs of workgroups
    int window_bytes;                                 // 0: all entries go through the buffer
    float slope;
};
// What the counts say: how many entries, and of each chunk how long its list is and which segment it ends before
struct FarCounted {
    uint32_t total, list[FAR_MAX_CHUNKS];
    int32_t end[FAR_MAX_CHUNKS];
};

// Calls take(column, place) for the entries of a workgroup's tiles outside its window
template <int SIGMA, typename VT, typename F>
__device__ __forceinline__ void far_each(const FarShape& f, int group, const uint32_t* __restrict__ tile_ptr, const int32_t* __restrict__ col_idx, F take) {
    constexpr uint32_t ROWMASK = Index<int32_t>::ROWMASK;
    constexpr int T = OMEGA * SIGMA, TILES = FAR_ENTRIES / T, EACH = FAR_ENTRIES / FAR_THREADS;
    const int tile0 = group * TILES, tiles = f.pc - tile0 < TILES ? f.pc - tile0 : TILES;
    const uint32_t window = uint32_t(window_first(tile_ptr[tile0] & ROWMASK, tile_ptr[tile0 + TILES < f.pc ? tile0 + TILES : f.pc] & ROWMASK,
                                                  f.slope, f.n * int(sizeof(VT)), int(sizeof(VT))));
    const auto cols = tile_buffer(col_idx + size_t(tile0) * T, tiles * T * 4);
    int32_t c[EACH];
#pragma unroll
    for (int u = 0; u < EACH; u++) c[u] = stream_from<int32_t, false>(cols, (u * FAR_THREADS + int(threadIdx.x)) * 4);
#pragma unroll
    for (int u = 0; u < EACH; u++) {
        const int place = u * FAR_THREADS + int(threadIdx.x);
        if (place < tiles * T && uint32_t(c[u]) * uint32_t(sizeof(VT)) - window >= uint32_t(f.window_bytes)) take(c[u], place);
    }
}

template <int SIGMA, typename VT>
__global__ void __launch_bounds__(FAR_THREADS)
k_far_count(const FarShape f, const uint32_t* __restrict__ tile_ptr, const int32_t* __restrict__ col_idx, uint16_t* __restrict__ counts, uint32_t* __restrict__ base) {
    __shared__ uint32_t count[FAR_MAX_BLOCKS], all;
    for (int b = threadIdx.x; b < f.blocks; b += FAR_THREADS) count[b] = 0;
    if (threadIdx.x == 0) all = 0;
    __syncthreads();
    const int group = int(xcd_order(blockIdx.x, uint32_t(f.groups), 0));
    far_each<SIGMA, VT>(f, group, tile_ptr, col_idx, [&](int32_t c, int) { atomicAdd(&count[c >> far_block_shift<VT>()], 1u); });
    __syncthreads();
    uint32_t mine = 0;
    for (int b = threadIdx.x; b < f.blocks; b += FAR_THREADS) {
        counts[size_t(group) * f.blocks + b] = uint16_t(count[b]);
        mine += count[b];
    }
    if (mine) atomicAdd(&all, mine);
    __syncthreads();
    if (threadIdx.x == 0) base[group] = all;
}

// Sums over FAR_SEGMENT workgroups.  The last workgroup: where each group's list begins.
__global__ void __launch_bounds__(SCAN_THREADS)
k_far_segments(const FarShape f, const uint16_t* __restrict__ counts, uint32_t* __restrict__ sums, uint32_t* __restrict__ base, FarCounted* __restrict__ counted) {
    if (int(blockIdx.x) == f.segments) {
        uint32_t carry = 0;
        for (int64_t at = 0; at < f.groups; at += SCAN_CHUNK) carry += scan_chunk<uint32_t>(base, at, f.groups, carry);
        if (threadIdx.x == 0) base[f.groups] = counted->total = carry;
        return;
    }
    const int g0 = blockIdx.x * FAR_SEGMENT, g1 = g0 + FAR_SEGMENT < f.groups ? g0 + FAR_SEGMENT : f.groups;
    for (int b = threadIdx.x; b < f.blocks; b += SCAN_THREADS) {
        uint32_t s = 0;
#pragma unroll 16
        for (int g = g0; g < g1; g++) s += counts[size_t(g) * f.blocks + b];
        sums[size_t(blockIdx.x) * f.blocks + b] = s;
    }
}

// A workgroup per chunk: in the chunk's list, by block of x, where each segment's share begins (in place of its sum), and where each
// block's does.
__global__ void __launch_bounds__(SCAN_THREADS)
k_far_bases(const FarShape f, int value_bytes, uint32_t* __restrict__ sums, uint32_t* __restrict__ range, const uint32_t* __restrict__ base, FarCounted* __restrict__ counted) {
    static_assert(FAR_MAX_BLOCKS == SCAN_THREADS, "a thread per block");
    const uint32_t total = counted->total;
    const int chunk = blockIdx.x, chunks = far_chunks(total, value_bytes);
    if (chunk >= chunks) return;
    __shared__ uint32_t wave_sum[SCAN_THREADS / OMEGA];
    const int lane = lane_id(), wave = threadIdx.x / OMEGA, b = threadIdx.x;
    const int s0 = far_chunk_segment(base, f.segments, total, chunks, chunk), s1 = far_chunk_segment(base, f.segments, total, chunks, chunk + 1);
    uint32_t all = 0;
    if (b < f.blocks) {
#pragma unroll 16
        for (int s = s0; s < s1; s++) all += sums[size_t(s) * f.blocks + b];
    }
    all = (all + FAR_PAD - 1) / FAR_PAD * FAR_PAD;
    uint32_t incl = all;
#pragma unroll
    for (int d = 1; d < OMEGA; d <<= 1) {
        const uint32_t up = __shfl_up(incl, d, OMEGA);
        if (lane >= d) incl += up;
    }
    if (lane == OMEGA - 1) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; w++) before += wave_sum[w];
    uint32_t at = before + incl - all;
    uint32_t* const my_range = range + size_t(chunk) * (f.blocks + 1);
    if (b < f.blocks) my_range[b] = at;
    if (b == f.blocks - 1) {
        my_range[f.blocks] = counted->list[chunk] = at + all;
        counted->end[chunk] = s1;
    }
    if (b < f.blocks) {
#pragma unroll 16
        for (int s = s0; s < s1; s++) {
            const uint32_t v = sums[size_t(s) * f.blocks + b];
            sums[size_t(s) * f.blocks + b] = at;
            at += v;
        }
    }
}

// Where in its chunk's list each workgroup's share of a block begins
__global__ void __launch_bounds__(FAR_THREADS)
k_far_starts(const FarShape f, const uint16_t* __restrict__ counts, const uint32_t* __restrict__ sums, uint32_t* __restrict__ starts) {
    const int g0 = blockIdx.x * FAR_SEGMENT, g1 = g0 + FAR_SEGMENT < f.groups ? g0 + FAR_SEGMENT : f.groups;
    for (int b = threadIdx.x; b < f.blocks; b += FAR_THREADS) {
        uint32_t at = sums[size_t(blockIdx.x) * f.blocks + b];
#pragma unroll 16
        for (int g = g0; g < g1; g++) {
            starts[size_t(g) * f.blocks + b] = at;
            at += counts[size_t(g) * f.blocks + b];
        }
    }
}

template <int SIGMA, typename VT>
__global__ void __launch_bounds__(FAR_THREADS)
k_far_place(const FarShape f, const uint32_t* __restrict__ tile_ptr, const int32_t* __restrict__ col_idx, const uint16_t* __restrict__ counts,
            const uint32_t* __restrict__ starts, const FarCounted* __restrict__ counted, const uint32_t* __restrict__ base, uint32_t* __restrict__ src,
            uint16_t* __restrict__ place, uint16_t* __restrict__ cols) {
    __shared__ uint32_t next[FAR_MAX_BLOCKS], from[FAR_MAX_BLOCKS], entry[FAR_ENTRIES], wave_sum[FAR_THREADS / OMEGA];
    __shared__ uint16_t block_of[FAR_ENTRIES];
    constexpr int SHIFT = far_block_shift<VT>(), EACH = FAR_MAX_BLOCKS / FAR_THREADS;
    static_assert(FAR_PLACE_BITS + SHIFT <= 32 && (1 << FAR_PLACE_BITS) == FAR_ENTRIES, "place and column in a word");
    const int group = int(xcd_order(blockIdx.x, uint32_t(f.groups), 0)), segment = group / FAR_SEGMENT;
    const int lane = lane_id(), wave = threadIdx.x / OMEGA;
    size_t first = 0;                                     // of the chunk's columns
    for (int chunk = 0; counted->end[chunk] <= segment; chunk++) first += counted->list[chunk];
    uint32_t n[EACH], at[EACH], s = 0;
#pragma unroll
    for (int u = 0; u < EACH; u++) {
        const int b = threadIdx.x * EACH + u;
        n[u] = at[u] = 0;
        if (b < f.blocks) {
            at[u] = starts[size_t(group) * f.blocks + b];
            n[u] = counts[size_t(group) * f.blocks + b];
        }
        s += n[u];
    }
    uint32_t incl = s;
#pragma unroll
    for (int d = 1; d < OMEGA; d <<= 1) {
        const uint32_t up = __shfl_up(incl, d, OMEGA);
        if (lane >= d) incl += up;
    }
    if (lane == OMEGA - 1) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t before = incl - s;
    for (int w = 0; w < wave; w++) before += wave_sum[w];
#pragma unroll
    for (int u = 0; u < EACH; u++) {
        const int b = threadIdx.x * EACH + u;
        next[b] = before;
        from[b] = at[u] - before;                         // of the chunk's list, less the place in the group's
        before += n[u];
    }
    __syncthreads();
    far_each<SIGMA, VT>(f, group, tile_ptr, col_idx, [&](int32_t c, int p) {
        const int b = c >> SHIFT;
        const uint32_t k = atomicAdd(&next[b], 1u);
        entry[k] = uint32_t(p) | (uint32_t(c) & ((1u << SHIFT) - 1)) << FAR_PLACE_BITS;
        block_of[k] = uint16_t(b);
    });
    __syncthreads();
    const uint32_t my = base[group], count = base[group + 1] - my;
    for (uint32_t k = threadIdx.x; k < count; k += FAR_THREADS) {
        const uint32_t e = entry[k], to = from[block_of[k]] + k;
        src[my + k] = to;
        place[my + k] = uint16_t(e & (FAR_ENTRIES - 1));
        cols[first + to] = uint16_t(e >> FAR_PLACE_BITS);
    }
}

constexpr int FAR_GATHER_THREADS = 1024, FAR_GATHER_AHEAD = 8;
template <typename VT>
__global__ void __launch_bounds__(FAR_GATHER_THREADS)
k_far_gather(int n, int pieces, const uint32_t* __restrict__ range, const uint16_t* __restrict__ cols, const VT* __restrict__ x, VT* __restrict__ values) {
    constexpr int SHIFT = far_block_shift<VT>(), WAVES = FAR_GATHER_THREADS / OMEGA, STEP = FAR_GATHER_THREADS * 2;
    constexpr uint32_t COLS = 1u << SHIFT;
    typedef VT pair_t __attribute__((ext_vector_type(2)));
    __shared__ __align__(16) char xs[FAR_BLOCK_BYTES];
    const int block = blockIdx.x / pieces, piece = blockIdx.x % pieces;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / OMEGA);
    const FarPiece mine(range[block], range[block + 1], piece, pieces);
    if (mine.empty()) return;
    const uint32_t begin = mine.begin, end = mine.end;
    const auto list = tile_buffer(cols + begin, int((end - begin) * 2));
    uint32_t c[FAR_GATHER_AHEAD];
    const auto ask = [&](uint32_t k0) {
#pragma unroll
        for (int u = 0; u < FAR_GATHER_AHEAD; u++) c[u] = stream_from<uint32_t, false>(list, int((k0 + uint32_t(u * STEP) + threadIdx.x * 2) * 2));
    };
    ask(0);
    const auto xbuf = tile_buffer(x, n * int(sizeof(VT)));
    const bool wide16 = (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    for (int at = wave * 1024; at < FAR_BLOCK_BYTES; at += WAVES * 1024) {
        const int64_t off = int64_t(block) * FAR_BLOCK_BYTES + at;
        if (wide16 && off + 1024 <= int64_t(n) * int64_t(sizeof(VT))) {
            to_lds_16(xbuf, xs + at, int(off) + lane * 16);
        } else if (off < int64_t(n) * int64_t(sizeof(VT))) {
#pragma unroll
            for (int q = 0; q < 4; q++) to_lds_4(xbuf, xs + at + q * 256, int(off) + q * 256 + lane * 4);
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(WAIT_LOADS);
    asm volatile("" ::: "memory");
    __syncthreads();
    for (uint32_t k0 = 0;;) {
        pair_t v[FAR_GATHER_AHEAD];
#pragma unroll
        for (int u = 0; u < FAR_GATHER_AHEAD; u++) {      // (the padding behind a block's columns holds anything)
            v[u].x = reinterpret_cast<const VT*>(xs)[c[u] & (COLS - 1)];
            v[u].y = reinterpret_cast<const VT*>(xs)[c[u] >> 16 & (COLS - 1)];
        }
        const uint32_t k1 = k0 + FAR_GATHER_AHEAD * STEP;
        const bool more = begin + k1 < end;
        if (more) ask(k1);
#pragma unroll
        for (int u = 0; u < FAR_GATHER_AHEAD; u++) {
            const uint32_t k = begin + k0 + uint32_t(u * STEP) + threadIdx.x * 2;
            if (k < end) *reinterpret_cast<pair_t*>(values + k) = v[u];
        }
        if (!more) break;
        k0 = k1;
    }
}

// Of a sample of entries (two neighbours in each column of FAR_SAMPLE_TILES tiles), how many lie far outside
// their window (answer[0]), and on how many lines of x (answer[1]).  One workgroup; only for matrices whose
// first sample (sample_window) speaks for it.
constexpr int FAR_SAMPLE_TILES = 128;
template <int SIGMA, typename VT>
__global__ void __launch_bounds__(SCAN_THREADS)
k_far_sample(const FarShape f, const uint32_t* __restrict__ tile_ptr, const int32_t* __restrict__ col_idx, uint32_t* __restrict__ answer) {
    constexpr uint32_t ROWMASK = Index<int32_t>::ROWMASK;
    constexpr int T = OMEGA * SIGMA, TILES = FAR_ENTRIES / T, PER_WAVE = FAR_SAMPLE_TILES / (SCAN_THREADS / OMEGA);
    constexpr int WORDS = FAR_BLOCK_BYTES / 128 * FAR_MAX_BLOCKS / 32;                // a bit per line of x
    __shared__ uint32_t seen[WORDS];
    __shared__ uint32_t far, lines;
    const int lane = lane_id(), wave = threadIdx.x / OMEGA;
    int32_t c[PER_WAVE][2];
    uint32_t window[PER_WAVE];
#pragma unroll
    for (int u = 0; u < PER_WAVE; u++) {
        const int q = wave * PER_WAVE + u, tile = int(int64_t(f.pc) * q / FAR_SAMPLE_TILES), tile0 = tile / TILES * TILES;
        const int j = (q + lane / 16 * SIGMA / 4) % (SIGMA - 1);
        const int32_t* const pair = col_idx + size_t(tile) * T + j * OMEGA + lane;
        c[u][0] = pair[0];
        c[u][1] = pair[OMEGA];
        window[u] = uint32_t(window_first(tile_ptr[tile0] & ROWMASK, tile_ptr[tile0 + TILES < f.pc ? tile0 + TILES : f.pc] & ROWMASK,
                                          f.slope, f.n * int(sizeof(VT)), int(sizeof(VT))));
    }
    for (int w = threadIdx.x; w < WORDS; w += SCAN_THREADS) seen[w] = 0;
    if (threadIdx.x == 0) far = lines = 0;
    __syncthreads();
    uint32_t my_far = 0, my_lines = 0;
#pragma unroll
    for (int u = 0; u < PER_WAVE; u++) {
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const uint32_t b = uint32_t(c[u][e]) * uint32_t(sizeof(VT));
            if (b - window[u] + FAR_REACH_BYTES >= uint32_t(2 * FAR_REACH_BYTES)) {
                const uint32_t bit = 1u << (b / 128 % 32);
                if (!(atomicOr(&seen[b / 4096], bit) & bit)) my_lines++;
                my_far++;
            }
        }
    }
    if (my_far) atomicAdd(&far, my_far);
    if (my_lines) atomicAdd(&lines, my_lines);
    __syncthreads();
    if (threadIdx.x == 0) {
        answer[0] = far;
        answer[1] = lines;
    }
}

struct RowSpan { int first, groups; };     // the workgroups a row touches

// part_bytes: of x, a multiple of 1024, at most STAGE_BYTES; parts * part_bytes covers x.
//
// WINDOW, for matrices most of whose entries lie near the diagonal but not in order: a band
// with random columns, wider than an L1 and narrower than LDS.  k_spmv takes a line from the
// L2 for each of those entries, too.  Here the workgroup keeps the one part of x around its
// rows' place on the diagonal (window_first), and the entries outside it come from memory as in
// k_spmv, asked for while the window is on its way.  Neighbouring workgroups run on one XCD
// (contiguous order), so that a window is read from memory once per L2.  Two workgroups of
// WINDOW_WAVES per CU, smaller than in the form above: nothing is read twice for it, and one has its
// loads in flight while the other walks.
// Bound by the stream and, where there are some, by the lines from outside the window.  Whole
// SpMV, before -> after: rows of 8-16 entries within +-5000 columns, 30 M 124.0 -> 92.7 us,
// 6 M 31.3 -> 23.6, single precision 4 M 18.3 -> 11.9; rows of 40-80, 45 M 154.5 -> 111.3; a
// fifth of the rows random (mixed), 12.6 M 83.9 -> 69.5, 34 M 270 -> 254, 136 M 1233 ->
// 1185 (59 M lines from memory are 1000 of it).
// Tried: 16 wavefronts of one tile at height 8: 500 000 rows of mixed 49.2 -> 50.5; 4 of four
// 54.2; 8 of three 48.9, but 23.2 -> 28.2 at 200 000 rows.
// Rows that cross workgroups: as above where the handle's slot has what that wants (meet),
// through the auxiliary array and k_spmv_fixup otherwise, one sum per workgroup.
//
// FORM_FAR: the window form, with the entries outside the window from the buffer of k_far_gather.
// FORM_ALL: all entries from there; no window, and the columns are not read.
constexpr int FORM_PARTS = 0, FORM_WINDOW = 1, FORM_FAR = 2, FORM_ALL = 3;
struct FarEntries {                // of FORM_FAR
    int first, count;              // the launch's workgroups
    const uint32_t* base;          // where a workgroup's share of the lists begins
    const uint32_t* src;           // an entry's place in the buffer
    const uint16_t* place;         // and among the workgroup's entries
    const void* values;            // the buffer
    int value_bytes;
};
template <int SIGMA, int WAVES, int K, int FORM, typename VT>
__global__ void __launch_bounds__(WAVES * OMEGA, FORM != FORM_PARTS ? WAVES * (LDS_BYTES / WINDOW_BYTES) / 4 : 1)
k_spmv_staged(int m, int n, int nnz, int pc, uint32_t groups, uint32_t has_tail, uint32_t zero_rows, int part_bytes, int parts,
              const int32_t* __restrict__ row_ptr, const uint32_t* __restrict__ tile_ptr,
              const uint32_t* __restrict__ tile_desc, const int32_t* __restrict__ eop, const int32_t* __restrict__ eo,
              const int32_t* __restrict__ col_idx, const VT* __restrict__ val, const VT* __restrict__ x, VT* __restrict__ y,
              VT* __restrict__ carry, uint64_t* __restrict__ meet, uint32_t* __restrict__ arrived,
              const uint32_t* __restrict__ tile_head, float slope, const FarEntries far) {
    constexpr bool ALL = FORM == FORM_ALL, FAR = FORM == FORM_FAR || ALL, WINDOW = FORM != FORM_PARTS;
    constexpr int AHEAD = ALL ? FAR_AHEAD_ALL : FAR_AHEAD;
    constexpr uint32_t ROWMASK = Index<int32_t>::ROWMASK, DIRTY = Index<int32_t>::DIRTY;
    constexpr int T = OMEGA * SIGMA, THREADS = WAVES * OMEGA, TILES = WAVES * K;
    constexpr int YSH = SIGMA + SBITS;
    static_assert(YSH + 32 - __builtin_clz(uint32_t(T - 1)) <= 32, "one descriptor word");
    static_assert(TILES <= OMEGA && (WINDOW ? WAVES * T * int(sizeof(VT)) <= WINDOW_BYTES : (WAVES + 1) / 2 * T * int(sizeof(VT)) <= STAGE_BYTES),
                  "one lane per tile; the segment sums in the stage's place");
    // two arrays, not the halves of one: the compiler has the reads of one wait for what is on its way to it only
    __shared__ __align__(16) char xs0[WINDOW ? WINDOW_BYTES : STAGE_BYTES], xs1[WINDOW ? 16 : STAGE_BYTES];
    __shared__ VT first_sum[TILES], last_sum[TILES];
    __shared__ uint32_t tile_bits[TILES];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / OMEGA);
    const int last_group = int(groups);            // the incomplete tile's
    const auto group_of = [&](int e) -> int { const int tile = e / T; return tile < pc ? tile / TILES : last_group; };
    const auto span_of = [&](uint32_t row) -> RowSpan {
        const int g0 = group_of(row_ptr[row]);
        return RowSpan{g0, group_of(row_ptr[row + 1] - 1) - g0 + 1};
    };
    if (blockIdx.x < has_tail) {
        const uint32_t row = tile_ptr[pc] & ROWMASK;
        const RowSpan s = row < uint32_t(m) ? span_of(row) : RowSpan{0, 1};
        spmv_tail<VT, int32_t>(m, nnz, pc * T, row, row_ptr, col_idx, val, x, y, carry + pc, WINDOW && !meet ? nullptr : carry, meet, arrived,
                               uint2{uint32_t(s.first), uint32_t(s.groups)}, nullptr, nullptr);
        return;
    }
    const int group = FAR ? far.first + int(xcd_order(blockIdx.x - has_tail, uint32_t(far.count), 0))
                          : int(WINDOW ? xcd_order(blockIdx.x - has_tail, groups, 0) : blockIdx.x - has_tail);
    const int tile0 = group * TILES, mine = tile0 + wave * K;
    int window = 0;
    if constexpr (WINDOW)
        window = window_first(tile_ptr[tile0] & ROWMASK, tile_ptr[tile0 + TILES < pc ? tile0 + TILES : pc] & ROWMASK, slope, n * int(sizeof(VT)), int(sizeof(VT)));

    // ---- x, first part; behind it the tiles' columns, the values of the first tile
    const auto xbuf = tile_buffer(x, n * int(sizeof(VT)));
    const bool wide16 = (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    const auto stage = [&](int part, char* to) {     // (what lies behind x reads as 0)
        for (int at = wave * 1024; at < part_bytes; at += WAVES * 1024) {
            const int off = (WINDOW ? window : part * part_bytes) + at;
            if (wide16 && off + 1024 <= n * int(sizeof(VT))) {
                to_lds_16(xbuf, to + at, off + lane * 16);
            } else {
#pragma unroll
                for (int q = 0; q < 4; q++) to_lds_4(xbuf, to + at + q * 256, off + q * 256 + lane * 4);
            }
        }
    };
    if constexpr (!WINDOW) stage(0, xs0);
    // Entries whose x comes through the buffer: where from and where to, the first AHEAD of each thread
    uint32_t far_count = 0;
    __amdgpu_buffer_rsrc_t far_src, far_place, far_values;
    uint32_t fs[AHEAD], fp[AHEAD];
    VT fv[AHEAD];
    const auto far_lists = [&](uint32_t k0) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            const uint32_t k = k0 + uint32_t(u * THREADS) + threadIdx.x;
            fs[u] = stream_from<uint32_t, false>(far_src, int(k * 4));         // (reads as 0 behind the end)
            fp[u] = uint32_t(stream_from<uint16_t, false>(far_place, int(k * 2)));
        }
    };
    const auto far_fetch = [&](uint32_t k0) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            const uint32_t k = k0 + uint32_t(u * THREADS) + threadIdx.x;
            fv[u] = stream_from<VT, true>(far_values, k < far_count ? int(fs[u] * uint32_t(sizeof(VT))) : INT32_MAX - 15);
        }
    };
    const auto far_put = [&](uint32_t k0) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            const uint32_t k = k0 + uint32_t(u * THREADS) + threadIdx.x;
            if (k < far_count) *reinterpret_cast<VT*>(xs0 + fp[u] * uint32_t(sizeof(VT))) = fv[u];
        }
    };
    if constexpr (FAR) {
        const uint32_t at = far.base[group];
        far_count = far.base[group + 1] - at;
        far_src = tile_buffer(far.src + at, int(far_count * 4));
        far_place = tile_buffer(far.place + at, int(far_count * 2));
        far_values = tile_buffer(static_cast<const VT*>(far.values), far.value_bytes);
    }
    asm volatile("" ::: "memory");
    int32_t c[K][SIGMA];               // (ALL: not used)
    uint32_t dw[K], tp[K], head[K + 1];
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int tile = mine + k;
        const auto cols = tile_buffer(col_idx + size_t(tile < pc ? tile : 0) * T, tile < pc ? T * 4 : 0);    // (an empty buffer reads as 0)
        const auto descs = tile_buffer(tile_desc + size_t(tile < pc ? tile : 0) * OMEGA, tile < pc ? OMEGA * 4 : 0);
#pragma unroll
        for (int j = 0; j < SIGMA; j++) c[k][j] = ALL ? 0 : stream_from<int32_t, false>(cols, (j * OMEGA + lane) * 4) * int(sizeof(VT));
        dw[k] = stream_from<uint32_t, false>(descs, lane * 4);
    }
    if constexpr (FAR) far_lists(0);
#pragma unroll
    for (int k = 0; k <= K; k++) {
        const int tile = mine + k < pc ? mine + k : pc;
        head[k] = tile_head[tile];
        if (k < K) tp[k] = tile_ptr[tile];
    }
    uint32_t row_in = 0, row_out = 0;
    RowSpan si = {0, 1}, so = {0, 1};
    if (wave == 0) {
        row_in = tile_ptr[tile0] & ROWMASK;
        row_out = tile_ptr[tile0 + TILES < pc ? tile0 + TILES : pc] & ROWMASK;
        if (!WINDOW || meet) {
            if (row_in < uint32_t(m)) si = span_of(row_in);
            if (row_out < uint32_t(m)) so = span_of(row_out);
        }
    }
    asm volatile("" ::: "memory");
    VT v[K][SIGMA];
    const auto load_v = [&](int k) {
        const int tile = mine + k;
        const auto vals = tile_buffer(val + size_t(tile < pc ? tile : 0) * T, tile < pc ? T * int(sizeof(VT)) : 0);
#pragma unroll
        for (int j = 0; j < SIGMA; j++) v[k][j] = stream_from<VT, false>(vals, (j * OMEGA + lane) * int(sizeof(VT)));
    };
    load_v(0);
    if constexpr (WINDOW) {
#pragma unroll
        for (int k = 1; k < K; k++) load_v(k);
        if constexpr (FAR) far_fetch(0);
        asm volatile("" ::: "memory");
        stage(0, xs0);
        asm volatile("" ::: "memory");
    }
    if (zero_rows) {
        for (RowShare r(m, uint32_t(group), groups, threadIdx.x); r.more(); r.next(THREADS))
            if (row_ptr[r.row] == row_ptr[r.row + 1]) y[r.row] = VT(0);
    }
    // ---- gather: every entry takes its x from the part that holds its column
    VT xv[K][SIGMA];
#pragma unroll
    for (int k = 0; k < K; k++)
#pragma unroll
        for (int j = 0; j < SIGMA; j++) xv[k][j] = VT(0);
    const auto take = [&](int part, const char* from, char* next) {
        // This part has arrived: what this wavefront asked for before the columns came before
        // them (loads return in order); later parts, and its reads of the part before (which the
        // compiler could move behind a wait that does not say that it is about memory).
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(WAIT_LDS);
        if (part > 0) __builtin_amdgcn_s_waitcnt(WAIT_LOADS);
        else asm volatile("" :: "v"(c[K - 1][SIGMA - 1]), "v"(dw[K - 1]) : "memory");
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();      // everybody's share of it, and nobody reads the part before any more
        asm volatile("" ::: "memory");
        if (part + 1 < parts) stage(part + 1, next);
        const uint32_t base = uint32_t(part * part_bytes);
#pragma unroll
        for (int k = 0; k < K; k++)
#pragma unroll
            for (int j = 0; j < SIGMA; j++) {
                const uint32_t at = uint32_t(c[k][j]) - base;
                if (at < uint32_t(part_bytes)) xv[k][j] = *reinterpret_cast<const VT*>(from + at);
            }
    };
    if constexpr (WINDOW) {
        // what lies outside the window comes from memory, on its way while the window is waited for
        if constexpr (!FAR) {
#pragma unroll
            for (int k = 0; k < K; k++)
#pragma unroll
                for (int j = 0; j < SIGMA; j++)
                    if (uint32_t(c[k][j]) - uint32_t(window) >= uint32_t(part_bytes))
                        xv[k][j] = *reinterpret_cast<const VT*>(reinterpret_cast<const char*>(x) + uint32_t(c[k][j]));
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(WAIT_LOADS);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (!ALL) {
#pragma unroll
            for (int k = 0; k < K; k++)
#pragma unroll
                for (int j = 0; j < SIGMA; j++) {
                    const uint32_t at = uint32_t(c[k][j]) - uint32_t(window);
                    if (at < uint32_t(part_bytes)) xv[k][j] = *reinterpret_cast<const VT*>(xs0 + at);
                }
        }
        if constexpr (FAR) {
            if constexpr (!ALL) __syncthreads();       // the other entries' values go where the window was, in the tiles' order
            far_put(0);
            for (uint32_t k0 = AHEAD * THREADS; k0 < far_count; k0 += AHEAD * THREADS) {
                far_lists(k0);
                far_fetch(k0);
                far_put(k0);
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K; k++)
#pragma unroll
                for (int j = 0; j < SIGMA; j++)
                    if (ALL || uint32_t(c[k][j]) - uint32_t(window) >= uint32_t(part_bytes))
                        xv[k][j] = *reinterpret_cast<const VT*>(xs0 + uint32_t(((wave * K + k) * T + j * OMEGA + lane) * int(sizeof(VT))));
        }
    } else {
        for (int part = 0; part < parts; part += 2) {
            take(part, xs0, xs1);
            if (part + 1 < parts) take(part + 1, xs1, xs0);
        }
    }
    __syncthreads();                   // the segment sums go where x was
    if constexpr (!WINDOW) {
#pragma unroll
        for (int k = 1; k < K; k++) load_v(k);
    }

    // ---- the tiles, one after the other, as in k_spmv
    VT* const yb = WINDOW ? reinterpret_cast<VT*>(xs0) + wave * T : reinterpret_cast<VT*>(wave % 2 ? xs1 : xs0) + wave / 2 * T;
#pragma unroll
    for (int k = 0; k < K; k++) {
        const int tile = mine + k;
        if (tile >= pc) {              // uniform
            if (lane == 0) tile_bits[wave * K + k] = 0;
            continue;
        }
        constexpr uint32_t FLAG_MASK = (1u << SIGMA) - 1;
        uint32_t nseg = walk_columns<SIGMA, VT>(dw[k] & FLAG_MASK, uint32_t(uint64_t(dw[k]) >> YSH), v[k], xv[k], yb, lane);
        if (nseg > uint32_t(T)) nseg = T;
        const bool dirty = (tp[k] & DIRTY) != 0;
        const uint32_t row0 = tp[k] & ROWMASK;
        const int32_t* eo_t = nullptr;
        if (dirty) {
            const int32_t e0 = eop[tile], e1 = eop[tile + 1];
            eo_t = eo + e0;
            if (nseg > uint32_t(e1 - e0)) nseg = uint32_t(e1 - e0);
        }
        wave_sync_lds();
        const bool cont0 = head[k] != 0, goes_on = head[k + 1] != 0;
        for (uint32_t s0 = 0; s0 < nseg; s0 += OMEGA) {
            const uint32_t sg = s0 + lane;
            if (sg < nseg) {
                const uint32_t row = row0 + (dirty ? uint32_t(eo_t[sg]) : sg);
                if (!(sg == 0 && cont0) && !(sg == nseg - 1 && goes_on) && row < uint32_t(m)) y[row] = yb[sg];
            }
        }
        if (lane == 0) {
            first_sum[wave * K + k] = nseg ? yb[0] : VT(0);
            last_sum[wave * K + k] = nseg ? yb[nseg - 1] : VT(0);
            tile_bits[wave * K + k] = 1u | (cont0 ? 2u : 0u) | (goes_on ? 4u : 0u) | (nseg == 1 ? 8u : 0u);
        }
        wave_sync_lds();
    }
    __syncthreads();
    if (wave != 0) return;

    // ---- rows that cross the workgroup's tiles, lane = tile: a tile inside a row passes
    // on what it got and its own sum
    const uint32_t bits = lane < TILES ? tile_bits[lane] : 0u;
    const bool live = bits & 1u, cont0 = bits & 2u, goes_on = bits & 4u, single = bits & 8u;
    const VT first = live ? first_sum[lane] : VT(0);
    const bool inside = live && single && cont0;                   // what it got goes through it
    VT sum = live ? (inside ? first : last_sum[lane]) : VT(0);
    const uint64_t begins = __ballot(live && !inside);
    const uint64_t upto = begins & (~0ull >> (OMEGA - 1 - lane));  // of the lanes up to this one
    const int from = upto ? OMEGA - 1 - __builtin_clzll(upto) : 0; // where the run of this lane begins
#pragma unroll
    for (int d = 1; d < OMEGA; d <<= 1) {
        const VT up = __shfl_up(sum, d, OMEGA);
        if (lane - d >= from) sum += up;
    }
    const VT before = __shfl_up(sum, 1, OMEGA);
    const VT total = lane > 0 ? before + first : first;
    const bool outside = cont0 && (begins & ((1ull << lane) - 1)) == 0;     // the row began before the workgroup
    const bool ends = cont0 && !(single && goes_on);
    const uint32_t my_row = live ? tile_ptr[tile0 + lane] & ROWMASK : 0u;
    if (ends && !outside && my_row < uint32_t(m)) y[my_row] = total;
    // what crosses the workgroup's own boundaries: at most one row at each
    const int lanes = __popcll(__ballot(live));
    const bool pub_in = (__ballot(cont0) & 1u) != 0;
    const bool pub_out = begins != 0 && ((__ballot(goes_on) >> (lanes - 1)) & 1u) != 0;
    if ((!WINDOW || meet) && !pub_in && !pub_out) return;
    const uint64_t ended = __ballot(ends && outside);
    const VT out_part = __shfl(sum, lanes - 1, OMEGA);
    const VT in_part = ended ? __shfl(total, __builtin_ctzll(ended), OMEGA) : out_part;
    if (WINDOW && !meet) {             // two kernels: to the auxiliary array, as the sum of the first tile
        if (live) carry[tile0 + lane] = lane == 0 && pub_in ? in_part : VT(0);
        if (lane == 0 && pub_out && row_out < uint32_t(m)) y[row_out] = out_part;
        return;
    }
    uint64_t other_in = MEET_EMPTY, other_out = MEET_EMPTY;
    uint32_t before_in = 0, before_out = 0;
    const bool count_row_in = pub_in && si.groups != 2, count_row_out = pub_out && so.groups != 2;
    if (lane == 0) {
        if (pub_in && !count_row_in) other_in = swap_in(meet_at(meet, si.first), meet_word(in_part));
        if (pub_out && !count_row_out) other_out = swap_in(meet_at(meet, group), meet_word(out_part));
        if (count_row_in) publish(carry + group, in_part);
        if (count_row_out) publish(meet_at(meet, group), meet_word(out_part));
        if (count_row_in || count_row_out) {
            wait_for_memory();
            if (count_row_in) before_in = count_in(arrived + si.first);
            if (count_row_out) before_out = count_in(arrived + group);
        }
        if (pub_in && !count_row_in && other_in != MEET_EMPTY) {
            if (row_in < uint32_t(m)) y[row_in] = meet_value<VT>(other_in) + in_part;
            publish(meet_at(meet, si.first), MEET_EMPTY);
        }
        if (pub_out && !count_row_out && other_out != MEET_EMPTY) {
            if (row_out < uint32_t(m)) y[row_out] = out_part + meet_value<VT>(other_out);
            publish(meet_at(meet, group), MEET_EMPTY);
        }
    }
    if (count_row_in && __shfl(before_in, 0, OMEGA) == uint32_t(si.groups - 1))
        assemble_row<VT>(carry, meet, arrived, si.first, si.first + si.groups - 1, y, row_in, m, lane);
    if (count_row_out && __shfl(before_out, 0, OMEGA) == uint32_t(so.groups - 1))
        assemble_row<VT>(carry, meet, arrived, group, group + so.groups - 1, y, row_out, m, lane);
}

// ----------------------------------------------------------------------------
// Second launch of an SpMV, needed only when some tile starts more than LOOK
// entries into a row: adds the carries (the global auxiliary array of Section 4).
// One thread per tile, tiles in order across the lanes.  Tiles whose first row
// is the same row R form a run (a row longer than a tile); a shuffle scan sums
// the carries of a run and its last lane adds the total to y[R], which already
// holds the part computed by the tile R starts in.  A run wholly inside one
// wavefront is a plain read-modify-write (nobody else touches y[R] now).  A run
// cut by a wavefront boundary uses atomic adds, which commute but arrive in any
// order, or, with FIXED, the wavefront that holds the run's first tile adds up the
// rest of the run by itself: the same bits on every call, for matrices that would
// have them from the one-launch form if their tiles were not taken by column
// (order_place).  The rest is usually shorter than a wavefront of tiles, which is
// asked for with the wavefront's own; beyond that it is a serial chain, RUN_AHEAD
// wavefronts of tiles per round trip.
// ----------------------------------------------------------------------------
constexpr int RUN_AHEAD = 16;

template <typename VT, typename IT, bool FIXED>
__global__ void __launch_bounds__(256)
k_spmv_fixup(int m, int ntiles,
             const typename Index<IT>::tp_t* __restrict__ tile_ptr, const VT* __restrict__ carry,
             VT* __restrict__ y, const uint32_t* __restrict__ status) {
    // rows are below 2^31 whatever the index width; 0xfff... marks "no tile"
    auto first_row = [&](int t) -> uint32_t {
        auto v = tile_ptr[t] & Index<IT>::ROWMASK;
        return v > 0x7fffffffu ? 0x7fffffffu : uint32_t(v);
    };
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = lane_id();
    const int t0 = gid - lane;                            // first tile of this wavefront
    const bool live = gid < ntiles;
    // Everything that does not depend on other loads is requested at once: the
    // kernel is a chain of memory round trips and nothing else.
    const uint32_t st = *status;
    const uint32_t R = live ? first_row(gid) : (0xfffffff0u - uint32_t(lane));
    VT cs = live ? carry[gid] : VT(0);
    const uint32_t r_after = (gid + 1 < ntiles) ? first_row(gid + 1) : 0xffffffffu;
    const uint32_t r_before = (t0 > 0 && t0 < ntiles) ? first_row(t0 - 1) : 0xffffffffu;
    uint32_t R2 = 0xffffffffu;                            // the next wavefront's tiles
    VT c2 = VT(0);
    if (FIXED && gid + OMEGA < ntiles) {
        R2 = first_row(gid + OMEGA);
        c2 = carry[gid + OMEGA];
    }
    if ((st & BAD_BITS) || t0 >= ntiles) return;
#pragma unroll
    for (int d = 1; d < OMEGA; d <<= 1) {
        VT up = __shfl_up(cs, d, OMEGA);
        uint32_t rup = __shfl_up(R, d, OMEGA);
        if (lane >= d && rup == R) cs += up;
    }
    const uint32_t rnext = __shfl_down(R, 1, OMEGA);
    const uint32_t rfirst = __shfl(R, 0, OMEGA);
    if constexpr (FIXED) {
        const uint32_t rlast = __shfl(R, OMEGA - 1, OMEGA);
        const bool began_before = rfirst == rlast && r_before == rlast;
        if (__shfl(r_after, OMEGA - 1, OMEGA) == rlast && !began_before) {      // uniform
            VT rest = R2 == rlast ? c2 : VT(0);
            bool goes_on = __shfl(R2, OMEGA - 1, OMEGA) == rlast;
            for (int t = t0 + 2 * OMEGA; goes_on; t += RUN_AHEAD * OMEGA) {     // behind the last tile every row is 0xfff...
                uint32_t r[RUN_AHEAD];
                VT c[RUN_AHEAD];
#pragma unroll
                for (int q = 0; q < RUN_AHEAD; q++) {
                    const int tile = t + q * OMEGA + lane;
                    r[q] = tile < ntiles ? first_row(tile) : 0xffffffffu;
                    c[q] = tile < ntiles ? carry[tile] : VT(0);
                }
#pragma unroll
                for (int q = 0; q < RUN_AHEAD; q++)
                    if (r[q] == rlast) rest += c[q];
                goes_on = __shfl(r[RUN_AHEAD - 1], OMEGA - 1, OMEGA) == rlast;
            }
            rest = wave_sum(rest);
            if (lane == OMEGA - 1) cs += rest;
        }
    }
    const bool run_end = live && ((lane == OMEGA - 1) || (rnext != R));
    if (run_end && cs != VT(0) && R < uint32_t(m)) {
        const bool ext_left = (rfirst == R) && (r_before == R);
        const bool ext_right = (lane == OMEGA - 1) && (r_after == R);
        if (FIXED) {
            if (!ext_left) y[R] += cs;                    // (else part of the wavefront's sum where the run begins)
        } else if (ext_left || ext_right) atomic_add_fp(&y[R], cs);
        else y[R] += cs;
    }
}

// ----------------------------------------------------------------------------
// Measurement aid: what the memory system charges for the tile kernel's streams
// alone.  One wavefront per complete tile, the same workgroup shape and tile
// order as the tile kernel's most common instantiation (by number also for a matrix
// that the tile kernel takes by column); it reads the tile's
// col_idx, val and descriptors with 16-byte non-temporal loads (all of a tile in
// flight at once up to sigma = 16) and, if asked, stores one value to every row
// the tile starts (the rows of y that tile's wavefront writes in an SpMV).  No
// gathers, no LDS, no arithmetic to speak of.
// ----------------------------------------------------------------------------
constexpr int FLOOR_WAVES = 4;
constexpr int FLOOR_LOADS = 12;            // 16-byte loads per lane and round

template <typename VT, typename IT>
__global__ void __launch_bounds__(FLOOR_WAVES * OMEGA)
k_stream_floor(int m, int pc, int sigma, int W, uint32_t nb_tiles, uint32_t xcd_chunk, int write_y,
               const typename Index<IT>::tp_t* __restrict__ tile_ptr, const uint32_t* __restrict__ tile_desc,
               const int32_t* __restrict__ col_idx, const VT* __restrict__ val, VT* __restrict__ y) {
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / OMEGA);
    const int tile = int(xcd_order(blockIdx.x, nb_tiles, xcd_chunk)) * FLOOR_WAVES + wave;
    if (tile >= pc) return;
    const int T = OMEGA * sigma;
    // the three streams of a tile as one sequence of 16-byte pieces
    const i32x4* c4 = reinterpret_cast<const i32x4*>(col_idx + size_t(tile) * T);
    const i32x4* v4 = reinterpret_cast<const i32x4*>(val + size_t(tile) * T);
    const i32x4* d4 = reinterpret_cast<const i32x4*>(tile_desc + size_t(tile) * W * OMEGA);
    const int n_c = T / 4, n_v = T * int(sizeof(VT)) / 16, n_d = W * OMEGA / 4;
    const int total = n_c + n_v + n_d;
    int32_t acc = 0;
    for (int base = 0; base < total; base += OMEGA * FLOOR_LOADS) {
        i32x4 r[FLOOR_LOADS];
#pragma unroll
        for (int u = 0; u < FLOOR_LOADS; u++) {
            const int idx = base + u * OMEGA + lane;
            const i32x4* src = idx < n_c ? c4 + idx : (idx < n_c + n_v ? v4 + (idx - n_c) : d4 + (idx - n_c - n_v));
            r[u] = i32x4{0, 0, 0, 0};
            if (idx < total) r[u] = __builtin_nontemporal_load(src);
        }
#pragma unroll
        for (int u = 0; u < FLOOR_LOADS; u++) acc ^= r[u].x ^ r[u].y ^ r[u].z ^ r[u].w;
    }
    if (write_y) {
        const uint32_t r0 = uint32_t(tile_ptr[tile] & Index<IT>::ROWMASK);
        uint32_t r1 = uint32_t(tile_ptr[tile + 1] & Index<IT>::ROWMASK);
        if (r1 > uint32_t(m)) r1 = uint32_t(m);
        for (uint32_t r = r0 + lane; r < r1; r += OMEGA) y[r] = VT(acc);
    } else if (acc == 0x5a17c0de) {
        y[0] = VT(acc);                    // keeps the loads alive; practically never taken (y is scratch here)
    }
}

// Whether the entries' x is gathered in pairs (gather_pairs), by a sample of neighbouring entries: of 100 of them, how many are
// one column on (blocks of 2 to 8 columns 50-87, 27-point stencil 67, 9-point 67, 5-point 40, all of which gain; 7-point 29, which
// gains 2 %; a star of 25 32, which loses 3 %), and how many a line of x and more (those 60-13; tridiagonal and five
// diagonals 0, which lose 5-7 %).  The sample is the window form's, so that matrices without it (window_fits: fewer than
// WINDOW_MIN_TILES tiles, other heights, an x below 80 KB or above WINDOW_MAX_X_BYTES) keep the gathers one by one.
constexpr uint32_t PAIR_NEXT_PERCENT = 36, PAIR_AWAY_PERCENT = 12;
inline bool pairs_pay(uint32_t sampled, uint32_t next, uint32_t away) {
    return sampled && next * 100 >= sampled * PAIR_NEXT_PERCENT && away * 100 >= sampled * PAIR_AWAY_PERCENT;
}

template <int SIGMA, typename VT, typename IT, int MODE>
hipError_t launch_spmv(bool keep, bool pairs, const Geom& g, int m, int n, IT nnz, const IT* row_ptr,
                       const typename Index<IT>::tp_t* tile_ptr,
                       const uint32_t* tile_desc, const IT* eop, const int32_t* eo,
                       const int32_t* col_idx, const VT* val, const VT* x, VT* y,
                       VT* carry, uint64_t* meet, uint32_t* arrived, const uint2* span, const uint32_t* status, const uint32_t* tile_head, const int32_t* last_col,
                       const VT* last_val, bool zero_rows, uint32_t far_mode,
                       const uint32_t* order, uint32_t order_second, uint32_t order_len, hipStream_t s) {
    constexpr int WAVES = TransposeShape<SIGMA>::WAVES;
    uint32_t nb_tiles = uint32_t((g.pc + WAVES - 1) / WAVES);
    if (MODE == MODE_CARRY && order) nb_tiles = (order_len + NUM_XCD * WAVES - 1) / (NUM_XCD * WAVES) * NUM_XCD;
    uint32_t has_tail = (int64_t(g.pc) * g.T < nnz) ? 1u : 0u;
    // rows without nonzeros: up to 512 workgroups stride over the rows
    size_t nb_zero = zero_rows ? (size_t(m) + WAVES * OMEGA - 1) / (WAVES * OMEGA) : 0;
    if (nb_zero > 512) nb_zero = 512;
    uint32_t nb = nb_tiles + has_tail + uint32_t(nb_zero);
    if (nb == 0) return hipSuccess;
    const size_t x_bytes = size_t(n) * sizeof(VT);
    uint32_t xcd_chunk = 0;                                        // contiguous eighths
    if (x_bytes > XCD_CONTIGUOUS_MAX_X_BYTES)                      // x too large for that to pay
        xcd_chunk = (int64_t(nnz) / (m > 0 ? m : 1) <= g.T / Y_LINE_ROWS) ? 1u : XCD_CHUNK;
    else if (x_bytes < XCD_CONTIGUOUS_MIN_X_BYTES)                 // x at home in every L2
        xcd_chunk = XCD_CHUNK;
    auto kernel = keep && rule_sigma(SIGMA) ? k_spmv<SIGMA, VT, IT, MODE, rule_sigma(SIGMA)> : k_spmv<SIGMA, VT, IT, MODE, false>;
    if constexpr (sizeof(VT) == 4 && rule_sigma(SIGMA) && MODE == MODE_LOOK)
        if (pairs) kernel = keep ? k_spmv<SIGMA, VT, IT, MODE, true, true> : k_spmv<SIGMA, VT, IT, MODE, false, true>;
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(WAVES * OMEGA), 0, s, m, int(x_bytes), nnz, g.pc, g.p, nb_tiles, has_tail,
                       xcd_chunk, far_mode, record_bytes(int64_t(nnz)), row_ptr, tile_ptr, tile_desc, eop, eo, col_idx, val, x, y, carry,
                       meet, arrived, span, status, tile_head, last_col, last_val, order, order_second, order_len);
    return hipGetLastError();
}

// The shapes of k_spmv_staged: as many tiles per wavefront as its registers hold.
constexpr int staged_most(int sigma, size_t value_bytes) { return sigma == RULE_SIGMA_SMALL ? (value_bytes == 8 ? 3 : 4) : 2; }
constexpr int staged_waves(int sigma, size_t value_bytes, int k) { return sigma == RULE_R && value_bytes == 8 && k == 2 ? 12 : 16; }
constexpr int STAGE_CUS = 256;
inline int staged_parts(int n, size_t value_bytes) { return int((int64_t(n) * int64_t(value_bytes) + STAGE_BYTES - 1) / STAGE_BYTES); }
inline int staged_rounds(const Geom& g, size_t value_bytes, int k) {       // of one workgroup per CU
    const int tiles = staged_waves(g.sigma, value_bytes, k) * k;
    return ((g.pc + tiles - 1) / tiles + (g.p > g.pc ? 1 : 0) + STAGE_CUS - 1) / STAGE_CUS;
}
// Tiles per wavefront for a matrix that may be one for k_spmv_staged, 0 for the others:
// the fewest that give the fewest rounds (8 M entries in single precision: 4 in one round 20.5 us, 2 in
// two 25.3, 3 in two 28.8).  Below STAGE_MIN_TILES too few CUs have work (1 M entries in
// rows of 100, x of 64 KB: 7.5 -> 8.3).
constexpr int STAGE_MIN_TILES = 3072;
constexpr int64_t STAGE_MIN_X = 16 << 10;
inline int staged_tiles(const Geom& g, int n, size_t value_bytes) {
    if (!rule_sigma(g.sigma) || g.p < STAGE_MIN_TILES || int64_t(n) * int64_t(value_bytes) < STAGE_MIN_X) return 0;
    int k = staged_most(g.sigma, value_bytes);
    const int fewest = staged_rounds(g, value_bytes, k);
    while (k > 1 && staged_rounds(g, value_bytes, k - 1) == fewest) k--;
    return k;
}
// The fewest entries that gather a line of their own for the kernel to pay.  What it costs is
// parts of x, one per round and STAGE_BYTES of x, 1.0-1.25 us each; such an entry costs k_spmv 3.4 us
// per million beyond its stream.  Measured at 1 to 28 M entries, x of 24 KB to 1.2 MB:
// with STAGE_MIN_ENTRIES per part it gains 8 % or more nearly everywhere (6 M entries, 15
// parts: 38.4 -> 35.3; 4 M in rows of 500, 10 parts: 25.1 -> 22.0), and what it passes by would gain no
// more (2 M, 6 parts: 14.6 -> 13.4) or lose (10 M, 15 parts in two rounds: 59.5 ->
// 66.5).  At height 16 in double precision several rounds cost more, there is no other workgroup to fill the
// gaps between them: 20 M entries, 6 parts in four rounds 98.1 -> 83.5, 12 parts 100.7 ->
// 115.6.
constexpr int64_t STAGE_MIN_ENTRIES = 400 * 1000, STAGE_MIN_ENTRIES_16 = 720 * 1000;
inline int64_t staged_min_entries(const Geom& g, int n, size_t value_bytes, int k) {
    const int rounds = staged_rounds(g, value_bytes, k);
    return int64_t(rounds) * staged_parts(n, value_bytes) * (g.sigma == RULE_R && value_bytes == 8 && rounds > 1 ? STAGE_MIN_ENTRIES_16 : STAGE_MIN_ENTRIES);
}

template <int SIGMA, int K, typename VT>
hipError_t launch_staged(const Geom& g, int m, int n, int nnz, const int32_t* row_ptr, const uint32_t* tile_ptr, const uint32_t* tile_desc,
                         const int32_t* eop, const int32_t* eo, const int32_t* col_idx, const VT* val, const VT* x, VT* y, VT* carry,
                         uint64_t* meet, uint32_t* arrived, const uint32_t* tile_head, bool zero_rows, hipStream_t s) {
    constexpr int WAVES = staged_waves(SIGMA, sizeof(VT), K);
    const uint32_t groups = uint32_t((g.pc + WAVES * K - 1) / (WAVES * K)), has_tail = g.p > g.pc ? 1u : 0u;
    const int bytes = n * int(sizeof(VT)), parts = staged_parts(n, sizeof(VT)), part_bytes = ((bytes + parts - 1) / parts + 1023) / 1024 * 1024;
    hipLaunchKernelGGL((k_spmv_staged<SIGMA, WAVES, K, FORM_PARTS, VT>), dim3(groups + has_tail), dim3(WAVES * OMEGA), 0, s, m, n, nnz, g.pc, groups, has_tail, zero_rows ? 1u : 0u,
                       part_bytes, parts, row_ptr, tile_ptr, tile_desc, eop, eo, col_idx, val, x, y, carry, meet, arrived, tile_head, 0.0f, FarEntries{});
    return hipGetLastError();
}

// The window form of k_spmv_staged: its shape, and the matrices it is for.  In entries per
// sample, rows of 8-16 entries unless said otherwise:
//  * At least half near the diagonal: with 0.7 4.8 M entries take 31.6 -> 28.7 us, with 0.4
//    32.2 -> 33.7, with 0.15 32.8 -> 38.9.
//  * Lines, of 128 entries near it in a tile: a band of +-1300 columns (0.67) 24 M 71.1 -> 71.2
//    and 3.6 M 15.4 -> 14.5, +-1600 (0.74) 76.0 -> 71.2, +-1000 (0.63) 67.0 -> 71.1; single
//    precision +-2000 58.9 -> 57.0, +-1600 54.3 -> 56.9; rows of 2000-4000 within +-5000 columns
//    (0.5) 103 -> 113.  Stencils have 0.25-0.4, and the L1 holds what they use.
//  * Tiles: below WINDOW_MIN_TILES of them some CUs have two workgroups and most have one
//    (mixed, 2.5 M entries 17.6 -> 18.0, 3.1 M 20.8 -> 21.3, 3.9 M 26.0 -> 22.9).
constexpr int WINDOW_WAVES = 8, WINDOW_MIN_TILES = 6400;
constexpr int64_t WINDOW_MAX_X_BYTES = 1 << 30;
static_assert(WINDOW_MAX_X_BYTES <= PAIR_NOWHERE, "gather_pairs");
constexpr uint32_t WINDOW_NEAR_PERCENT = 50, WINDOW_LINES_PERCENT = 70;
static_assert((WINDOW_WAVES & (WINDOW_WAVES - 1)) == 0, "window_sampled");
constexpr int window_tiles(int sigma) { return sigma == RULE_SIGMA_SMALL ? 2 : 1; }       // per wavefront
inline bool window_fits(const Geom& g, int n, size_t value_bytes) {
    const int64_t x_bytes = int64_t(n) * int64_t(value_bytes);
    return rule_sigma(g.sigma) && g.pc >= WINDOW_MIN_TILES && x_bytes >= WINDOW_BYTES && x_bytes <= WINDOW_MAX_X_BYTES;
}
inline bool window_pays(uint32_t samples, uint32_t near, uint32_t lines) {
    return near * 100 >= samples * WINDOW_NEAR_PERCENT && lines * 100 >= near * WINDOW_LINES_PERCENT;
}
// A band with entries elsewhere may suit both forms: a few of them make a tile wide for
// sample_columns.  A part costs a round about a microsecond whatever its entries are, the window's far
// entries 2 us per million, and one round of parts has 5.5 us less to wait for in front of it.  Parts, window, in
// us (k_spmv 24 to 57): 8.5 M entries in single precision, 2 rounds of 5 parts, a tenth far 33.7, 26.7,
// two fifths 33.5, 31.5; 12.7 M, 2 rounds of 8, a tenth 46.1, 33.4; 9.5 M in double precision, 2 rounds of 6, a fifth
// 40.7, 35.9, two fifths 40.5, 38.5 (left to the parts); 6.7 M, 2 rounds of 4, a tenth 28.9, 27.4, two
// fifths 28.8, 30.9; 4.3 M, one round of 6, a tenth 20.4, 21.2, two fifths 20.4, 23.8; 6 M in single
// precision, one round of 4, a tenth 17.5, 19.6.
inline bool window_rather(const Geom& g, int n, int64_t nnz, size_t value_bytes, int k, uint32_t far, uint32_t samples) {
    return 2 * (nnz * far / samples) + 5500 * 1000 < int64_t(staged_rounds(g, value_bytes, k)) * staged_parts(n, value_bytes) * 1000 * 1000;
}
template <int SIGMA, typename VT>
hipError_t launch_window(const Geom& g, int m, int n, int nnz, const int32_t* row_ptr, const uint32_t* tile_ptr, const uint32_t* tile_desc,
                         const int32_t* eop, const int32_t* eo, const int32_t* col_idx, const VT* val, const VT* x, VT* y, VT* carry,
                         uint64_t* meet, uint32_t* arrived, const uint32_t* tile_head, bool zero_rows, hipStream_t s) {
    constexpr int WAVES = WINDOW_WAVES, K = window_tiles(SIGMA), TILES = WAVES * K;
    const uint32_t groups = uint32_t((g.pc + TILES - 1) / TILES), has_tail = g.p > g.pc ? 1u : 0u;
    hipLaunchKernelGGL((k_spmv_staged<SIGMA, WAVES, K, FORM_WINDOW, VT>), dim3(groups + has_tail), dim3(WAVES * OMEGA), 0, s, m, n, nnz, g.pc, groups, has_tail, zero_rows ? 1u : 0u,
                       WINDOW_BYTES, 1, row_ptr, tile_ptr, tile_desc, eop, eo, col_idx, val, x, y, carry, meet, arrived, tile_head, float(n) / float(m), FarEntries{});
    return hipGetLastError();
}

// What a handle keeps for k_far_gather and FORM_FAR
struct FarPlan {
    void* tables;                          // hipMalloc'ed: what the conversion counts; released before it returns
    void* lists;                           // hipMalloc'ed: base, range, src, place, cols, the buffer; NULL: no plan
    FarShape shape;
    const uint32_t* base;
    const uint32_t* range;                 // per chunk: where the blocks' lists begin
    const uint32_t* src;
    const uint16_t* place;
    const uint16_t* cols;                  // in its block, of the buffer's entries
    char* values;                          // the buffer
    size_t values_bytes;
    std::mutex turn;                       // held while a product is enqueued: they go through the buffer one after the other,
    hipEvent_t done;                       // whatever their streams; behind the latest one's kernels
    int pieces;                            // workgroups per block
    int chunks;
    size_t first[FAR_MAX_CHUNKS + 1];      // of a chunk, in cols
    int end[FAR_MAX_CHUNKS];               // the segment that it ends before
};
// In how many products the plan has to come back, in what it costs a conversion and csr5_free (us per million
// entries, and in any case: allocation, release and waits, most of it the release of more than 64 MB) and gives a product (us per million
// entries further from their window than an L2 reaches).  Conversion and free longer by, product before -> after, hence back after so many
// products: mixed in double precision 34 M entries 540, 253 -> 170, 6.5 (not taken); 51 M 573, 405 -> 247, 3.6; 68 M 617, 556 -> 332, 2.8;
// 136 M 778, 1187 -> 688, 1.6; single precision 51 M 570, 313 -> 184, 4.4 (not taken); 68 M 614, 451 -> 234, 2.8; 136 M 764, 1020 -> 464, 1.4;
// random columns out of 3.3 M, 18 M entries 486, 297 -> 123, 2.8; out of 2 M, 30 M 531, 430 -> 191, 2.2; out of 4 M, 40 M 561, 682 -> 258, 1.3;
// single precision 555, 554 -> 167, 1.4.
// How many products follow is not known here; whoever makes fewer brings a workspace.
constexpr double FAR_PAYBACK = 4, FAR_COST = 450, FAR_COST_PER_M = 3.2, FAR_GAIN_PER_M = 8.5;
// Lines, of 100 entries far away (random columns 95-99, power-law ones 23-32; columns that all together are on fewer lines are in
// the caches), and tiles that spread them, of 100 (random 85-100; power-law columns and rows as long as several tiles 17).  Random
// ones over an x of 8 MB do not reach that: tiles at its ends have no 4 MB to spread over (2 M columns in single precision are
// left alone at 292 us a product, with the buffer 154).
constexpr uint32_t FAR_LINES_PERCENT = 85, FAR_SPREAD_PERCENT = 75;
// Near ones, of 100, for the window and the columns to be loaded.  48 M entries, a share near the diagonal, with the window
// and without: 0.1 356, 306 us; 0.3 326, 320; 0.4 269, 326; single precision 253, 205; 223, 204; 194, 203.
constexpr uint32_t FAR_WINDOW_PERCENT = 33;
inline bool far_pays(int64_t nnz, double far_share) {
    return FAR_COST + FAR_COST_PER_M * 1e-6 * double(nnz) <= FAR_PAYBACK * FAR_GAIN_PER_M * 1e-6 * double(nnz) * far_share;
}

// The caller holds plan.turn.
template <int SIGMA, typename VT>
hipError_t launch_far(const FarPlan& plan, const Geom& g, int m, int n, int nnz, const int32_t* row_ptr, const uint32_t* tile_ptr, const uint32_t* tile_desc,
                      const int32_t* eop, const int32_t* eo, const int32_t* col_idx, const VT* val, const VT* x, VT* y, VT* carry,
                      uint64_t* meet, uint32_t* arrived, const uint32_t* tile_head, bool zero_rows, hipStream_t s) {
    constexpr int WAVES = WINDOW_WAVES, K = window_tiles(SIGMA);
    static_assert(WAVES * K * SIGMA * OMEGA == FAR_ENTRIES && WAVES * OMEGA == FAR_THREADS, "a workgroup's entries");
    const FarShape& f = plan.shape;
    VT* const values = reinterpret_cast<VT*>(plan.values);
    hipError_t e = hipStreamWaitEvent(s, plan.done, 0);
    for (int c = 0, first = 0; c < plan.chunks && e == hipSuccess; c++) {
        hipLaunchKernelGGL(k_far_gather<VT>, dim3(uint32_t(f.blocks * plan.pieces)), dim3(FAR_GATHER_THREADS), 0, s, n, plan.pieces,
                           plan.range + size_t(c) * (f.blocks + 1), plan.cols + plan.first[c], x, values);
        const int last = c + 1 < plan.chunks ? plan.end[c] * FAR_SEGMENT : f.groups;
        const uint32_t has_tail = c == 0 && g.p > g.pc ? 1u : 0u;
        hipLaunchKernelGGL((f.window_bytes ? k_spmv_staged<SIGMA, WAVES, K, FORM_FAR, VT> : k_spmv_staged<SIGMA, WAVES, K, FORM_ALL, VT>), dim3(uint32_t(last - first) + has_tail), dim3(WAVES * OMEGA), 0, s, m, n, nnz, g.pc,
                           uint32_t(f.groups), has_tail, zero_rows ? 1u : 0u, f.window_bytes, 1, row_ptr, tile_ptr, tile_desc, eop, eo, col_idx, val, x, y, carry, meet,
                           arrived, tile_head, f.slope, FarEntries{first, last - first, plan.base, plan.src, plan.place, values, int(plan.values_bytes)});
        e = hipGetLastError();
        first = last;
    }
    return e;
}

template <int SIGMA, bool BACK, typename VT>
hipError_t launch_transpose(bool keep, const Geom& g, int n, int64_t nnz, int32_t* col_idx, VT* val,
                            uint32_t* status, int32_t* last_col, VT* last_val, const DescJob& job, hipStream_t s) {
    constexpr int WAVES = TransposeShape<SIGMA>::WAVES;
    uint32_t nb = uint32_t((g.pc + WAVES - 1) / WAVES);
    if (nb == 0) nb = BACK ? 0 : 1;   // forward pass still validates the tail's columns and collects the words of k_prepare
    if (nb == 0) return hipSuccess;
    const auto kernel = keep && rule_sigma(SIGMA) ? k_transpose<SIGMA, BACK, rule_sigma(SIGMA), VT> : k_transpose<SIGMA, BACK, false, VT>;
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(WAVES * OMEGA), 0, s, g.pc, n, nnz,
                       col_idx, val, status, last_col, last_val, record_bytes(nnz), job);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// CSR row-block baselines (Section 2.2.1), for the iteration-scenario comparison
// of Section 5.5: the cost of staying in CSR.  They read the untouched CSR
// arrays and have nothing to do with the CSR5 path.
//  * CSR-scalar (Algorithm 1): one thread per row.
//  * CSR-vector: LANES lanes per row (a power of two up to the wavefront),
//    lane-strided loads, shuffle reduction.
// ----------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_csr_scalar(int m, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
             const double* __restrict__ val, const double* __restrict__ x, double* __restrict__ y) {
    const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g >= int64_t(m)) return;
    const int r = int(g);
    double acc = 0.0;
    for (int k = row_ptr[r], e = row_ptr[r + 1]; k < e; k++) acc = fma(val[k], x[col_idx[k]], acc);
    y[r] = acc;
}

template <int LANES>
__global__ void __launch_bounds__(256)
k_csr_vector(int m, const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
             const double* __restrict__ val, const double* __restrict__ x, double* __restrict__ y) {
    const int64_t gid = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t r = gid / LANES;
    const int sub = int(gid % LANES);
    double acc = 0.0;
    if (r < int64_t(m))
        for (int64_t k = int64_t(row_ptr[r]) + sub, e = row_ptr[r + 1]; k < e; k += LANES)
            acc = fma(val[k], x[col_idx[k]], acc);
#pragma unroll
    for (int d = LANES / 2; d >= 1; d >>= 1) acc += __shfl_down(acc, d, LANES);
    if (r < int64_t(m) && sub == 0) y[r] = acc;
}

#define CSR5_FOR_SIGMA(X)                                                                          \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17)   \
    X(18) X(19) X(20) X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) X(32)      \
    X(33) X(34) X(35) X(36) X(37) X(38) X(39) X(40) X(41) X(42) X(43) X(44) X(45) X(46) X(47) X(48)

}  // namespace

// ----------------------------------------------------------------------------
// Scratch of csr5_spmv_static, the SpMV entry point that allocates nothing: the
// cross-tile auxiliary array lives here instead of in the handle.  Every GPU the
// library runs on holds its own copy of this array until the process ends.  In
// host code the array's NAME is only a stand-in; the memory is reached through
// the address hipGetSymbolAddress returns for the current device, resolved once
// per device (static_scratch) and passed to the kernels as an argument.
// ----------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[CSR5_STATIC_SCRATCH_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::atomic<void*> scratch_ptr[MAX_DEVICES];

// Address of `scratch` on device `dev`, which must be the current device.
// Threads that race here resolve the same address.
int static_scratch(int dev, void** out) {
    if (dev < 0 || dev >= MAX_DEVICES) return CSR5_ERANGE;
    void* p = scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return CSR5_EHIP;
        }
        scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return CSR5_OK;
}

}  // namespace

// ----------------------------------------------------------------------------
// handle
// ----------------------------------------------------------------------------
struct csr5_handle_s {
    int32_t m, n;
    int64_t nnz;
    Geom g;
    bool wide;             // 64-bit row_ptr, tile_ptr and empty_offset_ptr (csr5l_convert_ex)
    const void* row_ptr;   // int32_t* or int64_t*
    int32_t* col_idx;
    void* val;             // double* or float*, see dtype
    int dtype;             // CSR5_DTYPE_F64 / CSR5_DTYPE_F32
    void* tile_ptr;        // uint32_t* or uint64_t*
    uint32_t* tile_desc;
    void* eop;             // int32_t* or int64_t*
    int32_t* eo;
    uint32_t* status;
    // Cross-tile sums of an SpMV: one 8-byte entry per tile (incomplete one included),
    // CARRY_SLOTS such arrays taken in turn by successive calls, so that up to that
    // many SpMVs on one handle may be in flight at once (on different streams).
    void* carry;
    size_t carry_slot_bytes;
    std::atomic<uint32_t> carry_turn;      // SpMVs so far
    uint64_t number;       // of the handle, see use_latest
    std::atomic<bool> near;                // what reads the entries next has so far followed what wrote or read them last (keep_product)
    uint32_t* tile_head;   // per tile: entries of its first row that lie before it, saturated at 32 bits
    int aux_form;          // 0: the size rule decides how the auxiliary-array path adds its sums; 1: always the second kernel; 2: inside the tile kernel wherever span exists
    uint2* span;           // per tile: the groups of tiles that row touches (first, how many); NULL where the one-launch SpMV cannot run
    // CSR-order copy of the last LOOK entries of every tile group's last tile (NULL for
    // small and for large sigma): two views of one array of LAST_REC_BYTES-byte records
    int32_t* last_col;
    void* last_val;
    // The tile kernel's order of the tiles (order_place), in the place of the records; NULL: by number
    uint32_t* order;
    uint32_t order_second, order_len;
    int staged;            // tiles per wavefront of k_spmv_staged; 0: not for this matrix
    bool window;           // the window form of k_spmv_staged is for this matrix
    bool pairs;            // its entries' x may be gathered in pairs (gather_pairs)
    FarPlan far;           // lists != NULL: FORM_FAR is for this matrix
    void* owned;           // hipMalloc'ed block, or NULL when a workspace was given
    hipStream_t conv_stream;
    int device;            // HIP device that was current at conversion
    bool in_csr5_order;
    // The device-side status word once the host has read it (-1 before): tells
    // csr5_spmv* which launches this matrix needs.  Unknown means all of them.
    std::atomic<int32_t> status_host;
};

namespace {

constexpr int WORDS_RESERVED = 8192, ORDER_TOTAL_AT = WORDS_RESERVED - 2 * ORDER_BUCKETS;     // the sort's totals: the last of them
static_assert(PREP_TILE_WG + PREP_ROW_WG <= ORDER_TOTAL_AT, "words of k_prepare");

struct Layout {
    size_t off_tile_ptr, off_tile_head, off_span, off_desc, off_eop, off_eo, off_carry, off_last, off_scan, off_words, off_status, total;
    bool has_last;
    size_t ndesc, eo_cap, carry_slot_bytes;
};

Layout make_layout(int32_t m, int64_t nnz, const Geom& g, bool wide) {
    Layout L;
    const size_t isz = wide ? 8 : 4;   // bytes of one tile_ptr / empty_offset_ptr entry
    L.ndesc = size_t(g.pc) * g.W * OMEGA;
    size_t cap_a = size_t(m) + size_t(g.pc);
    size_t cap_b = size_t(g.pc) * g.T;
    L.eo_cap = cap_a < cap_b ? cap_a : cap_b;
    size_t o = 0;
    L.off_tile_ptr = o; o += align256((size_t(g.p) + 1) * isz);
    L.off_tile_head = o; o += align256((size_t(g.p) + 1) * 4);
    L.off_span = o;     o += one_launch_fits(g.sigma, g.p) ? align256((size_t(g.p) + 1) * 8) : 0;
    L.off_desc = o;     o += align256(L.ndesc * 4);
    L.off_eop = o;      o += align256((size_t(g.pc) + 1) * isz);
    L.off_eo = o;       o += align256(L.eo_cap * 4);
    // one slot per SpMV in flight: carry; where the one-launch form may run, also the meeting words and the counters
    L.carry_slot_bytes = align256((size_t(g.p) + 1) * 8);
    if (one_launch_fits(g.sigma, g.p)) L.carry_slot_bytes = slot_bytes_one(g, tile_group_waves(g.sigma));
    L.off_carry = o;    o += L.carry_slot_bytes * CARRY_SLOTS;
    L.has_last = look_sigma(g.sigma) && g.pc > 0;
    const size_t groups = (size_t(g.pc) + tile_group_waves(g.sigma) - 1) / tile_group_waves(g.sigma);
    L.off_last = o;     o += L.has_last ? align256(groups * size_t(record_bytes(nnz))) : 0;
    L.off_scan = o;     o += align256((size_t(g.pc) / SCAN_CHUNK + 1) * isz);   // chunk totals of the scan
    L.off_words = o;    o += size_t(WORDS_RESERVED) * 4;                          // one word per workgroup of k_prepare
    L.off_status = o;   o += 256;
    L.total = o;
    return L;
}

// Largest matrix the launches can address: one wavefront per tile and at most
// 2^32 - 1 threads in a grid; the row-parallel kernels add p_c threads to m, and
// all of them form m + 1 in 32 bits.
bool geometry_fits(int64_t m, int64_t nnz, int sigma) {
    if (m > int64_t(INT32_MAX) - 1) return false;
    const int64_t T = int64_t(OMEGA) * sigma;
    const int64_t p = (nnz + T - 1) / T;
    return p < (int64_t(1) << 26) - 4 && m + p < (int64_t(1) << 32) - 512;
}

}  // namespace

extern "C" {

const char* csr5_strerror(int code) {
    switch (code) {
        case CSR5_OK: return "ok";
        case CSR5_EINVAL: return "invalid argument";
        case CSR5_ENOMEM: return "out of memory or workspace too small";
        case CSR5_EHIP: return "HIP runtime error";
        case CSR5_ERANGE: return "sigma out of range, or matrix too large for the index width";
        default: return "unknown error";
    }
}

int32_t csr5_sigma_auto(int64_t nnz, int64_t m) {
    if (m <= 0 || nnz <= 0) return RULE_R;
    int64_t q = nnz / m;
    if (q > RULE_T) return RULE_U;
    int32_t sigma = q <= RULE_R ? RULE_R : (q <= RULE_S ? int32_t(q) : RULE_S);
    if (sigma > RULE_SIGMA_SMALL && nnz < RULE_MIN_TILES * OMEGA * sigma) sigma = RULE_SIGMA_SMALL;
    return sigma;
}

size_t csr5_workspace_bytes(int32_t m, int32_t nnz, int32_t sigma) {
    if (m < 0 || nnz < 0) return 0;
    if (sigma == 0) sigma = csr5_sigma_auto(nnz, m);
    if (sigma < CSR5_SIGMA_MIN || sigma > CSR5_SIGMA_MAX || !geometry_fits(m, nnz, sigma)) return 0;
    Geom g = make_geom(nnz, sigma);
    return make_layout(m, nnz, g, false).total;
}

size_t csr5l_workspace_bytes(int32_t m, int64_t nnz, int32_t sigma) {
    if (m < 0 || nnz < 0) return 0;
    if (sigma == 0) sigma = csr5_sigma_auto(nnz, m);
    if (sigma < CSR5_SIGMA_MIN || sigma > CSR5_SIGMA_MAX || !geometry_fits(m, nnz, sigma)) return 0;
    Geom g = make_geom(nnz, sigma);
    return make_layout(m, nnz, g, true).total;
}

}  // extern "C"

// The first `words` words at the handle's status word; notes the status for later calls.
static int read_status(csr5_handle_t h, uint32_t* got, int words) {
    if (hipMemcpyAsync(got, h->status, size_t(words) * 4, hipMemcpyDeviceToHost, h->conv_stream) != hipSuccess) return CSR5_EHIP;
    if (hipStreamSynchronize(h->conv_stream) != hipSuccess) return CSR5_EHIP;
    h->status_host.store(int32_t(got[0] & 0x7fffffffu), std::memory_order_relaxed);
    return CSR5_OK;
}

// Where the entries' next use is near, so that plain loads and stores leave them in the
// 256 MB memory-side cache for it instead of passing it by (the rule, see tile_buffer).  Near
// is what the order of the calls says: nothing else of the library was enqueued on the device in
// between (use_latest), and the stream is not being captured.
//  * The transposition, whose matrix is multiplied next, unless the call before was another
//    handle's conversion: several are converted first then.  One conversion, one product and the
//    way back, three matrices in turn, non-temporal throughout -> now: 100^3 stencil (318 MB) 319 -> 298 us,
//    90^3 246 -> 228, 75^3 162 -> 148, power-law of 2 M rows 245 -> 236, dense 4000^2 220 -> 203,
//    15 M random entries 370 -> 356.  With the product left non-temporal half of that or less
//    (100^3: 324), with only the stores or only the loads plain less or nothing.
//  * The product that follows it, if this handle's conversion was the call before.  Any first
//    product and any transposition plain: three matrices converted and then multiplied push each other
//    out, and the first product of each waits for the other ones' entries to be written (100^3 70 -> 86 us,
//    90^3 52 -> 67, power-law 66 -> 80; now 71, 55, 66).
//  * The second product in a row of a handle whose entries fit the L2s together brings them
//    there, where the later ones find them, plain or not: products 9 to 64 of dense 1500^2
//    9.4 -> 7.9, 40^3 6.6 -> 5.8, 1.2 M entries 10.4 -> 9.1.  With plain loads up to the eighth the same,
//    up to the 64th 40^3 5.6 and mixed of 1.7 M entries 11.2 -> 10.9, but power-law of 1.8 M 9.9 -> 11.0 and
//    45^3 7.7 -> 8.3.
//  * The way back is their last use: non-temporal, or it pushes out what comes next (75^3:
//    121 -> 134), except for the small, where the stores return sooner (dense 2000^2,
//    48 MB, 82 -> 76; 50^3, 40 MB, 55 -> 50; 60^3, 70 MB, 73.3 -> 72.1 but 78.9 with six
//    in turn).
// The upper line, entries with x and y: 387 MB (105^3) 336 -> 312 us, 409 MB (107^3) 380 -> 357,
// 390 MB (1.85 M rows, mixed) 539 -> 532, but 417 MB (power-law, 3.5 M rows) 399 -> 407, 445 MB
// (110^3) 381 -> 394, 570 MB (120^3) 487 -> 510.  The lower one, entries, the same cycle with one
// product: 20 MB (40^3) 63.5 -> 62.9, 27 MB (dense 1500^2) 70.9 -> 67.9, but 12 MB (dense 1000^2) 55.9 -> 58.4,
// 13 MB (35^3) 58.7 -> 60.1, 17 MB (dense 1200^2) 61.6 -> 64.1: what the transposition leaves in the
// L2s has to be written from there at its end.
// For the heights the automatic rule picks; the others keep one form, and so does k_spmv_staged (the
// product that follows a conversion, 12.6 M entries mixed 70.4 -> 78.3, in rows of 201 27.8 -> 28.0).
constexpr int64_t L2_BYTES = 32 << 20, KEEP_MIN_BYTES = 18 << 20, KEEP_MAX_BYTES = 384 << 20, KEEP_BACK_MAX_BYTES = 48 << 20;
static int64_t entry_bytes(int64_t nnz, size_t value_bytes) { return nnz * int64_t(value_bytes + 4); }
static bool keep_near(int32_t m, int32_t n, int64_t nnz, size_t value_bytes) {
    return entry_bytes(nnz, value_bytes) + (int64_t(m) + n) * int64_t(value_bytes) <= KEEP_MAX_BYTES;
}

// What the library enqueued last on a device: 2 * the handle's number, and 1 more if it was the
// handle's conversion.  Handles are numbered in the order of their conversions and no number is
// used twice.  Threads may race here: what they decide is a hint to the caches.
static std::atomic<uint64_t> handles_made, latest_use[MAX_DEVICES];
static uint64_t latest(int dev) { return dev >= 0 && dev < MAX_DEVICES ? latest_use[dev].load(std::memory_order_relaxed) : 0; }
static uint64_t use_latest(int dev, uint64_t use) {       // returns the one before
    const uint64_t before = latest(dev);
    if (before != use && dev >= 0 && dev < MAX_DEVICES) latest_use[dev].store(use, std::memory_order_relaxed);
    return before;
}

// A graph is replayed at any time, in turn with anything.  (An error is a capture elsewhere that forbids the question.)
static bool may_be_captured(hipStream_t s) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) == hipSuccess) return capture != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// before: what use_latest returned
static bool keep_product(csr5_handle_t h, uint32_t call, uint64_t before, hipStream_t s) {
    if (!h->near.load(std::memory_order_relaxed)) return false;
    const int64_t bytes = entry_bytes(h->nnz, h->dtype == CSR5_DTYPE_F32 ? 4 : 8);
    const bool soon = call == 0 ? bytes > KEEP_MIN_BYTES : call == 1 && bytes <= L2_BYTES;
    return soon && before / 2 == h->number && !may_be_captured(s);
}
static bool keep_back(int64_t nnz, size_t value_bytes) { return entry_bytes(nnz, value_bytes) > KEEP_MIN_BYTES && entry_bytes(nnz, value_bytes) <= KEEP_BACK_MAX_BYTES; }

// The plan of FORM_FAR.  Nothing is left where it does not pay or there is no memory for it.
static void far_release(csr5_handle_t h) {
    if (h->far.tables) (void)hipFree(h->far.tables);
    if (h->far.lists) (void)hipFree(h->far.lists);
    if (h->far.done) (void)hipEventDestroy(h->far.done);
    h->far.tables = h->far.lists = nullptr;
    h->far.done = nullptr;
}
static void* far_alloc(size_t bytes) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes) == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}
template <typename T>
static bool far_read(T* to, const T* from, int count, hipStream_t s) {
    return hipGetLastError() == hipSuccess && hipMemcpyAsync(to, from, count * sizeof(T), hipMemcpyDeviceToHost, s) == hipSuccess &&
           hipStreamSynchronize(s) == hipSuccess;
}
// Whether the plan is made; what was launched for it may still run if it is not.
template <int SIGMA, typename VT>
static bool far_make(csr5_handle_t h, hipStream_t s, int window_bytes, double far_share) {
    FarPlan& plan = h->far;
    FarShape& f = plan.shape;
    const int64_t x_bytes = int64_t(h->n) * int64_t(sizeof(VT));
    constexpr int tiles = FAR_ENTRIES / (SIGMA * OMEGA);
    f.pc = h->g.pc;
    f.n = h->n;
    f.groups = (h->g.pc + tiles - 1) / tiles;
    f.blocks = int((x_bytes + FAR_BLOCK_BYTES - 1) / FAR_BLOCK_BYTES);
    f.segments = (f.groups + FAR_SEGMENT - 1) / FAR_SEGMENT;
    f.window_bytes = window_bytes;
    f.slope = float(h->n) / float(h->m);
    const uint32_t* const tile_ptr = static_cast<const uint32_t*>(h->tile_ptr);
    uint32_t got[2];
    hipLaunchKernelGGL((k_far_sample<SIGMA, VT>), dim3(1), dim3(SCAN_THREADS), 0, s, f, tile_ptr, h->col_idx, h->status + FAR_ANSWER_AT);
    if (!far_read(got, h->status + FAR_ANSWER_AT, 2, s) || got[1] * 100 < got[0] * FAR_LINES_PERCENT) return false;
    const int most_chunks = far_chunks(uint32_t(h->nnz), sizeof(VT));
    const size_t counts_bytes = align256(size_t(f.groups) * f.blocks * 2), starts_bytes = align256(size_t(f.groups) * f.blocks * 4), sums_bytes = align256(size_t(f.segments) * f.blocks * 4);
    const size_t range_bytes = align256(size_t(most_chunks) * (f.blocks + 1) * 4), base_bytes = align256((size_t(f.groups) + 1) * 4), counted_bytes = align256(sizeof(FarCounted));
    const size_t tables_bytes = counts_bytes + starts_bytes + sums_bytes + range_bytes + base_bytes + counted_bytes;
    // not where it would take what the program may want itself: by what the sample says first, and by the counts
    size_t free_bytes = 0, device_bytes = 0;
    const double want = double(h->nnz) * far_share, want_buffer = want * sizeof(VT) < double(FAR_BUFFER_BYTES) ? want * sizeof(VT) : double(FAR_BUFFER_BYTES);
    if (hipMemGetInfo(&free_bytes, &device_bytes) != hipSuccess || tables_bytes + size_t(want * 8 + want_buffer) > free_bytes / 8) return false;
    plan.tables = far_alloc(tables_bytes);
    if (!plan.tables) return false;
    char* at = static_cast<char*>(plan.tables);
    FarCounted* const counted = reinterpret_cast<FarCounted*>(at);
    uint32_t* const base = reinterpret_cast<uint32_t*>(at += counted_bytes);
    uint32_t* const range = reinterpret_cast<uint32_t*>(at += base_bytes);
    uint32_t* const sums = reinterpret_cast<uint32_t*>(at += range_bytes);
    uint32_t* const starts = reinterpret_cast<uint32_t*>(at += sums_bytes);
    uint16_t* const counts = reinterpret_cast<uint16_t*>(at += starts_bytes);
    hipLaunchKernelGGL((k_far_count<SIGMA, VT>), dim3(uint32_t(f.groups)), dim3(FAR_THREADS), 0, s, f, tile_ptr, h->col_idx, counts, base);
    hipLaunchKernelGGL(k_far_segments, dim3(uint32_t(f.segments + 1)), dim3(SCAN_THREADS), 0, s, f, counts, sums, base, counted);
    hipLaunchKernelGGL(k_far_bases, dim3(uint32_t(most_chunks)), dim3(SCAN_THREADS), 0, s, f, int(sizeof(VT)), sums, range, base, counted);
    hipLaunchKernelGGL(k_far_starts, dim3(uint32_t(f.segments)), dim3(FAR_THREADS), 0, s, f, counts, sums, starts);
    FarCounted c;
    if (!far_read(&c, counted, 1, s)) return false;
    plan.chunks = far_chunks(c.total, sizeof(VT));
    plan.first[0] = 0;
    uint32_t most = 0;
    for (int k = 0; k < plan.chunks; k++) {
        plan.first[k + 1] = plan.first[k] + c.list[k];
        plan.end[k] = c.end[k];
        if (c.list[k] > most) most = c.list[k];
    }
    const size_t src_bytes = align256(size_t(c.total) * 4), place_bytes = align256(size_t(c.total) * 2), cols_bytes = align256(plan.first[plan.chunks] * 2);
    plan.values_bytes = align256(size_t(most) * sizeof(VT));
    const size_t bytes = base_bytes + range_bytes + src_bytes + place_bytes + cols_bytes + plan.values_bytes;
    if (plan.values_bytes > size_t(FAR_BUFFER_BYTES) || tables_bytes + bytes > free_bytes / 8) return false;
    if (hipEventCreateWithFlags(&plan.done, hipEventDisableTiming) != hipSuccess) {
        plan.done = nullptr;
        return false;
    }
    plan.lists = far_alloc(bytes);
    if (!plan.lists) return false;
    at = static_cast<char*>(plan.lists);
    plan.base = reinterpret_cast<uint32_t*>(at);
    plan.range = reinterpret_cast<uint32_t*>(at += base_bytes);
    uint32_t* const src = reinterpret_cast<uint32_t*>(at += range_bytes);
    uint16_t* const place = reinterpret_cast<uint16_t*>(at += src_bytes);
    uint16_t* const cols = reinterpret_cast<uint16_t*>(at += place_bytes);
    plan.values = at + cols_bytes;
    plan.src = src;
    plan.place = place;
    plan.cols = cols;
    plan.pieces = STAGE_CUS / f.blocks > 1 ? STAGE_CUS / f.blocks : 1;
    hipLaunchKernelGGL((k_far_place<SIGMA, VT>), dim3(uint32_t(f.groups)), dim3(FAR_THREADS), 0, s, f, tile_ptr, h->col_idx, counts, starts, counted, base, src, place, cols);
    if (hipGetLastError() != hipSuccess || hipMemcpyAsync(plan.lists, base, base_bytes + range_bytes, hipMemcpyDeviceToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) return false;
    (void)hipFree(plan.tables);
    plan.tables = nullptr;
    return true;
}
// near, far, spread: of `samples` entries, see WindowJob
template <typename VT>
static void far_plan(csr5_handle_t h, hipStream_t s, uint32_t samples, uint32_t near, uint32_t far, uint32_t spread) {
    const int64_t x_bytes = int64_t(h->n) * int64_t(sizeof(VT));
    if (x_bytes > int64_t(FAR_BLOCK_BYTES) * FAR_MAX_BLOCKS || spread * 100 < samples / (2 * OMEGA) * FAR_SPREAD_PERCENT ||
        !far_pays(h->nnz, double(far) / samples)) return;
    const int window = near * 100 >= samples * FAR_WINDOW_PERCENT ? WINDOW_BYTES : 0;
    const double share = window ? double(samples - near) / samples : 1.0;
    if (h->g.sigma == RULE_R ? far_make<RULE_R, VT>(h, s, window, share) : far_make<RULE_SIGMA_SMALL, VT>(h, s, window, share)) return;
    (void)hipGetLastError();
    (void)hipStreamSynchronize(s);         // before the memory goes
    far_release(h);
}

template <typename VT, typename IT>
static int convert_impl(int32_t m, int32_t n, IT nnz, const IT* row_ptr, int32_t* col_idx,
                        VT* val, int32_t sigma, void* workspace, size_t workspace_bytes,
                        void* hip_stream, uint32_t flags, csr5_handle_t* out) {
    using tp_t = typename Index<IT>::tp_t;
    constexpr bool wide = sizeof(IT) == 8;
    if (!out) return CSR5_EINVAL;
    *out = nullptr;
    if (m < 0 || n < 0 || nnz < 0) return CSR5_EINVAL;
    if (!row_ptr) return CSR5_EINVAL;                      // row_ptr has m+1 >= 1 entries
    if (nnz > 0 && (!col_idx || !val || m == 0 || n == 0)) return CSR5_EINVAL;
    // natural alignment of every element is all the kernels need
    if ((reinterpret_cast<uintptr_t>(col_idx) & 3) || (reinterpret_cast<uintptr_t>(val) & (sizeof(VT) - 1)) ||
        (reinterpret_cast<uintptr_t>(row_ptr) & (sizeof(IT) - 1))) return CSR5_EINVAL;
    if (sigma == 0) sigma = csr5_sigma_auto(nnz, m);
    if (sigma < CSR5_SIGMA_MIN || sigma > CSR5_SIGMA_MAX) return CSR5_ERANGE;
    if (!geometry_fits(m, nnz, sigma)) return CSR5_ERANGE;
    if ((flags & ~(CSR5_FLAG_NO_HOST_CHECK | CSR5_FLAG_AUX_TWO_KERNELS | CSR5_FLAG_AUX_ONE_KERNEL)) ||
        ((flags & CSR5_FLAG_AUX_TWO_KERNELS) && (flags & CSR5_FLAG_AUX_ONE_KERNEL))) return CSR5_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);

    Geom g = make_geom(nnz, sigma);
    Layout L = make_layout(m, nnz, g, wide);
    csr5_handle_s* h = new (std::nothrow) csr5_handle_s();
    if (!h) return CSR5_ENOMEM;
    char* basep = nullptr;
    if (workspace) {
        if (workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255)) {
            delete h;
            return workspace_bytes < L.total ? CSR5_ENOMEM : CSR5_EINVAL;
        }
        basep = static_cast<char*>(workspace);
        h->owned = nullptr;
    } else {
        void* ptr = nullptr;
        if (hipMalloc(&ptr, L.total) != hipSuccess) {
            (void)hipGetLastError();
            delete h;
            return CSR5_ENOMEM;
        }
        basep = static_cast<char*>(ptr);
        h->owned = ptr;
    }
    h->m = m; h->n = n; h->nnz = nnz; h->g = g; h->wide = wide;
    h->row_ptr = row_ptr; h->col_idx = col_idx; h->val = val;
    h->dtype = std::is_same<VT, float>::value ? CSR5_DTYPE_F32 : CSR5_DTYPE_F64;
    h->tile_ptr = basep + L.off_tile_ptr;
    h->tile_desc = reinterpret_cast<uint32_t*>(basep + L.off_desc);
    h->eop = basep + L.off_eop;
    h->eo = reinterpret_cast<int32_t*>(basep + L.off_eo);
    h->carry = basep + L.off_carry;
    h->carry_slot_bytes = L.carry_slot_bytes;
    h->carry_turn.store(0, std::memory_order_relaxed);
    h->tile_head = reinterpret_cast<uint32_t*>(basep + L.off_tile_head);
    h->aux_form = (flags & CSR5_FLAG_AUX_TWO_KERNELS) ? 1 : ((flags & CSR5_FLAG_AUX_ONE_KERNEL) ? 2 : 0);
    h->span = one_launch_fits(g.sigma, g.p) ? reinterpret_cast<uint2*>(basep + L.off_span) : nullptr;
    h->last_val = L.has_last ? basep + L.off_last : nullptr;                               // record + 0
    h->last_col = L.has_last ? reinterpret_cast<int32_t*>(basep + L.off_last + LOOK * 8) : nullptr;
    h->status = reinterpret_cast<uint32_t*>(basep + L.off_status);
    h->staged = 0;
    h->window = h->pairs = false;
    h->far.tables = h->far.lists = nullptr;
    h->far.done = nullptr;
    h->order = nullptr;
    h->order_second = h->order_len = 0;
    h->conv_stream = s;
    if (hipGetDevice(&h->device) != hipSuccess) {
        if (h->owned) (void)hipFree(h->owned);
        delete h;
        return CSR5_EHIP;
    }
    h->in_csr5_order = true;
    h->status_host.store(-1, std::memory_order_relaxed);
    h->number = handles_made.fetch_add(1, std::memory_order_relaxed) + 1;
    const bool among_conversions = use_latest(h->device, 2 * h->number + 1) & 1;
    const bool near = keep_near(m, n, nnz, sizeof(VT)) && !among_conversions && !may_be_captured(s);
    const bool keep = near && entry_bytes(nnz, sizeof(VT)) > KEEP_MIN_BYTES;
    h->near.store(near, std::memory_order_relaxed);
    {   // set-up time on this device: resolve the static scratch's address now, so
        // that csr5_spmv_static has nothing left to look up (failure is reported there)
        void* unused = nullptr;
        (void)static_scratch(h->device, &unused);
    }
    tp_t* const tile_ptr = static_cast<tp_t*>(h->tile_ptr);
    IT* const eop = static_cast<IT*>(h->eop);

    hipError_t e = hipSuccess;
    uint32_t* const words = reinterpret_cast<uint32_t*>(basep + L.off_words);
    // The tile order goes along with the scan where it may pay and the host will know of it (see below).  It sorts by
    // the tiles' first columns, which the transposition leaves in the first carry array, and takes the records' place.
    OrderJob order = {n, NUM_XCD * tile_group_waves(g.sigma), 0, nullptr, nullptr, nullptr, nullptr, h->status + 1};
    if (!(flags & CSR5_FLAG_NO_HOST_CHECK) && h->last_val && h->aux_form == 0 && g.pc >= ORDER_MIN_TILES &&
        size_t(n) * sizeof(VT) >= ORDER_MIN_X_BYTES) {
        order.slices = (g.pc + ORDER_SLICE - 1) / ORDER_SLICE < ORDER_MAX_SLICES ? (g.pc + ORDER_SLICE - 1) / ORDER_SLICE : ORDER_MAX_SLICES;
        order.first_col = static_cast<const int32_t*>(h->carry);
        order.total = words + ORDER_TOTAL_AT;
        order.order = static_cast<uint32_t*>(h->last_val);             // pc + align words
        order.base = order.order + g.pc + order.align;                 // 2 * ORDER_BUCKETS words per slice
        // the records are 24 words and more per tile: enough for the fewest tiles, and for every further slice
        constexpr int words_per_tile = NEAR_REC_BYTES / 4 / tile_group_waves(LOOK_MIN_SIGMA);
        static_assert(ORDER_MIN_TILES * words_per_tile >= ORDER_MIN_TILES + 64 + (ORDER_MIN_TILES / ORDER_SLICE + 1) * 2 * ORDER_BUCKETS &&
                      ORDER_SLICE * words_per_tile >= ORDER_SLICE + 2 * ORDER_BUCKETS, "list and bases in the records' place");
    }
    // Whether k_spmv_staged is for this matrix is looked up along with the scan where its size is right
    SampleJob sample = {nullptr, n, sigma, int(sizeof(VT)), h->status + 3};
    static_assert(STAGE_MIN_TILES >= SAMPLE_TILES && one_launch_fits(RULE_R, SCAN_SINGLE) && !one_launch_fits(RULE_R, SCAN_SINGLE + 1), "taken by k_scan_eop");
    const int staged = !wide && !(flags & CSR5_FLAG_NO_HOST_CHECK) && h->span && h->aux_form == 0 ? staged_tiles(g, n, sizeof(VT)) : 0;
    const int64_t staged_entries = staged ? staged_min_entries(g, n, sizeof(VT), staged) : 0;
    if (staged && int64_t(nnz) >= staged_entries && int64_t(n) * int64_t(sizeof(VT)) <= SAMPLE_MAX_LINES * 128) sample.col_idx = col_idx;
    WindowJob window = {nullptr, 0, WINDOW_WAVES * window_tiles(sigma), float(n) / float(m > 0 ? m : 1)};
    if (!wide && !(flags & CSR5_FLAG_NO_HOST_CHECK) && h->aux_form == 0 && window_fits(g, n, sizeof(VT))) {
        window.answer = h->status + WINDOW_ANSWER_AT;
        window.shift = window_shift(g.pc);
    }
    DescJob job = {m, wide ? 1 : 0, row_ptr, tile_ptr, h->tile_desc, eop, words, 0, 0, order.slices ? static_cast<int32_t*>(h->carry) : nullptr, window};
    {   // step 2a
        const size_t nb_tiles = (size_t(g.p) + 1 + PREP_THREADS - 1) / PREP_THREADS;
        const size_t nb_rows = (size_t(m) + PREP_THREADS * PREP_UNROLL - 1) / (PREP_THREADS * PREP_UNROLL);
        job.nb_tiles = int(nb_tiles < PREP_TILE_WG ? nb_tiles : PREP_TILE_WG);
        job.nb_rows = int(nb_rows < PREP_ROW_WG ? nb_rows : PREP_ROW_WG);
        hipLaunchKernelGGL(k_prepare<IT>, dim3(uint32_t(job.nb_tiles + job.nb_rows)), dim3(PREP_THREADS), 0, s, m, nnz, row_ptr, g.T, g.p, g.pc,
                           tile_group_waves(g.sigma), int64_t(nnz) <= LOOK_FAR_MAX_NNZ ? LOOK_MAX : LOOK, uint32_t(job.nb_tiles), tile_ptr,
                           h->tile_head, words,
                           reinterpret_cast<uint32_t*>(basep + L.off_carry + slot_off_arrived(g, tile_group_waves(g.sigma))),
                           reinterpret_cast<uint64_t*>(basep + L.off_carry + slot_off_meet(g)), L.carry_slot_bytes,
                           one_launch_fits(g.sigma, g.p) ? int(CARRY_SLOTS) : 0, reinterpret_cast<uint2*>(basep + L.off_span), h->status, order.total);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {            // steps 2b, 3a, 3b (descriptors, inside the same kernel) + 4
        switch (sigma) {
#define X(S) case S: e = launch_transpose<S, false, VT>(keep, g, n, nnz, col_idx, val, h->status, h->last_col,      \
                                                        static_cast<VT*>(h->last_val), job, s); break;
            CSR5_FOR_SIGMA(X)
#undef X
            default: e = hipErrorInvalidValue;
        }
    }
    if (e == hipSuccess && g.pc <= SCAN_SINGLE) {
        hipLaunchKernelGGL(k_scan_eop<IT>, dim3(1 + order.slices + (sample.col_idx ? 1 : 0)), dim3(SCAN_THREADS), 0, s,
                           g.pc, g.p, eop, tile_ptr, h->status, order, sample);
        e = hipGetLastError();
    } else if (e == hipSuccess) {
        IT* chunk_sum = reinterpret_cast<IT*>(basep + L.off_scan);
        const int nchunks = (g.pc + SCAN_CHUNK - 1) / SCAN_CHUNK;      // <= 2^26 / 2^13 = SCAN_CHUNK
        hipLaunchKernelGGL(k_scan_chunks<IT>, dim3(nchunks + order.slices), dim3(SCAN_THREADS), 0, s, g.pc, eop, chunk_sum,
                           tile_ptr, h->status, order);
        e = hipGetLastError();
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_scan_finish<IT>, dim3(nchunks), dim3(SCAN_THREADS), 0, s, g.pc, g.p, eop, chunk_sum,
                               tile_ptr, h->status);
            e = hipGetLastError();
        }
    }
    if (e == hipSuccess && g.pc > 0 && m > 0) {
        size_t threads = size_t(m) + size_t(g.pc);
        hipLaunchKernelGGL(k_empty_offset<IT>, dim3(uint32_t((threads + PLACE_THREADS - 1) / PLACE_THREADS) + uint32_t(order.slices)),
                           dim3(PLACE_THREADS), 0, s, m, row_ptr, g.sigma, g.T, g.W, g.pc, tile_ptr, h->tile_desc, eop, h->eo,
                           h->status, order);
        e = hipGetLastError();
    }
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(s);
        if (h->owned) (void)hipFree(h->owned);
        delete h;
        return CSR5_EHIP;
    }
    if (!(flags & CSR5_FLAG_NO_HOST_CHECK)) {
        // blocking variant: wait for the device-side verdict; on bad input undo the
        // transposition and refuse
        uint32_t got[WINDOW_ANSWER_AT + 3] = {};      // the status word, behind it the plan of the tile order and the answers on the columns
        int rc = read_status(h, got, window.answer ? WINDOW_ANSWER_AT + 3 : (sample.col_idx ? 4 : (order.slices ? 3 : 1)));
        if (rc == CSR5_OK && got[2]) {
            h->order = order.order;
            h->order_second = got[1];
            h->order_len = got[2];
        }
        const uint32_t samples = window.answer ? window_samples(window, g.pc) : 0u, near = got[WINDOW_ANSWER_AT] >> 16, lines = got[WINDOW_ANSWER_AT] & 0xffffu;
        h->window = rc == CSR5_OK && window.answer && !h->order && window_pays(samples, near, lines);
        if (rc == CSR5_OK && got[3] && int64_t(nnz) * got[3] >= staged_entries * SAMPLES &&
            !(h->window && window_rather(g, n, int64_t(nnz), sizeof(VT), staged, samples - near, samples))) {
            h->staged = staged;
            h->window = false;
        }
        if constexpr (!wide) {
            if (rc == CSR5_OK && !(got[0] & BAD_BITS) && window.answer && h->owned && !h->order && !h->staged)
                far_plan<VT>(h, s, samples, near, got[WINDOW_ANSWER_AT + 1] >> 16, got[WINDOW_ANSWER_AT + 1] & 0xffffu);
            // (the instantiation with the look-behind only)
            h->pairs = rc == CSR5_OK && sizeof(VT) == 4 && h->last_col && !(got[0] & STATUS_NEEDS_CARRY) && !h->staged && !h->window && !h->far.lists &&
                       pairs_pay(samples / 2, got[WINDOW_ANSWER_AT + 2] >> 16, got[WINDOW_ANSWER_AT + 2] & 0xffffu);
        }
        if (rc == CSR5_OK && (got[0] & BAD_BITS)) {
            (void)csr5_to_csr(h, hip_stream);
            (void)hipStreamSynchronize(s);
            rc = CSR5_EINVAL;
        }
        if (rc != CSR5_OK) {
            if (h->owned) (void)hipFree(h->owned);
            delete h;
            return rc;
        }
    }
    *out = h;
    return CSR5_OK;
}

extern "C" {

int csr5_convert_ex(int32_t m, int32_t n, int32_t nnz, const int32_t* row_ptr, int32_t* col_idx,
                    double* val, int32_t sigma, void* workspace, size_t workspace_bytes,
                    void* hip_stream, uint32_t flags, csr5_handle_t* out) {
    return convert_impl<double, int32_t>(m, n, nnz, row_ptr, col_idx, val, sigma, workspace, workspace_bytes,
                                         hip_stream, flags, out);
}

int csr5l_convert_ex(int32_t m, int32_t n, int64_t nnz, const int64_t* row_ptr, int32_t* col_idx,
                     double* val, int32_t sigma, void* workspace, size_t workspace_bytes,
                     void* hip_stream, uint32_t flags, csr5_handle_t* out) {
    return convert_impl<double, int64_t>(m, n, nnz, row_ptr, col_idx, val, sigma, workspace, workspace_bytes,
                                         hip_stream, flags, out);
}

int csr5s_convert_ex(int32_t m, int32_t n, int32_t nnz, const int32_t* row_ptr, int32_t* col_idx,
                     float* val, int32_t sigma, void* workspace, size_t workspace_bytes,
                     void* hip_stream, uint32_t flags, csr5_handle_t* out) {
    return convert_impl<float, int32_t>(m, n, nnz, row_ptr, col_idx, val, sigma, workspace, workspace_bytes,
                                        hip_stream, flags, out);
}

int csr5_convert(int32_t m, int32_t n, int32_t nnz, const int32_t* row_ptr, int32_t* col_idx,
                 double* val, csr5_handle_t* out) {
    return csr5_convert_ex(m, n, nnz, row_ptr, col_idx, val, 0, nullptr, 0, nullptr, CSR5_FLAG_NONE, out);
}

}  // extern "C"

// One SpMV: the tile kernel, then the carry fix-up if this matrix needs it.
// `which` selects the launches (measurement only): bit 0 the tile kernel, bit 1
// the fix-up.
constexpr int LAUNCH_TILES = 1, LAUNCH_FIXUP = 2, LAUNCH_BOTH = 3;

// Whether a product on the stream has far entries' x gathered into the handle's buffer.  Not one that is captured: its replays
// cannot be ordered with the handle's other products.
static bool gathered(csr5_handle_t h, hipStream_t s) { return h->far.lists && !may_be_captured(s); }

template <typename VT, typename IT>
static int spmv_launch_it(csr5_handle_t h, const VT* x, VT* y, hipStream_t s, int which, void* carry_mem) {
    using tp_t = typename Index<IT>::tp_t;
    const IT* row_ptr = static_cast<const IT*>(h->row_ptr);
    const tp_t* tile_ptr = static_cast<const tp_t*>(h->tile_ptr);
    const IT* eop = static_cast<const IT*>(h->eop);
    hipError_t e = hipSuccess;
    // a whole SpMV takes the next of the handle's carry arrays; partial launches (measurement) the first
    const uint32_t call = (which == LAUNCH_BOTH) ? h->carry_turn.fetch_add(1, std::memory_order_relaxed) : 0u, turn = call % CARRY_SLOTS;
    const uint64_t before = use_latest(h->device, 2 * h->number);
    const bool keep = which == LAUNCH_BOTH && keep_product(h, call, before, s);
    if (before / 2 != h->number) h->near.store(false, std::memory_order_relaxed);
    VT* carry = static_cast<VT*>(carry_mem ? carry_mem : static_cast<void*>(static_cast<char*>(h->carry) + turn * h->carry_slot_bytes));
    // What the matrix needs beyond its tiles is known once the host has seen the
    // status word of the conversion; until then everything is launched (the
    // kernels look at the status word themselves and return at once if idle).
    const int32_t known = h->status_host.load(std::memory_order_relaxed);
    const bool zero_rows = known < 0 || (uint32_t(known) & CSR5_STATUS_HAS_EMPTY_ROWS);
    const bool carries = known < 0 || (uint32_t(known) & STATUS_NEEDS_CARRY) || !h->last_col;
    // the instantiation without the look-behind when the matrix is known not to use it
    const bool can_look = h->last_col && (known < 0 || !(uint32_t(known) & STATUS_NEEDS_CARRY));
    // can the look-behind of this matrix need the far part of the records
    const uint32_t far_mode = (known < 0 || (uint32_t(known) & STATUS_FAR_HEADS)) ? 1u : 0u;
    // The auxiliary-array path in one launch: when the matrix is known to take that
    // path, is small enough for it to pay, and the call uses the handle's own slot
    // (whose counters the conversion cleared).
    const bool one_pays = h->g.p <= ONE_LAUNCH_ANY_TILES || h->nnz / (h->m > 0 ? h->m : 1) < ONE_LAUNCH_SHORT_ROWS;
    const bool one = !carry_mem && known >= 0 && !can_look && h->span && !h->order &&
                     (h->aux_form == 2 || (h->aux_form == 0 && one_pays));
    // A matrix whose tiles are taken by column and that would take that form otherwise has its sums added in a fixed
    // order as well (second kernel 2.8 us either way).  Not where two kernels are the rule anyway: a row of 29 000 tiles
    // took the chain 70 us with RUN_AHEAD = 8, the atomics 7.5.
    const bool fixed = h->order && h->span && one_pays;
    uint64_t* const meet = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(carry) + slot_off_meet(h->g));
    uint32_t* const arrived = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(carry) + slot_off_arrived(h->g, tile_group_waves(h->g.sigma)));
#define ARGS keep, h->pairs, h->g, h->m, h->n, IT(h->nnz), row_ptr, tile_ptr, h->tile_desc, eop, h->eo, h->col_idx,              \
             static_cast<const VT*>(h->val), x, y, carry, meet, arrived, h->span, h->status, h->tile_head, h->last_col, \
             static_cast<const VT*>(h->last_val), zero_rows, far_mode, h->order, h->order_second, h->order_len, s
    // x through LDS: one launch, which wants the handle's own slot like the one-launch form
    if constexpr (std::is_same<IT, int32_t>::value) {
        if (h->staged && !carry_mem) {
            if (!(which & LAUNCH_TILES)) return CSR5_OK;
#define STAGED(S, K) e = launch_staged<S, K, VT>(h->g, h->m, h->n, int(h->nnz), row_ptr, tile_ptr, h->tile_desc, eop, h->eo, h->col_idx, \
                                               static_cast<const VT*>(h->val), x, y, carry, meet, arrived, h->tile_head, zero_rows, s)
            if (h->g.sigma == RULE_R) {
                if (h->staged == 1) STAGED(RULE_R, 1);
                else STAGED(RULE_R, 2);
            } else if (h->staged == 1) STAGED(RULE_SIGMA_SMALL, 1);
            else if (h->staged == 2) STAGED(RULE_SIGMA_SMALL, 2);
            else if (h->staged == 3) STAGED(RULE_SIGMA_SMALL, 3);
            else if constexpr (staged_most(RULE_SIGMA_SMALL, sizeof(VT)) >= 4) STAGED(RULE_SIGMA_SMALL, 4);
#undef STAGED
            return e == hipSuccess ? CSR5_OK : CSR5_EHIP;
        }
    }
    // a window of x in LDS: one launch where the handle's slot has what that wants, otherwise two
    bool window = false, window_one = false, in_turn = false;
    std::unique_lock<std::mutex> far_turn(h->far.turn, std::defer_lock);
    if constexpr (std::is_same<IT, int32_t>::value) {
        const bool far = !carry_mem && gathered(h, s);
        in_turn = far && (which & LAUNCH_TILES);
        if (in_turn) far_turn.lock();
        window = h->window || far;
        window_one = window && h->span && !carry_mem;
        if (in_turn) {
#define FARRED(S) e = launch_far<S, VT>(h->far, h->g, h->m, h->n, int(h->nnz), row_ptr, tile_ptr, h->tile_desc, eop, h->eo, h->col_idx,            \
                                      static_cast<const VT*>(h->val), x, y, carry, window_one ? meet : nullptr, arrived, h->tile_head, zero_rows, s)
            if (h->g.sigma == RULE_R) FARRED(RULE_R);
            else FARRED(RULE_SIGMA_SMALL);
#undef FARRED
        } else if (window && (which & LAUNCH_TILES)) {
#define WINDOWED(S) e = launch_window<S, VT>(h->g, h->m, h->n, int(h->nnz), row_ptr, tile_ptr, h->tile_desc, eop, h->eo, h->col_idx,            \
                                             static_cast<const VT*>(h->val), x, y, carry, window_one ? meet : nullptr, arrived, h->tile_head, zero_rows, s)
            if (h->g.sigma == RULE_R) WINDOWED(RULE_R);
            else WINDOWED(RULE_SIGMA_SMALL);
#undef WINDOWED
        }
    }
    if ((which & LAUNCH_TILES) && !window) {
#define X(S) case S:                                                                                  \
        if (look_sigma(S) && can_look) e = launch_spmv<S, VT, IT, look_sigma(S) ? MODE_LOOK : MODE_CARRY>(ARGS); \
        else if (look_sigma(S) && one) e = launch_spmv<S, VT, IT, look_sigma(S) ? MODE_ONE : MODE_CARRY>(ARGS);  \
        else e = launch_spmv<S, VT, IT, MODE_CARRY>(ARGS);                                            \
        break;
        switch (h->g.sigma) {
            CSR5_FOR_SIGMA(X)
            default: e = hipErrorInvalidValue;
        }
#undef X
#undef ARGS
    }
    if (e != hipSuccess) {
        if (in_turn) (void)hipStreamSynchronize(s);       // what was launched may use the buffer
        return CSR5_EHIP;
    }
    if ((which & LAUNCH_FIXUP) && (window ? !window_one : carries && !one) && h->g.p > 0) {
        int ntiles = h->g.p;                                  // one thread per tile
        size_t nb = (size_t(ntiles) + 255) / 256;
        hipLaunchKernelGGL((fixed ? k_spmv_fixup<VT, IT, true> : k_spmv_fixup<VT, IT, false>), dim3(uint32_t(nb)), dim3(256), 0, s,
                           h->m, ntiles, tile_ptr, carry, y, h->status);
        if (hipGetLastError() != hipSuccess) return CSR5_EHIP;
    }
    // (where the event cannot be recorded, the next product could not be made to wait: this one does)
    if (in_turn && hipEventRecord(h->far.done, s) != hipSuccess && hipStreamSynchronize(s) != hipSuccess) return CSR5_EHIP;
    return CSR5_OK;
}

// The 64-bit index variant exists for double only.
template <typename VT>
static int spmv_launch(csr5_handle_t h, const VT* x, VT* y, hipStream_t s, int which = LAUNCH_BOTH,
                       void* carry_mem = nullptr) {
    if constexpr (std::is_same<VT, double>::value) {
        if (h->wide) return spmv_launch_it<double, int64_t>(h, x, y, s, which, carry_mem);
    }
    if (h->wide) return CSR5_EINVAL;
    return spmv_launch_it<VT, int32_t>(h, x, y, s, which, carry_mem);
}

template <typename VT>
static int spmv_checked(csr5_handle_t h, const VT* x, VT* y, void* hip_stream, bool static_carry = false) {
    constexpr int want = std::is_same<VT, float>::value ? CSR5_DTYPE_F32 : CSR5_DTYPE_F64;
    if (!h || !h->in_csr5_order || h->dtype != want) return CSR5_EINVAL;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return CSR5_EHIP;
    if (dev != h->device) return CSR5_EINVAL;              // the handle's arrays live on another device
    if (h->m > 0 && !y) return CSR5_EINVAL;
    if (h->nnz > 0 && !x) return CSR5_EINVAL;
    void* carry_mem = nullptr;
    if (static_carry) {
        // one 8-byte slot per tile, the incomplete one included, in the static array
        if ((size_t(h->g.p) + 1) * 8 > size_t(CSR5_STATIC_SCRATCH_BYTES)) return CSR5_ERANGE;
        const int rc = static_scratch(dev, &carry_mem);
        if (rc != CSR5_OK) return rc;
    }
    if (h->m == 0) return CSR5_OK;
    return spmv_launch<VT>(h, x, y, static_cast<hipStream_t>(hip_stream), LAUNCH_BOTH, carry_mem);
}

template <typename VT>
static int spmv_profile(csr5_handle_t h, const VT* x, VT* y, void* hip_stream, int reps, float* ms) {
    constexpr int want = std::is_same<VT, float>::value ? CSR5_DTYPE_F32 : CSR5_DTYPE_F64;
    if (!h || !h->in_csr5_order || h->dtype != want || !ms || reps <= 0 || reps > 100000) return CSR5_EINVAL;
    if (h->m == 0 || !y || (h->nnz > 0 && !x)) return CSR5_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    // Each kernel is launched `reps` times in a row between two events: consecutive
    // launches hide each other's dispatch latency, so elapsed / reps is the kernel's
    // duration (an event pair around a single launch would add that latency).
    // What the repeated launches leave in y is overwritten by the full SpMV at the end.
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    int rc = CSR5_OK;
    for (int k = 0; k < 3 && rc == CSR5_OK; k++)
        if (hipEventCreate(&ev[k]) != hipSuccess) rc = CSR5_EHIP;
    if (rc == CSR5_OK && hipEventRecord(ev[0], s) != hipSuccess) rc = CSR5_EHIP;
    for (int r = 0; rc == CSR5_OK && r < reps; r++) rc = spmv_launch<VT>(h, x, y, s, LAUNCH_TILES);
    if (rc == CSR5_OK && hipEventRecord(ev[1], s) != hipSuccess) rc = CSR5_EHIP;
    for (int r = 0; rc == CSR5_OK && r < reps; r++) rc = spmv_launch<VT>(h, x, y, s, LAUNCH_FIXUP);
    if (rc == CSR5_OK && hipEventRecord(ev[2], s) != hipSuccess) rc = CSR5_EHIP;
    if (rc == CSR5_OK) rc = spmv_launch<VT>(h, x, y, s);
    if (hipStreamSynchronize(s) != hipSuccess && rc == CSR5_OK) rc = CSR5_EHIP;
    float a = 0.f, b = 0.f;
    if (rc == CSR5_OK && (hipEventElapsedTime(&a, ev[0], ev[1]) != hipSuccess ||
                          hipEventElapsedTime(&b, ev[1], ev[2]) != hipSuccess))
        rc = CSR5_EHIP;
    for (int k = 0; k < 3; k++)
        if (ev[k]) (void)hipEventDestroy(ev[k]);
    if (rc == CSR5_OK) {
        ms[0] = a / float(reps);   // tile kernel
        ms[1] = b / float(reps);   // carry fix-up
    }
    return rc;
}

template <typename VT, typename IT>
static int stream_floor(csr5_handle_t h, VT* y, hipStream_t s, int reps, float* ms) {
    using tp_t = typename Index<IT>::tp_t;
    const Geom& g = h->g;
    const uint32_t nb_tiles = uint32_t((g.pc + FLOOR_WAVES - 1) / FLOOR_WAVES);
    // the SpMV's order by number for this matrix
    const size_t x_bytes = size_t(h->n) * sizeof(VT);
    uint32_t xcd_chunk = 0;
    if (x_bytes > XCD_CONTIGUOUS_MAX_X_BYTES)
        xcd_chunk = (h->nnz / (h->m > 0 ? h->m : 1) <= g.T / Y_LINE_ROWS) ? 1u : XCD_CHUNK;
    else if (x_bytes < XCD_CONTIGUOUS_MIN_X_BYTES)
        xcd_chunk = XCD_CHUNK;
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    int rc = CSR5_OK;
    for (int k = 0; k < 3 && rc == CSR5_OK; k++)
        if (hipEventCreate(&ev[k]) != hipSuccess) rc = CSR5_EHIP;
    for (int pass = 0; pass < 2 && rc == CSR5_OK; pass++) {      // reads only, then reads and the rows of y
        if (hipEventRecord(ev[pass], s) != hipSuccess) rc = CSR5_EHIP;
        for (int r = 0; rc == CSR5_OK && r < reps; r++) {
            hipLaunchKernelGGL((k_stream_floor<VT, IT>), dim3(nb_tiles), dim3(FLOOR_WAVES * OMEGA), 0, s, h->m, g.pc,
                               g.sigma, g.W, nb_tiles, xcd_chunk, pass, static_cast<const tp_t*>(h->tile_ptr),
                               h->tile_desc, h->col_idx, static_cast<const VT*>(h->val), y);
            if (hipGetLastError() != hipSuccess) rc = CSR5_EHIP;
        }
    }
    if (rc == CSR5_OK && hipEventRecord(ev[2], s) != hipSuccess) rc = CSR5_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess && rc == CSR5_OK) rc = CSR5_EHIP;
    float a = 0.f, b = 0.f;
    if (rc == CSR5_OK && (hipEventElapsedTime(&a, ev[0], ev[1]) != hipSuccess ||
                          hipEventElapsedTime(&b, ev[1], ev[2]) != hipSuccess))
        rc = CSR5_EHIP;
    for (int k = 0; k < 3; k++)
        if (ev[k]) (void)hipEventDestroy(ev[k]);
    if (rc == CSR5_OK) {
        ms[0] = a / float(reps);
        ms[1] = b / float(reps);
    }
    return rc;
}

extern "C" {

int csr5_stream_floor(csr5_handle_t h, void* y, size_t y_bytes, void* hip_stream, int reps, float* ms) {
    if (!h || !h->in_csr5_order || !y || !ms || reps <= 0 || reps > 100000) return CSR5_EINVAL;
    if (h->g.pc == 0 || h->m == 0) return CSR5_EINVAL;                     // no complete tile: nothing to stream
    if (y_bytes < size_t(h->m) * (h->dtype == CSR5_DTYPE_F32 ? 4 : 8)) return CSR5_EINVAL;
    if ((reinterpret_cast<uintptr_t>(h->col_idx) & 15) || (reinterpret_cast<uintptr_t>(h->val) & 15)) return CSR5_EINVAL;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return CSR5_EHIP;
    if (dev != h->device) return CSR5_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (h->dtype == CSR5_DTYPE_F32) return h->wide ? CSR5_EINVAL : stream_floor<float, int32_t>(h, static_cast<float*>(y), s, reps, ms);
    return h->wide ? stream_floor<double, int64_t>(h, static_cast<double*>(y), s, reps, ms)
                   : stream_floor<double, int32_t>(h, static_cast<double*>(y), s, reps, ms);
}

int csr5_spmv_ex(csr5_handle_t h, const double* x, double* y, void* hip_stream) {
    return spmv_checked<double>(h, x, y, hip_stream);
}
int csr5_spmv(csr5_handle_t h, const double* x, double* y) { return spmv_checked<double>(h, x, y, nullptr); }
int csr5_spmv_static(csr5_handle_t h, const double* x, double* y, void* hip_stream) {
    return spmv_checked<double>(h, x, y, hip_stream, true);
}
int csr5s_spmv_ex(csr5_handle_t h, const float* x, float* y, void* hip_stream) {
    return spmv_checked<float>(h, x, y, hip_stream);
}
int csr5_spmv_profile(csr5_handle_t h, const double* x, double* y, void* hip_stream, int reps, float* ms) {
    return spmv_profile<double>(h, x, y, hip_stream, reps, ms);
}
int csr5s_spmv_profile(csr5_handle_t h, const float* x, float* y, void* hip_stream, int reps, float* ms) {
    return spmv_profile<float>(h, x, y, hip_stream, reps, ms);
}

int csr5_to_csr(csr5_handle_t h, void* hip_stream) {
    if (!h) return CSR5_EINVAL;
    if (!h->in_csr5_order) return CSR5_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipSuccess;
    const bool keep = keep_back(h->nnz, h->dtype == CSR5_DTYPE_F32 ? 4 : 8);
    (void)use_latest(h->device, 2 * h->number);
    if (h->nnz > 0) {
        switch (h->g.sigma) {
#define X(S) case S: e = (h->dtype == CSR5_DTYPE_F32)                                                            \
        ? launch_transpose<S, true, float>(keep, h->g, h->n, h->nnz, h->col_idx, static_cast<float*>(h->val), h->status,     \
                                           nullptr, nullptr, DescJob{}, s)                                             \
        : launch_transpose<S, true, double>(keep, h->g, h->n, h->nnz, h->col_idx, static_cast<double*>(h->val), h->status,   \
                                            nullptr, nullptr, DescJob{}, s);                                            \
        break;
            CSR5_FOR_SIGMA(X)
#undef X
            default: e = hipErrorInvalidValue;
        }
    }
    if (e != hipSuccess) return CSR5_EHIP;
    h->in_csr5_order = false;
    return CSR5_OK;
}

int csr5_free(csr5_handle_t h) {
    if (!h) return CSR5_OK;
    int rc = CSR5_OK;
    if (h->owned && hipFree(h->owned) != hipSuccess) rc = CSR5_EHIP;
    far_release(h);
    delete h;
    return rc;
}

int csr5_status(csr5_handle_t h, uint32_t* status) {
    if (!h || !status) return CSR5_EINVAL;
    const int rc = read_status(h, status, 1);
    if (rc == CSR5_OK) *status &= STATUS_PUBLIC;
    return rc;
}

int csr5_get_info(csr5_handle_t h, int32_t* omega, int32_t* sigma, int32_t* p, int32_t* p_complete,
                  int32_t* desc_words_per_lane, int32_t* empty_offset_len) {
    if (!h) return CSR5_EINVAL;
    if (omega) *omega = OMEGA;
    if (sigma) *sigma = h->g.sigma;
    if (p) *p = h->g.p;
    if (p_complete) *p_complete = h->g.pc;
    if (desc_words_per_lane) *desc_words_per_lane = h->g.W;
    if (empty_offset_len) {
        int64_t v = 0;
        const size_t isz = h->wide ? 8 : 4;   // little-endian host: a 4-byte count lands in the low half
        const char* src = static_cast<const char*>(h->eop) + size_t(h->g.pc) * isz;
        if (hipMemcpyAsync(&v, src, isz, hipMemcpyDeviceToHost, h->conv_stream) != hipSuccess) return CSR5_EHIP;
        if (hipStreamSynchronize(h->conv_stream) != hipSuccess) return CSR5_EHIP;
        if (v < 0 || v > INT32_MAX) return CSR5_ERANGE;
        *empty_offset_len = int32_t(v);
    }
    return CSR5_OK;
}

int csr5_get_shape(csr5_handle_t h, int32_t* m, int32_t* n) {
    if (!h) return CSR5_EINVAL;
    if (m) *m = h->m;
    if (n) *n = h->n;
    return CSR5_OK;
}

int csr5_get_form(csr5_handle_t h, void* hip_stream, int32_t* kernel, int32_t* wave_tiles, int32_t* plain) {
    if (!h || !h->in_csr5_order) return CSR5_EINVAL;
    const bool far = gathered(h, static_cast<hipStream_t>(hip_stream));
    if (kernel) *kernel = h->staged ? CSR5_KERNEL_PARTS : (far ? CSR5_KERNEL_GATHERED : (h->window ? CSR5_KERNEL_WINDOW : (h->pairs ? CSR5_KERNEL_PAIRS : CSR5_KERNEL_TILES)));
    if (wave_tiles) *wave_tiles = h->staged ? h->staged : (h->window || far ? window_tiles(h->g.sigma) : 1);
    if (plain)
        *plain = !h->staged && !h->window && !far && rule_sigma(h->g.sigma) &&
                 keep_product(h, h->carry_turn.load(std::memory_order_relaxed), latest(h->device), static_cast<hipStream_t>(hip_stream));
    return CSR5_OK;
}

int csr5_get_arrays(csr5_handle_t h, const uint32_t** tile_ptr, const uint32_t** tile_desc,
                    const int32_t** empty_offset_ptr, const int32_t** empty_offset) {
    if (!h || h->wide) return CSR5_EINVAL;
    if (tile_ptr) *tile_ptr = static_cast<const uint32_t*>(h->tile_ptr);
    if (tile_desc) *tile_desc = h->tile_desc;
    if (empty_offset_ptr) *empty_offset_ptr = static_cast<const int32_t*>(h->eop);
    if (empty_offset) *empty_offset = h->eo;
    return CSR5_OK;
}

int csr5l_get_arrays(csr5_handle_t h, const uint64_t** tile_ptr, const uint32_t** tile_desc,
                     const int64_t** empty_offset_ptr, const int32_t** empty_offset) {
    if (!h || !h->wide) return CSR5_EINVAL;
    if (tile_ptr) *tile_ptr = static_cast<const uint64_t*>(h->tile_ptr);
    if (tile_desc) *tile_desc = h->tile_desc;
    if (empty_offset_ptr) *empty_offset_ptr = static_cast<const int64_t*>(h->eop);
    if (empty_offset) *empty_offset = h->eo;
    return CSR5_OK;
}

int csr5_baseline_csr_scalar(int32_t m, const int32_t* row_ptr, const int32_t* col_idx, const double* val,
                             const double* x, double* y, void* hip_stream) {
    if (m < 0 || !row_ptr || (m > 0 && !y)) return CSR5_EINVAL;
    if (m == 0) return CSR5_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipLaunchKernelGGL(k_csr_scalar, dim3(uint32_t((size_t(m) + 255) / 256)), dim3(256), 0, s, m, row_ptr,
                       col_idx, val, x, y);
    return hipGetLastError() == hipSuccess ? CSR5_OK : CSR5_EHIP;
}

int csr5_baseline_csr_vector(int32_t m, int32_t nnz, const int32_t* row_ptr, const int32_t* col_idx,
                             const double* val, const double* x, double* y, int32_t lanes_per_row,
                             void* hip_stream) {
    if (m < 0 || nnz < 0 || !row_ptr || (m > 0 && !y)) return CSR5_EINVAL;
    if (m == 0) return CSR5_OK;
    if (lanes_per_row == 0) {   // smallest power of two >= nnz/row, between 2 and 64
        int64_t q = nnz / m;
        lanes_per_row = 2;
        while (lanes_per_row < 64 && lanes_per_row < q) lanes_per_row *= 2;
    }
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    size_t threads = size_t(m) * size_t(lanes_per_row);
    dim3 grid(uint32_t((threads + 255) / 256)), block(256);
    if (threads / 256 >= 0x7fffffffull) return CSR5_EINVAL;
    switch (lanes_per_row) {
#define X(L) case L: hipLaunchKernelGGL(k_csr_vector<L>, grid, block, 0, s, m, row_ptr, col_idx, val, x, y); break;
        X(2) X(4) X(8) X(16) X(32) X(64)
#undef X
        default: return CSR5_EINVAL;
    }
    return hipGetLastError() == hipSuccess ? CSR5_OK : CSR5_EHIP;
}

int csr5_read_array(csr5_handle_t h, int which, void* dst_host, size_t bytes) {
    if (!h || (!dst_host && bytes)) return CSR5_EINVAL;
    const void* src = nullptr;
    size_t have = 0;
    switch (which) {
        case CSR5_ARRAY_TILE_PTR: src = h->tile_ptr; have = (size_t(h->g.p) + 1) * (h->wide ? 8 : 4); break;
        case CSR5_ARRAY_TILE_DESC: src = h->tile_desc; have = size_t(h->g.pc) * h->g.W * OMEGA * 4; break;
        case CSR5_ARRAY_EMPTY_OFFSET_PTR: src = h->eop; have = (size_t(h->g.pc) + 1) * (h->wide ? 8 : 4); break;
        case CSR5_ARRAY_EMPTY_OFFSET: {
            int32_t len = 0;
            int rc = csr5_get_info(h, nullptr, nullptr, nullptr, nullptr, nullptr, &len);
            if (rc != CSR5_OK) return rc;
            src = h->eo; have = size_t(len) * 4;
            break;
        }
        default: return CSR5_EINVAL;
    }
    if (bytes > have) return CSR5_EINVAL;
    if (bytes == 0) return CSR5_OK;
    if (hipMemcpyAsync(dst_host, src, bytes, hipMemcpyDeviceToHost, h->conv_stream) != hipSuccess) return CSR5_EHIP;
    if (hipStreamSynchronize(h->conv_stream) != hipSuccess) return CSR5_EHIP;
    return CSR5_OK;
}

}  // extern "C"
