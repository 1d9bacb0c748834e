// Internal declarations shared by the f3s HIP sources (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <atomic>

#include "f3s.h"

namespace f3s {

constexpr int kWindowRows = 16;   // r: rows per row window (Section 3.1)
constexpr int kBlockCols = 16;    // c: compacted columns per block
constexpr int kMaskWords = 8;     // 256-bit bitmap per 16x16 block
constexpr int kMaxD = 256;        // largest supported feature dimension

// Storage type of Q, K, V in the forward kernels.
constexpr int kInF16 = 0;
constexpr int kInBF16 = 1;
constexpr int kInFP8 = 2;     // OCP e4m3 (finite values up to 448)

// One unit of work for the fused kernel: a whole row window or one piece of
// a split window.  Blocks are absolute indices into the plan's block arrays.
struct WorkItem {
    int32_t window;
    int32_t blk_begin;
    int32_t blk_end;
    int32_t slot;  // partial-result slot of a piece, -1 for a whole window
};
static_assert(sizeof(WorkItem) == 16, "WorkItem must be 16 bytes");

// A plan's table of heavy items: heavy[j] counts the items of windows (or
// pieces) above heavy_blocks(j) blocks: 8, 10, 12, 14, 16, 20, 24, 28, 32, ...
constexpr int kHeavySteps = 32;
__host__ __device__ constexpr int32_t heavy_blocks(int j) { return (8 + 2 * (j & 3)) << (j >> 2); }
// Steps that k blocks exceed.
__host__ __device__ inline int heavy_level(int32_t k)
{
    int level = 0;
    while (level < kHeavySteps && k > heavy_blocks(level)) ++level;
    return level;
}

}  // namespace f3s

struct f3s_plan_s {
    int device = 0;
    int32_t N = 0;
    int32_t T = 0;               // row windows
    int64_t nnz_csr = 0;
    int64_t nnz = 0;             // distinct (row, col) pairs
    int64_t n_unique = 0;
    int64_t n_blocks = 0;
    int32_t max_blocks = 0;
    int32_t piece = 0;
    int32_t n_items = 0;
    int32_t n_split = 0;
    int32_t n_pieces = 0;
    int32_t flags = 0;           // bit 0: work list in window order; bit 1: narrow gathers;
                                 // bit 2: windows aligned to the graphs of a batch;
                                 // bit 3: split-row forward (ablation)
    int32_t heavy[f3s::kHeavySteps] = {};  // leading items above heavy_blocks(j) blocks
                                 // (heavy-first work lists)
    uint64_t id = 0;             // process-unique plan id
    uint64_t transpose_of = 0;   // id of the plan this one transposes (0: none)
    void *store = nullptr;       // one allocation: blk_off, cols, mask, items, merges,
                                 // shared with the transposed plan of a symmetric pattern
    std::atomic<int> *store_refs = nullptr;  // plans that hold it
    int64_t store_bytes = 0;
    void *part_store = nullptr;  // one allocation: part_o, part_ml
    int64_t part_bytes = 0;
    int32_t *blk_off = nullptr;  // [T + 1]
    int32_t *cols = nullptr;     // [16 * n_blocks]
    uint32_t *mask = nullptr;    // [8 * n_blocks]
    f3s::WorkItem *items = nullptr;  // [n_items]
    int32_t *merges = nullptr;   // [3 * n_split]
    int32_t *win_row = nullptr;  // [T + 1] first row of each window, then N (plans whose
                                 // windows follow the graphs of a batch; null: window w
                                 // is rows 16 w .. 16 w + 15)
    // Partial results of split windows for one launch group of nh heads
    // (nh * d <= part_row): slot (piece, head) = piece * nh + head.
    float *part_o = nullptr;     // [n_pieces * 16 * part_row]
    int32_t part_row = f3s::kMaxD;  // floats per piece row of part_o: kMaxD, or 4 kMaxD
                                 // with few pieces (transposed plans: twice that, for
                                 // the dK and dV partials)
    float *part_ml = nullptr;    // [n_pieces * (part_row/32) * 32]: 16 maxima, 16 sums
    int64_t device_bytes = 0;
    int64_t bsb_bytes = 0;
    double build_ms = 0.0;
};

namespace f3s {

// ---- plan kernels (plan_kernels.hip) ------------------------------------
// What places the items of a window in the work list.  Window w, R-th in the
// list's window order, starts at item
//   R + slot_base[w] - split_idx[w]    if its key is the largest (the split
//                                      windows', or all keys are equal)
//   R + n_pieces - n_split             otherwise:
// of the windows before it, the split ones have taken their pieces, the
// others one item each.
struct WorkListShape {
    const int32_t *blk_off;    // [T + 1]
    const int32_t *slot_base;  // [T + 1] pieces of the split windows before w
    const int32_t *split_idx;  // [T + 1] split windows before w
    int32_t piece, n_pieces, n_split;
};
// Items of a window of n blocks, and the k-th of them: the whole window, or
// piece k of np, which covers the block pairs [floor(k pairs / np),
// floor((k + 1) pairs / np)).
__host__ __device__ inline int32_t window_items(const WorkListShape &sh, int32_t n)
{
    return n <= sh.piece ? 1 : (n + sh.piece - 1) / sh.piece;
}
__host__ __device__ inline WorkItem window_item(const WorkListShape &sh, int32_t w, int32_t b0,
                                                int32_t n, int32_t k)
{
    if (n <= sh.piece) return WorkItem{w, b0, b0 + n, -1};
    const int32_t np = window_items(sh, n);
    const int64_t pairs = (n + 1) / 2;
    const int32_t a = 2 * (int32_t)((k * pairs) / np), b = 2 * (int32_t)(((k + 1) * pairs) / np);
    return WorkItem{w, b0 + a, b0 + (b < n ? b : n), sh.slot_base[w] + k};
}
// Writes window w's items from position pos on, one wavefront's lanes (or a
// workgroup's threads) sharing the pieces.
__host__ __device__ inline void place_window(const WorkListShape &sh, int32_t w, int32_t pos,
                                             int tid, int threads, WorkItem *items,
                                             int32_t *merges)
{
    const int32_t b0 = sh.blk_off[w], n = sh.blk_off[w + 1] - b0;
    const int32_t np = window_items(sh, n);
    if (n > sh.piece && tid == 0) {
        const int32_t s = sh.split_idx[w];
        merges[3 * s + 0] = w;
        merges[3 * s + 1] = sh.slot_base[w];
        merges[3 * s + 2] = np;
    }
    for (int32_t k = tid; k < np; k += threads) items[pos + k] = window_item(sh, w, b0, n, k);
}
// Whether item t of the list is what place_window put there, window w's items
// starting at pos[w] (pos null: window order).  An item names its window and
// its number among the window's items, and these name its position: if all
// n_items items are in place no two share a window's part, and as there are
// as many as the windows have parts, each part is in the list exactly once.
__host__ __device__ inline bool item_in_place(const WorkListShape &sh, const int32_t *pos,
                                              int32_t T, int32_t t, const WorkItem &it)
{
    const int32_t w = it.window;
    if (w < 0 || w >= T) return false;
    const int32_t b0 = sh.blk_off[w], n = sh.blk_off[w + 1] - b0, slot = sh.slot_base[w];
    const int32_t first = pos ? pos[w] : w + slot - sh.split_idx[w];
    const int32_t k = n > sh.piece ? it.slot - slot : 0;
    if (k < 0 || k >= window_items(sh, n) || t != first + k) return false;
    const WorkItem x = window_item(sh, w, b0, n, k);
    return it.blk_begin == x.blk_begin && it.blk_end == x.blk_end && it.slot == x.slot;
}
// The same of merge record s.
__host__ __device__ inline bool merge_in_place(const WorkListShape &sh, int32_t T, int32_t s,
                                               const int32_t *merges)
{
    const int32_t w = merges[3 * s];
    if (w < 0 || w >= T) return false;
    const int32_t n = sh.blk_off[w + 1] - sh.blk_off[w];
    return n > sh.piece && s == sh.split_idx[w] && merges[3 * s + 1] == sh.slot_base[w] &&
           merges[3 * s + 2] == window_items(sh, n);
}
// Workgroup order flags of the fused kernels: heads outermost (one pass over
// the work list per head), and consecutive ranges of the order per XCD.
constexpr uint32_t kOrderHead = 1u;
constexpr uint32_t kOrderXcd = 2u;
// Plans whose windows are nearly uniform: at least kUniformWindows windows,
// the largest holding at most twice the mean block count.  Their work list
// keeps window order (heavy-first sorting has nothing to balance, and sets
// windows that share rows of K and V apart), and launches of 1, 2, 4 or 8 heads
// give each XCD a consecutive range of it.  Sequences, forward and backward,
// sorted against window order with ranges: 30,000 tokens (1,875 windows), band
// 512, 3 heads of 64, 153.6 + 351 against 117.4 + 287 us; 24,000 (1,500), band
// 256, 2 heads of 128, 105.9 + 252 against 100.3 + 238, 1 head of 64, 30.9 + 75.2
// against 31.1 + 74.8; 20,000 (1,250) 4 heads of 128, 162 + 404 against 160 +
// 386, but 1 head of 64, 25.5 + 64.2 against 26.1 + 64.6; below, the ranges
// cost up to 0.5 us a launch and gain nothing.
constexpr int64_t kUniformWindows = 1280;
__host__ __device__ inline bool uniform_windows(int64_t windows, int64_t blocks, int64_t max_blocks)
{
    return windows >= kUniformWindows && max_blocks * windows <= 2 * blocks;
}
// Whether a launch of nh > 1 heads over plan p, whose K and V (all heads)
// hold kv_bytes, runs head by head instead of window-major (item * nh +
// head).  Window-major order shares a window's column lists and bitmaps
// among its heads, and with nh = 2, 4 or 8 round-robin dispatch still leaves
// each XCD one head (b mod 8 fixes b mod nh).  Head by head wins
// - when K and V exceed the 256 MB Infinity Cache: each head's gathers then
//   stream like a single head's;
// - when nh does not divide 8: window-major order then gives every XCD the
//   rows of every head (hub-heavy Chung-Lu graph, 3 heads: 97.1 -> 88.7 us
//   forward, 245.7 -> 226.7 us backward);
// - on nearly uniform plans, whose XCD ranges then hold one head's rows at a
//   time (3, 4 and 8 heads: 5-28% faster on the molecule batch and the
//   sequence workload; equal with 2).
// Window-major stays for skewed plans with 2, 4 or 8 heads (hub-heavy graph,
// 4 heads: 108.6 against 113.8 us head by head).  F3S_HEAD_MAJOR_BYTES=
// <bytes>, when set, replaces all three tests with kv_bytes > bytes (read at
// launch).
inline bool head_major_order(const f3s_plan_s &p, int32_t nh, uint64_t kv_bytes)
{
    if (nh <= 1) return false;
    const char *e = getenv("F3S_HEAD_MAJOR_BYTES");
    if (e && *e) return kv_bytes > (uint64_t)strtoull(e, nullptr, 10);
    return kv_bytes > ((uint64_t)256 << 20) || 8 % nh != 0 ||
           uniform_windows(p.n_items, p.n_blocks, p.max_blocks);
}
// Whether a launch of `heads` heads over plan p gives each XCD consecutive
// ranges of the work list (see workgroup_position): for nearly uniform plans
// (no XCD's range is then much heavier than another's), window-major with
// 1, 2, 4 or 8 heads, head-major with any.  With its window-order work list
// the molecule batch ran 18.8 -> 15.6 us forward and 52.8 -> 45.0 us
// backward with one head, 33.7 -> 26.4 us forward with two.  On skewed plans
// the ranges would give the heaviest items to one XCD (1.7x slower on the
// million-node graph).  Window-major ranges over all heads of a window would
// give every XCD the rows of every head, where round-robin order with 2, 4
// or 8 heads leaves each XCD one head (b mod 8 fixes b mod heads): that
// measured 45% slower with four heads of the sequence workload, so other
// head counts keep round-robin there.  F3S_XCD_CHUNKS=0 or 1 forces the
// choice where the ranges apply (read at launch).
inline bool xcd_chunks(const f3s_plan_s &p, int32_t heads, bool head_major = false)
{
    if (heads < 1 || (!head_major && 8 % heads != 0)) return false;
    const char *e = getenv("F3S_XCD_CHUNKS");
    if (e && *e) return atoi(e) != 0;
    return uniform_windows(p.n_items, p.n_blocks, p.max_blocks);
}
// Work-list piece size (even).  Pieces cost a partial result of 16 rows
// through memory and a merge launch (6 to 18 us a call on the hub-heavy
// graph when the pieces were a quarter of this), so a window stays whole as
// long as the 4 waves of a workgroup get through it while the launch runs:
// about 4 n_blocks / slots blocks (slots = 8 per CU), twice a resident wave's
// even share for each of the 4 waves; at least 64 blocks and 1.5 times the
// mean window, and 128 for nearly uniform windows (the largest at most twice
// the mean: all are as long and splitting balances nothing).  Never above the
// largest window (a larger value splits nothing and only widens the histogram
// of the work-list sort), nor a little below it.  forced >= 2 overrides the
// estimate.  Measured against pieces of n_blocks / slots, at least 16, and one
// wave per item: hub-heavy graph, N = 65,536, d = 64, forward 33.5 -> 29.3 us,
// 4 bf16 heads forward and backward 421 -> 372 us; sequence of 16,001 tokens, 2
// heads of d = 128, forward and backward 303 -> 233 us; ER graph of 10,007
// nodes, 16 neighbours, 2 heads 56 -> 37 us.
// Skewed windows listed in window order have no heavy items in front for a
// workgroup to share: the pieces stay n_blocks / slots, at least 16.  (The
// gather and split-row ablations take the pieces of the plans that they are
// compared with, bit for bit.)
__host__ __device__ inline int32_t plan_piece(int64_t n_blocks, int32_t max_blocks, int32_t T,
                                              int32_t forced, int32_t slots, bool window_order)
{
    const int64_t cap = ((int64_t)(max_blocks > 2 ? max_blocks : 2) + 1) & ~1LL;
    int64_t piece;
    const bool uniform = (int64_t)max_blocks * T <= 2 * n_blocks;
    if (forced >= 2) {
        piece = forced & ~1;
    } else if (window_order && !uniform) {
        piece = (n_blocks + slots - 1) / slots;
        if (piece < 16) piece = 16;
        piece = (piece + 1) & ~1LL;
    } else {
        int64_t least = uniform ? 128 : 64;
        if (2 * least * T < 3 * n_blocks) least = 3 * n_blocks / (2 * (int64_t)T);
        piece = (4 * n_blocks + slots - 1) / slots;
        if (piece < least) piece = least;
        piece = (piece + 1) & ~1LL;
        if (2 * cap <= 3 * piece) piece = cap;
    }
    return (int32_t)(piece < cap ? piece : cap);
}
// Waves per work item (forward and backward).  nw: waves of a workgroup; the
// first `shared` items are shared by the nw waves of a workgroup each, the
// others get one wave each, nw of them to a workgroup.
struct WaveSplit {
    int nw;
    int32_t shared;
};
// Nearly uniform plans (the largest window at most twice the mean item), and
// plans whose list keeps window order: all items by 4 waves while all of these
// fit the GPU at once (`resident`: the kernel's waves per SIMD x 1024 SIMDs),
// there are no more items x heads than SIMDs and the items average at least 4
// blocks; else all by 2 while these fit, there are at most 1.5 items x heads
// per SIMD and the items average at least 8 blocks (two pairs per wave); else
// one each.  More waves than fit at once run as a second round, and more waves
// than hide the latencies only spread the gathers over more of K and V at a
// time: windows in flight together walk their columns in step, so whole
// windows find each other's rows in the caches, halves and quarters of them
// less.  (Sequences, band 256 + 64 random keys, forward, 1 / 2 / 4 waves:
// d = 64, 1000 items x heads 23.4, 19.3, 19.3 us, 1500 30.1, 27.7, 27.9, 2000
// 34.7, 35.2, 36.6; d = 128, 500 28.2, 21.2, 19.1, 1001 43.8, 38.5, 47.7, 1250
// 53.3, 56.0, 64.2, 1500 55.4, 78.7, 83.8; d = 256, 375 73.1, 47.2, 54.2.)
// A last round that is nearly empty is not split off: one wave each still beats
// two waves or half windows as items at 24,000 tokens, 2 heads, d = 128 (3000
// over 2048, window order: 100, 127, 116 us; backward 238, 318, 298), and at
// 30,000 tokens, band 512, 3 heads of 64 (5625 over 4096: 117, 170, 131;
// backward 287, 391, 390).
// Skewed plans: 4 waves share the heavy items, the lighter ones take one wave
// each.  Left to one wave, items of up to T blocks outlast the launch by about T
// less a resident wave's even share of all blocks; shared, each costs three
// more waves' start, Q rows and combination, which the whole GPU pays: 16 items
// (times heads) cost as much as one block that a lone wave is left with.  T is
// the table's step with the least sum of both (or nothing is shared).  The 16
// was fitted, from 12 to 18, to 36 Chung-Lu graphs of 10,000 to 262,147 nodes, 1
// to 4 heads, d = 32 to 256, forward and backward at ten fixed T each: 1.8% above
// the best T on average, where T = the even share alone was 7.5% above it and
// up to 45%: nearly everything was shared where the mean item exceeded the
// share.  (40,000 nodes, exponent 2.6, d = 64, forward + backward, T = 10, the
// share: 24.5 + 68.8 us; 28: 19.7 + 48.2; 56: 26.9 + 65.3.  65,536 nodes,
// exponent 2.1: 14: 25.5 + 69.3, 20: 25.9 + 66.6, 40: 28.7 + 71.9.)
// F3S_WAVES_PER_ITEM=1, 2 or 4 forces one count for all items (read at launch).
inline WaveSplit wave_split(const f3s_plan_s &p, int32_t heads, int64_t resident)
{
    const char *e = getenv("F3S_WAVES_PER_ITEM");
    if (e && *e) {
        const int v = atoi(e);
        return WaveSplit{v == 4 ? 4 : v == 2 ? 2 : 1, p.n_items};
    }
    if (p.n_items <= 0) return WaveSplit{1, p.n_items};
    if ((p.flags & 1) || (int64_t)p.max_blocks * p.n_items <= 2 * p.n_blocks) {
        const int64_t waves = (int64_t)p.n_items * heads;
        if (waves <= 1024 && 4 * waves <= resident && p.n_blocks >= 4ll * p.n_items)
            return WaveSplit{4, p.n_items};
        if (waves <= 1536 && 2 * waves <= resident && p.n_blocks >= 8ll * p.n_items)
            return WaveSplit{2, p.n_items};
        return WaveSplit{1, p.n_items};
    }
    const int64_t share = p.n_blocks * heads / resident;
    const int32_t largest = p.max_blocks < p.piece ? p.max_blocks : p.piece;
    int64_t least = largest > share ? 16 * (largest - share) : 0;
    int32_t shared = 0;
    for (int j = 0; j < kHeavySteps && heavy_blocks(j) < largest; ++j) {
        const int32_t t = heavy_blocks(j);
        const int64_t cost = (t > share ? 16 * (t - share) : 0) + (int64_t)p.heavy[j] * heads;
        if (cost < least) {
            least = cost;
            shared = p.heavy[j];
        }
    }
    return shared > 0 ? WaveSplit{4, shared} : WaveSplit{1, p.n_items};
}
// Workgroups per head of such a launch.
inline int64_t wave_groups(const WaveSplit &ws, int32_t n_items)
{
    return ws.shared + ((int64_t)n_items - ws.shared + ws.nw - 1) / ws.nw;
}
// The item of wave wv of group g (workgroup / heads), and whether the
// workgroup's nw waves share it; false: no such item (device code).
template <int NW>
__device__ __forceinline__ bool wave_item(int g, int wv, int32_t shared_items, int32_t n_items,
                                          int *item, bool *shared)
{
    if constexpr (NW == 1) {  // a workgroup per item: no count to load first
        *shared = true;
        *item = g;
        return true;
    }
    *shared = g < shared_items;
    *item = *shared ? g : shared_items + (g - shared_items) * NW + wv;
    return *item < n_items;
}
// Byte offset of a row of row_bytes bytes in a table of less than 4 GiB, as 32
// bits (the products are unsigned: offsets of 2 GiB and more use the top bit).
__host__ __device__ inline int32_t row_offset(int32_t row, int32_t row_bytes)
{
    return (int32_t)((uint32_t)row * (uint32_t)row_bytes);
}
// First row and row count of window w: rows 16 w .. 16 w + 15 (the last
// window clipped at N), or those given by win_row (device code).
__device__ __forceinline__ void window_rows(const int32_t *win_row, int32_t N, int32_t w,
                                           int32_t *r0, int32_t *nr)
{
    if (win_row) {
        *r0 = win_row[w];
        *nr = win_row[w + 1] - *r0;
    } else {
        *r0 = w * kWindowRows;
        *nr = min(kWindowRows, N - *r0);
    }
}
// Inclusive sum over the 64 lanes of a wavefront (all active), with DPP row
// shifts (within rows of 16 lanes, out-of-row sources read 0) and the first
// three row totals by readlane (device code).
__device__ __forceinline__ int wave_inclusive_sum(int x, int lane)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);  // row_shr:8
    const int r0 = __builtin_amdgcn_readlane(x, 15), r1 = __builtin_amdgcn_readlane(x, 31);
    const int r2 = __builtin_amdgcn_readlane(x, 47);
    const int row = lane >> 4;
    return x + (row >= 1 ? r0 : 0) + (row >= 2 ? r1 : 0) + (row >= 3 ? r2 : 0);
}

// Device-side statistics of a plan build, read back with one copy each
// time the host needs them.
struct BuildStats {
    unsigned long long n_unique;  // sum of distinct columns over windows
    unsigned long long nnz;       // set bits of all bitmaps
    int32_t err;                  // kBuildBadCsr or kBuildBadValue
    int32_t bad_rows;             // err before any column was read
    int32_t nnz_csr;              // row_ptr[N]
    int32_t n_mid, n_big, n_heavy;  // windows listed by launch_classify
    int32_t max_blocks;
    int32_t n_blocks;
    int32_t piece;
    int32_t n_pieces;
    int32_t n_split;
    int32_t placed;               // see launch_shape
    int32_t invalid;              // plan integrity check
    int32_t heavy[kHeavySteps];   // items above heavy_blocks(j) blocks
};
constexpr int kBuildBadCsr = 1;    // malformed pattern
constexpr int kBuildBadValue = 2;  // entries but no col_idx, or more than nnz_cap
// Zeroes *st, reads nnz into it and checks it (also against the nnz_cap
// entries the scratch holds; has_cols: col_idx was given); then checks
// row_ptr and lists the windows with more than 512 CSR entries: mid up to
// 1024, big up to 4096, heavy above.
// win_row: the windows' first rows (null: 16-row windows); also below.
hipError_t launch_classify(const int32_t *row_ptr, int32_t N, const int32_t *win_row, int32_t T,
                           int64_t nnz_cap, bool has_cols, BuildStats *st, int32_t *mid,
                           int32_t *big, int32_t *heavy, hipStream_t s);
// Staging area of the window bitmaps, in 32-bit words, for nnz CSR entries.
int64_t mask_stage_words(int64_t nnz, int32_t T);
// Per window: sorted distinct columns into tmp_cols at the window's CSR
// offset, their count into u, the block bitmaps into the staging area, their
// set bits into bits.  Nothing if *st already holds an error.
hipError_t launch_windows(const int32_t *row_ptr, const int32_t *col_idx, int32_t N,
                          const int32_t *win_row, int32_t T, int64_t nnz_cap, BuildStats *st,
                          const int32_t *mid, const int32_t *big, const int32_t *heavy,
                          int32_t *tmp_cols, uint32_t *tmp_mask, int32_t *u, int32_t *bits,
                          hipStream_t s);
// Exclusive scan of n int32 into out[0..n], out[n] = total (in == out ok).
// total (may be null) also receives the total.
struct ScanArray {
    const int32_t *in = nullptr;
    int32_t *out = nullptr;
    int32_t *total = nullptr;
    int32_t *tile_sums = nullptr;  // set by the launcher (from tmp)
};
// tmp: scan_tmp_ints(n) ints of workspace.
int64_t scan_tmp_ints(int64_t n);
hipError_t launch_scan(ScanArray a, int32_t n, int32_t *tmp, hipStream_t s);
hipError_t launch_scan(const int32_t *in, int32_t *out, int32_t n, int32_t *tmp,
                       int32_t *total_out, hipStream_t s);
// Two independent scans of n ints each (one launch when n is small).
hipError_t launch_scan2(ScanArray a0, ScanArray a1, int32_t n, int32_t *tmp, hipStream_t s);
// The plan's blk_off, padded column lists and block bitmaps from the scratch;
// with `items` also the work list, window w's items from pos[w] on (pos null:
// in window order).
hipError_t launch_fill_windows(const int32_t *row_ptr, const int32_t *win_row, int32_t T,
                               const int32_t *tmp_cols, const uint32_t *tmp_mask,
                               const int32_t *u, int32_t *plan_off, int32_t *cols,
                               uint32_t *mask, const WorkListShape &shape,
                               const int32_t *pos, WorkItem *items, int32_t *merges,
                               hipStream_t s);
// Blocks per window and the shape of the work list, from u and bits: nb[w] =
// ceil(u[w] / 16) and its prefix blk_off[0..T]; the statistics (st->n_unique,
// nnz, n_blocks, max_blocks); the piece size (see plan_piece for forced and
// slots) in st->piece; per window the sort key, and
// over the split windows the prefixes of their pieces (slot_base[0..T]) and
// of their number (split_idx[0..T]); st->n_pieces and n_split.  order:
// kOrderAuto keeps window order for nearly uniform windows and sorts others,
// heavy first.  st->placed != 0: the list's order is decided, pos[w] is
// window w's first item and st->heavy is set (plans of up to kOnePlace
// windows, keys below kPlaceKeys); else launch_worklist has to follow.
// scan_tmp: scan_tmp_ints(T) ints.
constexpr int kOrderAuto = 0, kOrderSorted = 1, kOrderWindow = 2;
hipError_t launch_shape(const int32_t *u, const int32_t *bits, int32_t T, int32_t forced,
                        int32_t slots, int order, BuildStats *st, int32_t *nb,
                        int32_t *blk_off, int32_t *key, int32_t *slot_base, int32_t *split_idx,
                        int32_t *pos, int32_t *scan_tmp, hipStream_t s);

// ---- radix sort (radix.hip) -------------------------------------------------
// Stable sort of n (key, value) int32 pairs, keys in [0, max_key], ascending
// or descending; vals == nullptr stands for the values 0 .. n-1 (the sort
// then yields the sorting permutation).  The inputs are not written; the
// results end up in one of the two scratch pairs (*keys_out, *vals_out say
// which).
struct RadixScratch {
    int32_t *keys_a, *vals_a, *keys_b, *vals_b;  // [n] each
    int32_t *counts;                              // radix_count_ints(n)
    int32_t *scan_tmp;                            // scan_tmp_ints(max(n, radix_count_ints(n)))
};
int64_t radix_count_ints(int32_t n);
// Digit passes of a sort with keys up to max_key (the results of an odd
// count end up in keys_a / vals_a, of an even count in keys_b / vals_b).
int radix_passes(int32_t max_key);
hipError_t launch_radix_pairs(const int32_t *keys, const int32_t *vals, int32_t n,
                              int32_t max_key, bool descending, const RadixScratch &rs,
                              const int32_t **keys_out, const int32_t **vals_out,
                              hipStream_t s);

// ---- work list (worklist.hip) ----------------------------------------------
// Heavy-first work list from the keys of launch_shape where it did not place
// the windows itself: the windows stably sorted by key, largest first; whole
// windows as items, split windows as merge records and their pieces as
// items; pos[w]: window w's first item.  heavy: the table of heavy items
// (zeroed).
hipError_t launch_worklist(const int32_t *key, const WorkListShape &shape, int32_t T,
                           const RadixScratch &radix, WorkItem *items, int32_t *merges,
                           int32_t *pos, int32_t *heavy, hipStream_t s);

// ---- transposed pattern (transpose.hip) ----------------------------------
// CSR of A^T (rp[N+1], ci[nnz], each row in increasing column order) from a
// plan's bitmaps; scratch of transpose_scratch_bytes(p) bytes.
size_t transpose_scratch_bytes(const f3s_plan_s &p);
hipError_t launch_transpose_csr(const f3s_plan_s &p, void *scratch, size_t scratch_bytes,
                                int32_t *rp, int32_t *ci, hipStream_t s);
// Sets *asym to 0 if the plan's pattern is symmetric, to 1 otherwise,
// from the plan alone (binary searches in the windows' column lists; cheap
// on small patterns); win: scratch of n_blocks ints.
hipError_t launch_check_symmetric(const f3s_plan_s &p, int32_t *win, int32_t *asym,
                                  hipStream_t s);
// The same decision given the CSR of A^T, *asym zeroed by the caller (every
// row of A compared with the same row of A^T, position by position; cheaper on
// large patterns once A^T is sorted anyway).  win: n_blocks ints, pre: 16 *
// n_blocks ints of scratch.
hipError_t launch_compare_rows(const f3s_plan_s &p, const int32_t *rpt, const int32_t *cit,
                               int32_t *win, int32_t *pre, int32_t *asym, hipStream_t s);

// Sets *err when a finished plan is internally inconsistent: a block without
// a first column, a column out of range, a work list that does not hold every
// part of every window once (the windows' first items: pos, null for window
// order; shape and pos are the build's scratch).
hipError_t launch_validate_plan(const f3s_plan_s &p, const WorkListShape &shape,
                                const int32_t *pos, int32_t *err, hipStream_t s);

// ---- fused operator (fused3s.hip) ---------------------------------------
// H heads of size d; Q, K, V, O rows hold the heads back to back (stride H*d).
// lse (may be null): [N, H] natural-log log-sum-exp of each row's scores.
// in_type: kInF16, kInBF16 or kInFP8; out_f16: O is fp16 instead of fp32.
hipError_t launch_fused(const f3s_plan_s &p, const void *Q, const void *K,
                        const void *V, int in_type, void *O, bool out_f16, float *lse,
                        int32_t H, int32_t d, float scale_log2, hipStream_t s);
hipError_t launch_fused_bf16(const f3s_plan_s &p, const void *Q, const void *K,
                             const void *V, void *O, bool out_f16, float *lse, int32_t H,
                             int32_t d, float scale_log2, hipStream_t s);
// Measurement instance of the one-head fp16 -> fp32 forward: the same result
// in O, plus a 32-byte record per work item in trace (start and end times on
// the constant clock, hardware ids of the compute unit, record index).
hipError_t launch_fused_trace(const f3s_plan_s &p, const void *Q, const void *K,
                              const void *V, void *O, int32_t d, float sl2, uint32_t *trace,
                              hipStream_t s);
// Ablation: fp16 -> fp32 forward with 4-byte K/V gathers (plan flag bit 1).
hipError_t launch_fused_narrow(const f3s_plan_s &p, const void *Q, const void *K,
                               const void *V, void *O, float *lse, int32_t H, int32_t d,
                               float scale_log2, hipStream_t s);
// Ablation: fp16 -> fp32 forward with the split-row partition of a window
// among its waves (plan flag bit 3; d a multiple of 64, 32-bit addressing).
hipError_t launch_fused_split_row(const f3s_plan_s &p, const void *Q, const void *K,
                                  const void *V, float *O, float *lse, int32_t H, int32_t d,
                                  float scale_log2, hipStream_t s);
hipError_t launch_fused_fp8(const f3s_plan_s &p, const void *Q, const void *K,
                            const void *V, void *O, bool out_f16, float *lse, int32_t H,
                            int32_t d, float scale_log2, hipStream_t s);

// Records s as this thread's last error (f3s_last_error) and returns it.
f3s_status_t record_error(f3s_status_t s);

// Gradients (backward_kernel.h; fp16 inputs: backward.hip, bf16 inputs:
// backward_bf16.hip).  pt is the plan of the transposed pattern; row_stats:
// [N, H, 2] (base-2 lse, delta) written by the dQ pass.
hipError_t launch_backward(const f3s_plan_s &p, const f3s_plan_s &pt, const void *Q,
                           const void *K, const void *V, const float *O, const void *G,
                           const float *lse, float *row_stats, float *dQ, float *dK, float *dV,
                           int32_t H, int32_t d, float scale, hipStream_t s);
hipError_t launch_backward_bf16(const f3s_plan_s &p, const f3s_plan_s &pt, const void *Q,
                                const void *K, const void *V, const float *O, const void *G,
                                const float *lse, float *row_stats, float *dQ, float *dK,
                                float *dV, int32_t H, int32_t d, float scale, hipStream_t s);

}  // namespace f3s
