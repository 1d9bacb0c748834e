/*
 * The library's host-side rules, run on the CPU (built and run by
 * tests/test_host_rules.py, host code only).  Each check prints its name;
 * the run ends with "ok".
 */
#include <stdio.h>

#include <algorithm>
#include <numeric>
#include <random>
#include <vector>

#include "f3s_internal.h"

using namespace f3s;

#define CHECK(c)                                                           \
    do {                                                                   \
        if (!(c)) {                                                        \
            fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
            return 1;                                                      \
        }                                                                  \
    } while (0)

struct List {
    std::vector<int32_t> blk_off, slot_base, split_idx, pos, merges;
    std::vector<WorkItem> items;
    WorkListShape shape;
};

// The work list of windows of nb blocks, heavy first (stably) or in order.
static void make_list(const std::vector<int32_t> &nb, int32_t piece, bool sorted, List &l)
{
    const int32_t T = (int32_t)nb.size();
    l.blk_off.assign(1, 0);
    l.slot_base.assign(1, 0);
    l.split_idx.assign(1, 0);
    for (int32_t n : nb) {
        l.blk_off.push_back(l.blk_off.back() + n);
        l.slot_base.push_back(l.slot_base.back() + (n > piece ? (n + piece - 1) / piece : 0));
        l.split_idx.push_back(l.split_idx.back() + (n > piece));
    }
    l.shape = WorkListShape{l.blk_off.data(), l.slot_base.data(), l.split_idx.data(),
                            piece,            l.slot_base[T],     l.split_idx[T]};
    std::vector<int32_t> order(T);
    std::iota(order.begin(), order.end(), 0);
    if (sorted)
        std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
            return std::min(nb[a], piece) > std::min(nb[b], piece);
        });
    l.items.assign((size_t)T - l.shape.n_split + l.shape.n_pieces, WorkItem{-1, -1, -1, -1});
    l.merges.assign(3 * (size_t)l.shape.n_split, -1);
    l.pos.assign(T, -1);
    int32_t at = 0;
    for (int32_t w : order) {
        l.pos[w] = at;
        for (int tid = 0; tid < 3; ++tid)
            place_window(l.shape, w, at, tid, 3, l.items.data(), l.merges.data());
        at += window_items(l.shape, nb[w]);
    }
}

static bool whole(const List &l, int32_t T, bool window_order)
{
    for (size_t t = 0; t < l.items.size(); ++t)
        if (!item_in_place(l.shape, window_order ? nullptr : l.pos.data(), T, (int32_t)t,
                           l.items[t]))
            return false;
    for (int32_t s = 0; s < l.shape.n_split; ++s)
        if (!merge_in_place(l.shape, T, s, l.merges.data())) return false;
    return true;
}

// A list with every part of every window in its place passes, also in window
// order; one in which a window's item lies where another's should, or in
// which two windows were given one place, does not.
static int work_list_check()
{
    std::mt19937 rng(1);
    for (int32_t T : {1, 2, 63, 200}) {
        for (int32_t piece : {2, 6, 40}) {
            std::vector<int32_t> nb(T);
            for (int32_t &n : nb) n = (int32_t)(rng() % 50);
            for (bool sorted : {false, true}) {
                List l;
                make_list(nb, piece, sorted, l);
                CHECK(whole(l, T, false));
                if (!sorted) CHECK(whole(l, T, true));
                // every block in exactly one item
                std::vector<int> seen(l.blk_off[T], 0);
                for (const WorkItem &it : l.items)
                    for (int32_t b = it.blk_begin; b < it.blk_end; ++b) ++seen[b];
                for (int s : seen) CHECK(s == 1);
                const size_t n = l.items.size();
                if (n < 2) continue;
                for (int k = 0; k < 20; ++k) {
                    List bad = l;
                    bad.shape = l.shape;
                    const size_t a = rng() % n, b = (a + 1 + rng() % (n - 1)) % n;
                    switch (k % 4) {
                    case 0: bad.items[a] = bad.items[b]; break;  // one lost, one twice
                    case 1: std::swap(bad.items[a], bad.items[b]); break;
                    case 2: bad.items[a].blk_end += 2; break;
                    default: bad.items[a].slot += 1; break;
                    }
                    CHECK(!whole(bad, T, false));
                }
                if (l.shape.n_split > 0) {
                    List bad = l;
                    bad.merges[3 * (rng() % l.shape.n_split) + rng() % 3] += 1;
                    CHECK(!whole(bad, T, false));
                }
            }
            // two windows of one key given one place: the later one's item
            // overwrites the earlier one's, and a place keeps what the memory
            // held before -- here a plausible item, from a list built before
            for (int32_t w = 1; w < T; ++w) {
                if (nb[w] != nb[w - 1] || nb[w] > piece) continue;
                List l;
                make_list(nb, piece, true, l);
                const int32_t lost = l.pos[w];
                l.pos[w] = l.pos[w - 1];
                place_window(l.shape, w, l.pos[w], 0, 1, l.items.data(), l.merges.data());
                for (size_t t = 0; t < l.items.size(); ++t) {
                    l.items[lost] = l.items[t];
                    CHECK(!whole(l, T, false));
                }
            }
        }
    }
    printf("work list check\n");
    return 0;
}

// Waves per item of a nearly uniform plan of n windows of k blocks.
static int waves(int32_t n, int32_t k, int32_t heads, int64_t resident)
{
    f3s_plan_s p;
    p.n_items = p.T = n;
    p.n_blocks = (int64_t)n * k;
    p.max_blocks = k;
    const WaveSplit ws = wave_split(p, heads, resident);
    return ws.shared == n ? ws.nw : -1;
}

static int wave_rule()
{
    for (int64_t per_simd : {1, 2, 3, 4, 6}) {
        const int64_t resident = 1024 * per_simd;
        for (int32_t heads : {1, 2, 3, 8}) {
            int last = 4;
            for (int32_t n = 1; n * heads < 9000; n += 1 + n / 50) {
                const int nw = waves(n, 80, heads, resident);
                // the launch's waves fit at once, or nothing is shared; never
                // more waves an item for a larger launch
                CHECK(nw == 1 || (int64_t)nw * n * heads <= resident);
                CHECK(nw >= 1 && nw <= last);
                last = nw;
                // and no SIMD is left without a wave that could have one
                if (2ll * n * heads <= (resident < 2048 ? resident : 2048)) CHECK(nw >= 2);
                if (4ll * n * heads <= 1024) CHECK(nw == 4);
            }
        }
    }
    // one head of 16,001 tokens at d = 128: four waves a window were two rounds
    CHECK(waves(1001, 81, 1, 2048) == 2);
    CHECK(waves(375, 73, 1, 1024) == 2);
    CHECK(waves(500, 60, 1, 2048) == 4);
    // thin windows stay whole, more than one round too
    CHECK(waves(1000, 3, 1, 4096) == 1 && waves(1000, 7, 1, 2048) == 1);
    CHECK(waves(3000, 80, 1, 2048) == 1 && waves(1689, 24, 1, 4096) == 1);
    f3s_plan_s none;
    CHECK(wave_split(none, 4, 2048).nw == 1);
    printf("waves per item\n");
    return 0;
}

// A skewed plan from its items' block counts.
static f3s_plan_s skewed(const std::vector<int32_t> &size, int32_t piece)
{
    f3s_plan_s p;
    p.n_items = p.T = (int32_t)size.size();
    p.piece = piece;
    for (int32_t n : size) {
        p.n_blocks += n;
        p.max_blocks = std::max(p.max_blocks, n);
        for (int j = 0; j < kHeavySteps; ++j) p.heavy[j] += n > heavy_blocks(j);
    }
    return p;
}

// On skewed plans four waves share the few heaviest items: those whose one
// wave would outlast the launch, never the bulk of them, and none where every
// wave has more than the largest item to do anyway.
static int heavy_rule()
{
    // 2,500 items of about 17 blocks, some of up to 84 (40,000 nodes, exponent
    // 2.6): the even share of 4,096 waves, 10, is below nearly all of them
    std::vector<int32_t> size;
    for (int i = 0; i < 2500; ++i)
        size.push_back(i < 28 ? 60 : i < 54 ? 48 : i < 119 ? 33 : i < 402 ? 24 : i < 1365 ? 17 : 13);
    const f3s_plan_s mild = skewed(size, 84);
    const WaveSplit a = wave_split(mild, 1, 4096);
    CHECK(a.nw == 4 && a.shared >= 54 && a.shared <= 402);
    CHECK(wave_groups(a, 2500) == a.shared + (2500 - a.shared + 3) / 4);
    // hubs: 4,200 items of mean 13, up to 106
    size.clear();
    for (int i = 0; i < 4200; ++i)
        size.push_back(i < 49 ? 106 : i < 222 ? 70 : i < 384 ? 40 : i < 751 ? 20 : 7);
    const f3s_plan_s hubs = skewed(size, 106);
    const WaveSplit b = wave_split(hubs, 1, 4096), c = wave_split(hubs, 4, 4096);
    CHECK(b.nw == 4 && b.shared >= 222 && b.shared <= 751);
    CHECK(c.nw == 1 || c.shared <= b.shared);  // more heads: nothing more to share
    CHECK(wave_split(hubs, 64, 4096).nw == 1);
    // the items shared are a prefix of whole levels, at most all
    for (int32_t heads : {1, 2, 3, 8})
        for (int64_t resident : {1024, 2048, 3072, 4096, 6144})
            for (const f3s_plan_s *p : {&mild, &hubs}) {
                const WaveSplit ws = wave_split(*p, heads, resident);
                CHECK(ws.nw == 1 ? ws.shared == p->n_items
                                 : ws.nw == 4 && ws.shared > 0 && ws.shared < p->n_items);
            }
    printf("heavy items\n");
    return 0;
}

// Window order from 1,280 nearly uniform windows on.
static int order_rule()
{
    CHECK(uniform_windows(1500, 1500 * 80, 81) && uniform_windows(1280, 2560, 4));
    CHECK(!uniform_windows(1279, 1279 * 80, 81) && !uniform_windows(1500, 3000, 5));
    f3s_plan_s p;
    p.n_items = 1875;
    p.n_blocks = 1875 * 95;
    p.max_blocks = 96;
    CHECK(head_major_order(p, 3, 23 << 20) && xcd_chunks(p, 3, true) && xcd_chunks(p, 1));
    printf("window order\n");
    return 0;
}

static int piece_rule()
{
    const int32_t slots = 2048;
    // the hub-heavy graph: pieces for workgroups that share them, or, in window
    // order, for one wave each
    CHECK(plan_piece(67341, 1465, 4096, 0, slots, false) == 132);
    CHECK(plan_piece(67341, 1465, 4096, 0, slots, true) == 34);
    for (bool order : {false, true}) {
        // nearly uniform windows stay whole in either order
        CHECK(plan_piece(81081, 81, 1001, 0, slots, order) == 82);
        for (int32_t forced : {2, 7, 40}) {
            CHECK(plan_piece(67341, 1465, 4096, forced, slots, order) == (forced & ~1));
            CHECK(plan_piece(10, 5, 4, forced, slots, order) == (forced < 6 ? forced & ~1 : 6));
        }
        // even, at least 2, at most the largest window; also at the limits
        for (int64_t n : {0ll, 1ll, 100ll, 1ll << 20, 2147483647ll})
            for (int32_t T : {1, 3, 1000, 134217728})
                for (int32_t m : {0, 1, 2, 17, 65536, 134217727}) {
                    const int32_t piece = plan_piece(n, m, T, 0, slots, order);
                    CHECK(piece >= 2 && piece % 2 == 0 && piece <= (m > 2 ? m + (m & 1) : 2));
                }
    }
    printf("piece size\n");
    return 0;
}

// Offsets up to 4 GiB without overflow (the run checks for undefined
// behaviour), equal to the 64-bit product's low half.
static int offset_rule()
{
    for (int32_t bytes : {64, 256, 512, 56320})
        for (uint64_t off = 0; off < 0xFFFFFFF0ull; off += 0x0FFFFFF7ull) {
            const int32_t row = (int32_t)(off / bytes);
            CHECK((uint32_t)row_offset(row, bytes) == (uint32_t)((uint64_t)row * bytes));
        }
    CHECK((uint32_t)row_offset(16777214, 256) == 16777214u * 256u);
    printf("row offsets\n");
    return 0;
}

int main()
{
    if (offset_rule() || work_list_check() || wave_rule() || heavy_rule() || order_rule() || piece_rule()) return 1;
    printf("ok\n");
    return 0;
}
