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

static int piece_rule()
{
    const int32_t slots = 2048;
    // the hub-heavy graph: pieces for workgroups that share them, or not
    CHECK(plan_piece(67341, 1465, 4096, 0, slots, true, false) == 132);
    for (bool order : {false, true}) CHECK(plan_piece(67341, 1465, 4096, 0, slots, false, order) == 34);
    CHECK(plan_piece(67341, 1465, 4096, 0, slots, true, true) == 34);
    // nearly uniform windows stay whole in either order, unless a wave has
    // each item for itself
    for (bool order : {false, true}) CHECK(plan_piece(81081, 81, 1001, 0, slots, true, order) == 82);
    CHECK(plan_piece(81081, 81, 1001, 0, slots, false, true) == 40);
    for (bool shared : {false, true}) {
        for (int32_t forced : {2, 7, 40}) {
            CHECK(plan_piece(67341, 1465, 4096, forced, slots, shared, true) == (forced & ~1));
            CHECK(plan_piece(10, 5, 4, forced, slots, shared, true) == (forced < 6 ? forced & ~1 : 6));
        }
        // even, at least 2, at most the largest window; also at the limits
        for (int64_t n : {0ll, 1ll, 100ll, 1ll << 20, 2147483647ll})
            for (int32_t T : {1, 3, 1000, 134217728})
                for (int32_t m : {0, 1, 2, 17, 65536, 134217727}) {
                    const int32_t piece = plan_piece(n, m, T, 0, slots, shared, false);
                    CHECK(piece >= 2 && piece % 2 == 0 && piece <= (m > 2 ? m + (m & 1) : 2));
                }
    }
    printf("piece size\n");
    return 0;
}

int main()
{
    if (work_list_check() || piece_rule()) return 1;
    printf("ok\n");
    return 0;
}
