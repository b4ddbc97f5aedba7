// How an ordering call's plan of scratch memory gives way where memory is short (built and run by
// tests/test_order_native.py; no GPU).  A traversal takes 36 bytes a node, two bitmaps, and 6 bytes an edge of its window.
#include <cstdio>

#include "bgl_order_plan.h"

using namespace bgl;

static int64_t traversal(int64_t nodes, int64_t edges, int64_t window)
{
    return 36 * nodes + nodes / 4 + 6 * std::min(edges, window) + 400'000;
}

int main()
{
    int bad = 0;
    auto check = [&](bool ok, const char *what, int64_t nodes, int64_t edges, int sequences) {
        if (!ok) {
            printf("%s: %lld nodes, %lld edges, %d sequences\n", what, (long long)nodes, (long long)edges, sequences);
            bad = 1;
        }
    };
    for (int64_t nodes : {1ll, 100'000ll, 1'000'000ll, 2'000'000ll, 2'450'000ll, 5'000'000ll, 30'000'000ll, 111'000'000ll})
        for (int64_t edges : {0ll, 1ll << 20, 1ll << 23, (1ll << 23) + 1, 1ll << 24, 1ll << 27})
            for (int sequences : {1, 2, 3, 5, 10, 16, 17, 100}) {
                const int64_t shared = nodes / 8 + 4 * (nodes / 10);
                const auto plans = order_plans(sequences, edges, shared, [&](int64_t w) { return traversal(nodes, edges, w); });
                const int64_t least = traversal(nodes, edges, ORDER_SMALL_WINDOW);
                check(!plans.empty(), "no plan", nodes, edges, sequences);
                int64_t before = INT64_MAX;
                for (const OrderPlan &p : plans) {
                    const int64_t all = p.side * traversal(nodes, edges, p.window);
                    check(p.side >= 1 && p.side <= sequences && p.side <= ORDER_SIDE_BY_SIDE, "traversals", nodes, edges, sequences);
                    check(p.window == ORDER_WINDOW || p.window == ORDER_SMALL_WINDOW, "window", nodes, edges, sequences);
                    check(p.side == 1 || all <= ORDER_SIDE_BY_SIDE_BYTES, "more than they may take", nodes, edges, sequences);
                    check(all < before, "asked for as much again", nodes, edges, sequences);
                    before = all;
                }
                // what the graph can keep with one of the windows is kept
                const int all_of_them = std::min(sequences, ORDER_SIDE_BY_SIDE);
                if (shared + all_of_them * least <= ORDER_KEEP_BYTES)
                    check(plans[0].side == all_of_them && shared + all_of_them * traversal(nodes, edges, plans[0].window) <= ORDER_KEEP_BYTES,
                          "allocated in each call", nodes, edges, sequences);
                // nothing smaller would do: a call that fits with one traversal and the smaller window goes through
                check(before == least, "not the least a call can do with", nodes, edges, sequences);
                // no traversal is given up where the smaller window makes room
                for (size_t k = 1; k < plans.size(); ++k)
                    check(plans[k].side == plans[k - 1].side || plans[k - 1].window == ORDER_SMALL_WINDOW || edges <= ORDER_SMALL_WINDOW,
                          "a traversal is given up before the window", nodes, edges, sequences);
            }
    if (!bad) printf("ok\n");
    return bad;
}
