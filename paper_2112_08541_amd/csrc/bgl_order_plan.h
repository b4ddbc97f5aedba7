// How much scratch an ordering call takes: edges per step and traversals side by side.  Sizes only, no device code, so that
// it can be tested without a GPU.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace bgl {

// Edges per step at most: the larger window where the scratch of all traversals of a call fits then (fewer steps: two
// sequences on 2.45 M nodes 3.8 -> 3.6 ms, k_expand 2,390 -> 2,300 us, k_count 545 -> 460, k_append 480 -> 410; twice as
// large again 2,280 / 434 / 355), else the smaller one (ten on 1 M nodes, seven of them side by side: 6.1 -> 7.3).
constexpr int64_t ORDER_WINDOW = 1 << 24, ORDER_SMALL_WINDOW = 1 << 23;
constexpr int ORDER_SIDE_BY_SIDE = 16;                  // traversals that share their launches at most
constexpr int64_t ORDER_SIDE_BY_SIDE_BYTES = 1ll << 30;  // and the memory they may take together (one alone: whatever it needs)
constexpr int64_t ORDER_KEEP_BYTES = 512ll << 20;       // a graph keeps a scratch of at most this for its next call

struct OrderPlan {
    int64_t window;
    int side;  // traversals that run side by side
};

// The plans of a call of num_sequences on num_edges edges, the one to take first in front, each of the others for when there
// is no memory for the one before it: the larger window is given up before any traversal, and the last plan is one traversal
// with the smaller window.  bytes_of(window): scratch of one traversal; shared_bytes: what a call's traversals share.
//   The larger window is not taken either where it alone makes the scratch too large to be kept: allocating it in each call
// costs more than fewer steps give.  ms a call with the larger window, allocated / the smaller one, kept: three sequences on
// 2.45 M nodes / 122 M edges 4.10 / 3.50, on 3 M / 60 M 5.50 / 4.91, two on 5 M / 75 M 4.83 / 4.27, four on 2 M / 60 M 4.90 / 3.85,
// five on 1 M / 12 M 2.72 / 2.19.
template <typename Bytes>
std::vector<OrderPlan> order_plans(int32_t num_sequences, int64_t num_edges, int64_t shared_bytes, Bytes &&bytes_of)
{
    const int wanted = (int)std::min<int32_t>(num_sequences, ORDER_SIDE_BY_SIDE);
    const int64_t large = bytes_of(ORDER_WINDOW) * wanted, small = bytes_of(ORDER_SMALL_WINDOW) * wanted;
    const bool kept_if_small_only = shared_bytes + small <= ORDER_KEEP_BYTES && shared_bytes + large > ORDER_KEEP_BYTES;
    std::vector<OrderPlan> plans;
    if (large <= ORDER_SIDE_BY_SIDE_BYTES && !kept_if_small_only) plans.push_back({ORDER_WINDOW, wanted});
    // Side by side a traversal's small steps, which are launches and latency, cost next to nothing beside
    // the others'.  Where the memory for that is not there, fewer at a time.
    const int most = (int)std::max<int64_t>(1, std::min<int64_t>(wanted, ORDER_SIDE_BY_SIDE_BYTES / bytes_of(ORDER_SMALL_WINDOW)));
    for (int side = most;; side = (side + 1) / 2) {
        // (both windows hold all edges of a small graph: the same plan)
        if (plans.empty() || plans.back().side != side || num_edges > ORDER_SMALL_WINDOW) plans.push_back({ORDER_SMALL_WINDOW, side});
        if (side == 1) return plans;
    }
}

}  // namespace bgl
