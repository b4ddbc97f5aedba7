// Proximity-aware ordering of the training nodes (BGL paper, Sec. 3.2.2):
// several BFS sequences over the training nodes from given roots, each read from
// a given offset, merged into batches in turn.  The traversals run on the GPU;
// the merge (a strictly sequential scan over a few hundred thousand ids) and the
// shuffling-error statistic run on the host.
//
// BFS order is the first-in-first-out queue order (neighbors in CSR row order,
// restart at the smallest unvisited id).  Number the out-edges of a level's nodes
// in queue order, row by row: the next level is the not yet visited targets in the
// order of the first edge that reaches each.  So a level is
//   k_expand   every edge whose target is unvisited lowers the target's key to its
//              own number (atomicMin); the edges that lowered a key are the only
//              ones that can be a first edge and go to a candidate list
//   k_count    candidates whose number is still their target's key are the first
//              edges; totals (nodes, out-edges, training nodes) per workgroup
//   k_append   prefixes of those totals give every new node its place: the next
//              frontier and the training-node sequence are written in order
// No sort, and the sizes stay on the device: the host enqueues steps (three
// launches each) a few ahead of the one that the device says, in page-locked
// words, it has come to.
//   Every wavefront owns a contiguous run of EDGES, not of nodes: out-degrees are
// a power law, and with a fixed number of lanes per node the longest row sets the
// pace (16 lanes on a row of 20,000 edges: 1.9 ms for one level).  Measured, two
// sequences on 2.45 M nodes / 122 M edges: 26 to 28 ms with 16 lanes per node and a
// radix sort per level, 2.5 to 3.8 ms now, by the host (a graph handle's first call: OrderScratch; k_expand 2.3 ms,
// 100 G edges/s: 262 M reads that reach an L2, which serves random ones at 267 G/s when they hit and 58 G/s when they miss, 14 %
// of these, and 10 M atomics, which the chip does 27 G/s of wherever they go); five sequences on 100,000 nodes / 1 M edges,
// where launches and host round trips count: 14 to 19 and 0.46 to 0.50 ms.
//   The sequences of a call are independent traversals and share their launches (blockIdx.y): one after the
// other, the five took 1.7 ms, the two 4.8.
//   A level is handled in windows of at most WINDOW edges, which bounds the lists (6 bytes an edge) whatever the
// graph's size; a target reached in one window is visited in the next.
//   When the frontier is empty the same three kernels restart the traversal.
// Nodes all of whose out-neighbors are visited ("closed") would each be a one-node
// traversal; all closed nodes below the smallest open node are taken in one step,
// in id order, which is what the sequential rule does: k_expand finds the smallest
// open node, k_count and k_append walk the bitmap words below it.
#include <algorithm>
#include <climits>
#include <cstring>
#include <vector>

#include "bgl_internal.h"
#include "bgl_order_merge.h"

namespace {

using namespace bgl;

constexpr int BT = 256;
constexpr int BW = BT / kWave;               // wavefronts per workgroup
// Workgroups of a step's kernels for one or two traversals, half as many each where there are more (those without a share leave
// at once, but 40,000 of them cost a launch 10 us).  k_expand, two on 2.45 M nodes, with 1,024 / 2,048 / 4,096: 2,533 / 2,400 / 2,355 us.
constexpr int BLOCKS = 4096;
// Of all traversals of a launch together on a graph of few edges, whose steps are launches and latency: as many as run at a time.
// Before / with these, us a call: five on 100,000 nodes / 1 M edges 523 / 473, 3 M edges 612 / 497, 300,000 nodes / 6 M 1,153 / 1,016;
// ten 765 / 635, 906 / 700, 1,807 / 1,642; two on 6 M edges 710 / 668, 12 M 843 / 792.  Elsewhere the larger steps lose as much as the small
// ones gain (five on 24 M edges 3,001 / 3,120, two on 3 M 390 / 402, on 24 M 1,589 / 1,595), and one traversal is level throughout.
// Within, a few large steps lose too: two on 100,000 nodes / 16 M edges 390 / 413, sixteen on 400,000 / 7 M 4,150 / 4,250; three, four and
// seven on 0.2 to 8 M edges 250 to 2,410 / 256 to 2,240.
// (No multiple of 8 each, or the first workgroups of all traversals, in small steps the only ones with work, share an XCD: ten on
// 30,000 nodes / 0.3 M edges with 256 each 466 instead of 360.)
constexpr int RESIDENT_BLOCKS = 2048;
constexpr int WAVES = BLOCKS * BW;
constexpr int GROUPS = BLOCKS / kWave;       // groups of 64 workgroups whose totals are added up
static_assert(GROUPS <= kWave && BW >= 2, "a wavefront sums the groups, another one a group's workgroups");
constexpr int WTILE = 4 * kWave;             // edges a wavefront handles at a time, four per lane
constexpr int64_t WINDOW = ORDER_WINDOW;       // edges per step at most (bgl_order_plan.h)
constexpr int SEARCH_BLOCKS = 256;           // workgroups that look for the restart node
constexpr int SHORT_ROW = 32;                // edges of a row that one lane walks by itself
constexpr int64_t STEPS_AHEAD = 4;           // steps the host enqueues ahead of the device
constexpr int64_t MERGE_ENTRIES = 2048;      // entries the merge looks at (1.5 to 4 ns each) between two looks at how far the device is
constexpr int SIDE_BY_SIDE = ORDER_SIDE_BY_SIDE;
static_assert((1 << 23) / ((RESIDENT_BLOCKS / SIDE_BY_SIDE / 8 * 8 - 3) * BW) + WTILE <= 1 << 16, "a share's edges have 16 bits");
constexpr size_t PAGE_LOCKED_SEQ_BYTES = 32 << 20;  // sequences of a call that still go to page-locked memory
// A node's key: below WINDOW the smallest edge of the current window that reaches it (it is visited by the
// end of the step), else none, and the excess says how many leading edges of its own row are known to end
// at visited nodes (search_open; rows have fewer than 2^31 edges).
constexpr uint32_t NO_KEY = (uint32_t)WINDOW;

// What a step finds.  Step s reads copy s & 1; its last kernel writes the other.
struct Step {
    unsigned long long edges;       // out-edges of the current level's nodes
    unsigned long long win_lo;      // first one of this step's window
    unsigned long long next_edges;  // out-edges of the next level's nodes found so far
    uint32_t rows;                  // nodes of the current level that have out-edges; 0: restart
    uint32_t next_rows;             // the same for the next level so far
    int32_t seq_len;                // training nodes recorded so far
    int32_t scan_lo;                // every node below is visited
    uint32_t buf;                   // which frontier buffer holds the current level
    uint32_t done;
};

struct OrderDev {
    Step step[2];
    int open_min;   // restart: smallest unvisited node that has an unvisited out-neighbor
};

// What the host sees of a traversal (page-locked memory).
struct Progress {
    uint64_t begun;   // the last step that has begun to append, from 1, << 32 | training nodes that the steps before it have recorded
    uint32_t done;    // the traversal has ended
    int32_t seq_len;  // then: training nodes recorded
    int32_t status;   // of the call, in the first one's
};

// One level's nodes that have out-edges, in queue order.
struct Frontier {
    unsigned long long *off;   // edges before this node's row
    int64_t *base;             // the row's first column index - off
};

// New nodes of a window: how many have out-edges (upper half) and how many are training nodes (lower half; a
// window has fewer than 2^31 of either), and their out-edges.
struct Totals {
    unsigned long long nodes, edges;
    __device__ __forceinline__ uint32_t rows() const { return (uint32_t)(nodes >> 32); }
    __device__ __forceinline__ uint32_t train() const { return (uint32_t)nodes; }
    __device__ __forceinline__ Totals &operator+=(const Totals &o) { nodes += o.nodes; edges += o.edges; return *this; }
};

// The lists and totals of a step: one share per wavefront.
struct Lists {
    uint32_t *node;                // as many entries as a window has edges: k_expand: targets; k_count: new nodes
    uint16_t *edge;                // beside the targets: their edges, from the share's first one on
    uint32_t *n_cand, *n_win;      // per wavefront
    Totals *wave, *block;          // of a wavefront's, of a workgroup's first edges
    Totals *group;                 // of 64 workgroups'
};

// What one traversal works on.  The traversals of a call run side by side, blockIdx.y says which: their
// memory has the same layout, `stride` bytes apart.
struct Traversal {
    uint32_t *visited, *closed, *key;
    Frontier f0, f1;
    Lists li;
    OrderDev *dev;
    int32_t *seq;       // num_train ids each, densely packed (page-locked memory, unless they are too many)
    Progress *host;     // one each
    int64_t stride, num_train, window;
    int32_t blocks;     // workgroups that a step is dealt to, at most BLOCKS

    __device__ __forceinline__ uint32_t edges_of(const Step &st) const { return (uint32_t)min((unsigned long long)window, st.edges - st.win_lo); }
    __device__ __forceinline__ Traversal mine() const
    {
        Traversal t = *this;
        const int64_t by = (int64_t)blockIdx.y * stride;
        auto move = [&](auto *&p) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(reinterpret_cast<char *>(p) + by); };
        move(t.visited), move(t.closed), move(t.key);
        move(t.f0.off), move(t.f0.base), move(t.f1.off), move(t.f1.base);
        move(t.li.node), move(t.li.edge), move(t.li.n_cand), move(t.li.n_win);
        move(t.li.wave), move(t.li.block), move(t.li.group);
        move(t.dev);
        t.seq += (int64_t)blockIdx.y * num_train;
        t.host += blockIdx.y;
        return t;
    }
};
struct Roots {
    int32_t of[SIDE_BY_SIDE];
};

__device__ __forceinline__ bool test_bit(const uint32_t *bm, uint32_t v) { return (bm[v >> 5] >> (v & 31)) & 1u; }

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void k_set_bits(const int32_t *ids, int64_t n, int64_t num_nodes, uint32_t *bm, uint32_t *refused, Progress *host)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = ids[i];
    const uint32_t bit = 1u << (v & 31);
    if (v < 0 || (int64_t)v >= num_nodes || (atomicOr(&bm[(uint32_t)v >> 5], bit) & bit)) {  // foreign, or listed twice
        *refused = 1;
        host->status = BGL_EINVAL;
    }
}

// A fresh traversal from its root: no keys, nothing visited but the root (bits at and above num_nodes
// count as visited), the root's row as the first level.  Where the training ids have been refused (the word
// behind their bitmap) it is over before its first step.
template <typename RP>
__global__ __launch_bounds__(BT) void k_reset(const RP *__restrict__ row_ptr, Roots roots, int64_t words, int64_t num_nodes,
                                              const uint32_t *__restrict__ train, Traversal all)
{
    const Traversal me = all.mine();
    if (train[words]) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            me.dev->step[0] = me.dev->step[1] = Step{0, 0, 0, 0, 0, 0, 0, 0, 1};
            __hip_atomic_store(&me.host->done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return;
    }
    const int32_t root = roots.of[blockIdx.y];
    uint32_t *visited = me.visited, *closed = me.closed, *key = me.key;
    const Frontier f = me.f0;
    OrderDev *dev = me.dev;
    const int64_t t = (int64_t)blockIdx.x * BT + threadIdx.x, stride = (int64_t)gridDim.x * BT;
    for (int64_t w = t; w < words; w += stride) {
        uint32_t v = 0;
        const int64_t base = w * 32;
        if (base + 32 > num_nodes) v = num_nodes > base ? ~0u << (uint32_t)(num_nodes - base) : ~0u;
        if (w == root >> 5) v |= 1u << (root & 31);
        visited[w] = v;
        closed[w] = 0;
    }
    for (int64_t i = t; i < num_nodes; i += stride) key[i] = NO_KEY;
    if (t == 0) {
        const int64_t lo = (int64_t)row_ptr[root], d = (int64_t)row_ptr[root + 1] - lo;
        f.off[0] = 0;
        f.base[0] = lo;
        const bool tr = test_bit(train, (uint32_t)root);
        if (tr) me.seq[0] = root;
        dev->step[0] = Step{(unsigned long long)d, 0, 0, d > 0 ? 1u : 0u, 0, tr ? 1 : 0, 0, 0, 0};
        dev->open_min = INT_MAX;
    }
}

// The share of each wavefront in a step's window: a multiple of WTILE edges.
__device__ __forceinline__ uint32_t edges_per_wave(uint32_t win, int blocks)
{
    const uint32_t all = (uint32_t)blocks * (BW * WTILE);
    return (win + all - 1) / all * WTILE;
}

// Number of rows whose edges begin before x, by the whole wavefront: 64 probes a round.
__device__ __forceinline__ uint32_t rows_before(const unsigned long long *off, uint32_t rows, unsigned long long x)
{
    const uint32_t lane = threadIdx.x & (kWave - 1);
    uint32_t lo = 0, n = rows;  // the answer is in [lo, lo + n]
    while (n > 0) {
        const uint32_t s = (n + kWave - 1) / kWave;  // lane l looks at the last row of its part of s rows
        const uint32_t i = min(lane * s + s - 1, n - 1);
        const bool before = lane * s < n && off[lo + i] < x;
        const uint32_t parts = (uint32_t)__popcll(__ballot(before));  // parts that lie wholly before x
        const uint32_t skip = min(parts * s, n);
        lo += skip;
        n = min(s - 1, n - skip);
    }
    return lo;
}

// Does one of eight edges, e, e + step, ..., lead from v to an unvisited node other than v?  Edges from hi on
// read the last one again.  The eight reads are in flight together.
__device__ __forceinline__ bool open_edge(const int32_t *__restrict__ col, const uint32_t *__restrict__ visited, int64_t v,
                                          int64_t e, int step, int64_t hi)
{
    uint32_t u[8], seen[8];
    bool open = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) u[j] = (uint32_t)col[min(e + j * step, hi - 1)];
#pragma unroll
    for (int j = 0; j < 8; ++j) seen[j] = visited[u[j] >> 5] >> (u[j] & 31);
#pragma unroll
    for (int j = 0; j < 8; ++j) open |= (int64_t)u[j] != v && !(seen[j] & 1u);
    return open;
}

// The smallest unvisited node with an unvisited out-neighbor other than itself.  A wavefront takes
// 64 ids at a time, ascending: every lane walks one node's row if it is short, then 16 lanes walk each of
// the longer rows, eight reads in flight per lane (with 16 lanes for every row a wavefront looks at few
// nodes at a time: calls on 10 M nodes of one edge / 4 M of 20 edges, all closed, 2.5 / 1.7 ms, 1.1 / 0.9
// now); nobody
// goes on beyond the smallest open node found so far.  The visited set only grows, so a node found closed
// stays closed and is not looked at again, and the leading edges of a row that are known to end at visited
// nodes (their number is kept in the node's key) are not read again: a graph has a restart for every component that no other
// one leads to, some rows of the nodes in between are long, and over a traversal a row is walked once.
// (2.45 M nodes / 122 M edges, 110 restarts per traversal: 130 to 300 us a search that walks the closed
// nodes again each time with one read per lane, 30 to 55 now; five such traversals in a row 118 -> 40 ms.  A row of
// 200,000 edges, the last one open, behind 300 components of two nodes: 203 -> 26 ms.)
template <typename RP>
__device__ __forceinline__ void search_open(const RP *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                            const uint32_t *__restrict__ visited, uint32_t *closed, uint32_t *key,
                                            int64_t num_nodes, int64_t scan_lo, OrderDev *dev)
{
    const int blocks = min((int)gridDim.x, SEARCH_BLOCKS);
    if ((int)blockIdx.x >= blocks) return;
    const int lane = threadIdx.x & (kWave - 1), l = lane & 15, gshift = lane & ~15;
    const int64_t wave = (int64_t)blockIdx.x * BW + threadIdx.x / kWave;
    for (int64_t c = scan_lo / 64 + wave; c * 64 < num_nodes; c += blocks * BW) {
        const int found = __hip_atomic_load(&dev->open_min, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (c * 64 >= __builtin_amdgcn_readfirstlane(found)) return;
        // (the bitmaps end with a whole number of 64-bit pairs; bits beyond the last id count as visited)
        const int64_t word = c * 2 + (lane >> 5), own = c * 64 + lane;
        const bool look = !(((visited[word] | closed[word]) >> (lane & 31)) & 1u);
        // one row per lane where it is short
        bool open = false, rest = false;
        if (look) {
            const int64_t lo = (int64_t)row_ptr[own], hi = (int64_t)row_ptr[own + 1], e = lo + (key[own] - NO_KEY);
            rest = hi - e > SHORT_ROW;
            for (int64_t k = e; k < hi && !rest && !open; k += 8) open = open_edge(col, visited, own, k, 1, hi);
        }
        const uint64_t opens = __ballot(open);
        const uint64_t shuts = __ballot(look && !open && !rest);
        if (opens && lane == __ffsll((unsigned long long)opens) - 1) atomicMin(&dev->open_min, (int)own);
        const uint32_t shut_word = (uint32_t)(shuts >> (lane & 32));
        if ((lane & 31) == 0 && shut_word) atomicOr(&closed[word], shut_word);
        // the longer ones before the first open node: 16 lanes per row
        const uint64_t longs = __ballot(rest) & (opens ? (opens & (0ull - opens)) - 1ull : ~0ull);
        uint32_t todo = (uint32_t)(longs >> gshift) & 0xffffu, shut = 0;
        for (; todo; todo &= todo - 1) {
            const int64_t v = c * 64 + gshift + (__ffs(todo) - 1);
            const int64_t lo = (int64_t)row_ptr[v], hi = (int64_t)row_ptr[v + 1];
            int64_t e = lo + (key[v] - NO_KEY);
            bool found_one = false;
            while (e < hi) {
                const bool mine = open_edge(col, visited, v, e + l, 16, hi);
                found_one = ((__ballot(mine) >> gshift) & 0xffffull) != 0;
                if (found_one) break;
                e += 128;
            }
            if (found_one) {
                if (l == 0) {
                    key[v] = NO_KEY + (uint32_t)(e - lo);
                    atomicMin(&dev->open_min, (int)v);
                }
                break;
            }
            shut |= todo & (0u - todo);
        }
        if (shut && l == 0) atomicOr(&closed[c * 2 + (gshift >> 5)], shut << (gshift & 16));
    }
}

template <typename RP>
__global__ __launch_bounds__(BT) void k_expand(const RP *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                               int64_t num_nodes, Traversal all, int par)
{
    __shared__ uint32_t sh_start[BW][kWave];  // per wavefront: WTILE bytes, 1 where a row begins
    const Traversal me = all.mine();
    OrderDev *const dev = me.dev;
    const Lists &li = me.li;
    const uint32_t *__restrict__ visited = me.visited;
    uint32_t *const key = me.key;
    const Step st = dev->step[par];
    if (st.done) return;
    if (blockIdx.x == 0 && threadIdx.x < GROUPS) li.group[threadIdx.x] = Totals{0, 0};  // for k_count
    if (st.rows == 0) {
        search_open(row_ptr, col, visited, me.closed, key, num_nodes, st.scan_lo, dev);
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) dev->open_min = INT_MAX;  // for the next restart
    const Frontier f = st.buf ? me.f1 : me.f0;
    const uint32_t win = me.edges_of(st);
    const uint32_t per = edges_per_wave(win, me.blocks);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t wave = blockIdx.x * BW + w;
    const unsigned long long lo64 = (unsigned long long)wave * per;
    if (lo64 >= win) return;  // (no barrier in this kernel: wavefronts are on their own)
    const uint32_t lo = (uint32_t)lo64, hi = min(lo + per, win);
    uint8_t *start = reinterpret_cast<uint8_t *>(sh_start[w]);
    uint32_t before = rows_before(f.off, st.rows, st.win_lo + lo);  // rows that begin before the tile
    uint32_t n_cand = 0;
    for (uint32_t t0 = lo; t0 < hi; t0 += WTILE) {
        const unsigned long long x0 = st.win_lo + t0;
        sh_start[w][lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // rows that begin inside the tile (every row has an edge: at most WTILE of them)
        for (uint32_t j = 0; j < WTILE; j += kWave) {
            const uint32_t r = before + j + lane;
            const unsigned long long o = r < st.rows ? f.off[r] - x0 : (unsigned long long)WTILE;
            if (o < WTILE) start[o] = 1;
            if (__ballot(o < WTILE) != ~0ull) break;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t row[4], u[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t b = __ballot(start[j * kWave + lane] != 0);
            row[j] = before + (uint32_t)__popcll(b & (~0ull >> (63 - lane))) - 1;
            before += (uint32_t)__popcll(b);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint32_t row0 = __builtin_amdgcn_readfirstlane(row[0]);
        int64_t at[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // lanes beyond the end of the share read the tile's first edge again and drop it
            const uint32_t k = t0 + j * kWave + lane;
            at[j] = f.base[k < hi ? row[j] : row0] + (int64_t)(st.win_lo + (k < hi ? k : t0));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = (uint32_t)col[at[j]];
        uint32_t seen[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) seen[j] = visited[u[j] >> 5];
        bool cand[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t k = t0 + j * kWave + lane;
            cand[j] = false;
            // (a stale key can only be too large: then the atomic is made for nothing)
            if (k < hi && !((seen[j] >> (u[j] & 31)) & 1u) &&
                __hip_atomic_load(&key[u[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > k)
                cand[j] = atomicMin(&key[u[j]], k) > k;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t b = __ballot(cand[j]);
            if (cand[j]) {
                const uint32_t at = lo + n_cand + (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
                li.node[at] = u[j];
                li.edge[at] = (uint16_t)(t0 - lo + j * kWave + lane);
            }
            n_cand += (uint32_t)__popcll(b);
        }
    }
    if (lane == 0) li.n_cand[wave] = n_cand;
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}
__device__ __forceinline__ Totals wave_sum(const Totals &t) { return Totals{wave_sum(t.nodes), wave_sum(t.edges)}; }

// Restart: the bitmap words that may hold closed nodes to take, an equal run of them per workgroup.
struct WordRange {
    int64_t first, per, end;
    __device__ __forceinline__ WordRange(int64_t scan_lo, int open_min, int64_t words, int blocks)
    {
        first = scan_lo >> 5;
        end = open_min == INT_MAX ? words : ((int64_t)open_min >> 5) + 1;
        const int64_t n = end - first;
        per = (n + (int64_t)blocks * BT - 1) / ((int64_t)blocks * BT) * BT;
    }
    __device__ __forceinline__ int64_t begin_of(int64_t block) const { return first + block * per; }
    __device__ __forceinline__ int64_t end_of(int64_t block) const { return min(first + (block + 1) * per, end); }
};
// Unvisited ids of word w below the smallest open node: all of them are closed.
__device__ __forceinline__ uint32_t closed_bits(uint32_t visited_word, int64_t w, int open_min)
{
    uint32_t m = ~visited_word;
    if (w * 32 + 32 > (int64_t)open_min) m &= (1u << (uint32_t)(open_min - w * 32)) - 1u;
    return m;
}

template <typename RP>
__global__ __launch_bounds__(BT) void k_count(const RP *__restrict__ row_ptr, int64_t words,
                                              const uint32_t *__restrict__ train, Traversal all, int par)
{
    typedef RP Ends __attribute__((ext_vector_type(2), aligned(sizeof(RP))));  // of a row, with one read
    __shared__ Totals sh[BW];
    const Traversal me = all.mine();
    const OrderDev *const dev = me.dev;
    const Lists &li = me.li;
    const uint32_t *__restrict__ visited = me.visited;
    const uint32_t *__restrict__ key = me.key;
    const Step st = dev->step[par];
    if (st.done) return;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    Totals mine = {0, 0};
    if (st.rows == 0) {
        const WordRange wr(st.scan_lo, dev->open_min, words, me.blocks);
        if (wr.begin_of(blockIdx.x) >= wr.end) return;
        for (int64_t i = wr.begin_of(blockIdx.x) + threadIdx.x; i < wr.end_of(blockIdx.x); i += BT)
            mine.nodes += (uint32_t)__popc(closed_bits(visited[i], i, dev->open_min) & train[i]);
        mine = wave_sum(mine);
    } else {
        const uint32_t win = me.edges_of(st);
        const uint32_t per = edges_per_wave(win, me.blocks);
        if ((unsigned long long)blockIdx.x * BW * per >= win) return;  // whole workgroups
        const uint32_t wave = blockIdx.x * BW + w;
        const bool active = (unsigned long long)wave * per < win;
        const uint32_t lo = active ? wave * per : 0, n = active ? li.n_cand[wave] : 0;
        uint32_t n_win = 0;
        // The nodes of first edges move to the front of the wavefront's own list, in order.  Four groups of 64 candidates at a
        // time: their keys, then their rows, are in flight together.
        for (uint32_t i0 = 0; i0 < n; i0 += 4 * kWave) {
            uint32_t u[4], e[4], k[4], tr[4];
            bool first[4];
            Ends ends[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t at = lo + min(i0 + j * kWave + lane, n - 1);
                u[j] = li.node[at];
                e[j] = lo + li.edge[at];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) k[j] = key[u[j]];
#pragma unroll
            for (int j = 0; j < 4; ++j) {  // (candidates that are no first edge look at node 0)
                first[j] = i0 + j * kWave + lane < n && k[j] == e[j];
                const uint32_t v = first[j] ? u[j] : 0;
                ends[j] = *reinterpret_cast<const Ends *>(row_ptr + v);
                tr[j] = train[v >> 5] >> (v & 31) & 1u;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint64_t b = __ballot(first[j]);
                if (first[j]) {
                    li.node[lo + n_win + __popcll(b & ((1ull << lane) - 1ull))] = u[j];
                    const uint32_t degree = (uint32_t)(ends[j].y - ends[j].x);  // (less than 2^31: checked when the graph is loaded)
                    mine += Totals{(unsigned long long)(degree > 0) << 32 | tr[j], degree};
                }
                n_win += (uint32_t)__popcll(b);
            }
        }
        mine = wave_sum(mine);
        if (lane == 0) {
            li.n_win[wave] = n_win;
            li.wave[wave] = mine;
        }
    }
    if (lane == 0) sh[w] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        Totals all = {0, 0};
#pragma unroll
        for (int k = 0; k < BW; ++k) all += sh[k];
        li.block[blockIdx.x] = all;
        Totals *group = &li.group[blockIdx.x / kWave];
        if (all.nodes) atomicAdd(&group->nodes, all.nodes);
        if (all.edges) atomicAdd(&group->edges, all.edges);
    }
}

// Totals of the workgroups before this one and of all, by the whole workgroup: one wavefront sums the groups, another the
// workgroups before this one in its own group.  (With every workgroup adding up the totals of all 2,048, two
// traversals of 2.45 M nodes / 122 M edges spend 676 us in k_append and 500 in k_count, now 472 and 574.)
struct Before {
    Totals before, all;
    __device__ __forceinline__ Before(const Lists &li, uint32_t block, Totals *sh)  // sh: three
    {
        const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, group = block / kWave;
        if (w == 0) {
            const Totals g = lane < GROUPS ? li.group[lane] : Totals{0, 0};
            const Totals every = wave_sum(g), lower = wave_sum(lane < group ? g : Totals{0, 0});
            if (lane == 0) { sh[0] = every; sh[1] = lower; }
        } else if (w == 1) {
            const Totals own = wave_sum(group * kWave + lane < block ? li.block[group * kWave + lane] : Totals{0, 0});
            if (lane == 0) sh[2] = own;
        }
        __syncthreads();
        all = sh[0];
        before = sh[1];
        before += sh[2];
    }
};

template <typename RP>
__global__ __launch_bounds__(BT) void k_append(const RP *__restrict__ row_ptr, int64_t num_nodes, int64_t words,
                                               const uint32_t *__restrict__ train, Traversal all, int par, uint32_t step)
{
    typedef RP Ends __attribute__((ext_vector_type(2), aligned(sizeof(RP))));  // of a row, with one read
    __shared__ Totals sh[3];
    __shared__ int sh_scan[BW];
    const Traversal me = all.mine();
    OrderDev *const dev = me.dev;
    const Lists &li = me.li;
    uint32_t *const visited = me.visited;
    int32_t *const seq = me.seq;
    Progress *const host = me.host;
    const Step st = dev->step[par];
    Step &next = dev->step[par ^ 1];
    if (st.done) {
        if (blockIdx.x == 0 && threadIdx.x == 0) next = st;
        return;
    }
    // A workgroup beyond the others' says that the step is under way, so that the host may enqueue another, and what the
    // ones before it have recorded, so that the host may read that part of the sequence.
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x == 0)
            __hip_atomic_store(&host->begun, (uint64_t)step << 32 | (uint32_t)st.seq_len, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (st.rows == 0) {
        const int open = dev->open_min;
        const WordRange wr(st.scan_lo, open, words, me.blocks);
        if (blockIdx.x > 0 && wr.begin_of(blockIdx.x) >= wr.end) return;
        const Before t(li, blockIdx.x, sh);
        int32_t o = st.seq_len + (int32_t)t.before.train();
        for (int64_t i0 = wr.begin_of(blockIdx.x); i0 < wr.end_of(blockIdx.x); i0 += BT) {  // uniform in the workgroup
            const int64_t i = i0 + threadIdx.x;
            uint32_t m = 0;
            if (i < wr.end_of(blockIdx.x)) {
                const uint32_t v = visited[i];
                m = closed_bits(v, i, open);
                uint32_t now = v | m;
                if (open != INT_MAX && i == (int64_t)open >> 5) now |= 1u << (open & 31);
                if (now != v) visited[i] = now;
                m &= train[i];
            }
            int tot;
            int at = o + block_excl_scan<BT>(__popc(m), sh_scan, tot);
            for (; m; m &= m - 1) seq[at++] = (int32_t)(i * 32) + (__ffs(m) - 1);
            o += tot;
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            int32_t len = st.seq_len + (int32_t)t.all.train();
            if (open == INT_MAX) {  // everything that was left was closed
                next = Step{0, 0, 0, 0, 0, len, st.scan_lo, 0, 1};
                host->seq_len = len;
                __hip_atomic_store(&host->done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            } else {
                const int64_t lo = (int64_t)row_ptr[open], d = (int64_t)row_ptr[open + 1] - lo;
                me.f0.off[0] = 0;
                me.f0.base[0] = lo;
                if (test_bit(train, (uint32_t)open)) seq[len++] = open;
                next = Step{(unsigned long long)d, 0, 0, d > 0 ? 1u : 0u, 0, len, open, 0, 0};
            }
        }
        return;
    }
    const uint32_t win = me.edges_of(st);
    const uint32_t per = edges_per_wave(win, me.blocks);
    if ((unsigned long long)blockIdx.x * BW * per >= win) return;
    const Before t(li, blockIdx.x, sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        Step n = st;
        n.next_rows += t.all.rows();
        n.next_edges += t.all.edges;
        n.seq_len += (int32_t)t.all.train();
        n.win_lo += (unsigned long long)me.window;
        if (n.win_lo >= st.edges) {  // that was the level's last window
            n.edges = n.next_edges;
            n.rows = n.next_rows;
            n.win_lo = n.next_edges = 0;
            n.next_rows = 0;
            n.buf ^= 1;
        }
        next = n;
    }
    const uint32_t wave = blockIdx.x * BW + w;
    // Where many nodes are new, the bitmap is brought up to date from the keys, 64 nodes a wavefront at a time, instead of with
    // an atomic for each (the chip does 27 G/s): from a 32nd of the nodes on (2.45 M nodes, the largest steps 90 -> 52 us, all
    // 447 -> 410), if enough wavefronts have a share for it (48 of them on 100,000 nodes: 8 -> 42).
    const uint32_t waves = (win + per - 1) / per;
    const bool bulk = t.all.rows() > (uint32_t)words && (int64_t)waves * (4 * kWave) >= num_nodes;
    if (bulk) {
        uint64_t *const visited64 = reinterpret_cast<uint64_t *>(visited);
        for (int64_t i = wave; wave < waves && i * 64 < num_nodes; i += waves) {
            const int64_t v = i * 64 + lane;
            const uint64_t b = __ballot(v < num_nodes && me.key[v] < NO_KEY);
            if (lane == 0 && b) visited64[i] |= b;
        }
    }
    if ((unsigned long long)wave * per >= win) return;
    Totals at = t.before;
    for (uint32_t k = blockIdx.x * BW; k < wave; ++k) at += li.wave[k];  // the wavefronts before this one in its workgroup
    const Frontier f = st.buf ? me.f0 : me.f1;  // the next level's
    uint32_t row = st.next_rows + at.rows();
    unsigned long long edge = st.next_edges + at.edges;
    int32_t pos = st.seq_len + (int32_t)at.train();
    const uint32_t n = li.n_win[wave], lo = wave * per;
    for (uint32_t i0 = 0; i0 < n; i0 += 4 * kWave) {  // four groups of 64 at a time, as in k_count
        uint32_t nodes[4], trains[4];
        Ends ends[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) nodes[j] = li.node[lo + min(i0 + j * kWave + lane, n - 1)];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            ends[j] = *reinterpret_cast<const Ends *>(row_ptr + nodes[j]);
            trains[j] = train[nodes[j] >> 5] >> (nodes[j] & 31) & 1u;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool mine = i0 + j * kWave + lane < n;
            const uint32_t u = nodes[j], d = mine ? (uint32_t)(ends[j].y - ends[j].x) : 0u;
            const bool tr = mine && trains[j] != 0;
            const uint64_t has_row = __ballot(d > 0), is_train = __ballot(tr);
            const uint64_t below = (1ull << lane) - 1ull;
            unsigned long long inc = d;  // out-edges of the nodes up to this one
#pragma unroll
            for (int s = 1; s < kWave; s <<= 1) {
                const unsigned long long x = __shfl_up(inc, s, kWave);
                if (lane >= s) inc += x;
            }
            if (mine) {
                if (!bulk) atomicOr(&visited[u >> 5], 1u << (u & 31));
                if (d > 0) {
                    const uint32_t r = row + (uint32_t)__popcll(has_row & below);
                    f.off[r] = edge + inc - d;
                    f.base[r] = (int64_t)ends[j].x - (int64_t)(edge + inc - d);
                }
                if (tr) seq[pos + __popcll(is_train & below)] = (int32_t)u;
            }
            row += (uint32_t)__popcll(has_row);
            pos += (int32_t)__popcll(is_train);
            edge += __shfl(inc, kWave - 1, kWave);
        }
    }
}

struct OrderWork {
    const bgl_graph *g;
    Traversal t = {};            // of the first traversal
    int side = 1;                // traversals that run side by side
    uint32_t *train = nullptr;   // a bit per node, then a word that says whether the ids were refused
    int32_t *train_ids = nullptr;
    Progress *host = nullptr;    // page-locked, one per traversal
    int32_t *seqs = nullptr;     // host memory: num_train ids per sequence of the call
    int32_t *seqs_device = nullptr;  // the same as the device sees it, where it is page-locked: the kernels write there
    std::vector<int32_t> pageable;  // the same where they are too many to be page-locked
    bgl::OrderScratch scratch;   // what all of the above are carved from
    bool keep = false;           // nothing enqueued uses the scratch any more
    explicit OrderWork(const bgl_graph *g_) : g(g_) {}
    OrderWork(const OrderWork &) = delete;
    ~OrderWork()
    {
        if (!keep || !bgl::order_scratch_put(g, scratch)) bgl::order_scratch_free(scratch);
    }
};

int prepare(const bgl_graph *g, const int32_t *train_nodes, int64_t num_train, int num_sequences, OrderWork &w, hipStream_t st)
{
    const int64_t N = g->num_nodes, words = round_up(ceil_div(N, 32), 2);
    // one device allocation for the whole call, sized up front and carved into 256-byte aligned parts: what
    // the traversals share, then one equal part per traversal
    const size_t nt = (size_t)std::max<int64_t>(num_train, 1);
    const size_t seq_bytes = sizeof(int32_t) * nt * (size_t)num_sequences;
    size_t shared = 0, total = 0;
    char *at = nullptr;
    auto carve = [&](int side) {
        auto take = [&](auto *&p, size_t n) {
            p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(at + total);
            total += round_up(n * sizeof(*p), 256);
        };
        total = 0;
        take(w.train, (size_t)words + 1);
        take(w.train_ids, nt);
        if (seq_bytes > PAGE_LOCKED_SEQ_BYTES) take(w.t.seq, nt * (size_t)side);
        shared = total;
        take(w.t.visited, (size_t)words);
        take(w.t.closed, (size_t)words);
        take(w.t.key, (size_t)N);
        for (Frontier *f : {&w.t.f0, &w.t.f1}) {
            take(f->off, (size_t)N);
            take(f->base, (size_t)N);
        }
        const size_t win = (size_t)std::max<int64_t>(std::min<int64_t>(g->num_edges, w.t.window), 1);
        take(w.t.li.node, win);
        take(w.t.li.edge, win);
        take(w.t.li.n_cand, WAVES);
        take(w.t.li.n_win, WAVES);
        take(w.t.li.wave, WAVES);
        take(w.t.li.block, BLOCKS);
        take(w.t.li.group, GROUPS);
        take(w.t.dev, 1);
        w.t.stride = (int64_t)(total - shared);
        total = shared + (total - shared) * (size_t)side;
    };
    carve(1);  // (what is shared)
    const auto plans = order_plans(num_sequences, g->num_edges, (int64_t)shared, [&](int64_t window) {
        w.t.window = window;
        carve(1);
        return w.t.stride;
    });
    const size_t host_bytes = sizeof(Progress) * SIDE_BY_SIDE + (seq_bytes <= PAGE_LOCKED_SEQ_BYTES ? seq_bytes : 0);
    int rc = BGL_ENOMEM;
    for (size_t k = 0; k < plans.size() && rc == BGL_ENOMEM; ++k) {
        w.t.window = plans[k].window;
        w.side = plans[k].side;
        carve(w.side);
        rc = bgl::order_scratch_take(g, total, host_bytes, w.scratch);
    }
    if (rc != BGL_OK) return rc;
    at = static_cast<char *>(w.scratch.device);
    carve(w.side);
    w.t.num_train = num_train;
    w.host = static_cast<Progress *>(w.scratch.host);
    w.host[0].status = 0;
    BGL_HIP(hipHostGetDevicePointer((void **)&w.t.host, w.host, 0));
    const int32_t *ids = train_nodes;
    if (seq_bytes <= PAGE_LOCKED_SEQ_BYTES) {
        w.seqs = reinterpret_cast<int32_t *>(w.host + SIDE_BY_SIDE);
        w.seqs_device = reinterpret_cast<int32_t *>(w.t.host + SIDE_BY_SIDE);
        ids = static_cast<const int32_t *>(std::memcpy(w.seqs, train_nodes, sizeof(int32_t) * (size_t)num_train));
    } else {
        w.pageable.resize(nt * (size_t)num_sequences);
        w.seqs = w.pageable.data();
    }
    BGL_HIP(hipMemcpyAsync(w.train_ids, ids, sizeof(int32_t) * (size_t)num_train, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_fill_u32, dim3(std::min<int64_t>(ceil_div(words + 1, BT), 4096)), dim3(BT), 0, st, w.train, words + 1, 0u);
    // (nobody waits here: ids that are refused end the traversals before their first step, and the host looks then)
    hipLaunchKernelGGL(k_set_bits, dim3((unsigned)ceil_div(num_train, BT)), dim3(BT), 0, st, w.train_ids, num_train, N, w.train,
                       w.train + words, w.t.host);
    BGL_HIP(hipGetLastError());
    return BGL_OK;
}

// `count` <= w.side traversals side by side: sequences number first, first + 1, ... of the call.
template <typename RP>
int bfs_sequences(const bgl_graph *g, const int64_t *roots, int first, int count, int64_t num_train, OrderWork &w, hipStream_t st,
                  OrderMerge *merge)
{
    const int64_t N = g->num_nodes, words = round_up(ceil_div(N, 32), 2);
    const RP *rp = static_cast<const RP *>(g->row_ptr);
    const size_t one = (size_t)num_train;
    Traversal t = w.t;
    if (w.seqs_device) t.seq = w.seqs_device + one * (size_t)first;
    Roots r = {};
    for (int j = 0; j < count; ++j) {
        r.of[j] = (int32_t)roots[first + j];
        w.host[j].begun = w.host[j].done = 0;
    }
    const dim3 reset_grid((unsigned)std::min<int64_t>(ceil_div(N, BT), 4096), (unsigned)count);
    hipLaunchKernelGGL(k_reset<RP>, reset_grid, dim3(BT), 0, st, rp, r, words, N, w.train, t);
    // As many workgroups as the largest step of this graph has shares for.
    const int64_t shares = std::max({ceil_div(std::min(g->num_edges, w.t.window), WTILE * BW), ceil_div(words, BT),
                                     std::min<int64_t>(ceil_div(N, 64 * BW), SEARCH_BLOCKS), (int64_t)1});
    const bool small = count > 2 ? g->num_edges <= 1 << 23 : count == 2 && g->num_edges > 1 << 22 && g->num_edges <= 1 << 24;
    t.blocks = small ? RESIDENT_BLOCKS / count / 8 * 8 - 3 : count <= 2 ? BLOCKS : BLOCKS / 2;
    const dim3 grid((unsigned)std::min<int64_t>(shares, t.blocks), (unsigned)count);
    // The device says in page-locked words which step each traversal has come to and when it has ended; the
    // host stays STEPS_AHEAD steps ahead of the foremost, so the queue never runs empty and at most that many steps,
    // whose launches return at once, are enqueued beyond the end.  The calling thread merges what there is of the sequences
    // meanwhile (two of 204,800 on 2.45 M nodes: 4.25 -> 3.8 ms a call), or spins.  (A
    // synchronisation every 8 to 32 steps instead: 2.2 ms for five sequences of 13 steps on 100,000 nodes
    // one after the other, 1.7 with the words.)  Every step visits a
    // node or ends the traversal or is one of a level's windows.
    const int64_t most = 2 * N + g->num_edges / w.t.window + 4;
    auto word = [](const auto &x) { return __atomic_load_n(&x, __ATOMIC_ACQUIRE); };
    auto all_done = [&] {
        for (int j = 0; j < count; ++j)
            if (!word(w.host[j].done)) return false;
        return true;
    };
    auto come_to = [&] {
        uint64_t s = 0;
        for (int j = 0; j < count; ++j) {
            const uint64_t begun = word(w.host[j].begun);
            s = std::max(s, begun >> 32);
            if (merge && w.seqs_device) merge->there[(size_t)(first + j)] = (int64_t)(uint32_t)begun;
        }
        return (int64_t)s;
    };
    for (int64_t step = 1; !all_done(); ++step) {
        if (step > most + STEPS_AHEAD) BGL_FAIL(BGL_EHIP, "the traversal did not end");
        const int par = (int)((step - 1) & 1);
        hipLaunchKernelGGL(k_expand<RP>, grid, dim3(BT), 0, st, rp, g->col, N, t, par);
        hipLaunchKernelGGL(k_count<RP>, grid, dim3(BT), 0, st, rp, words, w.train, t, par);
        hipLaunchKernelGGL(k_append<RP>, dim3(grid.x + 1, grid.y), dim3(BT), 0, st, rp, N, words, w.train, t, par, (uint32_t)step);
        BGL_HIP(hipGetLastError());
        for (int64_t spins = 1; !all_done() && step - come_to() >= STEPS_AHEAD; ++spins) {
            if (!merge || merge->go_on(MERGE_ENTRIES) == 0) __builtin_ia32_pause();
            // a stream that has nothing left to do, or has failed, will not come to the step waited for
            if (spins % 65536 == 0) {
                const hipError_t e = hipStreamQuery(st);
                if (e == hipErrorNotReady) { (void)hipGetLastError(); continue; }
                BGL_HIP(e);
                if (!all_done() && step - come_to() >= STEPS_AHEAD)
                    BGL_FAIL(BGL_EHIP, "the traversal stopped at step %lld of %lld", (long long)come_to(), (long long)step);
            }
        }
    }
    if (!w.seqs_device)
        BGL_HIP(hipMemcpyAsync(w.seqs + one * (size_t)first, t.seq, sizeof(int32_t) * one * (size_t)count, hipMemcpyDeviceToHost, st));
    else if (merge)
        while (come_to(), merge->go_on(MERGE_ENTRIES) > 0) {}  // (while the last launches return)
    BGL_HIP(hipStreamSynchronize(st));  // the steps beyond the end too; w.host may be written anew
    if (w.host->status != 0) {
        w.keep = true;
        BGL_FAIL(BGL_EINVAL, "train_nodes holds an id outside [0, num_nodes) or a repeated id");
    }
    for (int j = 0; j < count; ++j)
        if (w.host[j].seq_len != num_train)
            BGL_FAIL(BGL_EHIP, "the traversal recorded %d of %lld training nodes", w.host[j].seq_len, (long long)num_train);
    if (merge) std::fill_n(merge->there.begin() + first, count, num_train);
    return BGL_OK;
}

// Behind prepare: leaves sequence j, num_train ids, at w.seqs[j * num_train].  A merge goes on meanwhile and may go to its end
// afterwards.
int compute_sequences(const bgl_graph_t *g, int64_t num_train, int32_t num_sequences, const int64_t *roots, hipStream_t st,
                      OrderWork &w, OrderMerge *merge)
{
    for (int j = 0; j < num_sequences; j += w.side) {
        const int count = std::min(num_sequences - j, w.side);
        const int rc = g->bits == 64 ? bfs_sequences<int64_t>(g, roots, j, count, num_train, w, st, merge)
                                     : bfs_sequences<int32_t>(g, roots, j, count, num_train, w, st, merge);
        if (rc != BGL_OK) return rc;
    }
    w.keep = true;
    return BGL_OK;
}

int check_order_args(const bgl_graph_t *g, const int32_t *train_nodes, int64_t num_train)
{
    if (!g) BGL_FAIL(BGL_EINVAL, "graph handle is null");
    if (num_train < 1 || num_train > g->num_nodes) BGL_FAIL(BGL_EINVAL, "num_train must be in [1, num_nodes]");
    if (!train_nodes) BGL_FAIL(BGL_EINVAL, "train_nodes is null");
    return BGL_OK;
}

}  // namespace

extern "C" int bgl_order_bfs_sequence(const bgl_graph_t *g, const int32_t *train_nodes, int64_t num_train,
                                      int64_t root, int32_t *seq, void *stream)
try {
    int rc = check_order_args(g, train_nodes, num_train);
    if (rc != BGL_OK) return rc;
    if (root < 0 || root >= g->num_nodes) BGL_FAIL(BGL_EINVAL, "root is outside [0, num_nodes)");
    if (!seq) BGL_FAIL(BGL_EINVAL, "seq is null");
    hipStream_t st = static_cast<hipStream_t>(stream);
    OrderWork w(g);
    if ((rc = prepare(g, train_nodes, num_train, 1, w, st)) != BGL_OK) return rc;
    if ((rc = compute_sequences(g, num_train, 1, &root, st, w, nullptr)) != BGL_OK) return rc;
    std::memcpy(seq, w.seqs, sizeof(int32_t) * (size_t)num_train);
    return BGL_OK;
} BGL_NOTHROW_END

namespace {

int check_proximity_args(const bgl_graph_t *g, const int32_t *train_nodes, int64_t num_train,
                         int32_t num_sequences, const int64_t *roots, const int64_t *shifts)
{
    int rc = check_order_args(g, train_nodes, num_train);
    if (rc != BGL_OK) return rc;
    if (num_sequences < 1 || !roots || !shifts) BGL_FAIL(BGL_EINVAL, "need at least one sequence with a root and a shift");
    for (int j = 0; j < num_sequences; ++j) {
        if (roots[j] < 0 || roots[j] >= g->num_nodes) BGL_FAIL(BGL_EINVAL, "roots[%d] is outside [0, num_nodes)", j);
        if (shifts[j] < 0 || shifts[j] >= num_train) BGL_FAIL(BGL_EINVAL, "shifts[%d] is outside [0, num_train)", j);
    }
    return BGL_OK;
}

}  // namespace

extern "C" int bgl_order_proximity(const bgl_graph_t *g, const int32_t *train_nodes, int64_t num_train,
                                   int32_t num_sequences, const int64_t *roots, const int64_t *shifts,
                                   int64_t num_out, int32_t *order, void *stream)
try {
    int rc = check_proximity_args(g, train_nodes, num_train, num_sequences, roots, shifts);
    if (rc != BGL_OK) return rc;
    if (num_out < 0 || num_out > num_train) BGL_FAIL(BGL_EINVAL, "num_out must be in [0, num_train]");
    if (num_out > 0 && !order) BGL_FAIL(BGL_EINVAL, "order is null");
    OrderWork w(g);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if ((rc = prepare(g, train_nodes, num_train, num_sequences, w, st)) != BGL_OK) return rc;
    OrderMerge merge(w.seqs, num_sequences, shifts, num_train, g->num_nodes, num_out, order, 0);
    if ((rc = compute_sequences(g, num_train, num_sequences, roots, st, w, &merge)) != BGL_OK) return rc;
    merge.finish();
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_order_choose_sequences(const bgl_graph_t *g, const int32_t *train_nodes, int64_t num_train,
                                          int32_t max_sequences, const int64_t *roots, const int64_t *shifts,
                                          int32_t batch, const int32_t *labels, int32_t num_classes,
                                          double threshold, int32_t *chosen, double *mean_tv_per_count,
                                          int32_t *order, void *stream)
try {
    int rc = check_proximity_args(g, train_nodes, num_train, max_sequences, roots, shifts);
    if (rc != BGL_OK) return rc;
    if (!labels || !chosen || !order) BGL_FAIL(BGL_EINVAL, "labels, chosen and order must not be null");
    OrderWork w(g);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if ((rc = prepare(g, train_nodes, num_train, max_sequences, w, st)) != BGL_OK) return rc;
    if ((rc = compute_sequences(g, num_train, max_sequences, roots, st, w, nullptr)) != BGL_OK) return rc;
    for (int32_t s = 1; s <= max_sequences; ++s) {
        OrderMerge(w.seqs, s, shifts, num_train, g->num_nodes, num_train, order, num_train).finish();
        double mean_tv = 0.0, max_tv = 0.0;
        rc = bgl_order_shuffling_error(order, num_train, batch, labels, g->num_nodes, num_classes, &mean_tv, &max_tv);
        if (rc != BGL_OK) return rc;
        if (mean_tv_per_count) mean_tv_per_count[s - 1] = mean_tv;
        *chosen = s;
        if (mean_tv <= threshold) break;   // `order` holds the order for this count
    }
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_order_shuffling_error(const int32_t *order, int64_t n, int32_t batch, const int32_t *labels,
                                         int64_t num_nodes, int32_t num_classes, double *mean_tv, double *max_tv)
try {
    if (!order || !labels || !mean_tv || !max_tv) BGL_FAIL(BGL_EINVAL, "null argument");
    if (n < 1 || batch < 1 || num_classes < 1 || num_nodes < 1) BGL_FAIL(BGL_EINVAL, "sizes must be positive");
    std::vector<int64_t> global((size_t)num_classes, 0), local((size_t)num_classes);
    for (int64_t i = 0; i < n; ++i) {
        if (order[i] < 0 || order[i] >= num_nodes) BGL_FAIL(BGL_EINVAL, "order[%lld] is not a node id", (long long)i);
        const int32_t c = labels[order[i]];
        if (c < 0 || c >= num_classes) BGL_FAIL(BGL_EINVAL, "label of node %d is outside [0, num_classes)", order[i]);
        global[(size_t)c] += 1;
    }
    double sum = 0.0, mx = 0.0;
    int64_t batches = 0;
    for (int64_t s = 0; s < n; s += batch, ++batches) {
        const int64_t e = std::min<int64_t>(s + batch, n);
        std::fill(local.begin(), local.end(), 0);
        for (int64_t i = s; i < e; ++i) local[(size_t)labels[order[i]]] += 1;
        double tv = 0.0;
        for (int32_t c = 0; c < num_classes; ++c) {
            const double pb = (double)local[(size_t)c] / (double)(e - s), pg = (double)global[(size_t)c] / (double)n;
            tv += 0.5 * (pb > pg ? pb - pg : pg - pb);
        }
        sum += tv;
        mx = std::max(mx, tv);
    }
    *mean_tv = sum / (double)batches;
    *max_tv = mx;
    return BGL_OK;
} BGL_NOTHROW_END
