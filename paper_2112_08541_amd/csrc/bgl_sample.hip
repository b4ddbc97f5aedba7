// k-hop fanout neighbor sampling with per-hop deduplication and relabelling
// (BGL paper, Sec. 3.1: samplers iteratively sample next-hop neighbors of the
// training nodes; Sec. 5.1: Neighbor Sampling with one fanout per hop).
//
// One call runs on one stream without any host round trip: a launch that clears
// the dedup map and removes repeated seeds, then three kernels per hop:
//   sample    a group of G lanes (G = power of two >= fanout) per frontier node
//             draws the node's edge positions (Floyd's subset algorithm resolved
//             with wavefront ballots), reads the neighbor ids and enters each in
//             the dedup map with the smallest position (node, slot) that holds it
//   mark      positions that are first occurrences of a new id: a bit each, and
//             how many precede every 64 positions
//   finalize  gives every new id its local id (old frontier size + rank),
//             appends it to the frontier, and writes the hop's CSR block
// The dedup map is an array indexed by node id where the graph is small enough
// for its clearing to cost less than hashing (k_sample_direct), else a hash table
// that a workgroup enters its ids into after removing repeats in LDS
// (k_sample_insert).  mark and finalize deal the positions to at most SHARES
// workgroups in contiguous shares, so that each of them can turn the shares'
// totals into prefixes itself, in LDS: no launch for a scan at any size.
//   What bounds a call: up to ~50,000 neighbors the launches, each 4 to 6 us of
// dependent reads; beyond, the random lines (row ends, column ids, map).  Measured
// per call, host included, with 11 to 15 launches and the hash table everywhere /
// now (7 to 10 launches): 512 seeds, fanout 10,5 on 10,000 nodes 91 / 55 us;
// 1,024 seeds, fanout 15,10,5 on 2.45 M nodes / 122 M edges 163 / 125 us; 4,096
// seeds, fanout 25,10 on 8 M nodes 124 / 95 us.
// Launches are sized by upper bounds; the real sizes stay on the device, and the
// last kernel stores them into the caller's page-locked counts.
#include "bgl_internal.h"

namespace {

using namespace bgl;

constexpr int TILE = 512;                      // threads (= padded positions) per workgroup
constexpr int SHARES = 1024;                   // workgroups of mark / finalize at most
constexpr int MARK_TILES = 4;                  // tiles a workgroup of mark has in flight
constexpr int SEEDS_LDS = 4096;                // seeds whose repeats one workgroup removes in LDS
constexpr int PREP = 1024;                     // threads per workgroup of k_prepare
constexpr int FILL_PER_THREAD = 4;             // 16-byte stores per thread that clears the map ...
// ... up to this many (28 MiB); a larger map is cleared with one non-temporal store per thread: its lines do not stay in the
// L2s, and the kernel's end waits for what is dirty in them.  Behind other work that has used the caches that is the
// faster way from 16 MB on, but one call right after the other then finds less of a map that the last-level cache
// could hold.  us, four stores / one non-temporal, behind other work | one call after the other:
//   nodes (degree)   4,096 seeds, 25,10          1,024 seeds, 15,10,5        4,096 seeds, 10
//   4.3 M (50)       72.9 / 71.8 | 63.6 / 67.3   83.2 / 82.4 | 81.7 / 81.2   31.4 / 30.7 | 25.3 / 24.7
//   6 M (14)         68.7 / 67.1 | 59.9 / 61.0   76.5 / 75.2 | 74.2 / 74.1   31.7 / 30.6 | 25.7 / 24.4
//   8 M (20)         73.2 / 70.6 | 61.7 / 62.4   82.7 / 81.4 | 80.7 / 80.8   33.5 / 32.1 | 26.6 / 24.7
//   12 M (10)        69.5 / 67.9 | 58.6 / 57.7   75.8 / 74.4 | 73.7 / 73.5   35.1 / 32.2 | 26.6 / 24.3
//   16 M (10)        70.8 / 67.9 | 59.0 / 57.9   78.9 / 77.4 | 74.1 / 74.4   35.0 / 32.7 | 26.9 / 24.6
constexpr int64_t FILL_CACHED_CHUNKS = 7 << 18;
constexpr uint64_t EMPTY64 = ~0ull;
constexpr uint32_t EMPTY32 = ~0u;
// Largest graph whose dedup map is indexed by node id.  Clearing it costs 4 bytes per node (4 us at
// 2.45 M nodes, 12 us at 16 M), the hash table's chains of probes and the removal of repeats in front
// of them 3 to 6 us per hop.  Measured on 16 M nodes, by id / hashed: 64 seeds, fanout 10,5: 53 / 59 us
// a call; 1,024 seeds, fanout 15,10,5: 139 / 155 us; 4,096 seeds, fanout 25,10: 94 / 109 us; at twice as
// many nodes the small calls would lose what the large ones gain.
constexpr int64_t DIRECT_MAX_NODES = 1 << 24;
constexpr uint32_t TENT = 0x80000000u;         // value is a tentative position, not yet a local id
constexpr uint64_t GOLDEN = 0x9E3779B97F4A7C15ull;
constexpr int STATUS = BGL_COUNTS_LEN - 1;
constexpr int NNZ0 = BGL_MAX_HOPS + 1;

// SplitMix64 output function (Steele, Lea, Flood 2014): the mixing step of the
// counter-based generator keyed on (call seed, hop, node, slot).
__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

// The dedup map.  Direct: value[id], 32 bits.  Hash: (id << 32 | value), 64 bits.  Either way the
// value is TENT | position while an id of the hop is new, later its local id, and an empty entry
// (all ones) is larger than any value.
template <bool DIRECT>
__device__ __forceinline__ uint32_t map_value(const void *tab, int32_t entry)
{
    // (cached: a value that is about to become a local id decodes to the same id in either form)
    if constexpr (DIRECT)
        return __hip_atomic_load(static_cast<const uint32_t *>(tab) + entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else
        return __hip_atomic_load(reinterpret_cast<const uint32_t *>(static_cast<const uint64_t *>(tab) + entry), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Start of a call: empty map, counts at zero.  With num_seeds > 0 (at most SEEDS_LDS) the first
// workgroup also writes frontier_0, the seeds without repeats (first occurrence kept): an LDS hash
// table of seed indices finds them.  The sample kernel of the first hop enters them in the map.
// LDS (dynamic): 2^tab_log >= 2 * num_seeds indices, then the seeds.
__global__ __launch_bounds__(PREP) void k_prepare(uint4 *p, int64_t n, int32_t *cnt, const int32_t *__restrict__ seeds,
                                                  int num_seeds, int tab_log, int64_t num_nodes, int32_t *frontier)
{
    constexpr int PER = SEEDS_LDS / PREP, NW = PREP / kWave;
    static_assert(PER * NW == kWave, "one count per lane");
    extern __shared__ uint32_t sh_tab[];
    __shared__ int sh_pop[kWave];
    if (blockIdx.x > 0) {
        typedef uint32_t Four __attribute__((ext_vector_type(4)));
        const Four empty = {EMPTY32, EMPTY32, EMPTY32, EMPTY32};
        Four *const to = reinterpret_cast<Four *>(p);
        if (n > FILL_CACHED_CHUNKS) {
            const int64_t at = (int64_t)(blockIdx.x - 1) * PREP + threadIdx.x;
            if (at < n) __builtin_nontemporal_store(empty, to + at);
        } else {
            const int64_t at = (int64_t)(blockIdx.x - 1) * (FILL_PER_THREAD * PREP) + threadIdx.x;
#pragma unroll
            for (int k = 0; k < FILL_PER_THREAD; ++k)
                if (at + k * PREP < n) to[at + k * PREP] = empty;
        }
        return;
    }
    if (threadIdx.x < BGL_COUNTS_LEN) cnt[threadIdx.x] = 0;
    if (num_seeds == 0) return;
    const uint32_t tab_mask = (1u << tab_log) - 1u;
    int32_t *sh_seed = reinterpret_cast<int32_t *>(sh_tab + tab_mask + 1);
    int32_t v[PER];
    uint32_t at[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = k * PREP + threadIdx.x;
        v[k] = i < num_seeds ? seeds[i] : -1;
        if (i < num_seeds) sh_seed[i] = v[k];
    }
    for (uint32_t i = threadIdx.x; i <= tab_mask; i += PREP) sh_tab[i] = EMPTY32;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = k * PREP + threadIdx.x;
        at[k] = 0;
        if (i >= num_seeds) continue;
        if (v[k] < 0 || (int64_t)v[k] >= num_nodes) {
            cnt[STATUS] = BGL_EINVAL;
            v[k] = -1;
            continue;
        }
        for (at[k] = hash32((uint32_t)v[k]) & tab_mask;; at[k] = (at[k] + 1) & tab_mask) {  // at most half full: ends
            const uint32_t old = atomicCAS(&sh_tab[at[k]], EMPTY32, (uint32_t)i);
            if (old == EMPTY32) break;
            if (sh_seed[old] == v[k]) {
                atomicMin(&sh_tab[at[k]], (uint32_t)i);
                break;
            }
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint64_t first[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        first[k] = __ballot(v[k] >= 0 && sh_tab[at[k]] == (uint32_t)(k * PREP + threadIdx.x));
        if (lane == 0) sh_pop[k * NW + w] = __popcll(first[k]);
    }
    __syncthreads();
    const int pop = sh_pop[lane], inc = wave_incl_scan(pop);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int before = __shfl(inc - pop, k * NW + w);
        if ((first[k] >> lane) & 1ull) frontier[before + __popcll(first[k] & ((1ull << lane) - 1ull))] = v[k];
    }
    if (threadIdx.x == kWave - 1) cnt[0] = inc;
}

// Enter (key, val) in the global table, keeping the smallest val per key.
// Entries are (key << 32 | val); returns the entry index.
__device__ __forceinline__ int table_insert_min(uint64_t *tab, uint32_t mask, uint32_t key,
                                                uint32_t val, int32_t *cnt)
{
    const uint64_t mine = ((uint64_t)key << 32) | val;
    uint32_t s = hash32(key) & mask;
    for (uint32_t tries = 0; tries <= mask; ++tries) {
        // (a stale entry is one that was still empty or held a larger value: the atomics decide)
        uint64_t cur = __hip_atomic_load(&tab[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == EMPTY64) {
            unsigned long long old = atomicCAS((unsigned long long *)&tab[s], EMPTY64, mine);
            if (old == EMPTY64) return (int)s;
            cur = old;
        }
        if ((uint32_t)(cur >> 32) == key) {
            if ((uint32_t)cur > val) atomicMin((unsigned long long *)&tab[s], mine);
            return (int)s;
        }
        s = (s + 1) & mask;
    }
    cnt[STATUS] = BGL_ECAPACITY;  // cannot happen: the table outsizes the frontier bound
    return -1;
}

// Second half of a sample/insert kernel: workgroup-local dedup in LDS, then one
// global insert per distinct id of the workgroup.  sh_tab (2*TILE entries) must
// be EMPTY64 and visible to the whole workgroup on entry.
__device__ __forceinline__ void dedup_and_insert(bool valid, uint32_t key, uint32_t p,
                                                 uint64_t *tab, uint32_t mask,
                                                 int32_t *slotidx, uint64_t *sh_tab,
                                                 int32_t *sh_gs, int32_t *cnt)
{
    constexpr uint32_t LM = 2 * TILE - 1;
    uint32_t ls = 0;
    if (valid) {
        const uint64_t mine = ((uint64_t)key << 32) | threadIdx.x;
        ls = (hash32(key) >> 8) & LM;
        for (;;) {
            unsigned long long old = atomicCAS((unsigned long long *)&sh_tab[ls], EMPTY64, mine);
            if (old == EMPTY64) break;
            if ((uint32_t)(old >> 32) == key) {
                atomicMin((unsigned long long *)&sh_tab[ls], mine);
                break;
            }
            ls = (ls + 1) & LM;
        }
    }
    __syncthreads();
    if (valid && (uint32_t)sh_tab[ls] == threadIdx.x)
        sh_gs[ls] = table_insert_min(tab, mask, key, TENT | p, cnt);
    __syncthreads();
    slotidx[p] = valid ? sh_gs[ls] : -1;
}

// More seeds than k_prepare takes: the seeds themselves are the keys, position = index in the seed list.
template <bool DIRECT>
__global__ __launch_bounds__(TILE) void k_seed_insert(const int32_t *seeds, int32_t num_seeds,
                                                      int64_t num_nodes, void *tab,
                                                      uint32_t mask, int32_t *slotidx,
                                                      int32_t *cnt)
{
    const uint32_t p = blockIdx.x * TILE + threadIdx.x;
    bool valid = p < (uint32_t)num_seeds;
    int32_t v = valid ? seeds[p] : 0;
    if (valid && (v < 0 || (int64_t)v >= num_nodes)) {
        cnt[STATUS] = BGL_EINVAL;
        valid = false;
    }
    if constexpr (DIRECT) {
        if (valid) atomicMin(static_cast<uint32_t *>(tab) + v, TENT | p);
        slotidx[p] = valid ? v : -1;
    } else {
        __shared__ uint64_t sh_tab[2 * TILE];
        __shared__ int32_t sh_gs[2 * TILE];
        for (int i = threadIdx.x; i < 2 * TILE; i += TILE) sh_tab[i] = EMPTY64;
        __syncthreads();
        dedup_and_insert(valid, (uint32_t)v, p, static_cast<uint64_t *>(tab), mask, slotidx, sh_tab, sh_gs, cnt);
    }
}

// One sampled position: group of G lanes per frontier node, lane s owns slot s.
template <int G, typename RP>
struct Draw {
    int i, s, c;     // frontier index, slot, neighbors the node gets
    uint32_t v;      // the node
    uint32_t u;      // the neighbor in this slot
    bool active, valid;

    // node: frontier[p / G], which the caller has read beside n_dst
    __device__ __forceinline__ Draw(const RP *__restrict__ row_ptr, const int32_t *__restrict__ col,
                                    int32_t node, uint32_t p, int n_dst, int fanout, uint64_t h0)
    {
        i = (int)(p / G);
        s = (int)(p & (G - 1));
        const int lane = threadIdx.x & (kWave - 1);
        const int gshift = lane & ~(G - 1);
        active = i < n_dst;
        int64_t lo = 0, d = 0;
        v = 0;
        if (active) {
            v = (uint32_t)node;
            // both ends of the row with one read (the pair is only 4 or 8 bytes aligned)
            typedef RP Ends __attribute__((ext_vector_type(2), aligned(sizeof(RP))));
            const Ends ends = *reinterpret_cast<const Ends *>(row_ptr + v);
            lo = (int64_t)ends.x;
            d = (int64_t)ends.y - lo;
        }
        c = (int)(d < (int64_t)fanout ? d : (int64_t)fanout);
        const bool need = active && d > (int64_t)fanout;  // Floyd's algorithm, else the whole row
        const int64_t J = d - fanout + s;
        uint32_t pos = (uint32_t)s;
        if (need && s < fanout) {
            const uint64_t h1 = mix64(h0 ^ (uint64_t)v);
            const uint64_t w = mix64(h1 + GOLDEN * (uint64_t)(s + 1));
            pos = (uint32_t)__umul64hi(w, (uint64_t)(J + 1));
        }
        if (__ballot(need) != 0) {
            // Slot q keeps its draw unless an earlier slot already holds that
            // position, in which case it takes J_q.  Lanes below q are final.
            for (int q = 1; q < fanout; ++q) {
                const uint32_t tq = __shfl(pos, q, G);
                const bool coll = need && s < q && pos == tq;
                const uint64_t bal = __ballot(coll);
                const bool any = (G == kWave) ? (bal != 0)
                                              : (((bal >> gshift) & ((1ull << (G & 63)) - 1ull)) != 0);
                if (need && s == q && any) pos = (uint32_t)J;
            }
        }
        valid = active && s < c;
        u = 0;
        if (valid) u = (uint32_t)col[lo + (int64_t)pos];
    }
};

// Hop `hop` with the direct map.  enter_frontier: the first hop after k_prepare has written frontier_0;
// its nodes get their local ids here (smaller than any position's value, so the order does not matter).
template <int G, typename RP>
__global__ __launch_bounds__(TILE) void k_sample_direct(
    const RP *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const int32_t *__restrict__ frontier, const int32_t *__restrict__ cnt, int hop, int fanout, uint64_t h0,
    uint32_t *tab, int32_t *slotidx, int32_t *lrow, int32_t *cbs, int enter_frontier)
{
    __shared__ int sh_scan[TILE / kWave];
    constexpr uint32_t LM = 2 * TILE - 1;
    __shared__ uint32_t sh_first[2 * TILE], sh_id[TILE];
    const uint32_t p = blockIdx.x * TILE + threadIdx.x;
    // (the grid ends less than a tile beyond the frontier's bound, and other arrays of the workspace follow it)
    const int32_t node = frontier[p / G];
    const int n_dst = cnt[hop];
    if ((int64_t)blockIdx.x * TILE >= (int64_t)n_dst * G) return;  // whole workgroup
    sh_first[threadIdx.x] = sh_first[threadIdx.x + TILE] = EMPTY32;
    const Draw<G, RP> d(row_ptr, col, node, p, n_dst, fanout, h0);
    const uint32_t seen = d.valid ? __hip_atomic_load(&tab[d.u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    if (enter_frontier && d.active && d.s == 0) atomicMin(&tab[d.v], (uint32_t)d.i);
    slotidx[p] = d.valid ? (int32_t)d.u : -1;
    sh_id[threadIdx.x] = d.u;
    // per-node counts -> row starts inside this tile, tile total
    int total;
    const int ex = block_excl_scan<TILE>((d.active && d.s == 0) ? d.c : 0, sh_scan, total);
    if (d.active && d.s == 0) lrow[d.i] = ex;
    if (threadIdx.x == 0) cbs[blockIdx.x] = total;
    // A repeat inside the workgroup need not go to the map: without its removal, a graph whose edges lead
    // to a few nodes for the most part makes every lane lower the same words, 7 ns each (10 % of the edges
    // to one node: 166 us a call of 16,384 seeds, fanout 10).  An LDS hash table of thread indices finds
    // the first thread of every id.  It has to resolve ids that meet in a slot: with one probe per id, two
    // heavy nodes of the same slot left one of them to the map (a quarter of the edges to each: 287 us,
    // 50 now, 79 with the hash table).
    // (block_excl_scan ended with a barrier: sh_first and sh_id are there for everyone)
    uint32_t at = 0;
    if (d.valid) {
        for (at = (hash32(d.u) >> 8) & LM;; at = (at + 1) & LM) {  // at most half full: ends
            const uint32_t first = atomicCAS(&sh_first[at], EMPTY32, threadIdx.x);
            if (first == EMPTY32) break;
            if (sh_id[first] == d.u) {
                if (first > threadIdx.x) atomicMin(&sh_first[at], threadIdx.x);
                break;
            }
        }
    }
    __syncthreads();
    if (d.valid && seen > (TENT | p) && sh_first[at] == threadIdx.x) atomicMin(&tab[d.u], TENT | p);
}

// The same with the hash table.
template <int G, typename RP>
__global__ __launch_bounds__(TILE) void k_sample_insert(
    const RP *__restrict__ row_ptr, const int32_t *__restrict__ col,
    const int32_t *__restrict__ frontier, int32_t *cnt, int hop, int fanout, uint64_t h0,
    uint64_t *tab, uint32_t mask, int32_t *slotidx, int32_t *lrow, int32_t *cbs, int enter_frontier)
{
    __shared__ uint64_t sh_tab[2 * TILE];
    __shared__ int32_t sh_gs[2 * TILE];
    __shared__ int sh_scan[TILE / kWave];

    const uint32_t p = blockIdx.x * TILE + threadIdx.x;
    // (the grid ends less than a tile beyond the frontier's bound, and other arrays of the workspace follow it)
    const int32_t node = frontier[p / G];
    const int n_dst = cnt[hop];
    if ((int64_t)blockIdx.x * TILE >= (int64_t)n_dst * G) return;  // whole workgroup

    for (int i = threadIdx.x; i < 2 * TILE; i += TILE) sh_tab[i] = EMPTY64;
    const Draw<G, RP> d(row_ptr, col, node, p, n_dst, fanout, h0);
    if (enter_frontier && d.active && d.s == 0) (void)table_insert_min(tab, mask, d.v, (uint32_t)d.i, cnt);
    // per-node counts -> row starts inside this tile, tile total
    int total;
    const int ex = block_excl_scan<TILE>((d.active && d.s == 0) ? d.c : 0, sh_scan, total);
    if (d.active && d.s == 0) lrow[d.i] = ex;
    if (threadIdx.x == 0) cbs[blockIdx.x] = total;
    // (block_excl_scan ended with a barrier: sh_tab is initialised for everyone)
    dedup_and_insert(d.valid, d.u, p, tab, mask, slotidx, sh_tab, sh_gs, cnt);
}

// How the tiles of a stage are dealt to the workgroups of mark and finalize: 2^log contiguous tiles each.
struct Shares {
    int64_t positions, tiles;
    int log;
    __device__ __forceinline__ Shares(int64_t positions_) : positions(positions_), tiles((positions_ + TILE - 1) / TILE), log(0)
    {
        while ((tiles + (1 << log) - 1) >> log > SHARES) ++log;
    }
    __device__ __forceinline__ int count() const { return (int)((tiles + (1 << log) - 1) >> log); }
    __device__ __forceinline__ int64_t first_tile(int share) const { return (int64_t)share << log; }
    __device__ __forceinline__ int64_t end_tile(int share) const { return min((int64_t)(share + 1) << log, tiles); }
};

// Which positions introduced a new id?  A bit per position, the number of bits before every 64
// positions inside the share, the share's total; and the share's number of sampled neighbors.
// ONE: the stage's bound is at most SHARES tiles, a share is a tile: its entries are read beside the
// stage's size (a workgroup beyond the stage's real end reads what earlier calls left there, or the
// map entry that is the nearest valid one, and drops it).
template <bool DIRECT, bool ONE>
__global__ __launch_bounds__(TILE) void k_mark(const int32_t *__restrict__ cnt, int stage, int logG, int32_t num_seeds,
                                               const void *tab, uint32_t tab_entries, const int32_t *__restrict__ slotidx,
                                               uint64_t *bits, int32_t *before, const int32_t *__restrict__ cbs, int32_t *fsum,
                                               int32_t *csum)
{
    constexpr int NW = TILE / kWave;
    constexpr int TILES = ONE ? 1 : MARK_TILES;
    __shared__ int sh_pop[TILES][NW];
    __shared__ int sh_scan[NW];
    int32_t gs[TILES];
    uint32_t val[TILES];
    if constexpr (ONE) {
        gs[0] = slotidx[(int64_t)blockIdx.x * TILE + threadIdx.x];
        val[0] = map_value<DIRECT>(tab, (int32_t)min((uint32_t)gs[0], tab_entries - 1));
    }
    const Shares sh(stage == 0 ? (int64_t)num_seeds : (int64_t)cnt[stage - 1] << logG);
    const int64_t t0 = ONE ? blockIdx.x : sh.first_tile(blockIdx.x), t1 = ONE ? min(t0 + 1, sh.tiles) : sh.end_tile(blockIdx.x);
    if (t0 >= t1) return;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int carry = 0;
    for (int64_t t = t0; t < t1; t += TILES) {
        uint64_t b[TILES];
        if constexpr (!ONE) {  // tiles beyond the share's end read its last tile again and drop it
#pragma unroll
            for (int k = 0; k < TILES; ++k) gs[k] = slotidx[min(t + k, t1 - 1) * TILE + threadIdx.x];
#pragma unroll
            for (int k = 0; k < TILES; ++k) val[k] = map_value<DIRECT>(tab, max(gs[k], 0));
        }
#pragma unroll
        for (int k = 0; k < TILES; ++k) {
            const int64_t p = (t + k) * TILE + threadIdx.x;
            b[k] = __ballot(t + k < t1 && p < sh.positions && gs[k] >= 0 && val[k] == (TENT | (uint32_t)p));
            if (lane == 0) sh_pop[k][w] = __popcll(b[k]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < TILES; ++k) {
            int mine = 0, all = 0;
#pragma unroll
            for (int x = 0; x < NW; ++x) {
                if (x < w) mine += sh_pop[k][x];
                all += sh_pop[k][x];
            }
            if (lane == 0 && t + k < t1) {
                const int64_t word = (t + k) * NW + w;
                bits[word] = b[k];
                before[word] = carry + mine;
            }
            carry += all;
        }
        if constexpr (!ONE) __syncthreads();
    }
    int total = 0;
    if constexpr (ONE) {
        if (stage > 0 && threadIdx.x == 0) total = cbs[t0];
    } else {
        int edges = 0;
        if (stage > 0)
            for (int64_t t = t0 + threadIdx.x; t < t1; t += TILE) edges += cbs[t];
        (void)block_excl_scan<TILE>(edges, sh_scan, total);
    }
    if (threadIdx.x == 0) {
        fsum[blockIdx.x] = carry;
        csum[blockIdx.x] = total;
    }
}

// Local ids, frontier append, CSR block.  Every workgroup scans the shares' totals in LDS; the first
// one publishes the stage's sizes and, after the last hop, stores all counts into the caller's
// page-locked copy.  last: nobody looks the hop's new ids up any more.  ONE: as in k_mark.
template <bool DIRECT, bool ONE>
__global__ __launch_bounds__(TILE) void k_finalize(int32_t *cnt, int stage, int logG, int32_t num_seeds, void *tab,
                                                   uint32_t tab_entries, const int32_t *__restrict__ slotidx,
                                                   const uint64_t *__restrict__ bits,
                                                   const int32_t *__restrict__ before, const int32_t *__restrict__ fsum,
                                                   const int32_t *__restrict__ csum, const int32_t *__restrict__ cbs,
                                                   const int32_t *__restrict__ lrow, int32_t *frontier,
                                                   int32_t *row_ptr_h, int32_t *col_local, int last, int32_t *counts_host)
{
    static_assert(SHARES == 2 * TILE, "two totals per thread");
    __shared__ int sh_scan[TILE / kWave];
    __shared__ int32_t sh_f[SHARES], sh_c[SHARES];
    const int t = threadIdx.x, lane = threadIdx.x & (kWave - 1);
    // what position p needs: its entry, its word of bits and the bits before it, its node's row start
    struct Position {
        int32_t gs, before, row;
        uint64_t own;
        uint32_t val;
    };
    auto read = [&](int64_t p) {
        Position x;
        x.gs = slotidx[p];
        x.own = bits[p / kWave];
        x.before = before[p / kWave];
        x.row = stage > 0 ? lrow[p >> logG] : 0;
        return x;
    };
    Position x;
    if constexpr (ONE) {  // (the last tile may end a little beyond lrow's bound: the tile counts follow it)
        x = read((int64_t)blockIdx.x * TILE + t);
        x.val = map_value<DIRECT>(tab, (int32_t)min((uint32_t)x.gs, tab_entries - 1));
    }
    int f0 = fsum[2 * t], f1 = fsum[2 * t + 1], c0 = csum[2 * t], c1 = csum[2 * t + 1];
    const int n_dst = stage == 0 ? 0 : cnt[stage - 1];
    const Shares sh(stage == 0 ? (int64_t)num_seeds : (int64_t)n_dst << logG);
    // (whole workgroups; the one that publishes the sizes stays, also for an empty stage)
    if ((int)blockIdx.x >= sh.count() && blockIdx.x > 0) return;
    {
        const int n = sh.count();
        if (2 * t >= n) f0 = c0 = 0;
        if (2 * t + 1 >= n) f1 = c1 = 0;
        int tf, tc;
        const int ef = block_excl_scan<TILE>(f0 + f1, sh_scan, tf);
        const int ec = block_excl_scan<TILE>(c0 + c1, sh_scan, tc);
        sh_f[2 * t] = ef;
        sh_f[2 * t + 1] = ef + f0;
        sh_c[2 * t] = ec;
        sh_c[2 * t + 1] = ec + c0;
        if (blockIdx.x == 0) {
            if (t == 0) {
                cnt[stage] = n_dst + tf;
                if (stage > 0) {
                    cnt[NNZ0 + stage - 1] = tc;
                    row_ptr_h[n_dst] = tc;
                }
            }
            __syncthreads();
            if (counts_host && t < BGL_COUNTS_LEN) counts_host[t] = cnt[t];
        }
        __syncthreads();
    }
    int edges = sh_c[blockIdx.x];
    const int64_t t0 = ONE ? blockIdx.x : sh.first_tile(blockIdx.x), t1 = ONE ? min(t0 + 1, sh.tiles) : sh.end_tile(blockIdx.x);
    for (int64_t tile = t0; tile < t1; ++tile) {
        const int64_t p64 = tile * TILE + t;
        if (p64 < sh.positions) {
            const uint32_t p = (uint32_t)p64;
            if constexpr (!ONE) x = read(p64);
            int local = -1;
            if ((x.own >> lane) & 1ull) {
                local = n_dst + sh_f[blockIdx.x] + x.before + __popcll(x.own & ((1ull << lane) - 1ull));
                if constexpr (DIRECT) {
                    frontier[local] = x.gs;
                    if (!last) __hip_atomic_store(static_cast<uint32_t *>(tab) + x.gs, (uint32_t)local, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    uint32_t *e = reinterpret_cast<uint32_t *>(static_cast<uint64_t *>(tab) + x.gs);
                    frontier[local] = (int32_t)e[1];
                    // Other positions of the same id may read the entry while it
                    // turns from "first position" into "local id"; both forms
                    // decode to the same local id.
                    if (!last) __hip_atomic_store(e, (uint32_t)local, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            } else if (x.gs >= 0) {
                const uint32_t val = ONE ? x.val : map_value<DIRECT>(tab, x.gs);
                if (val & TENT) {
                    const uint32_t q = val & ~TENT;  // first position of this id
                    local = n_dst + sh_f[(q / TILE) >> sh.log] + before[q / kWave] +
                            __popcll(bits[q / kWave] & ((1ull << (q & (kWave - 1))) - 1ull));
                } else {
                    local = (int)val;
                }
            }
            if (stage > 0) {
                const int i = (int)(p >> logG);
                const int s = (int)(p & ((1u << logG) - 1));
                const int base = edges + x.row;
                if (s == 0) row_ptr_h[i] = base;
                if (x.gs >= 0) col_local[base + s] = local;
            }
        }
        if (!ONE && stage > 0) edges += cbs[tile];
    }
}

// ------------------------------------------------------------------ host side
struct Layout {
    int K;
    int G[BGL_MAX_HOPS], logG[BGL_MAX_HOPS];
    int64_t ubf[BGL_MAX_HOPS + 1], ube[BGL_MAX_HOPS];
    int64_t P[BGL_MAX_HOPS + 1];  // padded positions per stage
    bool direct;                  // the dedup map is indexed by node id
    int64_t table_entries;
    size_t table_bytes;
    size_t off_counts, off_frontier, off_row_ptr[BGL_MAX_HOPS], off_col[BGL_MAX_HOPS];
    size_t off_table, off_slotidx, off_bits, off_before, off_lrow, off_cbs, off_fsum, off_csum;
    size_t bytes;
};

int make_layout(int32_t num_seeds, const int32_t *fanouts, int32_t num_hops, int64_t num_nodes,
                Layout &L)
{
    if (num_seeds < 1) BGL_FAIL(BGL_EINVAL, "num_seeds must be >= 1 (got %d)", num_seeds);
    if (num_hops < 1 || num_hops > BGL_MAX_HOPS)
        BGL_FAIL(BGL_EINVAL, "num_hops must be in [1, %d] (got %d)", BGL_MAX_HOPS, num_hops);
    if (!fanouts) BGL_FAIL(BGL_EINVAL, "fanouts is null");
    if (num_nodes < 1 || num_nodes > INT32_MAX) BGL_FAIL(BGL_EINVAL, "num_nodes out of range");
    L.K = num_hops;
    L.ubf[0] = num_seeds < num_nodes ? num_seeds : num_nodes;
    L.P[0] = num_seeds;
    int64_t pmax = num_seeds, fmax = L.ubf[0];
    for (int h = 0; h < num_hops; ++h) {
        const int f = fanouts[h];
        if (f < 1) BGL_FAIL(BGL_EINVAL, "fanouts[%d] = %d must be >= 1", h, f);
        if (f > BGL_MAX_FANOUT)
            BGL_FAIL(BGL_EUNSUPPORTED, "fanouts[%d] = %d exceeds BGL_MAX_FANOUT = %d", h, f,
                     BGL_MAX_FANOUT);
        int g = 4, lg = 2;
        while (g < f) { g <<= 1; ++lg; }
        L.G[h] = g;
        L.logG[h] = lg;
        L.ube[h] = L.ubf[h] * f;
        L.P[h + 1] = L.ubf[h] * g;
        int64_t nxt = L.ubf[h] * (1 + (int64_t)f);
        L.ubf[h + 1] = nxt < num_nodes ? nxt : num_nodes;
        if (L.P[h + 1] > pmax) pmax = L.P[h + 1];
        if (L.ubf[h] > fmax) fmax = L.ubf[h];
        if (L.P[h + 1] >= (int64_t)TENT || L.ube[h] >= (int64_t)TENT)
            BGL_FAIL(BGL_EUNSUPPORTED, "hop %d is too large for 31-bit positions", h);
    }
    int64_t need = L.ubf[num_hops] + L.ubf[num_hops] / 3 + 1;
    int64_t ts = 1024;
    while (ts < need) ts <<= 1;
    L.direct = num_nodes <= DIRECT_MAX_NODES;
    L.table_entries = L.direct ? (int64_t)bgl::round_up((size_t)num_nodes, 4) : ts;
    L.table_bytes = L.direct ? sizeof(uint32_t) * (size_t)L.table_entries : sizeof(uint64_t) * (size_t)ts;
    const int64_t nbmax = bgl::ceil_div(pmax, TILE) + 1;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += bgl::round_up(bytes, 256); return o; };
    L.off_counts = take(sizeof(int32_t) * BGL_COUNTS_LEN);
    L.off_frontier = take(sizeof(int32_t) * (size_t)L.ubf[num_hops]);
    for (int h = 0; h < num_hops; ++h) {
        L.off_row_ptr[h] = take(sizeof(int32_t) * (size_t)(L.ubf[h] + 1));
        L.off_col[h] = take(sizeof(int32_t) * (size_t)L.ube[h]);
    }
    L.off_table = take(L.table_bytes);
    const size_t ppad = bgl::round_up((size_t)pmax, TILE);
    L.off_slotidx = take(sizeof(int32_t) * ppad);
    L.off_bits = take(sizeof(uint64_t) * (ppad / kWave));
    L.off_before = take(sizeof(int32_t) * (ppad / kWave));
    L.off_lrow = take(sizeof(int32_t) * (size_t)fmax);
    L.off_cbs = take(sizeof(int32_t) * (size_t)nbmax);
    L.off_fsum = take(sizeof(int32_t) * SHARES);
    L.off_csum = take(sizeof(int32_t) * SHARES);
    L.bytes = off;
    return BGL_OK;
}

// What the kernels of one call share.
struct Call {
    const bgl_graph *g;
    bool direct;
    void *tab;
    uint32_t mask;
    int32_t *cnt, *frontier, *slotidx, *lrow, *cbs;
    hipStream_t st;
};

template <int G, typename RP>
void launch_sample(const Call &k, int blocks, int hop, int fanout, uint64_t h0, int enter_frontier)
{
    const RP *rp = static_cast<const RP *>(k.g->row_ptr);
    if (k.direct)
        hipLaunchKernelGGL((k_sample_direct<G, RP>), dim3(blocks), dim3(TILE), 0, k.st, rp, k.g->col, k.frontier, k.cnt, hop, fanout,
                           h0, static_cast<uint32_t *>(k.tab), k.slotidx, k.lrow, k.cbs, enter_frontier);
    else
        hipLaunchKernelGGL((k_sample_insert<G, RP>), dim3(blocks), dim3(TILE), 0, k.st, rp, k.g->col, k.frontier, k.cnt, hop, fanout,
                           h0, static_cast<uint64_t *>(k.tab), k.mask, k.slotidx, k.lrow, k.cbs, enter_frontier);
}

template <typename RP>
void launch_sample_g(int G, const Call &k, int blocks, int hop, int fanout, uint64_t h0, int enter_frontier)
{
    switch (G) {
    case 4: launch_sample<4, RP>(k, blocks, hop, fanout, h0, enter_frontier); break;
    case 8: launch_sample<8, RP>(k, blocks, hop, fanout, h0, enter_frontier); break;
    case 16: launch_sample<16, RP>(k, blocks, hop, fanout, h0, enter_frontier); break;
    case 32: launch_sample<32, RP>(k, blocks, hop, fanout, h0, enter_frontier); break;
    default: launch_sample<64, RP>(k, blocks, hop, fanout, h0, enter_frontier); break;
    }
}

}  // namespace

extern "C" int bgl_sample_workspace_bytes(int32_t num_seeds, const int32_t *fanouts,
                                          int32_t num_hops, int64_t num_nodes, size_t *bytes)
try {
    if (!bytes) BGL_FAIL(BGL_EINVAL, "bytes is null");
    Layout L;
    int rc = make_layout(num_seeds, fanouts, num_hops, num_nodes, L);
    if (rc != BGL_OK) return rc;
    *bytes = L.bytes;
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_sample_khop(const bgl_graph_t *g, const int32_t *seeds, int32_t num_seeds,
                               const int32_t *fanouts, int32_t num_hops, uint64_t rng_seed,
                               void *workspace, size_t workspace_bytes, bgl_subgraph_t *out,
                               int32_t *counts_host, void *stream)
try {
    if (!g) BGL_FAIL(BGL_EINVAL, "graph handle is null");
    if (!seeds) BGL_FAIL(BGL_EINVAL, "seeds is null");
    if (!out) BGL_FAIL(BGL_EINVAL, "out is null");
    if (!workspace || !bgl::aligned(workspace, 256))
        BGL_FAIL(BGL_EINVAL, "workspace is null or not 256-byte aligned");
    Layout L;
    int rc = make_layout(num_seeds, fanouts, num_hops, g->num_nodes, L);
    if (rc != BGL_OK) return rc;
    if (workspace_bytes < L.bytes)
        BGL_FAIL(BGL_ECAPACITY, "workspace has %zu bytes, %zu needed", workspace_bytes, L.bytes);

    hipStream_t st = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    int32_t *cnt = reinterpret_cast<int32_t *>(ws + L.off_counts);
    int32_t *frontier = reinterpret_cast<int32_t *>(ws + L.off_frontier);
    void *tab = ws + L.off_table;
    int32_t *slotidx = reinterpret_cast<int32_t *>(ws + L.off_slotidx);
    uint64_t *bits = reinterpret_cast<uint64_t *>(ws + L.off_bits);
    int32_t *before = reinterpret_cast<int32_t *>(ws + L.off_before);
    int32_t *lrow = reinterpret_cast<int32_t *>(ws + L.off_lrow);
    int32_t *cbs = reinterpret_cast<int32_t *>(ws + L.off_cbs);
    int32_t *fsum = reinterpret_cast<int32_t *>(ws + L.off_fsum);
    int32_t *csum = reinterpret_cast<int32_t *>(ws + L.off_csum);
    const uint32_t mask = (uint32_t)(L.table_entries - 1);
    // page-locked counts are stored by the last kernel; anything else is copied to behind it
    int32_t *counts_dev = nullptr;
    if (counts_host) {
        hipPointerAttribute_t attr;
        if (hipPointerGetAttributes(&attr, counts_host) == hipSuccess && attr.type == hipMemoryTypeHost)
            counts_dev = static_cast<int32_t *>(attr.devicePointer);
        else
            (void)hipGetLastError();
    }

    out->num_hops = num_hops;
    out->input_nodes = frontier;
    out->counts = cnt;
    for (int h = 0; h <= BGL_MAX_HOPS; ++h) out->cap_nodes[h] = h <= num_hops ? L.ubf[h] : 0;
    for (int h = 0; h < BGL_MAX_HOPS; ++h) {
        out->row_ptr[h] = h < num_hops ? reinterpret_cast<int32_t *>(ws + L.off_row_ptr[h]) : nullptr;
        out->col_local[h] = h < num_hops ? reinterpret_cast<int32_t *>(ws + L.off_col[h]) : nullptr;
        out->cap_edges[h] = h < num_hops ? L.ube[h] : 0;
    }

    const Call k{g, L.direct, tab, mask, cnt, frontier, slotidx, lrow, cbs, st};
    // mark and finalize of one stage
    auto place = [&](int stage, int logG, int64_t positions, int32_t *row_ptr_h, int32_t *col_local, bool last) {
        const int blocks = (int)std::min<int64_t>(bgl::ceil_div(positions, TILE), SHARES);
        const bool one = bgl::ceil_div(positions, TILE) <= SHARES;
        const uint32_t entries = (uint32_t)std::min<int64_t>(L.table_entries, INT32_MAX);
        auto mark = L.direct ? (one ? k_mark<true, true> : k_mark<true, false>) : (one ? k_mark<false, true> : k_mark<false, false>);
        auto finalize = L.direct ? (one ? k_finalize<true, true> : k_finalize<true, false>)
                                 : (one ? k_finalize<false, true> : k_finalize<false, false>);
        hipLaunchKernelGGL(mark, dim3(blocks), dim3(TILE), 0, st, cnt, stage, logG, num_seeds, tab, entries,
                           slotidx, bits, before, cbs, fsum, csum);
        hipLaunchKernelGGL(finalize, dim3(blocks), dim3(TILE), 0, st, cnt, stage, logG, num_seeds, tab, entries,
                           slotidx, bits, before, fsum, csum, cbs, lrow, frontier, row_ptr_h, col_local, last ? 1 : 0,
                           last ? counts_dev : nullptr);
    };
    const bool few_seeds = num_seeds <= SEEDS_LDS;
    const int64_t chunks = (int64_t)(L.table_bytes / 16);
    int tab_log = 10;
    while ((1 << tab_log) < 2 * std::min(num_seeds, SEEDS_LDS)) ++tab_log;
    const size_t lds = few_seeds ? sizeof(uint32_t) * (((size_t)1 << tab_log) + (size_t)num_seeds) : 0;
    hipLaunchKernelGGL(k_prepare, dim3(1 + (unsigned)bgl::ceil_div(chunks, chunks > FILL_CACHED_CHUNKS ? PREP : FILL_PER_THREAD * PREP)), dim3(PREP), lds, st,
                       static_cast<uint4 *>(tab), chunks, cnt, seeds, few_seeds ? num_seeds : 0, tab_log, g->num_nodes, frontier);
    if (!few_seeds) {
        hipLaunchKernelGGL((L.direct ? k_seed_insert<true> : k_seed_insert<false>), dim3((unsigned)bgl::ceil_div(L.P[0], TILE)),
                           dim3(TILE), 0, st, seeds, num_seeds, g->num_nodes, tab, mask, slotidx, cnt);
        place(0, 0, L.P[0], nullptr, nullptr, false);
    }
    for (int h = 0; h < num_hops; ++h) {
        const int blocks = (int)bgl::ceil_div(L.P[h + 1], TILE);
        const uint64_t h0 = mix64(rng_seed + GOLDEN * (uint64_t)(h + 1));
        const int enter = h == 0 && few_seeds;
        if (g->bits == 64) launch_sample_g<int64_t>(L.G[h], k, blocks, h, fanouts[h], h0, enter);
        else launch_sample_g<int32_t>(L.G[h], k, blocks, h, fanouts[h], h0, enter);
        place(h + 1, L.logG[h], L.P[h + 1], out->row_ptr[h], out->col_local[h], h == num_hops - 1);
    }
    BGL_HIP(hipGetLastError());
    if (counts_host && !counts_dev)
        BGL_HIP(hipMemcpyAsync(counts_host, cnt, sizeof(int32_t) * BGL_COUNTS_LEN,
                               hipMemcpyDeviceToHost, st));
    return BGL_OK;
} BGL_NOTHROW_END
