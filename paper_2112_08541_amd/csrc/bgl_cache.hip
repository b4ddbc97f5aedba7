// GPU-resident FIFO feature cache (BGL paper, Sec. 3.2: dynamic FIFO policy,
// cache map + cache buffer per GPU, lookup / gather / fetch / update workflow;
// Sec. 4 "Feature Cache Engine": circular buffer addressed through a running
// tail, the occupant of the next position is evicted from the map and its row
// overwritten, cache work on a dedicated stream).
//
// Cache map: open addressing over 128-byte buckets.  A bucket is 16 64-bit
// words = exactly one cache line: words 0..14 hold (node id << 32 | slot) or
// EMPTY, word 15 counts the live entries that rest in a later bucket although
// their id hashes to this one or to an earlier one, i.e. whose walk from their
// home bucket to their resting bucket passed over this bucket.  A lookup reads
// its id's bucket (one line) and goes on to the next bucket only while that
// count is not zero (one id per lane: a wavefront keeps 64 independent line
// reads in flight; a 16-lanes-per-id lookup that found the id with a ballot was
// measured at half the speed, the lookup being latency bound).  An insertion
// (one per lane too) reads the bucket, claims a free word with a CAS, and raises
// the count of every full bucket it walks past by one.  An eviction blanks its
// word (slot_to_entry[slot] remembers the word that maps a slot's occupant, so
// no search) and lowers the counts of the buckets between the evicted id's home
// bucket (recomputed from the id) and that word's bucket: what one insertion
// added, the eviction of the same entry takes away.  So the counts always say
// exactly which buckets a live entry was pushed past, however long the cache
// has been churning under the FIFO policy: no tombstones, no rebuilds, and the
// length of a lookup depends on the load only (full buckets are rare at load
// <= 1/2 of 15 words per bucket), not on the cache's age.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include <hip/hip_ext.h>

#include "bgl_host_tier.h"
#include "bgl_internal.h"

namespace {

using namespace bgl;

constexpr uint64_t EMPTY64 = ~0ull;
constexpr int BUCKET = 16;       // 64-bit words per bucket (15 entries + the count of entries pushed past it)
constexpr int KEYS_PER_TILE = 256;  // ids per workgroup in probe / miss-list kernels
constexpr int PROF_RING = 4096;

struct CacheDev {          // device-resident scalars
    // tail is kept twice: FIFO update number k reads tail[k & 1] in every
    // workgroup while one lane writes tail[(k + 1) & 1], so no launch is needed
    // just to advance it.  The host counts the updates (bgl_cache::insert_calls).
    unsigned long long tail[2];
    unsigned long long lookups, hits;
    long long n_miss_last;  // miss count of the most recent lookup
    long long n_miss_gen[2];  // the same, kept per call parity for early lookups (the previous call's fetch still reads its own)
    long long n_hit_last;   // hit count of the most recent lookup
    int status;
    unsigned long long probe_lines;  // bucket lines read by all map lookups so far
    unsigned long long census[2];    // bgl_cache_map_stats: buckets with a count, sum of the counts
};

}  // namespace

struct bgl_cache {
    int64_t capacity = 0;
    int32_t row_bytes = 0;
    int64_t num_nodes = 0;
    const char *features = nullptr;  // device-visible backing store
    bool features_in_hbm = false;    // backing store is device memory (then the fetch is an HBM gather)
    int device = 0;
    int64_t rows = 0;                // row positions of the buffer: capacity + spare positions (see RowRing)
    char *buffer = nullptr;          // rows * row_bytes
    uint64_t *table = nullptr;       // num_buckets * BUCKET words
    uint32_t num_buckets = 0;        // power of two
    int32_t *slot_to_node = nullptr;  // capacity
    uint32_t *slot_to_entry = nullptr;
    CacheDev *dev = nullptr;
    int32_t *mbs = nullptr;          // per-tile miss counts of the most recent lookup (mbs_cap of them), then mbs_cap prefixes,
                                     // then mbs_cap counts of bucket lines read
    int64_t mbs_cap = 0;
    int32_t *hit_pos = nullptr;      // hits of the most recent lookup: hit_cap positions, then hit_cap slots
    int64_t hit_cap = 0;
    int64_t last_n = 0;              // n of the most recent lookup
    int32_t *mpos_copy[2] = {nullptr, nullptr};  // early lookups: the library's own copy of miss_pos, alternating between calls
    int64_t mpos_cap[2] = {0, 0};
    int32_t *src_of[2] = {nullptr, nullptr};  // assembled output: where each position's row comes from, alternating between calls
    int64_t src_cap[2] = {0, 0};
    uint64_t lookup_calls = 0;
    uint64_t insert_calls = 0;       // FIFO updates enqueued so far (selects the live copy of tail)
    hipStream_t own_side = nullptr;  // the miss fetch's stream when the caller names none; created on first use
                                     // (a process has few hardware queues: a stream that is never used should not take one)
    // Ordering between streams.  ev_listed: lists and hit rows of the last lookup are complete
    // (recorded on that lookup's main stream); ev_miss: its miss rows are complete and so are its hit
    // rows (recorded on the stream the fetch ran on, behind the hit gather: whoever waits for the rows,
    // or is behind the call in that stream, has all of them; not recorded where rows_split); ev_map: the last FIFO update is complete
    // (recorded on the update's stream), or ev_map_local: map_event says which (see LONG_LOOKUP_BYTES).
    // ev_fetched: a fetch that ran beside the hit gather is complete, whatever the gather does (for work
    // that is behind the gather anyway, and where rows_split for everyone, together with ev_listed).  ev_behind: nothing
    // waits for it (see BESIDE_BYTES).
    hipEvent_t ev_listed = nullptr, ev_miss = nullptr, ev_map = nullptr, ev_fetched = nullptr, ev_behind = nullptr;
    hipEvent_t ev_map_local = nullptr, map_event = nullptr;
    hipEvent_t ev_ids = nullptr;     // the lists of a lookup are complete (tiered: the missed ids have reached the host)
    hipEvent_t ev_lists = nullptr;   // the same for this cache's own miss fetch on the side stream
    hipStream_t last_main = nullptr, fetch_stream = nullptr, map_stream = nullptr;
    bool fetch_pending = false;      // ev_miss marks a miss fetch that later work may have to wait for
    bool rows_joined = false;        // a FIFO update on the lookup's main stream has made it wait for that fetch
    bool rows_split = false;         // ev_miss marks neither: ev_fetched the fetch, ev_listed the hit gather beside it
    bool fetch_beside = false;       // that fetch ran beside its hit gather: ev_fetched marks its own end
    bool fetch_reads_caller_lists = true;  // that fetch reads the caller's miss_pos (not the library's copy)
    bool map_pending = false;        // map_event marks a FIFO update the next lookup has to wait for
    bool ev_listed_valid = false;    // a lookup has recorded ev_listed
    bool streaming = false;          // the caller enqueues batch after batch and waits for no stream meanwhile (the overlapped loop)
    bool write_through = false;      // the miss fetch also fills the cache buffer (see bgl_cache_set_write_through)
    bool awaiting_insert = false;    // write-through: a lookup's misses are in the buffer but not in the map yet
    const void *wt_ids = nullptr, *wt_miss_pos = nullptr;  // arguments of that lookup
    // A tiered lookup between its two halves (bgl_cache_lookup_tiered_begin / _finish): the host threads
    // are packing its rows, the kernels that take them to their places have not been enqueued yet.
    struct TieredCall {
        bool active = false;
        bgl_host_tier *t = nullptr;
        bgl::TierPlan plan;
        hipStream_t ms = nullptr, ss = nullptr, ls = nullptr;
        const int32_t *ids = nullptr, *mpos = nullptr, *src_of = nullptr;
        int32_t *miss_pos = nullptr;
        void *out_rows = nullptr;
        int64_t n = 0;
        int par = 0, gen = 0;
        bool in_place = false;
    } tiered;
    // profiling
    unsigned profiling = 0;          // bit s set: stage s is timed
    hipEvent_t timed_start = nullptr, timed_stop = nullptr;  // events the next launch() hands to the kernel dispatch itself
    std::vector<hipEvent_t> prof_ev;  // pairs
    struct Rec { int stage; int ev; };
    std::vector<Rec> prof_rec;
    double prof_overhead_ms = 0;     // event pair around an (almost) empty kernel
    int64_t prof_dropped = 0;        // timed launches that got no events (event creation failed)
    int prof_every[BGL_NUM_STAGES];  // stage s is timed only in calls whose ordinal is a multiple of this
    double prof_ms[BGL_NUM_STAGES] = {};
    int64_t prof_n[BGL_NUM_STAGES] = {};

    bgl_cache() { std::fill(prof_every, prof_every + BGL_NUM_STAGES, 1); }
};

namespace {

// ------------------------------------------------------------------ kernels
__global__ void k_fill_u64(uint64_t *p, int64_t n, uint64_t v, int mark_stride)
{
    // every mark_stride-th word (the buckets' pushed-past counts) starts at 0
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = ((i % mark_stride) == mark_stride - 1) ? 0ull : v;
}

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

// Map lookup, one id per lane.  A lane reads its id's whole bucket (one 128-byte
// line, eight 16-byte loads issued together) and compares the 15 entries in
// registers; the chain continues only past a bucket whose pushed-past count is
// not zero.  A wavefront thus keeps 64 independent line reads in flight, which is
// what a latency-bound random lookup needs.  The misses of a wavefront are
// counted with one ballot; the bucket lines read are summed per workgroup for
// the map statistics (the list kernel adds the sums up).  own_slot: a second copy of the slots for a fetch on another stream
// (k_fetch_slots), or null.
__global__ __launch_bounds__(KEYS_PER_TILE) void k_probe(const int32_t *__restrict__ ids, int64_t n,
                                                         int64_t num_nodes,
                                                         const uint64_t *__restrict__ table,
                                                         uint32_t bucket_mask, int32_t *out_slot, int32_t *own_slot,
                                                         int32_t *mbs, int32_t *tile_lines, CacheDev *dev)
{
    __shared__ int sh_miss[KEYS_PER_TILE / kWave];
    __shared__ int sh_lines[KEYS_PER_TILE / kWave];
    const int64_t i = (int64_t)blockIdx.x * KEYS_PER_TILE + threadIdx.x;
    int slot = -1;
    int lines = 0;
    if (i < n) {
        const int32_t id = ids[i];
        if (id < 0 || (int64_t)id >= num_nodes) {
            dev->status = BGL_EINVAL;
        } else {
            const uint32_t key = (uint32_t)id;
            uint32_t b = hash32(key) & bucket_mask;
            for (uint32_t tries = 0; tries <= bucket_mask; ++tries) {
                const ulonglong2 *bp = reinterpret_cast<const ulonglong2 *>(table + (size_t)b * BUCKET);
                ulonglong2 w[BUCKET / 2];
#pragma unroll
                for (int k = 0; k < BUCKET / 2; ++k) w[k] = bp[k];
                bool found = false;
#pragma unroll
                for (int k = 0; k < BUCKET / 2; ++k) {
                    if ((uint32_t)(w[k].x >> 32) == key) { slot = (int)(uint32_t)w[k].x; found = true; }
                    if (k < BUCKET / 2 - 1 && (uint32_t)(w[k].y >> 32) == key) {
                        slot = (int)(uint32_t)w[k].y;
                        found = true;
                    }
                }
                ++lines;
                if (found || w[BUCKET / 2 - 1].y == 0) break;  // count zero: no live entry was pushed past this bucket
                b = (b + 1) & bucket_mask;
            }
        }
        out_slot[i] = slot;
        if (own_slot) own_slot[i] = slot;
    }
    const uint64_t missed = __ballot(i < n && slot < 0);
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) lines += __shfl_down(lines, d, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        sh_miss[threadIdx.x / kWave] = __popcll(missed);
        sh_lines[threadIdx.x / kWave] = lines;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0, ln = 0;
#pragma unroll
        for (int k = 0; k < KEYS_PER_TILE / kWave; ++k) { t += sh_miss[k]; ln += sh_lines[k]; }
        mbs[blockIdx.x] = t;
        tile_lines[blockIdx.x] = ln;  // (summed by the list kernel: one atomic per workgroup on one counter
                                      // costs this kernel a third of its time)
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const int32_t *mbs, int64_t tiles, int32_t *prefix)
{
    __shared__ int sh[kScanThreads / kWave];
    scan_tile_counts<kScanThreads>(mbs, tiles, prefix, sh);
}

// Counters of an empty lookup (n = 0); with n > 0 k_split_list publishes them.
__global__ void k_empty_lookup(CacheDev *dev, int64_t *n_hit_host, int gen)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        dev->n_miss_last = 0;
        dev->n_miss_gen[gen] = 0;
        dev->n_hit_last = 0;
        if (n_hit_host) *n_hit_host = 0;
    }
}

// Where the rows live.  The cache buffer has `rows` >= capacity row positions.  Insertion
// number k (counted from the cache's creation, k = tail at the time) is written to position
// k mod rows, while its slot, which is what the map, out_slot and slot_to_node speak of, is
// k mod capacity.  With rows == capacity the two are the same number.  With spare positions
// (bgl_cache_set_spare_rows) a batch's new rows go to positions that hold no live row as long
// as the batch has no more misses than there are spare positions: the rows its own
// insertions evict stay readable until the next batch, so nothing has to be read "before it
// is overwritten".  The live rows are the last min(tail, capacity) insertions; slot and
// position of a live row follow from each other and tail by additions alone.
__device__ __forceinline__ unsigned long long uniform(unsigned long long v)  // keeps the divisions below off the vector unit
{
    return (unsigned long long)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
struct RowRing {
    int64_t capacity, rows;
    int64_t newest_slot, newest_pos;  // of insertion tail - 1 (tail > 0)
    // this call's insertions: ranks start <= r < start + count stay, rank r goes to position first_pos + (r - start)
    int64_t start, count, first_pos;
    // (tail and n_miss are the same for all lanes)
    __device__ __forceinline__ RowRing(unsigned long long tail, int64_t capacity_, int64_t rows_, int64_t n_miss = 0)
        : capacity(capacity_), rows(rows_)
    {
        tail = uniform(tail);
        n_miss = (int64_t)uniform((unsigned long long)n_miss);
        const unsigned long long newest = tail > 0 ? tail - 1 : 0;
        newest_slot = (int64_t)(newest % (unsigned long long)capacity);
        newest_pos = (int64_t)(newest % (unsigned long long)rows);
        start = n_miss > capacity ? n_miss - capacity : 0;
        count = n_miss - start;
        first_pos = (int64_t)((tail + (unsigned long long)start) % (unsigned long long)rows);
    }
    __device__ __forceinline__ int64_t pos_of_slot(int64_t slot) const  // an occupied slot
    {
        int64_t age = newest_slot - slot;  // insertions since
        if (age < 0) age += capacity;
        const int64_t pos = newest_pos - age;
        return pos < 0 ? pos + rows : pos;
    }
    __device__ __forceinline__ int64_t pos_of_rank(int64_t r) const  // start <= r < start + count
    {
        const int64_t pos = first_pos + (r - start);
        return pos >= rows ? pos - rows : pos;
    }
    __device__ __forceinline__ bool overwritten(int64_t pos) const  // by this call's insertions
    {
        int64_t d = pos - first_pos;
        if (d < 0) d += rows;
        return d < count;
    }
};

// What the list kernels read and write.
struct Lists {
    const int32_t *out_slot;
    int64_t n;
    const int32_t *mbs, *tile_prefix, *tile_lines;  // of tiles of KEYS_PER_TILE ids: misses, misses before, bucket lines read
    int32_t *miss_pos, *hit_pos, *hit_slot;
    CacheDev *dev;
    int64_t *n_hit_host;
    const int32_t *ids;
    int64_t num_nodes;
    int32_t *miss_ids_host, *miss_pos_copy;
    int gen;
    int32_t *src_of;
    int64_t capacity, rows;
    int par;
};

// Ordered lists of the miss positions and (HITS) of the hits (position and slot side by
// side, so the gather needs no dependent lookup).  A hit's rank is its position
// minus the number of misses before it.  Every workgroup sums the miss counts of
// the tiles before it (a few thousand ints at most), or reads the sum from
// tile_prefix where the call has so many tiles that k_scan_tiles ran first; the
// last one also publishes the call's counters.
template <bool HITS>
__device__ __forceinline__ void list_tile(const Lists &l, int block, int blocks)
{
    __shared__ int sh_scan[KEYS_PER_TILE / kWave];
    __shared__ int sh_base;
    int tot;
    if (l.tile_prefix) {
        if (threadIdx.x == 0) sh_base = l.tile_prefix[block];
    } else {
        int part = 0;
        for (int t = threadIdx.x; t < block; t += KEYS_PER_TILE) part += l.mbs[t];
        (void)block_excl_scan<KEYS_PER_TILE>(part, sh_scan, tot);
        if (threadIdx.x == 0) sh_base = tot;
    }
    const int64_t i = (int64_t)block * KEYS_PER_TILE + threadIdx.x;
    const int slot = i < l.n ? l.out_slot[i] : 0;
    const int flag = (i < l.n && slot < 0) ? 1 : 0;
    const int ex = block_excl_scan<KEYS_PER_TILE>(flag, sh_scan, tot);  // its barriers publish sh_base
    const int mrank = sh_base + ex;
    if (flag) {
        l.miss_pos[mrank] = (int32_t)i;
        if (HITS && l.miss_pos_copy) l.miss_pos_copy[mrank] = (int32_t)i;
        if (HITS && l.miss_ids_host) {  // a host tier that keeps nothing: it only wants the ids of the misses, in order
            const int32_t id = l.ids[i];
            l.miss_ids_host[mrank] = id;
            if (id < 0 || (int64_t)id >= l.num_nodes) l.n_hit_host[3] = 1;  // the host refuses the batch
        }
    } else if (HITS && i < l.n) {
        // the kernels that read the row get its position in the cache buffer (see RowRing)
        const int32_t pos = l.rows == l.capacity ? slot : (int32_t)RowRing(l.dev->tail[l.par], l.capacity, l.rows).pos_of_slot(slot);
        if (!l.src_of) {
            l.hit_pos[i - mrank] = (int32_t)i;
            l.hit_slot[i - mrank] = pos;
        } else {
            l.src_of[i] = pos;
        }
    }
    // assembled output (k_assemble_rows): the source of every position's row, a row position of the
    // cache buffer (>= 0) or, as -(r + 1), miss number r, whose row comes in with the packed miss rows
    if (HITS && l.src_of && flag) l.src_of[i] = -(mrank + 1);
    if (block != blocks - 1) return;
    // the last workgroup publishes the call's counters
    int lines = 0, all_lines;
    for (int t = threadIdx.x; t < blocks; t += KEYS_PER_TILE) lines += l.tile_lines[t];
    (void)block_excl_scan<KEYS_PER_TILE>(lines, sh_scan, all_lines);
    if (threadIdx.x == 0) {
        CacheDev *const dev = l.dev;
        const long long n_miss = sh_base + tot;
        dev->probe_lines += (unsigned long long)all_lines;
        dev->n_miss_last = n_miss;
        dev->n_miss_gen[l.gen] = n_miss;
        dev->n_hit_last = l.n - n_miss;
        dev->lookups += (unsigned long long)l.n;
        dev->hits += (unsigned long long)(l.n - n_miss);
        // page-locked host memory: visible to the host once the kernel has completed
        if (l.n_hit_host) *l.n_hit_host = l.n - n_miss;
        if (HITS && l.miss_ids_host) {  // the tier's counts: nothing found there, everything to be brought in
            l.n_hit_host[1] = 0;
            l.n_hit_host[2] = n_miss;
        }
    }
}

__global__ __launch_bounds__(KEYS_PER_TILE) void k_split_list(Lists l) { list_tile<true>(l, blockIdx.x, gridDim.x); }

// Row copies move 16-byte chunks; a row has Q = row_bytes / 16 of them.  Chunk
// index -> (row, chunk in row) with a compile-time Q where the width is a
// common one, so the division is a multiply.
template <int Q>
struct RowSplit {
    __device__ __forceinline__ static void split(int64_t idx, int q, int64_t &row, int &c)
    {
        if constexpr (Q > 0) { row = idx / Q; c = (int)(idx - row * Q); }
        else { row = idx / q; c = (int)(idx - row * q); }
    }
};

constexpr int COPY_THREADS = 256;
constexpr int MAP_THREADS = 64;  // rows per workgroup of the map update: a short batch spreads over many CUs
constexpr int COPY_UNROLL = 4;  // (the kernels name the four chunks of a lane by hand)
// Workgroups of a kernel that reads rows over the host link.  Each lane keeps
// four 16-byte loads in flight, so 64 x 256 lanes hold 1 MiB: that saturates
// the link for rows read in place (whole 128-byte lines, partly unused), and
// much more queues host reads in front of the concurrent kernels' HBM reads and
// slows those by an order of magnitude.  The packed ring is read densely and
// needs half as much in flight; with 64 workgroups there the next batch's
// lookup, and with it the packing of its rows, starts late.
constexpr int FETCH_BLOCKS = 64;
// Misses a wavefront of k_fetch_slots may have queued: less than a round of its fetch, and 64 more.
__host__ __device__ constexpr int slots_queue(int q) { return COPY_UNROLL * (kWave / q) + kWave; }
constexpr int RING_FETCH_BLOCKS = 32;
// The overlapped loop's small batches (write-through mode, FIFO updates on another stream than the fetches:
// the update and the next batch's sampling run beside the fetch): the bytes a lookup asks for at most, and
// the workgroups.  Every host read in
// flight beyond what the link needs delays the other kernels' HBM reads (with 64 workgroups the map
// update of 315 K rows took 700 us beside the fetch, with 24 it took 85), and a small batch is bound by
// those kernels' launches as much as by the link.  Microseconds per batch with 8 / 16 / 24 / 64
// workgroups: 2.6 MB asked 106 / 112 / 121 / 124; 4.2 MB 160 / 141 / 155 / 164; 8.4 MB 278 / 228 / 232 /
// 246; 16.8 MB 517 / 404 / 406 / 412.  A larger batch is bound by the fetch alone, which takes 7 % longer
// with 16 workgroups (3,270 against 3,055 us at 128 MB of misses), and so is a small one with nothing beside
// it (16 MB asked, fetch with 16 / 64 workgroups: 400-byte rows 427 / 391 us, 528 bytes 433 / 369, 1,024
// bytes 317 / 301).  (More workgroups where lanes stay idle, so that as many bytes are in flight: 528-byte
// rows 16 MB 374 -> 369 us, but 64 MB 1,448 -> 1,483.)
// Below 3 MiB fewer still, one for every 192 KiB: us a batch with 8 / 10 / 12 / 16 workgroups, 0.4 MB asked for 59.4 / 59.7 / 59.3 / 60.8, 0.7 MB
// 48.2 / 48.7 / 49.1 / 48.8, 1.6 MB 67.9 / 67.9 / 66.9 / 67.2, 2.3 MB 68.3 / 67.5 / 70.5 / 74.6, 2.4 MB 84.1 / 77.4 / 77.1 / 79.2, 3.3 MB
// 109.9 / 98.3 / 95.5 / 92.3, 6.1 MB 143 / 130 / 124 / 122.
constexpr int64_t SMALL_LOOKUP_BYTES = 16 << 20;
constexpr int SMALL_FETCH_BLOCKS = 16, LEAST_FETCH_BLOCKS = 8;
constexpr int64_t SMALL_FETCH_BYTES_PER_BLOCK = 192 << 10;
// Tiered lookup: rows the host threads copy per chunk before that chunk's fetch is launched.
constexpr int64_t TIER_CHUNK_ROWS = 49152;
constexpr int64_t TIER_FIRST_CHUNK_ROWS = 3072;
// Copy-engine transport without the early lookup: bytes that are worth a copy of their own (35 us on the
// link, beside some 10 us that a copy costs whatever its size).  Where it lies matters little: with 1, 2 and 4 MiB, rows of 16 to
// 1,024 bytes and 500 to 150,000 ids differ by 2 % or less.  Against chunks that double up to TIER_CHUNK_ROWS no size lost (272 B x
// 150,000 ids 1,074 -> 995 us, 400 B 1,449 -> 1,340, 528 B 1,871 -> 1,708, 60,000 ids x 528 B 891 -> 832; 5,000 ids and fewer: the same).
constexpr int64_t LINK_CHUNK_BYTES = 2 << 20;
// Lookups that ask for more bytes than this keep the GPU busy for longer than the host takes to enqueue
// them.  Three things pay only there:
//  - the FIFO update's event without a release to the system (only this library's kernels on this device
//    wait for it).  A row of calls saves 5 us of each (lookup + update of 302,709 hits of 1,024 bytes), but a host that waits for a stream whose last command it is enqueues another one first: 500
//    ids of 400 bytes, each call waited for, 63 / 70 us; hidden once the kernels outlast the host.  (Always
//    without it where the updates have a stream of their own, as in the overlapped loop: 512 seeds on
//    10,000 nodes, 20 batches 2,110 / 2,060 us.)
//  - the miss fetch beside the hit gather, in a cache that can hold every node.  It saves the update two
//    hand-overs between streams behind the gather, and overlaps a short fetch with a long gather; costs the
//    host three more calls.  Lookup + update behind / beside, microseconds: 2 MB of hits, each call waited
//    for 60 / 83, one after the other 59 / 67; 41 MB 71 / 86, 70 / 66; 82 MB 80 / 95, 75 / 70; 120 MB 101 /
//    100, 90 / 80; 205 MB 114 / 110, 101 / 94; with 2 % misses 120 MB 157 / 135, 205 MB 187 / 150; with half
//    of the ids missed the link sets the time either way.
//  - the own event of a fetch behind the gather: 100,000 ids x 400 B, all hits, 70 / 62 with an event behind it, 74 / 59
//    with its own; 250,000 x 64 B 70 / 68, 76 / 63.
constexpr int64_t LONG_LOOKUP_BYTES = 100ll << 20;
// Lookups of up to this many bytes whose miss fetch has the cache's own side stream start it beside the hit
// gather.  Its end is the launch's own event, which the update waits for, and an event that nothing waits for is recorded
// behind it, so that a host that waits finds one (see launch_marked).  Lookup + update, each waited for / one after the
// other, us: fetch behind the gather with no own event | beside, event behind | beside, own event | beside, both:
//   ids x bytes   10 % hits                                   50 % hits                               all hits
//   500 x 400     75 / 71 | 75 / 69 | 71 / 61 | 63 / 58       71 / 68 | 70 / 64 | 60 / 53 | 57 / 56   70 / 68 | 55 / 56 | 62 / 55 | 54 / 57
//   2,000 x 400   76 / 71 | 75 / 72 | 75 / 71 | 75 / 72       68 / 70 | 73 / 70 | 79 / 70 | 74 / 70   70 / 67 | 55 / 57 | 62 / 55 | 55 / 58
//   5,000 x 400   103 / 92 | 97 / 84 | 97 / 81 | 98 / 81      84 / 75 | 80 / 71 | 82 / 70 | 80 / 72   72 / 66 | 55 / 55 | 61 / 55 | 55 / 56
//   20,000 x 400  230 / 219 | 227 / 213 | 224 / 209 | 224 / 209   154 / 143 | 150 / 136 | 149 / 133 | 148 / 133   72 / 67 | 56 / 56 | 62 / 54 | 55 / 55
//   10,000 x 1024 226 / 216 | 223 / 211 | 221 / 206 | 221 / 206   153 / 142 | 149 / 136 | 147 / 133 | 147 / 132   72 / 62 | 63 / 57 | 61 / 53 | 55 / 55
//   30,000 x 64   148 / 135 | 144 / 127 | 144 / 124 | 144 / 123   110 / 97 | 108 / 89 | 110 / 86 | 109 / 88   63 / 72 | 61 / 62 | 69 / 61 | 62 / 63
// (no lower bound: 200 ids x 64 / 400 / 1,024 B, 10 % hits, behind | beside 67 / 67 | 62 / 61, 66 / 61 | 62 / 57, 73 / 74 | 71 / 69;
// 160,000 ids x 400 B 1,441 / 1,439 | 1,420 / 1,419.)  Beyond, a short gather is held up by the host reads (428,377 ids x 400 B 20 -> 140 us)
// and the whole gains nothing.
constexpr int64_t BESIDE_BYTES = 64 << 20;
constexpr int64_t FROM_SLOTS_BYTES = 32 << 20;  // of those, the ones whose fetch reads the probe's slots (lookup_gather_impl)
// Hit gather: largest output (of the hits) whose rows are read and written with ordinary accesses, and largest one that is not
// written non-temporally (the size of the last-level cache).
constexpr int64_t GATHER_CACHED_ROWS_BYTES = 64ll << 20;
constexpr int64_t GATHER_CACHED_OUTPUT_BYTES = 256ll << 20;
// Assembled output: largest out_rows of a call that is still written with ordinary stores.
constexpr int64_t ASSEMBLE_CACHED_OUTPUT_BYTES = 128ll << 20;

// 16-byte accesses that say "not needed again soon" (NT) or nothing.
template <bool NT>
__device__ __forceinline__ void st16(uint4 *p, const uint4 &v)
{
    if (NT) __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(p));
    else *p = v;
}
template <bool NT>
__device__ __forceinline__ uint4 ld16(const uint4 *p)
{
    if (NT) {
        const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        return uint4{t.x, t.y, t.z, t.w};
    }
    return *p;
}

// How the gathered rows are stored.
enum Stores { ORDINARY, THROUGH, NON_TEMPORAL };
template <int S>
__device__ __forceinline__ void st_gathered(uint4 *out, int64_t at, const uint4 &v)
{
    if constexpr (S == THROUGH) store16_through(out, (uint32_t)at * 16u, v);
    else st16<S == NON_TEMPORAL>(out + at, v);
}
// The accesses for `bytes` of gathered rows in an output of out_bytes (both the same for all lanes; a buffer store's offset has 32 bits).
template <typename F>
__device__ __forceinline__ void by_gather_size(int64_t bytes, int64_t out_bytes, F &&copy)
{
    using std::integral_constant;
    if (bytes <= GATHER_CACHED_ROWS_BYTES) copy(std::false_type{}, integral_constant<int, ORDINARY>{});
    else if (bytes > GATHER_CACHED_OUTPUT_BYTES) copy(std::true_type{}, integral_constant<int, NON_TEMPORAL>{});
    else if (out_bytes > (int64_t)UINT32_MAX) copy(std::true_type{}, integral_constant<int, ORDINARY>{});
    else copy(std::true_type{}, integral_constant<int, THROUGH>{});
}

// out[i] = the cached row of ids[i] for every hit i (taken from the hit list, which holds the
// rows' positions in the cache buffer, so the work is proportional to the hits).  Consecutive lanes take consecutive
// 16-byte chunks of a row, so the loads and stores of one row are contiguous;
// four independent chunks per lane keep loads in flight.  The grid is sized for
// n rows; workgroups beyond the hit count leave at once.
//   What the caches keep: a row is read once per launch, so beyond GATHER_CACHED_ROWS_BYTES its loads say
// so and leave the last-level cache (256 MB) to the output; output beyond GATHER_CACHED_OUTPUT_BYTES would
// not stay there either and is stored non-temporally too.  Microseconds, loads and stores ordinary / loads
// non-temporal / stores non-temporal / both; launches in a row with other ids | a 512 MiB copy before each:
//   72 MB from a buffer of 196 MB   25 / 27 / 23 / 31 | 35 / 29 / 39 / 31
//   102 MB from 614 MB              31 / 30 / 33 / 38 | 43 / 34 / 50 / 38
//   160 MB (400-byte rows) from 800 68 / 53 / 59 / 65 | 72 / 59 / 84 / 65
//   256 MB from 256 MB              96 / 69 / 70 / 89 | 99 / 75 / 119 / 89
//   310 MB from 614 MB              120 / 117 / 102 / 108 | 119 / 92 / 138 / 108
//   512 MB from 1,024 MB            196 / 184 / 185 / 179 | 195 / 164 / 210 / 179
//   1.6 GB (400 bytes), 4.1 GB      after a copy: 688 / 649 / 661 / 626, 1,584 / 1,522 / 1,556 / 1,484
// (Non-temporal stores alone are the fastest where nothing else has used the caches since the last launch,
// and the slowest where something has.)
//   Between the two bounds the rows are written through the L2s (store16_through): launches in a row | behind a copy | launch and
// a reader of its output, loads non-temporal, stores ordinary / through:
//   72 MB from 614 MB               25.1 / 22.9 | 28.4 / 25.6 | 36.8 / 34.3
//   160 MB (400 bytes) from 800     58.0 / 54.3 | 64.1 / 58.9 | 81.4 / 77.7
//   256 MB from 614 MB              76.6 / 73.5 | 81.0 / 77.5 | 113 / 110
//   (the kernel alone) 102, 205 MB (512 bytes) from 12.8 GB  35.2 / 33.4, 63.6 / 61.1 | 35.9 / 34.9, 64.9 / 62.2 | 35.6 / 34.0, 63.3 / 61.6
// Below 64 MB ordinary accesses are as fast (44 MB 16.4 / 17.2 | 24.5 / 19.8 | 24.4 / 25.3); beyond 256 MB non-temporal stores written
// through or not differ by 1 %.
template <int Q>
__global__ __launch_bounds__(COPY_THREADS) void k_gather_hits(
    const int32_t *__restrict__ hit_pos, const int32_t *__restrict__ hit_slot, int q,
    const uint4 *__restrict__ buffer, uint4 *__restrict__ out, int64_t out_bytes, const CacheDev *dev)
{
    static_assert(COPY_UNROLL == 4, "the four chunks of a lane are written out by hand");
    const int qq = Q > 0 ? Q : q;
    const int64_t total = (int64_t)dev->n_hit_last * qq;
    const int64_t base = (int64_t)blockIdx.x * (COPY_THREADS * COPY_UNROLL) + threadIdx.x;
    if (base - threadIdx.x >= total) return;
    // Three phases without a branch in between, so that the four list reads of a lane are in flight
    // together, then its four row reads, then its stores: chunk numbers beyond the end are clamped
    // to the last chunk, which those lanes then copy once more (same bytes to the same place).
    // (Written chunk by chunk with a branch each, every read waited for the one before it; with only
    // the stores under a branch the compiler moved reads back in there; and as an array `uint4 v[4]`
    // the values were put into LDS instead of registers.)
    const int64_t last = total - 1;
    int64_t r0, r1, r2, r3;
    int c0, c1, c2, c3;
    RowSplit<Q>::split(min(base, last), q, r0, c0);
    RowSplit<Q>::split(min(base + COPY_THREADS, last), q, r1, c1);
    RowSplit<Q>::split(min(base + 2 * COPY_THREADS, last), q, r2, c2);
    RowSplit<Q>::split(min(base + 3 * COPY_THREADS, last), q, r3, c3);
    const int32_t s0 = hit_slot[r0], s1 = hit_slot[r1], s2 = hit_slot[r2], s3 = hit_slot[r3];
    const int32_t p0 = hit_pos[r0], p1 = hit_pos[r1], p2 = hit_pos[r2], p3 = hit_pos[r3];
    by_gather_size(total * 16, out_bytes, [&](auto nt_loads, auto stores) {
        // (the markers keep the compiler from merging the branches' accesses into ordinary ones)
        asm volatile("; rows");
        const uint4 v0 = ld16<nt_loads.value>(&buffer[(int64_t)s0 * qq + c0]);
        const uint4 v1 = ld16<nt_loads.value>(&buffer[(int64_t)s1 * qq + c1]);
        const uint4 v2 = ld16<nt_loads.value>(&buffer[(int64_t)s2 * qq + c2]);
        const uint4 v3 = ld16<nt_loads.value>(&buffer[(int64_t)s3 * qq + c3]);
        st_gathered<stores.value>(out, (int64_t)p0 * qq + c0, v0);
        st_gathered<stores.value>(out, (int64_t)p1 * qq + c1, v1);
        st_gathered<stores.value>(out, (int64_t)p2 * qq + c2, v2);
        st_gathered<stores.value>(out, (int64_t)p3 * qq + c3, v3);
        asm volatile("; end of rows");
    });
}

// The miss list and the hit gather in one launch: the first workgroups are k_split_list's without the list of the hits, the
// others copy the rows in the order of the positions, from the slots that the probe has left.  The gather then need not wait
// for the lists, which are 4 to 6 us and a launch.  For calls that ask for little or hit for the most part: the positions of
// misses cost reads and idle lanes, and the hits' number, which k_gather_hits chooses its accesses by, is not known: here
// that is the number asked for.
template <int Q>
__global__ __launch_bounds__(COPY_THREADS) void k_list_and_hits(Lists l, int tiles, int q, const uint4 *__restrict__ buffer,
                                                                uint4 *__restrict__ out)
{
    static_assert(COPY_THREADS == KEYS_PER_TILE && COPY_UNROLL == 4, "both kinds of workgroups have one size");
    if ((int)blockIdx.x < tiles) {
        list_tile<false>(l, blockIdx.x, tiles);
        return;
    }
    const int qq = Q > 0 ? Q : q;
    const int64_t last = l.n * qq - 1;
    const int64_t base = (int64_t)(blockIdx.x - tiles) * (COPY_THREADS * COPY_UNROLL) + threadIdx.x;
    // Phase by phase, as in k_gather_hits; positions of misses read a row that is not stored.
    const int64_t x0 = min(base, last), x1 = min(base + COPY_THREADS, last), x2 = min(base + 2 * COPY_THREADS, last),
                  x3 = min(base + 3 * COPY_THREADS, last);
    int64_t i0, i1, i2, i3;
    int c0, c1, c2, c3;
    RowSplit<Q>::split(x0, q, i0, c0);
    RowSplit<Q>::split(x1, q, i1, c1);
    RowSplit<Q>::split(x2, q, i2, c2);
    RowSplit<Q>::split(x3, q, i3, c3);
    const int32_t s0 = l.out_slot[i0], s1 = l.out_slot[i1], s2 = l.out_slot[i2], s3 = l.out_slot[i3];
    int64_t p0 = max(s0, 0), p1 = max(s1, 0), p2 = max(s2, 0), p3 = max(s3, 0);
    if (l.rows != l.capacity) {  // uniform
        const RowRing ring(l.dev->tail[l.par], l.capacity, l.rows);
        p0 = s0 < 0 ? 0 : ring.pos_of_slot(s0);
        p1 = s1 < 0 ? 0 : ring.pos_of_slot(s1);
        p2 = s2 < 0 ? 0 : ring.pos_of_slot(s2);
        p3 = s3 < 0 ? 0 : ring.pos_of_slot(s3);
    }
    by_gather_size((last + 1) * 16, l.n * qq * 16, [&](auto nt_loads, auto stores) {
        // (the markers keep the compiler from merging the branches' accesses into ordinary ones)
        asm volatile("; rows");
        const uint4 v0 = ld16<nt_loads.value>(&buffer[p0 * qq + c0]);
        const uint4 v1 = ld16<nt_loads.value>(&buffer[p1 * qq + c1]);
        const uint4 v2 = ld16<nt_loads.value>(&buffer[p2 * qq + c2]);
        const uint4 v3 = ld16<nt_loads.value>(&buffer[p3 * qq + c3]);
        if (s0 >= 0) st_gathered<stores.value>(out, x0, v0);
        if (s1 >= 0) st_gathered<stores.value>(out, x1, v1);
        if (s2 >= 0) st_gathered<stores.value>(out, x2, v2);
        if (s3 >= 0) st_gathered<stores.value>(out, x3, v3);
        asm volatile("; end of rows");
    });
}

// out[miss_pos[r]] = features[ids[miss_pos[r]]] for every miss r; the loads cross
// the host link when the backing store is page-locked host memory.  The link
// needs little data in flight compared with HBM, and waves blocked on it would
// otherwise hold the wave slots the concurrent hit gather needs, so this kernel
// runs as a small fixed grid that strides over the miss list.
//
// Write-through variant (WT): the same loaded chunk is also stored into the cache
// buffer slot the row will get from the FIFO update that follows, so that update
// needs no row copy: miss r goes to slot (tail + r) mod capacity, ranks that a
// later miss of the same batch would overwrite are skipped.
template <int Q, bool WT>
__global__ __launch_bounds__(COPY_THREADS) void k_fetch_miss(
    const int32_t *__restrict__ miss_pos, const int32_t *__restrict__ ids, int q,
    int64_t num_nodes, const uint4 *__restrict__ features, uint4 *__restrict__ out,
    const CacheDev *dev, uint4 *__restrict__ buffer, int64_t capacity, int64_t rows, int par, int gen)
{
    static_assert(COPY_UNROLL == 4, "the four chunks of a lane are written out by hand");
    const int qq = Q > 0 ? Q : q;
    const int64_t n_miss = dev->n_miss_gen[gen];
    const int64_t total = n_miss * qq;
    const int64_t last = total - 1;
    // (the ranks that stay cover less than one turn of the buffer: the wrap-around is one subtraction)
    const RowRing ring(WT ? dev->tail[par] : 0ull, capacity, rows, n_miss);
    const int64_t start = ring.start;
    const int64_t step = (int64_t)gridDim.x * (COPY_THREADS * COPY_UNROLL);
    for (int64_t base = (int64_t)blockIdx.x * (COPY_THREADS * COPY_UNROLL) + threadIdx.x;
         base - threadIdx.x < total; base += step) {
        // Phase by phase for the lane's four chunks, as in k_gather_hits: positions, ids, rows, stores;
        // chunk numbers beyond the end are clamped to the last chunk, which is then copied again.
        int64_t r0, r1, r2, r3;
        int c0, c1, c2, c3;
        RowSplit<Q>::split(min(base, last), q, r0, c0);
        RowSplit<Q>::split(min(base + COPY_THREADS, last), q, r1, c1);
        RowSplit<Q>::split(min(base + 2 * COPY_THREADS, last), q, r2, c2);
        RowSplit<Q>::split(min(base + 3 * COPY_THREADS, last), q, r3, c3);
        const int32_t m0 = miss_pos[r0], m1 = miss_pos[r1], m2 = miss_pos[r2], m3 = miss_pos[r3];
        const int32_t i0 = ids[m0], i1 = ids[m1], i2 = ids[m2], i3 = ids[m3];
        // an id outside the table (reported by the lookup) reads row 0 and stores nothing
        const bool ok0 = i0 >= 0 && (int64_t)i0 < num_nodes, ok1 = i1 >= 0 && (int64_t)i1 < num_nodes;
        const bool ok2 = i2 >= 0 && (int64_t)i2 < num_nodes, ok3 = i3 >= 0 && (int64_t)i3 < num_nodes;
        uint4 v0 = features[(int64_t)(ok0 ? i0 : 0) * qq + c0];
        uint4 v1 = features[(int64_t)(ok1 ? i1 : 0) * qq + c1];
        uint4 v2 = features[(int64_t)(ok2 ? i2 : 0) * qq + c2];
        uint4 v3 = features[(int64_t)(ok3 ? i3 : 0) * qq + c3];
        // (the four reads stay above the branches that follow: the values are needed here)
        asm volatile("" : "+v"(v0.x), "+v"(v0.y), "+v"(v0.z), "+v"(v0.w), "+v"(v1.x), "+v"(v1.y), "+v"(v1.z), "+v"(v1.w),
                          "+v"(v2.x), "+v"(v2.y), "+v"(v2.z), "+v"(v2.w), "+v"(v3.x), "+v"(v3.y), "+v"(v3.z), "+v"(v3.w));
        auto store = [&](bool ok, int64_t r, int32_t m, int c, const uint4 &v) {
            if (!ok) return;
            out[(int64_t)m * qq + c] = v;
            if (WT && r >= start) buffer[ring.pos_of_rank(r) * qq + c] = v;
        };
        store(ok0, r0, m0, c0, v0);
        store(ok1, r1, m1, c1, v1);
        store(ok2, r2, m2, c2, v2);
        store(ok3, r3, m3, c3, v3);
    }
}

// The same over the host link.  The link moves whole 128-byte lines and a wavefront asks for each line
// it touches, so a row must not be dealt to two wavefronts: 64 consecutive 16-byte chunks of a list of
// 400-byte rows begin and end inside a row, and the two lines there cross the link twice (+ 9 %).  Here
// the lanes of a wavefront take whole rows, 64 / q of them at a time (rows of up to 64 chunks), four
// such groups in flight, and the next rows' ids are read while these are on the link.  Measured on
// 319 K misses of 400 bytes in page-locked memory: 3,077 us dealt chunk by chunk, 2,982 now (55 GB/s of
// whole lines; 96 or 128 workgroups: the same); the lanes that stay idle (14 of 64 with 400-byte rows)
// cost nothing, the link is the bound.  The chunk's place in its row needs no division in the loop.
template <bool WT>
__global__ __launch_bounds__(COPY_THREADS) void k_fetch_link(
    const int32_t *__restrict__ miss_pos, const int32_t *__restrict__ ids, int q,
    int64_t num_nodes, const uint4 *__restrict__ features, uint4 *__restrict__ out,
    const CacheDev *dev, uint4 *__restrict__ buffer, int64_t capacity, int64_t rows, int par, int gen)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t n_miss = dev->n_miss_gen[gen];
    const int group = kWave / q;                // rows side by side
    const int sub = lane / q, c = lane - sub * q;
    if (sub >= group) return;
    const RowRing ring(WT ? dev->tail[par] : 0ull, capacity, rows, n_miss);
    const int64_t step = (int64_t)gridDim.x * (COPY_THREADS / kWave) * COPY_UNROLL * group;
    const int64_t last = n_miss - 1;
    int64_t base = ((int64_t)blockIdx.x * (COPY_THREADS / kWave) + threadIdx.x / kWave) * COPY_UNROLL * group + sub;
    if (base - sub >= n_miss) return;
    // Phase by phase for the lane's four chunks, as in k_gather_hits; row numbers beyond the end are
    // clamped to the last row, which is then copied again.  The next rows' positions and ids are read
    // while this round's rows are on the link.
    int32_t m0 = miss_pos[min(base, last)], m1 = miss_pos[min(base + group, last)], m2 = miss_pos[min(base + 2 * group, last)],
            m3 = miss_pos[min(base + 3 * group, last)];
    int32_t i0 = ids[m0], i1 = ids[m1], i2 = ids[m2], i3 = ids[m3];
    for (;;) {
        // an id outside the table (reported by the lookup) reads row 0 and stores nothing
        const bool ok0 = i0 >= 0 && (int64_t)i0 < num_nodes, ok1 = i1 >= 0 && (int64_t)i1 < num_nodes;
        const bool ok2 = i2 >= 0 && (int64_t)i2 < num_nodes, ok3 = i3 >= 0 && (int64_t)i3 < num_nodes;
        uint4 v0 = features[(int64_t)(ok0 ? i0 : 0) * q + c];
        uint4 v1 = features[(int64_t)(ok1 ? i1 : 0) * q + c];
        uint4 v2 = features[(int64_t)(ok2 ? i2 : 0) * q + c];
        uint4 v3 = features[(int64_t)(ok3 ? i3 : 0) * q + c];
        const int64_t next = base + step;
        const int32_t p0 = miss_pos[min(next, last)], p1 = miss_pos[min(next + group, last)],
                      p2 = miss_pos[min(next + 2 * group, last)], p3 = miss_pos[min(next + 3 * group, last)];
        int32_t j0 = ids[p0], j1 = ids[p1], j2 = ids[p2], j3 = ids[p3];
        // (all these reads stay above the branches that follow: the values are needed here)
        asm volatile("" : "+v"(v0.x), "+v"(v0.y), "+v"(v0.z), "+v"(v0.w), "+v"(v1.x), "+v"(v1.y), "+v"(v1.z), "+v"(v1.w),
                          "+v"(v2.x), "+v"(v2.y), "+v"(v2.z), "+v"(v2.w), "+v"(v3.x), "+v"(v3.y), "+v"(v3.z), "+v"(v3.w),
                          "+v"(j0), "+v"(j1), "+v"(j2), "+v"(j3));
        auto store = [&](bool ok, int64_t r, int32_t m, const uint4 &v) {
            if (!ok) return;
            out[(int64_t)m * q + c] = v;
            if (WT && r >= ring.start) buffer[ring.pos_of_rank(r) * q + c] = v;
        };
        store(ok0, min(base, last), m0, v0);
        store(ok1, min(base + group, last), m1, v1);
        store(ok2, min(base + 2 * group, last), m2, v2);
        store(ok3, min(base + 3 * group, last), m3, v3);
        base = next;
        if (base - sub >= n_miss) return;
        m0 = p0; m1 = p1; m2 = p2; m3 = p3;
        i0 = j0; i1 = j1; i2 = j2; i3 = j3;
    }
}

// k_fetch_link without a list, for rows that go to out alone: a wavefront takes `per` positions at a time (at most 64) and
// queues the misses among them in LDS, so that the fetch need not wait for the lists (4 us and a launch), and fetches them
// as many at a time as k_fetch_link does.  (Every 64 positions' misses by themselves, the last few with lanes to spare: 20,000 ids of
// 400 bytes, 90 % missed, 204.9 -> 209.9 us a call.)
__global__ __launch_bounds__(COPY_THREADS) void k_fetch_slots(
    const int32_t *__restrict__ own_slot, const int32_t *__restrict__ ids, int64_t n, int per, int q, int64_t num_nodes,
    const uint4 *__restrict__ features, uint4 *__restrict__ out)
{
    extern __shared__ int2 sh_queue[];          // (id, position); slots_queue(q) per wavefront
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int group = kWave / q, round = COPY_UNROLL * group;  // rows side by side, rows at a time
    const int sub = lane / q, c = lane - sub * q;
    int2 *const queue = sh_queue + w * slots_queue(q);
    const int64_t step = (int64_t)gridDim.x * (COPY_THREADS / kWave) * per;
    int64_t first = ((int64_t)blockIdx.x * (COPY_THREADS / kWave) + w) * per;
    auto mine = [&](int64_t at) { return lane < per && at + lane < n ? at + lane : -1; };
    int64_t i = mine(first);
    int32_t slot = i >= 0 ? own_slot[i] : 0, id = i >= 0 ? ids[i] : 0;
    int queued = 0;
    while (first < n) {
        // (an id outside the table has been reported by the lookup: nothing is fetched for it)
        const bool miss = slot < 0 && id >= 0 && (int64_t)id < num_nodes;
        const uint64_t mask = __ballot(miss);
        if (miss) queue[queued + __popcll(mask & ((1ull << lane) - 1ull))] = int2{id, (int)i};
        queued += __popcll(mask);
        first += step;
        i = mine(first);  // the next positions' slots are read while these rows are on the link
        slot = i >= 0 ? own_slot[i] : 0;
        id = i >= 0 ? ids[i] : 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        int r = 0;
        for (; queued - r >= round || (first >= n && r < queued); r += round) {
            const int r0 = r + sub, r1 = r0 + group, r2 = r1 + group, r3 = r2 + group;
            const bool ok0 = sub < group && r0 < queued, ok1 = sub < group && r1 < queued, ok2 = sub < group && r2 < queued,
                       ok3 = sub < group && r3 < queued;
            const int2 none = {0, 0};
            const int2 m0 = ok0 ? queue[r0] : none, m1 = ok1 ? queue[r1] : none, m2 = ok2 ? queue[r2] : none, m3 = ok3 ? queue[r3] : none;
            uint4 v0 = {0, 0, 0, 0}, v1 = v0, v2 = v0, v3 = v0;
            if (ok0) v0 = features[(int64_t)m0.x * q + c];
            if (ok1) v1 = features[(int64_t)m1.x * q + c];
            if (ok2) v2 = features[(int64_t)m2.x * q + c];
            if (ok3) v3 = features[(int64_t)m3.x * q + c];
            // (the four reads stay above the branches that follow: the values are needed here)
            asm volatile("" : "+v"(v0.x), "+v"(v0.y), "+v"(v0.z), "+v"(v0.w), "+v"(v1.x), "+v"(v1.y), "+v"(v1.z), "+v"(v1.w),
                              "+v"(v2.x), "+v"(v2.y), "+v"(v2.z), "+v"(v2.w), "+v"(v3.x), "+v"(v3.y), "+v"(v3.z), "+v"(v3.w));
            if (ok0) out[(int64_t)m0.y * q + c] = v0;
            if (ok1) out[(int64_t)m1.y * q + c] = v1;
            if (ok2) out[(int64_t)m2.y * q + c] = v2;
            if (ok3) out[(int64_t)m3.y * q + c] = v3;
        }
        // what is left, less than a round, moves to the front (r is 0, or at least a round: the two parts do not overlap)
        queued = max(queued - r, 0);
        if (r > 0)
            for (int k = lane; k < queued; k += kWave) queue[k] = queue[r + k];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Tiered lookup, rows that the host tier holds, read where they lie in its page-locked ring: the h-th
// listed rank's row, h < count, is ring row hit_ring[h].  Whole rows per wavefront, as in k_fetch_link; for rows of
// whole 128-byte lines, which cross the link in place as fast as packed.  The launch needs no host thread, so it is
// under way while the first of the other rows are being packed, and it fills the moments between their copies.
// Measured, 150,001 ids x 512 B of which 25,600 in the tier, copy engine 1,600 -> 1,390 us a call, kernels
// reading the packed rows 1,560 -> 1,374; 100,000 ids x 1,024 B 1,960 -> 1,720; 20,000 ids x 512 B 387 -> 320; 60,000 x 128 B
// 306 -> 280; 5,000 ids x 128 / 512 / 1,024 B 164 / 192 / 260 -> 159 / 163 / 213; 500 ids the same.
template <bool WT>
__global__ __launch_bounds__(COPY_THREADS) void k_fetch_ring(
    const int32_t *__restrict__ hit_rank, const int32_t *__restrict__ hit_ring, int64_t count, const int32_t *__restrict__ miss_pos,
    int q, const uint4 *__restrict__ ring_rows, uint4 *__restrict__ out, const CacheDev *dev, uint4 *__restrict__ buffer,
    int64_t capacity, int64_t rows, int par, int64_t n_miss)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int group = kWave / q;                // rows side by side
    const int sub = lane / q, c = lane - sub * q;
    if (sub >= group) return;
    const RowRing ring(WT ? dev->tail[par] : 0ull, capacity, rows, n_miss);
    const int64_t step = (int64_t)gridDim.x * (COPY_THREADS / kWave) * COPY_UNROLL * group;
    const int64_t last = count - 1;
    for (int64_t base = ((int64_t)blockIdx.x * (COPY_THREADS / kWave) + threadIdx.x / kWave) * COPY_UNROLL * group + sub;
         base - sub < count; base += step) {
        // Phase by phase for the lane's four chunks, as in k_gather_hits; numbers beyond the end are clamped
        // to the last row, which is then copied again.
        const int64_t h0 = min(base, last), h1 = min(base + group, last), h2 = min(base + 2 * group, last), h3 = min(base + 3 * group, last);
        const int32_t r0 = hit_rank[h0], r1 = hit_rank[h1], r2 = hit_rank[h2], r3 = hit_rank[h3];
        const int32_t p0 = hit_ring[h0], p1 = hit_ring[h1], p2 = hit_ring[h2], p3 = hit_ring[h3];
        const int32_t m0 = miss_pos[r0], m1 = miss_pos[r1], m2 = miss_pos[r2], m3 = miss_pos[r3];
        uint4 v0 = ring_rows[(int64_t)p0 * q + c];
        uint4 v1 = ring_rows[(int64_t)p1 * q + c];
        uint4 v2 = ring_rows[(int64_t)p2 * q + c];
        uint4 v3 = ring_rows[(int64_t)p3 * q + c];
        // (the four reads stay above the branches that follow: the values are needed here)
        asm volatile("" : "+v"(v0.x), "+v"(v0.y), "+v"(v0.z), "+v"(v0.w), "+v"(v1.x), "+v"(v1.y), "+v"(v1.z), "+v"(v1.w),
                          "+v"(v2.x), "+v"(v2.y), "+v"(v2.z), "+v"(v2.w), "+v"(v3.x), "+v"(v3.y), "+v"(v3.z), "+v"(v3.w));
        auto store = [&](int32_t r, int32_t m, const uint4 &v) {
            out[(int64_t)m * q + c] = v;
            if (WT && r >= ring.start) buffer[ring.pos_of_rank(r) * q + c] = v;
        };
        store(r0, m0, v0);
        store(r1, m1, v1);
        store(r2, m2, v2);
        store(r3, m3, v3);
    }
}

// Tiered lookup: out[miss_pos[r]] = rows[(first + l) mod ring] for listed misses
// l0 <= l < l0 + count of the GPU cache, r = rank[l] (r = l without a list: a tier
// that keeps nothing lists every miss).  rows are page-locked host rows that the
// host threads have just packed in list order: the host tier's ring (rows it
// brought in from the store) or its staging rows (rows it held), or the device
// memory the copy engine has moved those rows to (NT: these are read once, and
// what is written is for a later kernel, so neither should displace the lines
// the next hit gather works on; measured, that gather takes 24 instead of 28
// microseconds and this kernel 69 instead of 74).  Same launch shape and
// write-through rule as k_fetch_miss.
template <int Q, bool WT, bool NT>
__global__ __launch_bounds__(COPY_THREADS) void k_fetch_rows(
    const int32_t *__restrict__ rank, int64_t l0, int64_t count, unsigned long long first, int64_t ring,
    const int32_t *__restrict__ miss_pos, int q, const uint4 *__restrict__ rows, uint4 *__restrict__ out,
    const CacheDev *dev, uint4 *__restrict__ buffer, int64_t capacity, int64_t buffer_rows, int par, int64_t n_miss)
{
    static_assert(COPY_UNROLL == 4, "the four chunks of a lane are written out by hand");
    const int qq = Q > 0 ? Q : q;
    const int64_t total = count * qq;
    const int64_t last = total - 1;
    // the two wrap-arounds without a division per chunk: the launch covers less than one turn of
    // the ring, and the ranks it stores (start <= r < n_miss) less than one turn of the buffer
    const int64_t first_pos = (int64_t)((first + (unsigned long long)l0) % (unsigned long long)ring) - l0;
    const RowRing dst(WT ? dev->tail[par] : 0ull, capacity, buffer_rows, n_miss);
    const int64_t start = dst.start;
    const int64_t step = (int64_t)gridDim.x * (COPY_THREADS * COPY_UNROLL);
    for (int64_t base = (int64_t)blockIdx.x * (COPY_THREADS * COPY_UNROLL) + threadIdx.x;
         base - threadIdx.x < total; base += step) {
        // Phase by phase for the lane's four chunks, as in k_gather_hits: ranks, positions, rows,
        // stores; chunk numbers beyond the end are clamped to the last chunk, which is then copied again.
        int64_t l_0, l_1, l_2, l_3;
        int c0, c1, c2, c3;
        RowSplit<Q>::split(min(base, last), q, l_0, c0);
        RowSplit<Q>::split(min(base + COPY_THREADS, last), q, l_1, c1);
        RowSplit<Q>::split(min(base + 2 * COPY_THREADS, last), q, l_2, c2);
        RowSplit<Q>::split(min(base + 3 * COPY_THREADS, last), q, l_3, c3);
        l_0 += l0; l_1 += l0; l_2 += l0; l_3 += l0;
        int64_t r0 = l_0, r1 = l_1, r2 = l_2, r3 = l_3;
        if (rank) { r0 = rank[l_0]; r1 = rank[l_1]; r2 = rank[l_2]; r3 = rank[l_3]; }
        const int32_t m0 = miss_pos[r0], m1 = miss_pos[r1], m2 = miss_pos[r2], m3 = miss_pos[r3];
        auto wrapped = [](int64_t x, int64_t turn) { return x >= turn ? x - turn : x; };
        uint4 v0 = ld16<NT>(&rows[wrapped(first_pos + l_0, ring) * qq + c0]);
        uint4 v1 = ld16<NT>(&rows[wrapped(first_pos + l_1, ring) * qq + c1]);
        uint4 v2 = ld16<NT>(&rows[wrapped(first_pos + l_2, ring) * qq + c2]);
        uint4 v3 = ld16<NT>(&rows[wrapped(first_pos + l_3, ring) * qq + c3]);
        st16<NT>(&out[(int64_t)m0 * qq + c0], v0);
        st16<NT>(&out[(int64_t)m1 * qq + c1], v1);
        st16<NT>(&out[(int64_t)m2 * qq + c2], v2);
        st16<NT>(&out[(int64_t)m3 * qq + c3], v3);
        if (WT) {
            if (start == 0) {  // every rank gets a slot (the usual case: fewer misses than slots)
                st16<NT>(&buffer[dst.pos_of_rank(r0) * qq + c0], v0);
                st16<NT>(&buffer[dst.pos_of_rank(r1) * qq + c1], v1);
                st16<NT>(&buffer[dst.pos_of_rank(r2) * qq + c2], v2);
                st16<NT>(&buffer[dst.pos_of_rank(r3) * qq + c3], v3);
            } else {
                if (r0 >= start) st16<NT>(&buffer[dst.pos_of_rank(r0) * qq + c0], v0);
                if (r1 >= start) st16<NT>(&buffer[dst.pos_of_rank(r1) * qq + c1], v1);
                if (r2 >= start) st16<NT>(&buffer[dst.pos_of_rank(r2) * qq + c2], v2);
                if (r3 >= start) st16<NT>(&buffer[dst.pos_of_rank(r3) * qq + c3], v3);
            }
        }
    }
}

// ---- assembled output
// With the packed miss rows of a call already in device memory (the copy engine
// has landed them, in miss order), one pass over the output in its own order can
// write every row: a hit's row comes from the cache buffer, a miss's row from the
// landed rows, and the miss rows also go to the buffer slots the FIFO rule gives
// them (write-through).  Every output line is then written whole by one stream of
// stores, and the hit gather and the scatter of the landed rows are one launch
// large enough to fill the memory system.  One hazard: a hit whose row lies
// where this call's own misses are written must be read before it is
// overwritten.  Those rows (few when a batch's misses are few against the
// capacity, all of the hits when they outnumber it) are copied by
// k_assemble_pre, which runs first; k_assemble_rows leaves them alone.
// With enough spare row positions in the buffer (RowRing) no live row lies where this call
// writes, and the first pass is not launched at all.
// The hits inside the window, copied before the window is written.  Each wavefront scans 64
// positions (one per lane), packs the ones concerned into LDS with a ballot and copies their rows
// with all its lanes, four 16-byte chunks in flight per lane.
template <int Q>
__global__ __launch_bounds__(COPY_THREADS) void k_assemble_pre(
    const int32_t *__restrict__ src_of, int64_t n, int q, const uint4 *__restrict__ buffer,
    uint4 *__restrict__ out, const CacheDev *dev, int64_t capacity, int64_t rows, int par, int64_t n_miss)
{
    constexpr int WAVES = COPY_THREADS / kWave;
    __shared__ int32_t sh_pos[WAVES][kWave];
    __shared__ int32_t sh_slot[WAVES][kWave];
    const int qq = Q > 0 ? Q : q;
    const RowRing ring(dev->tail[par], capacity, rows, n_miss);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t step = (int64_t)gridDim.x * COPY_THREADS;
    for (int64_t base = (int64_t)blockIdx.x * COPY_THREADS + wave * kWave; base < n; base += step) {
        const int64_t i = base + lane;
        const int32_t s = i < n ? src_of[i] : -1;
        const bool mine = s >= 0 && ring.overwritten(s);
        const uint64_t mask = __ballot(mine);
        if (mask == 0) continue;  // (uniform in the wavefront)
        const int m = __popcll(mask);
        if (mine) {
            const int at = __popcll(mask & ((1ull << lane) - 1ull));
            sh_pos[wave][at] = (int32_t)i;
            sh_slot[wave][at] = s;
        }
        // (the lists are written and read by this wavefront only)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int total = m * qq;
        for (int k0 = 0; k0 < total; k0 += 4 * kWave) {
            const int last = total - 1;
            const int k[4] = {min(k0 + lane, last), min(k0 + kWave + lane, last), min(k0 + 2 * kWave + lane, last),
                              min(k0 + 3 * kWave + lane, last)};
            int j[4], cc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (Q > 0) { j[u] = k[u] / Q; cc[u] = k[u] - j[u] * Q; }
                else { j[u] = k[u] / q; cc[u] = k[u] - j[u] * q; }
            }
            const uint4 v0 = buffer[(int64_t)sh_slot[wave][j[0]] * qq + cc[0]];
            const uint4 v1 = buffer[(int64_t)sh_slot[wave][j[1]] * qq + cc[1]];
            const uint4 v2 = buffer[(int64_t)sh_slot[wave][j[2]] * qq + cc[2]];
            const uint4 v3 = buffer[(int64_t)sh_slot[wave][j[3]] * qq + cc[3]];
            out[(int64_t)sh_pos[wave][j[0]] * qq + cc[0]] = v0;
            out[(int64_t)sh_pos[wave][j[1]] * qq + cc[1]] = v1;
            out[(int64_t)sh_pos[wave][j[2]] * qq + cc[2]] = v2;
            out[(int64_t)sh_pos[wave][j[3]] * qq + cc[3]] = v3;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Every other row, in output order: chunk number -> (position, chunk in row); the position's
// source decides where the chunk is read.  Phases as in k_gather_hits: the four sources of a lane,
// then its four chunks, then the stores; chunk numbers beyond the end are clamped to the last
// chunk, which is then copied again.  A chunk of a hit inside the window is read (from a slot that
// may be changing: the value is not used) and not stored.
template <int Q, bool NTO>
__global__ __launch_bounds__(COPY_THREADS) void k_assemble_rows(
    const int32_t *__restrict__ src_of, int64_t n, int q, const uint4 *__restrict__ landed,
    uint4 *buffer, uint4 *__restrict__ out, const CacheDev *dev, int64_t capacity, int64_t rows, int par,
    int64_t n_miss)
{
    static_assert(COPY_UNROLL == 4, "the four chunks of a lane are written out by hand");
    const int qq = Q > 0 ? Q : q;
    const int64_t total = n * qq;
    const int64_t last = total - 1;
    const RowRing ring(dev->tail[par], capacity, rows, n_miss);
    const int64_t step = (int64_t)gridDim.x * (COPY_THREADS * COPY_UNROLL);
    for (int64_t base = (int64_t)blockIdx.x * (COPY_THREADS * COPY_UNROLL) + threadIdx.x;
         base - threadIdx.x < total; base += step) {
        const int64_t x0 = min(base, last), x1 = min(base + COPY_THREADS, last),
                      x2 = min(base + 2 * COPY_THREADS, last), x3 = min(base + 3 * COPY_THREADS, last);
        int64_t i0, i1, i2, i3;
        int c0, c1, c2, c3;
        RowSplit<Q>::split(x0, q, i0, c0);
        RowSplit<Q>::split(x1, q, i1, c1);
        RowSplit<Q>::split(x2, q, i2, c2);
        RowSplit<Q>::split(x3, q, i3, c3);
        const int32_t s0 = src_of[i0], s1 = src_of[i1], s2 = src_of[i2], s3 = src_of[i3];
        auto source = [&](int32_t s, int c) -> const uint4 * {
            return s >= 0 ? buffer + (int64_t)s * qq + c : landed + (int64_t)(-s - 1) * qq + c;
        };
        uint4 v0 = *source(s0, c0);
        uint4 v1 = *source(s1, c1);
        uint4 v2 = *source(s2, c2);
        uint4 v3 = *source(s3, c3);
        // (the four reads stay above the branches that follow: the values are needed here)
        asm volatile("" : "+v"(v0.x), "+v"(v0.y), "+v"(v0.z), "+v"(v0.w), "+v"(v1.x), "+v"(v1.y), "+v"(v1.z), "+v"(v1.w),
                          "+v"(v2.x), "+v"(v2.y), "+v"(v2.z), "+v"(v2.w), "+v"(v3.x), "+v"(v3.y), "+v"(v3.z), "+v"(v3.w));
        auto store = [&](int32_t s, int c, int64_t x, const uint4 &v) {
            if (s >= 0) {
                if (!ring.overwritten(s)) st16<NTO>(&out[x], v);
            } else {
                st16<NTO>(&out[x], v);
                const int64_t r = -(int64_t)s - 1;
                if (r >= ring.start) st16<true>(&buffer[ring.pos_of_rank(r) * qq + c], v);
            }
        };
        store(s0, c0, x0, v0);
        store(s1, c1, x1, v1);
        store(s2, c2, x2, v2);
        store(s3, c3, x3, v3);
    }
}

// Map update, one inserted row per lane.  Evict the slot's occupant (blank its word, found through
// slot_to_entry, and take one off the pushed-past count of every bucket from the evicted id's home
// bucket up to the word's bucket), then read the new id's bucket whole (as k_probe does), and claim a
// free word with a CAS; a bucket without a free word gets one added to its count before the lane moves
// on.  Counts change by atomic adds only and no lookup runs beside an update, so after the launch every
// count is exact whatever the order of the lanes.  The bucket may be read from a cache that does not
// see other lanes' changes: a word that looks free is decided by the CAS, and one that looks taken and
// is being blanked is passed over.  The update is bound by dependent random accesses, so what counts is
// how many rows are in flight and how often a CAS is lost: a batch brings several ids per bucket (4.8 at
// 315 K misses, 65,536 buckets), so every lane starts at a word of its own choice.  Measured, against
// 16 lanes per row, four rows per wavefront, all starting at the first free word: 315 K rows 49 -> 34 us,
// 100 K rows 22 -> 19, 4 K rows (an overlapped loop's small batches) 10.6 -> 6.7.
__device__ __forceinline__ void insert_map_part(
    int64_t r, const int32_t *__restrict__ ids, const int32_t *__restrict__ miss_pos,
    int64_t start, unsigned long long tail, int64_t capacity, int64_t num_nodes,
    uint64_t *table, uint32_t bucket_mask, int32_t *slot_to_node, uint32_t *slot_to_entry,
    CacheDev *dev)
{
    // (the ranks from start on cover at most one turn of the slots)
    int64_t slot = (int64_t)((tail + (unsigned long long)start) % (unsigned long long)capacity) + (r - start);
    if (slot >= capacity) slot -= capacity;
    const int32_t key = ids[miss_pos[r]];
    const int32_t old = slot_to_node[slot];
    const bool ok = key >= 0 && (int64_t)key < num_nodes;
    uint32_t b = hash32((uint32_t)key) & bucket_mask;
    if (old >= 0) {
        const uint32_t word = slot_to_entry[slot];
        __hip_atomic_store(&table[word], EMPTY64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // the buckets this entry had been pushed past (none for an entry in its home bucket)
        const uint32_t rest = word / BUCKET;
        for (uint32_t p = hash32((uint32_t)old) & bucket_mask; p != rest; p = (p + 1) & bucket_mask)
            atomicAdd((unsigned long long *)&table[(size_t)p * BUCKET + (BUCKET - 1)], ~0ull);  // -1
    }
    if (!ok) {
        // reported by the lookup already: the slot's row will be overwritten, so
        // leave the slot unmapped rather than mapped to the wrong bytes
        slot_to_node[slot] = -1;
        dev->status = BGL_EINVAL;
        return;
    }
    const uint64_t mine = ((uint64_t)(uint32_t)key << 32) | (uint32_t)slot;
    const uint32_t first = (hash32((uint32_t)key) >> 27) % (BUCKET - 1);  // (bucket numbers use the low bits)
    // a table at load <= 1/2 always has a bucket with a free word
    for (uint32_t tries = 0; tries <= bucket_mask; ++tries) {
        const ulonglong2 *bp = reinterpret_cast<const ulonglong2 *>(table + (size_t)b * BUCKET);
        uint32_t free_words = 0;
#pragma unroll
        for (int k = 0; k < BUCKET / 2; ++k) {
            const ulonglong2 w = bp[k];
            free_words |= (w.x == EMPTY64 ? 1u : 0u) << (2 * k);
            if (k < BUCKET / 2 - 1) free_words |= (w.y == EMPTY64 ? 1u : 0u) << (2 * k + 1);
        }
        while (free_words) {
            const uint32_t after = free_words >> first << first;
            const uint32_t t = (uint32_t)__ffs(after ? after : free_words) - 1u;
            const unsigned long long prev =
                atomicCAS((unsigned long long *)&table[(size_t)b * BUCKET + t], EMPTY64, (unsigned long long)mine);
            if (prev == EMPTY64) {
                slot_to_node[slot] = key;
                slot_to_entry[slot] = b * BUCKET + t;
                return;
            }
            free_words &= ~(1u << t);  // another lane has it now
        }
        // full: this entry will rest beyond bucket b (its eviction takes the one off again)
        atomicAdd((unsigned long long *)&table[(size_t)b * BUCKET + (BUCKET - 1)], 1ull);
        b = (b + 1) & bucket_mask;
    }
    dev->status = BGL_ECAPACITY;
}

// buffer[(tail + r) % capacity] = out[miss_pos[r]]: the destination is a
// contiguous (wrapping) run of slots, so the stores stream.
template <int Q>
__device__ __forceinline__ void insert_rows_part(
    int64_t block, const int32_t *__restrict__ miss_pos, int64_t n_miss, int64_t start,
    unsigned long long tail, int64_t capacity, int64_t rows, int q, const uint4 *__restrict__ out,
    uint4 *__restrict__ buffer)
{
    static_assert(COPY_UNROLL == 4, "the four chunks of a lane are written out by hand");
    const int qq = Q > 0 ? Q : q;
    const int64_t total = (n_miss - start) * qq;
    const int64_t base = block * (COPY_THREADS * COPY_UNROLL) + threadIdx.x;
    if (base - threadIdx.x >= total) return;
    // Phase by phase for the lane's four chunks, as in k_gather_hits: positions, rows, stores; chunk
    // numbers beyond the end are clamped to the last chunk, which is then copied again.
    const int64_t last = total - 1;
    // (start <= r < n_miss covers at most one turn of the buffer: the wrap-around is one subtraction)
    const RowRing ring(tail, capacity, rows, n_miss);
    int64_t r0, r1, r2, r3;
    int c0, c1, c2, c3;
    RowSplit<Q>::split(min(base, last), q, r0, c0);
    RowSplit<Q>::split(min(base + COPY_THREADS, last), q, r1, c1);
    RowSplit<Q>::split(min(base + 2 * COPY_THREADS, last), q, r2, c2);
    RowSplit<Q>::split(min(base + 3 * COPY_THREADS, last), q, r3, c3);
    const int32_t m0 = miss_pos[start + r0], m1 = miss_pos[start + r1], m2 = miss_pos[start + r2],
                  m3 = miss_pos[start + r3];
    const uint4 v0 = out[(int64_t)m0 * qq + c0];
    const uint4 v1 = out[(int64_t)m1 * qq + c1];
    const uint4 v2 = out[(int64_t)m2 * qq + c2];
    const uint4 v3 = out[(int64_t)m3 * qq + c3];
    buffer[ring.pos_of_rank(start + r0) * qq + c0] = v0;
    buffer[ring.pos_of_rank(start + r1) * qq + c1] = v1;
    buffer[ring.pos_of_rank(start + r2) * qq + c2] = v2;
    buffer[ring.pos_of_rank(start + r3) * qq + c3] = v3;
}

// The FIFO update is two launches because only the row copy needs the fetched
// rows: the map update is enqueued ahead of the wait for the miss fetch and runs
// while the host link is still busy.  Both read tail[par]; the row copy stores the
// advanced value in tail[par ^ 1] for the next update.
__global__ __launch_bounds__(MAP_THREADS) void k_insert_map(
    const int32_t *__restrict__ ids, const int32_t *__restrict__ miss_pos, int64_t n_miss_arg,
    int64_t capacity, int64_t num_nodes, uint64_t *table, uint32_t bucket_mask,
    int32_t *slot_to_node, uint32_t *slot_to_entry, CacheDev *dev, int par, int advance)
{
    const int64_t n_miss = n_miss_arg >= 0 ? n_miss_arg : dev->n_miss_last;
    const int64_t start = n_miss > capacity ? n_miss - capacity : 0;  // earlier ranks would be overwritten
    const unsigned long long tail = dev->tail[par];
    // write-through mode has no row-copy launch: then this one advances tail
    if (advance && blockIdx.x == 0 && threadIdx.x == 0) dev->tail[par ^ 1] = tail + (unsigned long long)n_miss;
    const int64_t r = start + (int64_t)blockIdx.x * MAP_THREADS + threadIdx.x;
    if (r < n_miss)
        insert_map_part(r, ids, miss_pos, start, uniform(tail), capacity, num_nodes, table, bucket_mask, slot_to_node,
                        slot_to_entry, dev);
}

template <int Q>
__global__ __launch_bounds__(COPY_THREADS) void k_insert_rows(
    const int32_t *__restrict__ miss_pos, int64_t n_miss_arg, int64_t capacity, int64_t rows, int q,
    const uint4 *__restrict__ out, uint4 *__restrict__ buffer, CacheDev *dev, int par)
{
    const int64_t n_miss = n_miss_arg >= 0 ? n_miss_arg : dev->n_miss_last;
    const int64_t start = n_miss > capacity ? n_miss - capacity : 0;
    const unsigned long long tail = dev->tail[par];
    if (blockIdx.x == 0 && threadIdx.x == 0) dev->tail[par ^ 1] = tail + (unsigned long long)n_miss;
    insert_rows_part<Q>(blockIdx.x, miss_pos, n_miss, start, tail, capacity, rows, q, out, buffer);
}

// Both in one launch, for caches that can hold every node: once such a cache is warm its updates find little or nothing to
// do, and a map update ahead of the wait for the fetch hides nothing.  Lookup + update of 302,709 hits of 1,024 bytes 138.2 -> 136.5 us,
// each waited for 168 -> 166; a first lookup, all missed, 5,000 x 400 B 109 -> 107, 300,000 the same.
template <int Q>
__global__ __launch_bounds__(COPY_THREADS) void k_insert_both(
    const int32_t *__restrict__ ids, const int32_t *__restrict__ miss_pos, int64_t n_miss_arg, int map_blocks, int64_t capacity,
    int64_t rows, int64_t num_nodes, uint64_t *table, uint32_t bucket_mask, int32_t *slot_to_node, uint32_t *slot_to_entry, int q,
    const uint4 *__restrict__ out, uint4 *__restrict__ buffer, CacheDev *dev, int par)
{
    const int64_t n_miss = n_miss_arg >= 0 ? n_miss_arg : dev->n_miss_last;
    const int64_t start = n_miss > capacity ? n_miss - capacity : 0;
    const unsigned long long tail = dev->tail[par];
    if (blockIdx.x == 0 && threadIdx.x == 0) dev->tail[par ^ 1] = tail + (unsigned long long)n_miss;
    if ((int)blockIdx.x >= map_blocks) {
        insert_rows_part<Q>(blockIdx.x - map_blocks, miss_pos, n_miss, start, tail, capacity, rows, q, out, buffer);
        return;
    }
    const int64_t r = start + (int64_t)blockIdx.x * MAP_THREADS + threadIdx.x;  // (as many rows a workgroup as k_insert_map)
    if (threadIdx.x < MAP_THREADS && r < n_miss)
        insert_map_part(r, ids, miss_pos, start, uniform(tail), capacity, num_nodes, table, bucket_mask, slot_to_node, slot_to_entry, dev);
}

// FIFO update when the launches above are skipped (nothing can be inserted).
__global__ void k_advance_tail(CacheDev *dev, int64_t n_miss_arg, int par)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        const long long n = n_miss_arg >= 0 ? n_miss_arg : dev->n_miss_last;
        dev->tail[par ^ 1] = dev->tail[par] + (unsigned long long)n;
    }
}

__global__ void k_noop() {}

// Census of the pushed-past counts for bgl_cache_map_stats: how many buckets a
// lookup would walk past, and how many (entry, bucket) pairs that is.
__global__ void k_map_census(const uint64_t *__restrict__ table, uint32_t num_buckets, CacheDev *dev)
{
    unsigned long long nz = 0, sum = 0;
    for (uint32_t b = blockIdx.x * blockDim.x + threadIdx.x; b < num_buckets; b += gridDim.x * blockDim.x) {
        const uint64_t cnt = table[(size_t)b * BUCKET + (BUCKET - 1)];
        nz += cnt != 0;
        sum += cnt;
    }
    if (nz) atomicAdd(&dev->census[0], nz);
    if (sum) atomicAdd(&dev->census[1], sum);
}

// ------------------------------------------------------------------ host helpers
// Stage timers.  A stage that is one kernel is timed by the dispatch itself: the
// pair of events goes into the launch (launch() below) and records the kernel's
// own begin and end on the device.  A stage of several launches (exact = false)
// is bracketed by two event records on the stream, which also times the launch
// gaps around it.
// Is a stage timed in this lookup or update?  `call` counts the lookups or the updates, from 1.
bool timed(const bgl_cache *c, int stage, uint64_t call)
{
    return (c->profiling & (1u << stage)) && (c->prof_every[stage] <= 1 || call % (uint64_t)c->prof_every[stage] == 0);
}
struct Prof {
    bgl_cache *c;
    hipStream_t st;
    int ev = -1;
    bool exact;
    Prof(bgl_cache *c_, int stage, hipStream_t st_, bool exact_ = true) : c(c_), st(st_), exact(exact_)
    {
        const bool of_update = stage == BGL_STAGE_INSERT_MAP || stage == BGL_STAGE_INSERT_ROWS;
        if (!timed(c, stage, of_update ? c->insert_calls + 1 : c->lookup_calls)) return;
        if (2 * (c->prof_rec.size() + 1) > c->prof_ev.size()) {  // more timed launches than events: add some
            const size_t old = c->prof_ev.size();
            c->prof_ev.resize(old + 2 * PROF_RING, nullptr);
            for (size_t k = old; k < c->prof_ev.size(); ++k)
                if (hipEventCreate(&c->prof_ev[k]) != hipSuccess) {
                    for (size_t j = old; j < k; ++j) (void)hipEventDestroy(c->prof_ev[j]);
                    c->prof_ev.resize(old);
                    c->prof_dropped += 1;
                    return;
                }
        }
        ev = (int)c->prof_rec.size() * 2;
        c->prof_rec.push_back({stage, ev});
        if (exact) {
            c->timed_start = c->prof_ev[ev];
            c->timed_stop = c->prof_ev[ev + 1];
        } else {
            (void)hipEventRecord(c->prof_ev[ev], st);
        }
    }
    ~Prof()
    {
        if (ev < 0) return;
        if (exact) c->timed_start = c->timed_stop = nullptr;  // (already taken by the launch)
        else (void)hipEventRecord(c->prof_ev[ev + 1], st);
    }
};

struct Grid {
    dim3 grid;
    size_t lds;  // dynamic
    Grid(dim3 grid_, size_t lds_ = 0) : grid(grid_), lds(lds_) {}
};

// Kernel launch; inside a Prof scope of a one-kernel stage the dispatch records its
// own begin and end into that scope's events.
template <typename... P, typename... A>
void launch(bgl_cache *c, hipStream_t st, void (*kernel)(P...), const Grid &grid, dim3 block, A &&...a)
{
    if (c->timed_start) {
        hipEvent_t e0 = c->timed_start, e1 = c->timed_stop;
        c->timed_start = c->timed_stop = nullptr;
        hipExtLaunchKernelGGL(kernel, grid.grid, block, grid.lds, st, e0, e1, 0, static_cast<P>(a)...);
    } else {
        hipLaunchKernelGGL(kernel, grid.grid, block, grid.lds, st, static_cast<P>(a)...);
    }
}

// The same, and `mark` says when the kernel is over: with `own` as the launch's own completion event, else (and
// where the launch is captured or timed) as a command behind it.  Its own event reaches a stream that waits for it
// 2 us earlier (a 5 us kernel, a hand-over, a 5 us kernel, a hand-over back, a 5 us kernel: 43 instead of 47 us).
// But a host that waits for a stream whose last event is a kernel's own enqueues another command first, and waits 4 to
// 15 us longer.  So an event is recorded behind as well where the launch is the last of its stream (BESIDE_BYTES), and where the
// updates have a stream of their own no launch marks its end itself unless the calls stream (bgl_cache::streaming): lookup
// + update on another stream, each waited for / one after the other, none own | all own: 500 ids x 400 B, half hits, 71 / 70 |
// 85 / 66 us; 2,000 ids, all hits, 70 / 68 | 85 / 66; 20,000 ids x 1,024 B, half hits, 257 / 234 | 265 / 232.  The overlapped loop, us
// a batch of 512 seeds, fanout 10,5: 10,000 nodes x 400 B 82.0 | 79.7, x 64 B 72.5 | 67.1; 100 seeds, fanout 8,4, 90,000 nodes 74.8 | 69.0.
// (The same loop written in Python over the public calls, which nothing tells apart from calls that are waited for, keeps the first of the
// two: 512 seeds, 10,000 nodes x 400 B 99 | 92.)
template <typename... P, typename... A>
int launch_marked(bgl_cache *c, hipStream_t st, hipEvent_t mark, bool own, void (*kernel)(P...), const Grid &grid, dim3 block, A &&...a)
{
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (own && hipStreamIsCapturing(st, &capture) != hipSuccess) {
        (void)hipGetLastError();
        own = false;
    }
    if (!own || c->timed_start || capture != hipStreamCaptureStatusNone) {
        launch(c, st, kernel, grid, block, std::forward<A>(a)...);
        BGL_HIP(hipEventRecord(mark, st));
    } else {
        hipExtLaunchKernelGGL(kernel, grid.grid, block, grid.lds, st, nullptr, mark, 0, static_cast<P>(a)...);
    }
    return BGL_OK;
}

void drain_profile(bgl_cache *c)
{
    for (auto &r : c->prof_rec) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->prof_ev[r.ev], c->prof_ev[r.ev + 1]) == hipSuccess) {
            c->prof_ms[r.stage] += ms;
            c->prof_n[r.stage] += 1;
        }
    }
    c->prof_rec.clear();
}

template <typename F>
void dispatch_q(int q, F &&f)
{
    switch (q) {
    case 25: f(std::integral_constant<int, 25>{}); break;  // 100 x fp32
    case 32: f(std::integral_constant<int, 32>{}); break;  // 128 x fp32
    case 64: f(std::integral_constant<int, 64>{}); break;  // 512 x bf16
    default: f(std::integral_constant<int, 0>{}); break;
    }
}

int copy_blocks(int64_t rows, int q)
{
    return (int)bgl::ceil_div(rows * q, (int64_t)COPY_THREADS * COPY_UNROLL);
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" int bgl_cache_create(int64_t capacity_rows, int32_t row_bytes,
                                const void *host_features, int64_t num_nodes, bgl_cache_t **out)
try {
    if (!out) BGL_FAIL(BGL_EINVAL, "out is null");
    *out = nullptr;
    if (capacity_rows < 1 || capacity_rows > INT32_MAX)
        BGL_FAIL(BGL_EINVAL, "capacity_rows must be in [1, 2^31) (got %lld)", (long long)capacity_rows);
    if (row_bytes < 16 || row_bytes % 16 != 0)
        BGL_FAIL(BGL_EINVAL, "row_bytes must be a positive multiple of 16 (got %d)", row_bytes);
    if (num_nodes < 1 || num_nodes > INT32_MAX) BGL_FAIL(BGL_EINVAL, "num_nodes out of range");
    if (!bgl::aligned(host_features, 16)) BGL_FAIL(BGL_EINVAL, "host_features is not 16-byte aligned");

    hipPointerAttribute_t attr;
    attr.type = hipMemoryTypeHost;
    const char *feat_dev = nullptr;
    if (host_features) {  // null: misses are served through a host tier only
        if (hipPointerGetAttributes(&attr, host_features) != hipSuccess) {
            (void)hipGetLastError();
            BGL_FAIL(BGL_EINVAL, "host_features is neither page-locked host memory nor device memory");
        }
        if (attr.type == hipMemoryTypeHost || attr.type == hipMemoryTypeDevice ||
            attr.type == hipMemoryTypeManaged) {
            feat_dev = static_cast<const char *>(attr.devicePointer);
        }
        if (!feat_dev)
            BGL_FAIL(BGL_EINVAL, "host_features is neither page-locked host memory nor device memory");
    }

    bgl_cache *c = new (std::nothrow) bgl_cache();
    if (!c) BGL_FAIL(BGL_ENOMEM, "out of host memory");
    c->capacity = capacity_rows;
    c->rows = capacity_rows;
    c->row_bytes = row_bytes;
    c->num_nodes = num_nodes;
    c->features = feat_dev;
    c->features_in_hbm = attr.type == hipMemoryTypeDevice;
    // load <= 1/2 of the 15 usable words per bucket
    uint64_t nbk = 1;
    while (nbk * 15 < (uint64_t)capacity_rows * 2) nbk <<= 1;
    c->num_buckets = (uint32_t)nbk;

    auto fail = [&](int code) { bgl_cache_destroy(c); return code; };
    hipError_t e;
    if (hipGetDevice(&c->device) != hipSuccess) { bgl::set_error("hipGetDevice failed"); return fail(BGL_EHIP); }
#define TRY_ALLOC(ptr, bytes)                                                              \
    if ((e = hipMalloc((void **)&(ptr), (bytes))) != hipSuccess) {                         \
        bgl::set_error("hipMalloc of %zu bytes failed: %s", (size_t)(bytes), hipGetErrorString(e)); \
        return fail(e == hipErrorOutOfMemory ? BGL_ENOMEM : BGL_EHIP);                     \
    }
    TRY_ALLOC(c->buffer, (size_t)c->rows * row_bytes);
    TRY_ALLOC(c->table, (size_t)nbk * BUCKET * sizeof(uint64_t));
    TRY_ALLOC(c->slot_to_node, (size_t)capacity_rows * sizeof(int32_t));
    TRY_ALLOC(c->slot_to_entry, (size_t)capacity_rows * sizeof(uint32_t));
    TRY_ALLOC(c->dev, sizeof(CacheDev));
#undef TRY_ALLOC
    if (hipEventCreateWithFlags(&c->ev_listed, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_miss, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_fetched, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_behind, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_map, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_ids, hipEventDisableTiming) != hipSuccess ||
        // only this library's kernels on this device wait for these two: no release to the system (LONG_LOOKUP_BYTES)
        hipEventCreateWithFlags(&c->ev_lists, hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_map_local, hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess) {
        bgl::set_error("stream/event creation failed");
        return fail(BGL_EHIP);
    }
    hipLaunchKernelGGL(k_fill_u64, dim3(2048), dim3(256), 0, 0, c->table, (int64_t)nbk * BUCKET,
                       EMPTY64, BUCKET);
    hipLaunchKernelGGL(k_fill_i32, dim3(1024), dim3(256), 0, 0, c->slot_to_node, capacity_rows, -1);
    if (hipMemset(c->dev, 0, sizeof(CacheDev)) != hipSuccess ||
        hipMemset(c->buffer, 0, (size_t)c->rows * row_bytes) != hipSuccess ||
        hipDeviceSynchronize() != hipSuccess) {
        bgl::set_error("cache initialisation failed: %s", hipGetErrorString(hipGetLastError()));
        return fail(BGL_EHIP);
    }
    *out = c;
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_destroy(bgl_cache_t *c)
try {
    if (!c) return BGL_OK;
    (void)hipDeviceSynchronize();
    for (auto ev : c->prof_ev) (void)hipEventDestroy(ev);
    if (c->ev_listed) (void)hipEventDestroy(c->ev_listed);
    if (c->ev_miss) (void)hipEventDestroy(c->ev_miss);
    if (c->ev_fetched) (void)hipEventDestroy(c->ev_fetched);
    if (c->ev_behind) (void)hipEventDestroy(c->ev_behind);
    if (c->ev_map) (void)hipEventDestroy(c->ev_map);
    if (c->ev_map_local) (void)hipEventDestroy(c->ev_map_local);
    if (c->ev_ids) (void)hipEventDestroy(c->ev_ids);
    if (c->ev_lists) (void)hipEventDestroy(c->ev_lists);
    if (c->own_side) (void)hipStreamDestroy(c->own_side);
    (void)hipFree(c->buffer);
    (void)hipFree(c->table);
    (void)hipFree(c->slot_to_node);
    (void)hipFree(c->slot_to_entry);
    (void)hipFree(c->dev);
    (void)hipFree(c->mbs);
    (void)hipFree(c->hit_pos);
    (void)hipFree(c->mpos_copy[0]);
    (void)hipFree(c->mpos_copy[1]);
    (void)hipFree(c->src_of[0]);
    (void)hipFree(c->src_of[1]);
    delete c;
    return BGL_OK;
} BGL_NOTHROW_END

namespace {

// The lists one lookup leaves for its own later kernels: per-tile miss counts (mbs_cap of them)
// followed by mbs_cap prefixes and mbs_cap counts of bucket lines read, and the hits as hit_cap
// positions followed by hit_cap slots.
struct LookupLists {
    int32_t *mbs;
    int64_t mbs_cap;
    int32_t *hit_pos;
    int64_t hit_cap;
};

// What the hit gather of a lookup needs of its lists.
struct HitList {
    const int32_t *pos = nullptr, *slot = nullptr;
    const int32_t *src_of = nullptr;  // assembled output: there is no hit gather
    bool with_lists = false;          // the lists are made in the gather's launch (k_list_and_hits)
    Lists lists = {};
};

// Make stream st wait for what a lookup that has not been joined yet still does on other streams: its miss
// fetch, and its hit gather unless st is that lookup's main stream (then st is behind it).
int join_rows(bgl_cache *c, hipStream_t st)
{
    if (!c->fetch_pending || c->fetch_stream == st) return BGL_OK;
    if (c->rows_split) {
        BGL_HIP(hipStreamWaitEvent(st, c->ev_fetched, 0));
        if (st != c->last_main) BGL_HIP(hipStreamWaitEvent(st, c->ev_listed, 0));
    } else {
        BGL_HIP(hipStreamWaitEvent(st, c->fetch_beside && st == c->last_main ? c->ev_fetched : c->ev_miss, 0));
    }
    return BGL_OK;
}

// First half of a lookup: map lookup and lists on stream ls, with a host tier its
// lookup for the misses (followed by ev_ids).  gather_phase enqueues the hit gather on stream ms,
// ev_listed.  ls == ms unless the lookup runs early (see the tiered call): then
// the lists go to *mpos_used, the library's own copy of miss_pos, because the
// caller's miss_pos of the previous call is still being read by that call's
// fetch while this one's lists are written.
int lookup_phase(bgl_cache *c, const int32_t *ids, int64_t n, int32_t *out_slot, int32_t *miss_pos, int64_t *n_hit_dev, hipStream_t ms, hipStream_t ls, bgl_host_tier *tier,
                 const int32_t **mpos_used, int *gen_used, HitList *hits, const LookupLists *fixed = nullptr,
                 bool assemble = false, bool record_lists = false, bool lists_with_hits = false, bool record_slots = false)
{
    const bool early = ls != ms;
    const int gen = (int)(c->lookup_calls & 1);  // which copy of the per-call device state this call owns
    *gen_used = gen;
    const int64_t tiles = bgl::ceil_div(n, KEYS_PER_TILE);
    // the per-call lists: the cache's own, grown on demand, or the ones the caller of this function brings
    if (!fixed && tiles + 1 > c->mbs_cap) {
        BGL_HIP(hipDeviceSynchronize());
        (void)hipFree(c->mbs);
        c->mbs = nullptr;
        c->mbs_cap = 0;
        const int64_t cap = std::max<int64_t>(2 * tiles + 1, 1024);
        BGL_HIP(hipMalloc((void **)&c->mbs, 3 * sizeof(int32_t) * (size_t)cap));  // counts, their prefixes, lines read
        c->mbs_cap = cap;
    }
    if (!fixed && n > c->hit_cap) {
        BGL_HIP(hipDeviceSynchronize());
        (void)hipFree(c->hit_pos);
        c->hit_pos = nullptr;
        c->hit_cap = 0;
        const int64_t cap = std::max<int64_t>(n + n / 2, 4096);
        BGL_HIP(hipMalloc((void **)&c->hit_pos, 2 * sizeof(int32_t) * (size_t)cap));  // positions, then slots
        c->hit_cap = cap;
    }
    int32_t *mpos_copy = nullptr;
    if (early) {
        const int g = gen;
        if (n > c->mpos_cap[g]) {
            BGL_HIP(hipDeviceSynchronize());
            (void)hipFree(c->mpos_copy[g]);
            c->mpos_copy[g] = nullptr;
            c->mpos_cap[g] = 0;
            const int64_t cap = std::max<int64_t>(n + n / 2, 4096);
            BGL_HIP(hipMalloc((void **)&c->mpos_copy[g], sizeof(int32_t) * (size_t)cap));
            c->mpos_cap[g] = cap;
        }
        mpos_copy = c->mpos_copy[g];
    }
    *mpos_used = early ? mpos_copy : miss_pos;
    // Assembled output (the caller launches k_assemble_pre / k_assemble_rows once the miss rows have
    // landed): the list kernel records every position's source, and there is no hit gather here.
    int32_t *src_of = nullptr;
    if (assemble) {
        const int g = gen;
        if (n > c->src_cap[g]) {
            BGL_HIP(hipDeviceSynchronize());
            (void)hipFree(c->src_of[g]);
            c->src_of[g] = nullptr;
            c->src_cap[g] = 0;
            const int64_t cap = std::max<int64_t>(n + n / 2, 4096);
            BGL_HIP(hipMalloc((void **)&c->src_of[g], sizeof(int32_t) * (size_t)cap));
            c->src_cap[g] = cap;
        }
        src_of = c->src_of[g];
    }
    int32_t *const mbs = fixed ? fixed->mbs : c->mbs;
    const int64_t mbs_cap = fixed ? fixed->mbs_cap : c->mbs_cap;
    int32_t *const hit_pos = fixed ? fixed->hit_pos : c->hit_pos;
    const int64_t hit_cap = fixed ? fixed->hit_cap : c->hit_cap;
    *hits = HitList{hit_pos, hit_pos + hit_cap, src_of, false, {}};
    c->lookup_calls += 1;
    c->last_n = n;
    if (tier) bgl::tier_prepare(tier);
    if (c->map_pending && c->map_stream != ls) BGL_HIP(hipStreamWaitEvent(ls, c->map_event, 0));
    int rc = BGL_OK;
    // the previous call's fetch still reads that call's lists
    if (!early && (rc = join_rows(c, ms)) != BGL_OK) return rc;
    // so does it when that call was not an early one: then this one cannot be early either
    if (early && c->fetch_reads_caller_lists && (rc = join_rows(c, ls)) != BGL_OK) return rc;
    if (n > 0) {
        {
            Prof p(c, BGL_STAGE_PROBE, ls);
            auto probe = [&](auto &&launch_it, int32_t *own_slot) {
                return launch_it(k_probe, dim3((unsigned)tiles), dim3(KEYS_PER_TILE), ids, n, c->num_nodes, c->table,
                                 c->num_buckets - 1, out_slot, own_slot, mbs, mbs + 2 * mbs_cap, c->dev);
            };
            if (record_slots)  // (the hits' list has no other use then)
                rc = probe([&](auto kernel, auto &&...a) { return launch_marked(c, ls, c->ev_lists, true, kernel, a...); }, hit_pos);
            else
                probe([&](auto kernel, auto &&...a) { launch(c, ls, kernel, a...); }, (int32_t *)nullptr);
            if (rc != BGL_OK) return rc;
        }
        {
            Prof p(c, BGL_STAGE_MISS_LIST, ls, false);
            int32_t *tile_prefix = nullptr;
            if (tiles >= kSelfSumTiles) {
                tile_prefix = mbs + mbs_cap;
                hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(kScanThreads), 0, ls, mbs, tiles, tile_prefix);
            }
            const Lists lists{out_slot, n, mbs, tile_prefix, mbs + 2 * mbs_cap, miss_pos, hit_pos, hit_pos + hit_cap, c->dev, n_hit_dev, ids,
                              c->num_nodes, tier ? bgl::tier_ids_device_if_passthrough(tier) : nullptr, mpos_copy, gen, src_of,
                              c->capacity, c->rows, (int)(c->insert_calls & 1)};
            if (lists_with_hits) {
                hits->with_lists = true;
                hits->lists = lists;
            } else if (record_lists) {
                rc = launch_marked(c, ls, c->ev_lists, true, k_split_list, dim3((unsigned)tiles), dim3(KEYS_PER_TILE), lists);
            } else {
                launch(c, ls, k_split_list, dim3((unsigned)tiles), dim3(KEYS_PER_TILE), lists);
            }
            if (rc != BGL_OK) return rc;
        }
    } else {
        hipLaunchKernelGGL(k_empty_lookup, dim3(1), dim3(64), 0, ls, c->dev, n_hit_dev, gen);
    }
    if (tier) {
        const int rc = bgl::tier_enqueue_lookup(tier, ids, miss_pos, &c->dev->n_miss_last, n, gen, ls);
        if (rc != BGL_OK) return rc;
    }
    if (tier || early) BGL_HIP(hipEventRecord(c->ev_ids, ls));  // the lists are complete
    if (early) {
        // the hit gather reads rows the previous fetch may still be writing, and needs the lists
        if ((rc = join_rows(c, ms)) != BGL_OK) return rc;
        BGL_HIP(hipStreamWaitEvent(ms, c->ev_ids, 0));
    }
    c->fetch_pending = false;
    c->rows_joined = false;
    c->map_pending = false;
    c->last_main = ms;
    return BGL_OK;
}

int gather_phase(bgl_cache *c, int64_t n, void *out_rows, hipStream_t ms, const HitList &hits, bool own)
{
    const int q = c->row_bytes / 16;
    c->ev_listed_valid = true;
    if (n > 0 && !hits.src_of) {
        Prof p(c, BGL_STAGE_GATHER_HIT, ms);
        int rc = BGL_OK;
        dispatch_q(q, [&](auto Q) {
            if (hits.with_lists) {
                const int tiles = (int)bgl::ceil_div(n, KEYS_PER_TILE);
                rc = launch_marked(c, ms, c->ev_listed, own, k_list_and_hits<decltype(Q)::value>, dim3(tiles + copy_blocks(n, q)),
                                   dim3(COPY_THREADS), hits.lists, tiles, q, reinterpret_cast<const uint4 *>(c->buffer),
                                   reinterpret_cast<uint4 *>(out_rows));
                return;
            }
            rc = launch_marked(c, ms, c->ev_listed, own, k_gather_hits<decltype(Q)::value>, dim3(copy_blocks(n, q)), dim3(COPY_THREADS),
                               hits.pos, hits.slot, q, reinterpret_cast<const uint4 *>(c->buffer),
                               reinterpret_cast<uint4 *>(out_rows), n * c->row_bytes, c->dev);
        });
        return rc;
    }
    BGL_HIP(hipEventRecord(c->ev_listed, ms));
    return BGL_OK;
}

// The miss rows of the last lookup, for work that is behind its hit gather.
hipEvent_t misses_event(const bgl_cache *c) { return c->fetch_beside ? c->ev_fetched : c->ev_miss; }

// The stream of the miss fetch: the caller's, or one of the cache's own.
int side_stream_of(bgl_cache *c, void *side_stream, hipStream_t *out)
{
    if (side_stream) {
        *out = static_cast<hipStream_t>(side_stream);
        return BGL_OK;
    }
    if (!c->own_side) BGL_HIP(hipStreamCreateWithFlags(&c->own_side, hipStreamNonBlocking));
    *out = c->own_side;
    return BGL_OK;
}

int check_lookup_args(bgl_cache *c, const int32_t *ids, int64_t n, void *out_rows, int32_t *out_slot,
                      int32_t *miss_pos)
{
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (n < 0 || n > INT32_MAX) BGL_FAIL(BGL_EINVAL, "n must be in [0, 2^31) (got %lld)", (long long)n);
    if (n > 0 && (!ids || !out_rows || !out_slot || !miss_pos))
        BGL_FAIL(BGL_EINVAL, "ids, out_rows, out_slot and miss_pos must not be null");
    if (!bgl::aligned(out_rows, 16)) BGL_FAIL(BGL_EINVAL, "out_rows is not 16-byte aligned");
    if (c->tiered.active)
        BGL_FAIL(BGL_EINVAL, "a tiered lookup has been begun: bgl_cache_lookup_tiered_finish comes first");
    if (c->write_through && c->awaiting_insert)
        BGL_FAIL(BGL_EINVAL, "write-through mode: the previous lookup's misses have not been inserted yet");
    return BGL_OK;
}

}  // namespace

namespace {

int lookup_gather_impl(bgl_cache_t *c, const int32_t *ids, int64_t n, void *out_rows, int32_t *out_slot,
                       int32_t *miss_pos, int64_t *n_hit_host, void *main_stream, void *side_stream,
                       void *lookup_stream, bool early, const LookupLists *fixed = nullptr)
{
    int rc = check_lookup_args(c, ids, n, out_rows, out_slot, miss_pos);
    if (rc != BGL_OK) return rc;
    if (early && !c->write_through)
        BGL_FAIL(BGL_EINVAL, "an early lookup needs write-through mode");
    if (!c->features) BGL_FAIL(BGL_EINVAL, "the cache has no backing store: use bgl_cache_lookup_gather_tiered");
    hipStream_t ms = static_cast<hipStream_t>(main_stream);
    hipStream_t ss = nullptr;
    if (fixed) {
        ss = side_stream ? static_cast<hipStream_t>(side_stream) : ms;  // (no stream is created here)
    } else {
        rc = side_stream_of(c, side_stream, &ss);
        if (rc != BGL_OK) return rc;
    }
    // the hit count goes straight into the caller's page-locked word (no copy launch)
    int64_t *n_hit_dev = nullptr;
    if (n_hit_host) {
        hipPointerAttribute_t attr;
        if (hipPointerGetAttributes(&attr, n_hit_host) != hipSuccess || attr.type != hipMemoryTypeHost ||
            !attr.devicePointer) {
            (void)hipGetLastError();
            BGL_FAIL(BGL_EINVAL, "n_hit_host must be page-locked host memory");
        }
        n_hit_dev = static_cast<int64_t *>(attr.devicePointer);
    }
    const int q = c->row_bytes / 16;
    hipStream_t ls = early ? static_cast<hipStream_t>(lookup_stream) : ms;
    const int32_t *mpos = nullptr;
    int gen = 0;
    // On a stream of its own the miss fetch starts once the hit gather is done: its host reads would hold
    // up the gather's HBM reads (428,377 ids, three quarters of them missed: gather 20 -> 140 us), and a
    // fetch of milliseconds loses nothing by waiting for it.  A cache that can hold every node misses a
    // node once: there the fetch of a large lookup starts as soon as the lists are there, beside the gather,
    // so that the FIFO update finds its (mostly empty) work done when the gather ends instead of waiting for
    // two more hand-overs between streams.
    // (Write-through mode: the fetch overwrites rows that the gather may have to read.)
    const bool beside = ss != ms && !c->write_through && c->capacity >= c->num_nodes && n * c->row_bytes > LONG_LOOKUP_BYTES;
    const bool update_beside = c->map_pending && c->map_stream != ms;  // the FIFO updates run on a stream of their own
    // So does the fetch of a small one on the cache's own side stream: there the host's calls set the pace, and
    // those for the side stream come before the gather's.
    const bool few_bytes = ss != ms && !side_stream && !c->write_through && !c->features_in_hbm && n * c->row_bytes <= BESIDE_BYTES;
    const bool mostly_hits = c->capacity >= c->num_nodes;
    // A fetch over the link beside the gather waits for the slots alone (k_fetch_slots), unless it may be long: then the lists
    // deal the misses more evenly (60,000 ids of 1,024 bytes, 90 % missed, from the slots / from lists: 1,084 / 1,077 us).
    // Lookup + update from lists | from slots with k_list_and_hits, each waited for / one after the other, us: 200 x 400 B 57 / 54 |
    // 54 / 49; 5,000 x 400 B, 90 % missed 97 / 83 | 93 / 77, half 83 / 70 | 77 / 64, none 59 / 59 | 56 / 54; 20,000 x 64 B, half 94 / 77 |
    // 89 / 70; 20,000 x 400 B, 90 % missed 220 / 205 | 220 / 204; 302,709 hits of 1,024 B 163 / 144 | 161 / 140.
    // (Stages timed in this call have launches of their own; the lists that allocate nothing are read until the gather has ended, no
    // longer.)
    const uint64_t call = c->lookup_calls + 1;
    const bool timed_lists = timed(c, BGL_STAGE_MISS_LIST, call) || timed(c, BGL_STAGE_GATHER_HIT, call);
    const bool from_slots = (beside || few_bytes) && !timed_lists && !fixed && !c->features_in_hbm && q <= kWave && n > 0 &&
                            (mostly_hits || n * c->row_bytes <= FROM_SLOTS_BYTES);
    // The lists in the gather's launch (k_list_and_hits), unless the fetch waits for them beside it.
    const bool with_hits = !early && !timed_lists && (from_slots || !(beside || few_bytes)) &&
                           (mostly_hits || n * c->row_bytes <= GATHER_CACHED_ROWS_BYTES);
    HitList hits;
    rc = lookup_phase(c, ids, n, out_slot, miss_pos, n_hit_dev, ms, ls, nullptr, &mpos, &gen, &hits, fixed, false,
                      (beside || few_bytes) && n > 0 && !from_slots, with_hits, from_slots);
    if (rc != BGL_OK) return rc;
    const hipEvent_t fetched = beside || few_bytes ? c->ev_fetched : c->ev_miss;
    // (see launch_marked)
    const bool own = update_beside || c->streaming ? c->streaming : few_bytes || n * c->row_bytes > LONG_LOOKUP_BYTES;
    auto fetch = [&]() -> int {
        {
            Prof p(c, BGL_STAGE_FETCH_MISS, ss);
            // The small grid and the dealing of whole rows to wavefronts are for the host link only; an
            // HBM-resident store wants the whole chip and every lane, and a row of more than 64 chunks is
            // dealt to several wavefronts either way.
            const int par = (int)(c->insert_calls & 1);
            const uint4 *features = reinterpret_cast<const uint4 *>(c->features);
            uint4 *out = reinterpret_cast<uint4 *>(out_rows), *buffer = reinterpret_cast<uint4 *>(c->buffer);
            if (from_slots) {
                // as many positions for every wavefront, and for each of its turns
                const int64_t waves = (int64_t)FETCH_BLOCKS * (COPY_THREADS / kWave), turns = bgl::ceil_div(n, waves * kWave);
                const int per = (int)bgl::ceil_div(n, waves * turns);
                const int blocks = (int)std::min<int64_t>(bgl::ceil_div(n, (int64_t)per * (COPY_THREADS / kWave)), FETCH_BLOCKS);
                const size_t lds = sizeof(int2) * (size_t)slots_queue(q) * (COPY_THREADS / kWave);
                rc = launch_marked(c, ss, fetched, own, k_fetch_slots, Grid(dim3(blocks), lds), dim3(COPY_THREADS), hits.pos, ids, n, per, q,
                                   c->num_nodes, features, out);
            } else if (!c->features_in_hbm && q <= kWave) {
                const bool few = c->write_through && update_beside && n * c->row_bytes <= SMALL_LOOKUP_BYTES;
                const int64_t rows_per_block = (int64_t)(COPY_THREADS / kWave) * COPY_UNROLL * (kWave / q);
                const int64_t most = !few ? FETCH_BLOCKS
                                          : std::clamp<int64_t>(bgl::ceil_div(n * c->row_bytes, SMALL_FETCH_BYTES_PER_BLOCK), LEAST_FETCH_BLOCKS,
                                                                SMALL_FETCH_BLOCKS);
                const int blocks = (int)std::min<int64_t>(bgl::ceil_div(n, rows_per_block), most);
                rc = launch_marked(c, ss, fetched, own, c->write_through ? k_fetch_link<true> : k_fetch_link<false>, dim3(blocks),
                                   dim3(COPY_THREADS), mpos, ids, q, c->num_nodes, features, out, c->dev, buffer, c->capacity,
                                   c->rows, par, gen);
            } else {
                const int blocks = (int)std::min<int64_t>(copy_blocks(n, q), c->features_in_hbm ? 8192 : FETCH_BLOCKS);
                dispatch_q(q, [&](auto Q) {
                    auto k = c->write_through ? k_fetch_miss<decltype(Q)::value, true>
                                              : k_fetch_miss<decltype(Q)::value, false>;
                    rc = launch_marked(c, ss, fetched, own, k, dim3(blocks), dim3(COPY_THREADS), mpos, ids, q, c->num_nodes, features,
                                       out, c->dev, buffer, c->capacity, c->rows, par, gen);
                });
            }
        }
        return rc;
    };
    if (n > 0 && (beside || few_bytes)) {
        BGL_HIP(hipStreamWaitEvent(ss, c->ev_lists, 0));
        if ((rc = fetch()) != BGL_OK) return rc;
    }
    if ((rc = gather_phase(c, n, out_rows, ms, hits, !update_beside || c->streaming)) != BGL_OK) return rc;
    if (n > 0) {
        if (!beside && !few_bytes) {
            if (ss != ms) BGL_HIP(hipStreamWaitEvent(ss, c->ev_listed, 0));
            if ((rc = fetch()) != BGL_OK) return rc;
        } else if (beside) {
            // (ev_miss, and whatever the caller enqueues on the side stream, come behind the gather as well)
            BGL_HIP(hipStreamWaitEvent(ss, c->ev_listed, 0));
            BGL_HIP(hipEventRecord(c->ev_miss, ss));
        } else if (own) {
            BGL_HIP(hipEventRecord(c->ev_behind, ss));
        }
        c->fetch_pending = true;
        c->fetch_beside = beside || few_bytes;
        c->rows_split = few_bytes && !beside;
        c->fetch_stream = ss;
        c->fetch_reads_caller_lists = mpos == miss_pos;
    }
    BGL_HIP(hipGetLastError());
    if (c->write_through) {
        c->awaiting_insert = true;
        c->wt_ids = ids;
        c->wt_miss_pos = miss_pos;
    }
    return BGL_OK;
}

}  // namespace

extern "C" int bgl_cache_lookup_gather(bgl_cache_t *c, const int32_t *ids, int64_t n,
                                       void *out_rows, int32_t *out_slot, int32_t *miss_pos,
                                       int64_t *n_hit_host, void *main_stream, void *side_stream)
try {
    return lookup_gather_impl(c, ids, n, out_rows, out_slot, miss_pos, n_hit_host, main_stream, side_stream,
                              nullptr, false);
} BGL_NOTHROW_END

// ---- the lookup that allocates nothing
// Its lists live in a fixed array in device memory that is part of the library's code object
// (every GPU the library runs on holds its own copy until the process ends).  The array's name
// is only a host-side stand-in: the address the kernels get is asked for once per device.
namespace {

constexpr int64_t NOALLOC_MAX_IDS = BGL_NOALLOC_MAX_IDS;
constexpr int64_t NOALLOC_TILES = (NOALLOC_MAX_IDS + KEYS_PER_TILE - 1) / KEYS_PER_TILE + 1;
constexpr size_t NOALLOC_MBS_BYTES = (3 * sizeof(int32_t) * (size_t)NOALLOC_TILES + 255) / 256 * 256;
constexpr size_t NOALLOC_BYTES = NOALLOC_MBS_BYTES + 2 * sizeof(int32_t) * (size_t)NOALLOC_MAX_IDS;
constexpr int NOALLOC_MAX_DEVICES = 64;

static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

void *g_scratch_ptr[NOALLOC_MAX_DEVICES];  // device address of `scratch` on each device, once asked for
std::mutex g_scratch_mutex;

int scratch_of_current_device(int device, void **out)
{
    if (device < 0 || device >= NOALLOC_MAX_DEVICES) BGL_FAIL(BGL_EUNSUPPORTED, "device ordinal %d is out of range", device);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        BGL_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) BGL_FAIL(BGL_EHIP, "hipGetSymbolAddress returned a null address");
        g_scratch_ptr[device] = ptr;
    }
    *out = g_scratch_ptr[device];
    return BGL_OK;
}

}  // namespace

extern "C" int bgl_cache_lookup_gather_noalloc(bgl_cache_t *c, const int32_t *ids, int64_t n,
                                               void *out_rows, int32_t *out_slot, int32_t *miss_pos,
                                               int64_t *n_hit_host, void *main_stream, void *side_stream)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (n > NOALLOC_MAX_IDS)
        BGL_FAIL(BGL_ECAPACITY, "n = %lld exceeds BGL_NOALLOC_MAX_IDS = %lld: use bgl_cache_lookup_gather",
                 (long long)n, (long long)NOALLOC_MAX_IDS);
    int device = -1;
    BGL_HIP(hipGetDevice(&device));
    if (device != c->device)
        BGL_FAIL(BGL_EINVAL, "the cache lives on device %d, the current device is %d", c->device, device);
    void *ptr = nullptr;
    int rc = scratch_of_current_device(device, &ptr);
    if (rc != BGL_OK) return rc;
    unsigned char *base = static_cast<unsigned char *>(ptr);
    const LookupLists lists{reinterpret_cast<int32_t *>(base), NOALLOC_TILES,
                            reinterpret_cast<int32_t *>(base + NOALLOC_MBS_BYTES), NOALLOC_MAX_IDS};
    // (a timed launch may have to create events: this call's kernels are not timed)
    struct Untimed {
        bgl_cache *c;
        unsigned saved;
        explicit Untimed(bgl_cache *c_) : c(c_), saved(c_->profiling) { c->profiling = 0; }
        ~Untimed() { c->profiling = saved; }
    } untimed(c);
    return lookup_gather_impl(c, ids, n, out_rows, out_slot, miss_pos, n_hit_host, main_stream, side_stream,
                              nullptr, false, &lists);
} BGL_NOTHROW_END

extern "C" int bgl_cache_lookup_gather_early(bgl_cache_t *c, const int32_t *ids, int64_t n,
                                             void *out_rows, int32_t *out_slot, int32_t *miss_pos,
                                             int64_t *n_hit_host, void *main_stream, void *side_stream,
                                             void *lookup_stream)
try {
    return lookup_gather_impl(c, ids, n, out_rows, out_slot, miss_pos, n_hit_host, main_stream, side_stream,
                              lookup_stream, static_cast<hipStream_t>(lookup_stream) != static_cast<hipStream_t>(main_stream));
} BGL_NOTHROW_END

namespace {

// The packed rows of one tiered lookup on their way to out_rows (and, in write-through mode, to the
// cache buffer).  Host threads pack them as one sequence: first the rows the tier holds (into its
// staging rows, in list order), then the others (from the store into consecutive ring positions).
struct TieredRows {
    bgl_cache *c;
    bgl_host_tier *t;
    const bgl::TierPlan *plan;
    hipStream_t ss;        // the stream of the kernels that write the rows to their places
    const int32_t *mpos;   // this call's miss positions (the caller's list, or the library's copy)
    void *out_rows;
    int64_t n;
    int64_t staged() const { return in_place ? 0 : plan->n_hit; }  // leading rows of the packed sequence that the tier holds
    int par;               // which copy of the cache's tail the kernels read
    bool early;            // the lookup ran early: the host is ahead of the link
    bool in_place;         // kernels read the rows the tier holds in its ring: only its misses are packed
    const int32_t *src_of; // assembled output: the source of every position's row (else null)

    // out[mpos[rank[l]]] = base[(first + l) mod ring] for l0 <= l < l0 + count.  landed: the rows are in
    // device memory (whole chip; rows read once, and written for a later kernel: non-temporal accesses, so
    // that they do not push the cache buffer's and the output's lines out of the chip's caches in front of
    // the next hit gather); else they are read over the host link (small grid).
    void launch_rows(const char *base, unsigned long long first, int64_t ring, const int32_t *rank, int64_t l0,
                     int64_t count, bool landed) const
    {
        if (count == 0) return;
        const int q = c->row_bytes / 16;
        Prof p(c, BGL_STAGE_FETCH_MISS, ss);
        const int blocks = (int)std::min<int64_t>(copy_blocks(count, q), landed ? 8192 : RING_FETCH_BLOCKS);
        dispatch_q(q, [&](auto Q) {
            constexpr int QQ = decltype(Q)::value;
            auto k = landed ? (c->write_through ? k_fetch_rows<QQ, true, true> : k_fetch_rows<QQ, false, true>)
                            : (c->write_through ? k_fetch_rows<QQ, true, false> : k_fetch_rows<QQ, false, false>);
            launch(c, ss, k, dim3(blocks), dim3(COPY_THREADS), rank, l0, count, first, ring, mpos, q,
                   reinterpret_cast<const uint4 *>(base), reinterpret_cast<uint4 *>(out_rows), c->dev,
                   reinterpret_cast<uint4 *>(c->buffer), c->capacity, c->rows, par, n - plan->n_hit_gpu);
        });
    }
    // The rows the tier holds, read in its ring.
    void launch_ring() const
    {
        const int q = c->row_bytes / 16;
        Prof p(c, BGL_STAGE_FETCH_MISS, ss);
        const int64_t rows_per_block = (int64_t)(COPY_THREADS / kWave) * COPY_UNROLL * (kWave / q);
        const int blocks = (int)std::min<int64_t>(bgl::ceil_div(plan->n_hit, rows_per_block), FETCH_BLOCKS);
        launch(c, ss, c->write_through ? k_fetch_ring<true> : k_fetch_ring<false>, dim3(blocks), dim3(COPY_THREADS), plan->hit_rank,
               plan->hit_ring, plan->n_hit, mpos, q, reinterpret_cast<const uint4 *>(bgl::tier_rows_device(t)),
               reinterpret_cast<uint4 *>(out_rows), c->dev, reinterpret_cast<uint4 *>(c->buffer), c->capacity, c->rows, par,
               n - plan->n_hit_gpu);
    }
    // Assembled output, first launch: the hits whose slots this call's misses are about to take.
    void launch_assemble_pre() const
    {
        const int q = c->row_bytes / 16;
        Prof p(c, BGL_STAGE_ASSEMBLE_PRE, ss);
        const int blocks = (int)std::min<int64_t>(bgl::ceil_div(n, COPY_THREADS), 2048);
        dispatch_q(q, [&](auto Q) {
            launch(c, ss, k_assemble_pre<decltype(Q)::value>, dim3(blocks), dim3(COPY_THREADS), src_of, n, q,
                   reinterpret_cast<const uint4 *>(c->buffer), reinterpret_cast<uint4 *>(out_rows), c->dev,
                   c->capacity, c->rows, par, n - plan->n_hit_gpu);
        });
    }
    // Second launch, once the packed miss rows are in `land`: every other row of the output, and
    // the miss rows into the cache buffer.
    void launch_assemble_rows(const char *land) const
    {
        const int q = c->row_bytes / 16;
        Prof p(c, BGL_STAGE_ASSEMBLE, ss);
        // One workgroup per 1,024 chunks (a grid capped at 8,192 workgroups that strides was measured 2 % slower
        // on 400- and 1,024-byte rows).  The output is written with ordinary stores while a batch's rows fit
        // the chip's last-level cache with room to spare (the next batch overwrites them there, and whoever
        // consumes them reads them there), with non-temporal ones beyond that; the rows that go into the
        // cache buffer are always written non-temporally.  (Measured, fraction of HBM peak with ordinary /
        // non-temporal output stores: 61 MB of output 0.68 / 0.64, 102 MB 0.77 / 0.67, 171 MB 0.66 / 0.66,
        // 310 MB 0.68 / 0.70.)
        const bool nto = (int64_t)n * c->row_bytes > ASSEMBLE_CACHED_OUTPUT_BYTES;
        const int blocks = (int)std::min<int64_t>(copy_blocks(n, q), 1 << 20);
        dispatch_q(q, [&](auto Q) {
            constexpr int QQ = decltype(Q)::value;
            auto k = nto ? k_assemble_rows<QQ, true> : k_assemble_rows<QQ, false>;
            launch(c, ss, k, dim3(blocks), dim3(COPY_THREADS), src_of, n, q,
                   reinterpret_cast<const uint4 *>(land), reinterpret_cast<uint4 *>(c->buffer),
                   reinterpret_cast<uint4 *>(out_rows), c->dev, c->capacity, c->rows, par, n - plan->n_hit_gpu);
        });
    }
};

// Copy-engine transport: the packed rows go to device memory (`land`) with plain copies on the tier's
// copy stream, as soon as they are packed and whatever the kernels of this cache are doing (the
// previous call's rows may still be on their way); kernels then scatter them from there, after the
// hit gather.  The link carries one batch after the other.
int rows_by_copy_engine(const TieredRows &r, char *land)
{
    bgl_cache *c = r.c;
    bgl_host_tier *t = r.t;
    const bgl::TierPlan &plan = *r.plan;
    const int64_t staged = r.staged(), total = staged + plan.n_miss;
    const size_t rb = (size_t)c->row_bytes;
    hipStream_t cs = bgl::tier_copy_stream(t);
    const char *ring_rows = bgl::tier_rows_device(t);
    auto copy = [&](char *dst, const char *src, int64_t count) -> int {
        Prof p(c, BGL_STAGE_LINK_COPY, cs, false);
        BGL_HIP(hipMemcpyAsync(dst, src, (size_t)count * rb, hipMemcpyDefault, cs));
        return BGL_OK;
    };
    // rows x0 <= x < x1 of the packed sequence: the tier's hits (staging rows), then its misses (ring)
    auto copy_rows = [&](int64_t x0, int64_t x1) -> int {
        if (x0 < staged) {
            const int64_t e = std::min(x1, staged);
            const int r1 = copy(land + (size_t)x0 * rb, plan.stage + (size_t)x0 * rb, e - x0);
            if (r1 != BGL_OK) return r1;
        }
        const int64_t a = std::max(x0, staged) - staged, b = x1 - staged;
        if (b > a) {
            const int64_t pos = (int64_t)((plan.ptail + (uint64_t)a) % (uint64_t)plan.ring);
            const int64_t len1 = std::min(b - a, plan.ring - pos);  // up to the end of the ring
            const int r1 = copy(land + (size_t)(staged + a) * rb, ring_rows + (size_t)pos * rb, len1);
            if (r1 != BGL_OK) return r1;
            if (len1 < b - a) {
                const int r2 = copy(land + (size_t)(staged + a + len1) * rb, ring_rows, b - a - len1);
                if (r2 != BGL_OK) return r2;
            }
        }
        return BGL_OK;
    };
    // A copy costs the link a few microseconds whatever its size, so while earlier copies (the
    // previous call's, or this call's) still occupy the link the packed rows pile up for one larger
    // copy; when the link is free a chunk goes at once.
    // (`land` was last read by the kernels of the call before the previous one.  They are over: this call's
    // lists, which the host has just waited for, follow the previous call's map update, which follows that
    // call's lists, which were recorded behind the wait for those kernels.)
    // (an early lookup is ahead of the link as a rule: large chunks from the start, but a short batch is
    // not held back for one)
    int64_t chunk = r.early ? std::min(TIER_CHUNK_ROWS, std::max<int64_t>(total / 4, 4 * TIER_FIRST_CHUNK_ROWS))
                            : TIER_FIRST_CHUNK_ROWS;
    bool link_busy = bgl::tier_copy_event_recorded(t);
    for (int64_t launched = 0; launched < total;) {
        const int64_t ready = bgl::tier_copy_progress(t);
        bool go = ready > launched && ready == total;
        if (!go && ready - launched >= chunk) {
            if (link_busy) {
                link_busy = hipEventQuery(bgl::tier_copy_event(t)) != hipSuccess;
                (void)hipGetLastError();  // "not ready" is no error
            }
            go = !link_busy;
        }
        if (go) {
            const int rc = copy_rows(launched, ready);
            if (rc != BGL_OK) return rc;
            BGL_HIP(hipEventRecord(bgl::tier_copy_event(t), cs));
            bgl::tier_set_copy_event_recorded(t);
            link_busy = true;
            launched = ready;
            // (without an early lookup what has piled up while a copy was on the link goes behind it: waiting for
            // larger and larger chunks left the link idle between them.  150,001 ids x 512 B, 67 MB: 1,690 -> 1,600 us)
            chunk = r.early ? std::min<int64_t>(2 * chunk, TIER_CHUNK_ROWS) : bgl::ceil_div(LINK_CHUNK_BYTES, (int64_t)rb);
        } else if (!bgl::tier_copy_help(t)) {  // nothing to send: pack a few rows too
            __builtin_ia32_pause();
        }
    }
    bgl::tier_copy_wait(t);
    if (r.src_of) {  // (the tier keeps nothing: plan.n_hit == 0, the landed rows are in miss order)
        // The first pass is needed only if this call's rows may land on live ones: not when the buffer
        // has a spare position for every miss of the call (the misses that do not stay advance the
        // position too).  (It needs no landed row: it runs while the copies are still on their way.)
        if (r.n - plan.n_hit_gpu > c->rows - c->capacity) r.launch_assemble_pre();
        BGL_HIP(hipStreamWaitEvent(r.ss, bgl::tier_copy_event(t), 0));
        r.launch_assemble_rows(land);
        return BGL_OK;
    }
    BGL_HIP(hipStreamWaitEvent(r.ss, bgl::tier_copy_event(t), 0));  // (recorded behind the last copy)
    r.launch_rows(land, 0ull, (int64_t)INT64_MAX, plan.hit_rank, 0, staged, true);
    r.launch_rows(land + (size_t)staged * rb, 0ull, (int64_t)INT64_MAX, plan.miss_rank, 0, plan.n_miss, true);
    return BGL_OK;
}

// Kernel transport: the kernels read the page-locked rows over the host link themselves, chunk by
// chunk as the rows are packed.  Small chunks first, so that the link starts early; the copy threads
// outrun the link only by a little, so the chunks grow until a launch is a few per cent of its kernel.
int rows_by_kernels(const TieredRows &r)
{
    bgl_cache *c = r.c;
    bgl_host_tier *t = r.t;
    const bgl::TierPlan &plan = *r.plan;
    const int64_t staged = r.staged(), total = staged + plan.n_miss;
    const char *ring_rows = bgl::tier_rows_device(t);
    // (an early lookup is ahead of the link anyway: full chunks from the start)
    int64_t chunk = r.early ? TIER_CHUNK_ROWS : TIER_FIRST_CHUNK_ROWS;
    bool gather_done = false;
    for (int64_t launched = 0; launched < total;) {
        const int64_t ready = bgl::tier_copy_progress(t);
        // a chunk does not straddle the two kinds of rows
        const int64_t limit = launched < staged ? std::min(ready, staged) : ready;
        bool go = limit > launched && (limit == staged || limit == total);
        if (!go && limit - launched >= chunk) {
            // An early lookup's fetch cannot start before its hit gather has run, which waits for
            // the previous call's fetch: until then the packed rows pile up for one larger launch.
            if (r.early && !gather_done) {
                gather_done = hipEventQuery(c->ev_listed) == hipSuccess;
                (void)hipGetLastError();  // "not ready" is no error
            }
            go = gather_done || !r.early;
        }
        if (go) {
            if (launched < staged)
                r.launch_rows(plan.stage, 0ull, (int64_t)INT64_MAX, plan.hit_rank, launched, limit - launched,
                              false);
            else
                r.launch_rows(ring_rows, (unsigned long long)plan.ptail, plan.ring, plan.miss_rank,
                              launched - staged, limit - launched, false);
            launched = limit;
            chunk = std::min<int64_t>(2 * chunk, TIER_CHUNK_ROWS);
        } else if (!bgl::tier_copy_help(t)) {  // nothing to send: pack a few rows too
            __builtin_ia32_pause();
        }
    }
    bgl::tier_copy_wait(t);
    return BGL_OK;
}

}  // namespace

namespace {

// First half of a tiered lookup: the map lookup and the lists (and, unless one pass will write the whole
// output, the hit gather) are enqueued, the host waits for the lists and its threads start packing rows.
int tiered_begin(bgl_cache_t *c, bgl_host_tier_t *t, const int32_t *ids, int64_t n, void *out_rows,
                 int32_t *out_slot, int32_t *miss_pos, void *main_stream, void *side_stream, void *lookup_stream,
                 int early_lookup)
{
    int rc = check_lookup_args(c, ids, n, out_rows, out_slot, miss_pos);
    if (rc != BGL_OK) return rc;
    if (!t) BGL_FAIL(BGL_EINVAL, "tier handle is null");
    if (bgl::tier_row_bytes(t) != c->row_bytes || bgl::tier_num_nodes(t) != c->num_nodes)
        BGL_FAIL(BGL_EINVAL, "cache and host tier differ in row_bytes or num_nodes");
    if (n > bgl::tier_max_batch(t))
        BGL_FAIL(BGL_ECAPACITY, "n = %lld exceeds the tier's max_batch_rows", (long long)n);
    hipStream_t ms = static_cast<hipStream_t>(main_stream);
    hipStream_t ss = nullptr;
    rc = side_stream_of(c, side_stream, &ss);
    if (rc != BGL_OK) return rc;
    // Early lookup: only in write-through mode (otherwise the previous call's row copy still reads
    // the caller's miss_pos).
    hipStream_t ls = ms;
    if (early_lookup && static_cast<hipStream_t>(lookup_stream) != ms) {
        if (!c->write_through) BGL_FAIL(BGL_EINVAL, "early_lookup needs write-through mode");
        ls = static_cast<hipStream_t>(lookup_stream);
    }
    const int32_t *mpos = nullptr;
    int gen = 0;
    // One pass that writes the whole output (k_assemble_rows) instead of a hit gather now and a scatter of
    // the landed miss rows later: when the tier was asked for it, keeps nothing (its packed rows are then
    // in miss order), lands them in device memory, and the cache is in write-through mode.
    const bool assemble = bgl::tier_assemble(t) && bgl::tier_capacity(t) == 0 && c->write_through &&
                          bgl::tier_landing(t, (int)(c->lookup_calls & 1)) != nullptr;
    const int32_t *src_of = nullptr;
    HitList hits;
    rc = lookup_phase(c, ids, n, out_slot, miss_pos, bgl::tier_count_device(t), ms, ls, t, &mpos, &gen, &hits, nullptr, assemble);
    if (rc != BGL_OK) return rc;
    src_of = hits.src_of;
    if ((rc = gather_phase(c, n, out_rows, ms, hits, false)) != BGL_OK) return rc;
    BGL_HIP(hipGetLastError());
    struct Guard {  // whatever goes wrong below, the copy threads are released and the batch is dropped
        bgl_host_tier *t;
        bool armed = true;
        ~Guard() { if (armed) bgl::tier_abort(t); }
    } guard{t};
    // the host continues as soon as the lists are there; the hit gather runs meanwhile
    BGL_HIP(hipEventSynchronize(c->ev_ids));
    bgl_cache::TieredCall &tc = c->tiered;
    rc = bgl::tier_begin(t, n, &tc.plan);
    if (rc != BGL_OK) return rc;
    // (Waking the copy threads earlier, to have them spin until the ids arrive, was measured:
    // slower, the spinning threads get in the way of the wait for the lookup.)
    if (ss != ms) BGL_HIP(hipStreamWaitEvent(ss, c->ev_listed, 0));
    // Rows of whole lines that the tier holds are read in its ring, by a launch that nothing on the host has to
    // wait for.  (An early lookup's rows are packed a batch ahead of the link; there the copies alone keep it busy.)
    tc.in_place = ls == ms && tc.plan.n_hit > 0 && c->row_bytes % 128 == 0 && c->row_bytes / 16 <= kWave;
    if ((tc.in_place ? 0 : tc.plan.n_hit) + tc.plan.n_miss > 0) {
        rc = bgl::tier_copy_start(t, tc.in_place);  // host threads start packing
        if (rc != BGL_OK) return rc;
    }
    if (tc.in_place)
        TieredRows{c, t, &tc.plan, ss, mpos, out_rows, n, (int)(c->insert_calls & 1), false, true, nullptr}.launch_ring();
    BGL_HIP(hipGetLastError());
    guard.armed = false;
    tc.active = true;
    tc.t = t;
    tc.ms = ms;
    tc.ss = ss;
    tc.ls = ls;
    tc.ids = ids;
    tc.mpos = mpos;
    tc.src_of = src_of;
    tc.miss_pos = miss_pos;
    tc.out_rows = out_rows;
    tc.n = n;
    tc.par = (int)(c->insert_calls & 1);  // (the map update of this batch may be enqueued before the second half)
    tc.gen = gen;
    if (c->write_through) {
        c->awaiting_insert = true;
        c->wt_ids = ids;
        c->wt_miss_pos = miss_pos;
    }
    return BGL_OK;
}

// Second half: the packed rows go on their way as the host threads finish them, and the kernels that take
// them to their places are enqueued.  Returns when the last row is packed and everything is enqueued.
int tiered_finish(bgl_cache_t *c, int64_t *n_hit)
{
    bgl_cache::TieredCall &tc = c->tiered;
    bgl_host_tier *t = tc.t;
    tc.active = false;
    struct Guard {
        bgl_host_tier *t;
        bool armed = true;
        ~Guard() { if (armed) bgl::tier_abort(t); }
    } guard{t};
    const bgl::TierPlan &plan = tc.plan;
    const TieredRows rows{c, t, &plan, tc.ss, tc.mpos, tc.out_rows, tc.n, tc.par, tc.ls != tc.ms, tc.in_place, tc.src_of};
    int rc;
    if (rows.staged() + plan.n_miss > 0) {
        char *land = bgl::tier_landing(t, tc.gen);  // device memory the copy engine fills, if that transport is on
        rc = land ? rows_by_copy_engine(rows, land) : rows_by_kernels(rows);
        if (rc != BGL_OK) return rc;
    } else if (tc.src_of && tc.n > 0) {
        rows.launch_assemble_rows(nullptr);  // every id hit: the pass only gathers (no landed row is read)
    }
    BGL_HIP(hipEventRecord(c->ev_miss, tc.ss));
    // the tier's map changes after this call's lists are final and before the next lookup,
    // which runs on the lookup stream
    rc = bgl::tier_enqueue_update(t, tc.ids, tc.miss_pos, tc.ls);
    if (rc != BGL_OK) return rc;
    guard.armed = false;
    BGL_HIP(hipGetLastError());
    c->fetch_pending = true;
    c->fetch_beside = c->rows_split = false;
    c->fetch_stream = tc.ss;
    c->fetch_reads_caller_lists = tc.mpos == tc.miss_pos;
    if (n_hit) {
        n_hit[0] = plan.n_hit_gpu;
        n_hit[1] = plan.n_hit;
    }
    return BGL_OK;
}

}  // namespace

extern "C" int bgl_cache_lookup_gather_tiered(bgl_cache_t *c, bgl_host_tier_t *t, const int32_t *ids,
                                              int64_t n, void *out_rows, int32_t *out_slot,
                                              int32_t *miss_pos, int64_t *n_hit, void *main_stream,
                                              void *side_stream, void *lookup_stream, int early_lookup)
try {
    const int rc = tiered_begin(c, t, ids, n, out_rows, out_slot, miss_pos, main_stream, side_stream, lookup_stream,
                                early_lookup);
    if (rc != BGL_OK) return rc;
    return tiered_finish(c, n_hit);
} BGL_NOTHROW_END

extern "C" int bgl_cache_lookup_tiered_begin(bgl_cache_t *c, bgl_host_tier_t *t, const int32_t *ids, int64_t n,
                                             void *out_rows, int32_t *out_slot, int32_t *miss_pos,
                                             int64_t *n_hit, void *main_stream, void *side_stream,
                                             void *lookup_stream, int early_lookup)
try {
    const int rc = tiered_begin(c, t, ids, n, out_rows, out_slot, miss_pos, main_stream, side_stream, lookup_stream,
                                early_lookup);
    if (rc != BGL_OK) return rc;
    if (n_hit) {  // known already: the lists are on the host
        n_hit[0] = c->tiered.plan.n_hit_gpu;
        n_hit[1] = c->tiered.plan.n_hit;
    }
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_lookup_tiered_finish(bgl_cache_t *c)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (!c->tiered.active) BGL_FAIL(BGL_EINVAL, "no tiered lookup has been begun");
    return tiered_finish(c, nullptr);
} BGL_NOTHROW_END

namespace {

// The event that marks the end of a FIFO update on st for the next lookup (on every stream: that lookup may
// run on another one than this call's lookup did).
hipEvent_t update_event(const bgl_cache *c, hipStream_t st)
{
    const bool local = st != c->last_main || c->last_n * c->row_bytes > LONG_LOOKUP_BYTES;
    return local ? c->ev_map_local : c->ev_map;
}

}  // namespace

void bgl::cache_streaming(bgl_cache *c, bool on) { c->streaming = on; }

extern "C" int bgl_cache_insert_fifo(bgl_cache_t *c, const int32_t *ids, const int32_t *miss_pos,
                                     int64_t n_miss, const void *out_rows, void *stream)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (n_miss < -1 || n_miss > INT32_MAX) BGL_FAIL(BGL_EINVAL, "n_miss out of range");
    const int64_t bound = n_miss >= 0 ? n_miss : c->last_n;  // launch size
    if (bound > 0 && (!ids || !miss_pos || !out_rows))
        BGL_FAIL(BGL_EINVAL, "ids, miss_pos and out_rows must not be null");
    if (!bgl::aligned(out_rows, 16)) BGL_FAIL(BGL_EINVAL, "out_rows is not 16-byte aligned");
    if (c->tiered.active && !c->write_through)
        BGL_FAIL(BGL_EINVAL, "a tiered lookup has been begun: without write-through mode the FIFO update copies "
                             "rows that bgl_cache_lookup_tiered_finish has yet to bring in");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int q = c->row_bytes / 16;
    const int64_t eff = std::min<int64_t>(bound, c->capacity);
    const int par = (int)(c->insert_calls & 1);
    const bool other_stream = st != c->last_main;
    const hipEvent_t done = update_event(c, st);
    const bool own = done == c->ev_map_local && (!other_stream || c->streaming);  // (see launch_marked)
    int rc = BGL_OK;
    auto enqueued = [&]() -> int {
        c->insert_calls += 1;
        if (rc != BGL_OK) return rc;
        BGL_HIP(hipGetLastError());
        c->map_event = done;
        c->map_pending = true;
        c->map_stream = st;
        return BGL_OK;
    };
    if (other_stream && c->ev_listed_valid) BGL_HIP(hipStreamWaitEvent(st, c->ev_listed, 0));  // the lookup's lists
    if (c->write_through) {
        // the rows are already on their way into the buffer: only the map changes here,
        // and nothing has to wait for the miss fetch
        if (!c->awaiting_insert || n_miss != -1 || ids != c->wt_ids || miss_pos != c->wt_miss_pos)
            BGL_FAIL(BGL_EINVAL, "write-through mode: insert_fifo must follow its lookup_gather with the same "
                                 "ids and miss_pos and n_miss = -1");
        c->awaiting_insert = false;
        if (eff > 0) {
            Prof p(c, BGL_STAGE_INSERT_MAP, st);
            rc = launch_marked(c, st, done, own, k_insert_map, dim3((unsigned)bgl::ceil_div(eff, MAP_THREADS)),
                               dim3(MAP_THREADS), ids, miss_pos, n_miss, c->capacity, c->num_nodes, c->table,
                               c->num_buckets - 1, c->slot_to_node, c->slot_to_entry, c->dev, par, 1);
        } else {
            rc = launch_marked(c, st, done, own, k_advance_tail, dim3(1), dim3(64), c->dev, n_miss, par);
        }
        return enqueued();
    }
    const uint64_t call = c->insert_calls + 1;
    const bool timed_parts = timed(c, BGL_STAGE_INSERT_MAP, call) || timed(c, BGL_STAGE_INSERT_ROWS, call);
    if (eff > 0 && c->capacity >= c->num_nodes && !other_stream && !timed_parts) {
        if (c->fetch_pending && c->fetch_stream != st) BGL_HIP(hipStreamWaitEvent(st, misses_event(c), 0));
        const int map_blocks = (int)bgl::ceil_div(eff, MAP_THREADS);
        dispatch_q(q, [&](auto Q) {
            rc = launch_marked(c, st, done, own, k_insert_both<decltype(Q)::value>, dim3(map_blocks + copy_blocks(eff, q)), dim3(COPY_THREADS),
                               ids, miss_pos, n_miss, map_blocks, c->capacity, c->rows, c->num_nodes, c->table, c->num_buckets - 1,
                               c->slot_to_node, c->slot_to_entry, q, reinterpret_cast<const uint4 *>(out_rows),
                               reinterpret_cast<uint4 *>(c->buffer), c->dev, par);
        });
    } else if (eff > 0) {
        {
            Prof p(c, BGL_STAGE_INSERT_MAP, st);
            launch(c, st, k_insert_map, dim3((unsigned)bgl::ceil_div(eff, MAP_THREADS)),
                   dim3(MAP_THREADS), ids, miss_pos, n_miss, c->capacity, c->num_nodes, c->table,
                   c->num_buckets - 1, c->slot_to_node, c->slot_to_entry, c->dev, par, 0);
        }
        if (c->fetch_pending && c->fetch_stream != st)  // rows of the misses (st is behind the hit gather, see above)
            BGL_HIP(hipStreamWaitEvent(st, misses_event(c), 0));
        {
            Prof p(c, BGL_STAGE_INSERT_ROWS, st);
            dispatch_q(q, [&](auto Q) {
                rc = launch_marked(c, st, done, own, k_insert_rows<decltype(Q)::value>, dim3(copy_blocks(eff, q)), dim3(COPY_THREADS),
                                   miss_pos, n_miss, c->capacity, c->rows, q, reinterpret_cast<const uint4 *>(out_rows),
                                   reinterpret_cast<uint4 *>(c->buffer), c->dev, par);
            });
        }
    } else {
        if (c->fetch_pending && c->fetch_stream != st) BGL_HIP(hipStreamWaitEvent(st, misses_event(c), 0));
        rc = launch_marked(c, st, done, own, k_advance_tail, dim3(1), dim3(64), c->dev, n_miss, par);
    }
    if (st == c->last_main) c->rows_joined = true;
    return enqueued();
} BGL_NOTHROW_END

extern "C" int bgl_cache_set_spare_rows(bgl_cache_t *c, int64_t spare_rows)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (spare_rows < 0 || c->capacity + spare_rows > INT32_MAX)
        BGL_FAIL(BGL_EINVAL, "spare_rows must be >= 0 and capacity + spare_rows < 2^31 (got %lld)", (long long)spare_rows);
    if (c->insert_calls != 0 || c->awaiting_insert || c->tiered.active)
        BGL_FAIL(BGL_EINVAL, "the spare rows can only be set before the first insertion");
    BGL_HIP(hipDeviceSynchronize());
    const int64_t rows = c->capacity + spare_rows;
    if (rows == c->rows) return BGL_OK;
    char *buf = nullptr;
    const hipError_t e = hipMalloc((void **)&buf, (size_t)rows * c->row_bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        bgl::set_error("hipMalloc of %zu bytes failed: %s", (size_t)rows * c->row_bytes, hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? BGL_ENOMEM : BGL_EHIP;
    }
    if (hipMemset(buf, 0, (size_t)rows * c->row_bytes) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        (void)hipFree(buf);
        BGL_FAIL(BGL_EHIP, "clearing the cache buffer failed: %s", hipGetErrorString(hipGetLastError()));
    }
    (void)hipFree(c->buffer);
    c->buffer = buf;
    c->rows = rows;
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_set_write_through(bgl_cache_t *c, int enable)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (c->awaiting_insert) BGL_FAIL(BGL_EINVAL, "a lookup's misses are still waiting for their insert_fifo");
    if (c->tiered.active) BGL_FAIL(BGL_EINVAL, "a tiered lookup has been begun: bgl_cache_lookup_tiered_finish comes first");
    c->write_through = enable != 0;
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_wait_rows(bgl_cache_t *c, void *stream)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    hipStream_t st = static_cast<hipStream_t>(stream);
    // (a FIFO update that copies rows has made the main stream wait for them already: a wait costs the host 10 us)
    if (c->rows_joined && st == c->last_main) return BGL_OK;
    return join_rows(c, st);
} BGL_NOTHROW_END

extern "C" int bgl_cache_wait_lists(bgl_cache_t *c, void *stream)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (c->ev_listed_valid && st != c->last_main)
        BGL_HIP(hipStreamWaitEvent(st, c->ev_listed, 0));
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_export_state(bgl_cache_t *c, int32_t *slot_to_node, uint64_t *tail,
                                      void *buffer)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    BGL_HIP(hipDeviceSynchronize());
    if (slot_to_node)
        BGL_HIP(hipMemcpy(slot_to_node, c->slot_to_node, sizeof(int32_t) * (size_t)c->capacity,
                          hipMemcpyDeviceToHost));
    if (tail) {
        CacheDev h;
        BGL_HIP(hipMemcpy(&h, c->dev, sizeof(h), hipMemcpyDeviceToHost));
        *tail = h.tail[c->insert_calls & 1];
    }
    if (buffer) {
        // rows by slot: the live rows are the last min(tail, capacity) insertions, insertion k sits at
        // position k mod rows and belongs to slot k mod capacity; runs of consecutive insertions are
        // copied whole (they break where either number wraps), empty slots read as zeros
        CacheDev h;
        BGL_HIP(hipMemcpy(&h, c->dev, sizeof(h), hipMemcpyDeviceToHost));
        const uint64_t t = h.tail[c->insert_calls & 1];
        const uint64_t cap = (uint64_t)c->capacity, rows = (uint64_t)c->rows, rb = (uint64_t)c->row_bytes;
        const uint64_t live = std::min<uint64_t>(t, cap);
        char *dst = static_cast<char *>(buffer);
        if (live < cap) std::memset(dst + live * rb, 0, (size_t)((cap - live) * rb));  // (then t < capacity: slots 0 .. t-1 are live)
        for (uint64_t k = t - live; k < t;) {
            const uint64_t slot = k % cap, pos = k % rows;
            const uint64_t run = std::min<uint64_t>(std::min<uint64_t>(cap - slot, rows - pos), t - k);
            BGL_HIP(hipMemcpy(dst + slot * rb, c->buffer + pos * rb, (size_t)(run * rb), hipMemcpyDeviceToHost));
            k += run;
        }
    }
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_stats(bgl_cache_t *c, uint64_t *lookups, uint64_t *hits, uint64_t *inserts,
                               uint64_t *evictions, int32_t *status)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    BGL_HIP(hipDeviceSynchronize());
    CacheDev h;
    BGL_HIP(hipMemcpy(&h, c->dev, sizeof(h), hipMemcpyDeviceToHost));
    if (lookups) *lookups = h.lookups;
    if (hits) *hits = h.hits;
    const uint64_t tail = h.tail[c->insert_calls & 1];
    if (inserts) *inserts = tail;  // every insertion advances tail by one
    // every insertion beyond the first `capacity` ones overwrote an occupied slot
    if (evictions) *evictions = tail > (uint64_t)c->capacity ? tail - (uint64_t)c->capacity : 0;
    if (status) *status = h.status;
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_map_stats(bgl_cache_t *c, uint64_t *ids_looked_up, uint64_t *bucket_lines_read,
                                   uint64_t *num_buckets, uint64_t *buckets_passed, uint64_t *passes)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    BGL_HIP(hipDeviceSynchronize());
    CacheDev h;
    if (buckets_passed || passes) {
        BGL_HIP(hipMemset(&c->dev->census[0], 0, sizeof(h.census)));
        hipLaunchKernelGGL(k_map_census, dim3(256), dim3(256), 0, 0, c->table, c->num_buckets, c->dev);
        BGL_HIP(hipGetLastError());
        BGL_HIP(hipDeviceSynchronize());
    }
    BGL_HIP(hipMemcpy(&h, c->dev, sizeof(h), hipMemcpyDeviceToHost));
    if (ids_looked_up) *ids_looked_up = h.lookups;
    if (bucket_lines_read) *bucket_lines_read = h.probe_lines;
    if (num_buckets) *num_buckets = c->num_buckets;
    if (buckets_passed) *buckets_passed = h.census[0];
    if (passes) *passes = h.census[1];
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_set_profiling(bgl_cache_t *c, int enable)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    BGL_HIP(hipDeviceSynchronize());
    if (enable && c->prof_ev.empty()) {
        c->prof_ev.resize(2 * PROF_RING, nullptr);
        for (auto &ev : c->prof_ev) BGL_HIP(hipEventCreate(&ev));
    }
    c->prof_rec.clear();
    c->prof_rec.reserve(PROF_RING);
    c->prof_dropped = 0;
    for (int s = 0; s < BGL_NUM_STAGES; ++s) { c->prof_ms[s] = 0; c->prof_n[s] = 0; }
    c->profiling = (unsigned)enable;
    if (enable) {
        // What an event pair reads for a kernel that does nothing:
        // the launch gap that every bracketed stage time includes.
        double sum = 0;
        const int reps = 16;
        for (int r = 0; r < reps + 2; ++r) {
            BGL_HIP(hipEventRecord(c->prof_ev[0], 0));
            hipLaunchKernelGGL(k_noop, dim3(1), dim3(64), 0, 0);
            BGL_HIP(hipEventRecord(c->prof_ev[1], 0));
            BGL_HIP(hipEventSynchronize(c->prof_ev[1]));
            float ms = 0.f;
            BGL_HIP(hipEventElapsedTime(&ms, c->prof_ev[0], c->prof_ev[1]));
            if (r >= 2) sum += ms;
        }
        c->prof_overhead_ms = sum / reps;
    }
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_set_profiling_every(bgl_cache_t *c, int stage, int every)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (stage < 0 || stage >= BGL_NUM_STAGES) BGL_FAIL(BGL_EINVAL, "unknown stage %d", stage);
    if (every < 1) BGL_FAIL(BGL_EINVAL, "every must be >= 1 (got %d)", every);
    c->prof_every[stage] = every;
    return BGL_OK;
} BGL_NOTHROW_END

extern "C" int bgl_cache_profile(bgl_cache_t *c, int stage, double *total_ms, int64_t *launches)
try {
    if (!c) BGL_FAIL(BGL_EINVAL, "cache handle is null");
    if (stage == BGL_STAGE_EVENT_OVERHEAD) {
        if (total_ms) *total_ms = c->prof_overhead_ms;
        if (launches) *launches = 1;
        return BGL_OK;
    }
    if (stage < 0 || stage >= BGL_NUM_STAGES) BGL_FAIL(BGL_EINVAL, "unknown stage %d", stage);
    BGL_HIP(hipDeviceSynchronize());
    drain_profile(c);
    if (c->prof_dropped > 0)
        BGL_FAIL(BGL_ENOMEM, "%lld timed launches could not get events; the stage totals are incomplete",
                 (long long)c->prof_dropped);
    if (total_ms) *total_ms = c->prof_ms[stage];
    if (launches) *launches = c->prof_n[stage];
    return BGL_OK;
} BGL_NOTHROW_END
