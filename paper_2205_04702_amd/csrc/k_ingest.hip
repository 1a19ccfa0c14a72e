// Window ingest: a batch that becomes visible to the planner is turned into
// sorted (table,row) keys, its unique keys, the inverse map and the runs of
// equal keys that the backward pass coalesces (gradient duplication and
// coalescing, Sec. II-B).  Everything here runs once per batch, when the batch
// enters the look-forward window.
#include <algorithm>

#include "sp_device.h"
#include "sp_internal.h"

namespace sp {

// ---------------------------------------------------------------- small fills

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

void launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s,
                       p, n, v);
}

void launch_zero_i32(int32_t *p, int64_t n, hipStream_t s) { launch_fill_i32(p, n, 0, s); }

// ---------------------------------------------------------------- bags

// Bag bookkeeping of a batch.  One wave takes 64 consecutive bags, lane i
// their i-th: it validates the offsets (non-decreasing, from 0 to nnz;
// ERR_OFFSETS otherwise, ranges clamped into [0, nnz)), copies them into the
// window ring (when they are read from the caller's device memory) and checks
// each table's ID count against max_table_ids (when set, ERR_TABLE_IDS); then
// the wave walks the positions its bags cover, 64 at a time, and writes
// bag_of for them, each lane finding its position's bag among the 64 offsets
// by a search over the lanes.  Stores are whole 256-byte lines; one thread per
// bag writing its positions one by one took 0.24 ms alone (0.9 ms beside the
// training kernels) for 21M IDs.  Where few bags hold many IDs, `parts` waves
// share the positions of the 64 bags (wave `part` takes every parts-th 64 of
// them, wave 0 validates and copies): bag_parts.
__device__ __forceinline__ void mark_bags(int64_t first, int part, int parts, const int32_t *bag_off,
                                          int32_t *bag_off_copy, int32_t B, int64_t nnz,
                                          int64_t nbags, int64_t max_table_ids, int32_t *bag_of,
                                          int32_t *err)
{
    const int lane = lane_id();
    const int64_t g = first + lane;
    const bool in = g < nbags;
    const int64_t gc = in ? g : nbags - 1;
    int64_t lo = bag_off[gc], hi = bag_off[gc + 1];
    int32_t bad = 0;
    if (in && part == 0) {
        if (bag_off_copy != bag_off) {
            bag_off_copy[g] = (int32_t)lo;
            if (g == nbags - 1) bag_off_copy[g + 1] = (int32_t)hi;
        }
        if (lo > hi || lo < 0 || hi > nnz || (g == 0 && lo != 0) || (g == nbags - 1 && hi != nnz))
            bad |= ERR_OFFSETS;
        if (max_table_ids > 0 && g % B == 0 && (int64_t)bag_off[g + B] - lo > max_table_ids)
            bad |= ERR_TABLE_IDS;
    }
    if (bad) atomicOr(err, bad);
    lo = lo < 0 ? 0 : (lo > nnz ? nnz : lo);
    hi = hi < 0 ? 0 : (hi > nnz ? nnz : hi);
    if (part == 0 && __ballot(in && hi - lo > FWD_LONG) && lane == 0 &&
        !(__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & BATCH_LONG_BAG))
        atomicOr(err, BATCH_LONG_BAG);
    if (!in) lo = hi;  // lanes past the last bag start where it ends
    const int32_t lo32 = (int32_t)lo;
    const int64_t p0 = __shfl(lo32, 0, WAVE), p1 = __shfl((int32_t)hi, WAVE - 1, WAVE);
    for (int64_t base = p0 + part * WAVE; base < p1; base += (int64_t)parts * WAVE) {
        const int32_t p = (int32_t)(base + lane);
        int k = 0;  // the last of the 64 bags that starts at or before p
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) {
            const int32_t x = __shfl(lo32, k + o, WAVE);
            if (x <= p) k += o;
        }
        const int64_t bag = first + k < nbags ? first + k : nbags - 1;
        if (p < p1) bag_of[p] = (int32_t)bag;
    }
}

__global__ void __launch_bounds__(BLOCK) k_bags(const int32_t *bag_off, int32_t *bag_off_copy,
                                                int32_t B, int64_t nnz, int64_t nbags,
                                                int64_t max_table_ids, int32_t *bag_of,
                                                int32_t *err)
{
    const int64_t first = ((int64_t)blockIdx.x * (BLOCK / WAVE) + wave_id()) * WAVE;
    if (first < nbags)
        mark_bags(first, 0, 1, bag_off, bag_off_copy, B, nnz, nbags, max_table_ids, bag_of, err);
}

// Waves per 64 bags: a wave's walk is a chain of some 0.3 us per 64 positions,
// so it is cut to about BAG_STEPS steps for bags of the mean length, unless the
// waves fill the chip as it is.  An ingest of 64 bags of 2000 IDs takes 0.60 ms
// with one wave for them, 0.066 cut to 32 steps, 0.060 to 8 and 0.060 to 2;
// 4096 bags of 300 IDs 0.20, 0.126, 0.126 and 0.123; 106k bags of 40 IDs 0.317
// each way.
constexpr int64_t BAG_STEPS = 8, BAG_WAVES = 4096;
static int bag_parts(int64_t nnz, int64_t nbags)
{
    const int64_t waves = (nbags + WAVE - 1) / WAVE;
    const int64_t steps = (nnz + waves * WAVE - 1) / (waves * WAVE);
    const int64_t parts = std::min((steps + BAG_STEPS - 1) / BAG_STEPS, (BAG_WAVES + waves - 1) / waves);
    return (int)std::max<int64_t>(parts, 1);
}

// ---------------------------------------------------------------- general path: segmented sort
//
// A batch arrives table by table, so its keys (table << row_bits | row) only
// have to be put in order within each table: a stable LSD radix sort of every
// table's IDs by the bits its row count needs, all tables in the same
// launches.  Table t takes ceil(bits / SORT_BITS) passes of equal digits; the
// tables that need fewer passes join at a later launch, so all of them end in
// the same buffer.  A table's first pass reads the caller's IDs themselves
// (validated: rows out of range raise ERR_ID_RANGE and become row 0), later
// ones 64-bit entries key << 32 | position.  A pass is two launches over tiles
// of each table's span:
//  * k_sort_hist: digit counts of every tile and of every group of G tiles
//    (one block per group);
//  * k_sort_scatter: one block per tile.  It adds up its digit's group counts
//    and the tile counts of its own group (no scan in between: a thread adds
//    its table's groups and up to G tiles, sort_group), ranks its
//    entries with wave ballots, puts them in digit order in LDS and writes
//    each digit's entries as one run.
// What bounds it: HBM traffic, 8 bytes read and written per entry and pass
// plus 8 for the counts: alone a pass takes 0.05 + 0.10 ms for 21M IDs and
// 0.02 + 0.03 ms for 4.3M.  Before (11-bit digits of the whole key, entries
// scattered one by one to 2048 bins, a scan launch per pass) 21M IDs took 3
// passes of 0.43 ms, 4.3M IDs 2 of 0.38 ms.
constexpr int SORT_BITS = 9;
constexpr int SORT_BINS = 1 << SORT_BITS;

// Spans, tiles and groups of the tables of a batch, from its offsets, by one
// wave (lane t: table t) into LDS.  Offsets that go back or leave [0, nnz] (an
// error raised by mark_bags) give disjoint spans inside it all the same.
struct SortLay {
    int32_t beg[MAX_TABLES + 1], tile0[MAX_TABLES + 1], group0[MAX_TABLES + 1];
};
static_assert(MAX_TABLES == WAVE, "one table per lane");
__device__ __forceinline__ void sort_layout(SortLay &l, const int32_t *bag_off, int32_t T,
                                            int32_t B, int64_t nnz, int tile_len, int G)
{
    const int lane = lane_id();
    int64_t end = lane < T ? bag_off[(int64_t)(lane + 1) * B] : 0;
    end = end < 0 ? 0 : (end > nnz ? nnz : end);
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const int32_t x = __shfl_up((int32_t)end, o, WAVE);
        if (lane >= o && x > end) end = x;
    }
    int32_t prev = __shfl_up((int32_t)end, 1, WAVE);
    if (lane == 0) prev = 0;
    const int32_t tiles = (int32_t)((end - prev + tile_len - 1) / tile_len);
    const int32_t ti = wave_incl_scan(tiles), gi = wave_incl_scan((tiles + G - 1) / G);
    l.beg[lane + 1] = (int32_t)end;
    l.tile0[lane + 1] = ti;
    l.group0[lane + 1] = gi;
    if (lane == 0) l.beg[0] = l.tile0[0] = l.group0[0] = 0;
}
// The table whose tiles (or groups) hold index i: the number of tables that end at or
// before it.  first: the array's first of MAX_TABLES + 1 entries.
__device__ __forceinline__ int sort_table(const int32_t *first, int64_t i)
{
    return __popcll(__ballot((int64_t)first[lane_id() + 1] <= i));
}

// The digit of table t in launch q of `passes`: false when the table starts
// later.  first: this launch is the table's first.
__device__ __forceinline__ bool sort_digit(int64_t rows, int q, int passes, int &shift, int &dbits,
                                           bool &first)
{
    const int bits = rows > 2 ? 64 - __clzll((unsigned long long)(rows - 1)) : 1;
    const int np = (bits + SORT_BITS - 1) / SORT_BITS;
    const int p = q - (passes - np);
    dbits = (bits + np - 1) / np;
    shift = p * dbits;
    first = p == 0;
    return p >= 0;
}

// ITEMS entries of a table, at(r) clamped into its span by the caller: its IDs
// as entries, or what an earlier pass left.  No branch around a load, so all
// are in flight together.
template <int ITEMS, class At>
__device__ __forceinline__ void sort_entries(uint64_t (&e)[ITEMS], bool first, const int32_t *ids,
                                             const uint64_t *in, int t, int row_bits, int64_t rows,
                                             At at, bool &bad)
{
    if (first) {  // uniform over the block
        int32_t row[ITEMS];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) row[r] = ids[at(r)];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const bool out = row[r] < 0 || (int64_t)row[r] >= rows;
            bad |= out;
            const uint32_t key = ((uint32_t)t << row_bits) | (uint32_t)(out ? 0 : row[r]);
            e[r] = (uint64_t)key << 32 | (uint64_t)(uint32_t)at(r);
        }
    } else {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) e[r] = in[at(r)];
    }
}

// NT * ITEMS entries per tile.  Blocks past `groups` of the first launch mark
// the bags instead, `parts` waves each 64.
template <int NT, int ITEMS>
__global__ void __launch_bounds__(NT) k_sort_hist(Tables tb, const int32_t *ids,
                                                  const int32_t *bag_off, int32_t *bag_off_copy,
                                                  int32_t B, int64_t nnz, int64_t nbags,
                                                  int64_t max_table_ids, int32_t *bag_of,
                                                  int32_t parts, int32_t groups,
                                                  const uint64_t *in, int q,
                                                  int passes, int G, uint32_t *thist,
                                                  uint32_t *ghist, int32_t *err)
{
    constexpr int TILE = NT * ITEMS;
    constexpr int PER = (SORT_BINS + NT - 1) / NT;
    __shared__ SortLay lay;
    __shared__ uint32_t h[SORT_BINS];
    __shared__ int32_t t_s;
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= groups) {
        const int64_t u = (int64_t)(blockIdx.x - groups) * (NT / WAVE) + wave_id();
        const int64_t first = u / parts * WAVE;
        if (first < nbags)
            mark_bags(first, (int)(u % parts), parts, bag_off, bag_off_copy, B, nnz, nbags,
                      max_table_ids, bag_of, err);
        return;
    }
    // consecutive groups (one table's) on one XCD, as in the scatter
    const int64_t gr = xcd_block(blockIdx.x, groups);
    if (tid < WAVE) {
        sort_layout(lay, bag_off, tb.T, B, nnz, TILE, G);
        const int t = sort_table(lay.group0, gr);
        if (tid == 0) t_s = t;
    }
    for (int d = tid; d < SORT_BINS; d += NT) h[d] = 0;
    __syncthreads();
    const int t = t_s;
    if (t >= tb.T) return;  // past the last group (uniform)
    const int64_t rows = tb.rows[t];
    int shift, dbits;
    bool first, bad = false;
    if (!sort_digit(rows, q, passes, shift, dbits, first)) return;
    const int bins = 1 << dbits;
    const uint32_t mask = (uint32_t)bins - 1u;
    const int64_t end = lay.beg[t + 1];
    const int tile_a = lay.tile0[t] + (int)(gr - lay.group0[t]) * G;
    const int tile_b = tile_a + G < lay.tile0[t + 1] ? tile_a + G : lay.tile0[t + 1];
    uint32_t sum[PER] = {};
    for (int tile = tile_a; tile < tile_b; ++tile) {
        const int64_t base = (int64_t)lay.beg[t] + (int64_t)(tile - lay.tile0[t]) * TILE;
        uint64_t e[ITEMS];
        sort_entries(e, first, ids, in, t, tb.row_bits, rows,
                     [&](int r) {
                         const int64_t i = base + r * NT + tid;
                         return i < end ? i : end - 1;
                     },
                     bad);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (base + r * NT + tid < end)
                atomicAdd(&h[(uint32_t)(e[r] >> (32 + shift)) & mask], 1u);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int d = k * NT + tid;
            if (d < bins) {
                const uint32_t c = h[d];
                thist[(int64_t)tile * SORT_BINS + d] = c;
                sum[k] += c;
                h[d] = 0;
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = k * NT + tid;
        if (d < bins) ghist[gr * SORT_BINS + d] = sum[k];
    }
    if (bad) atomicOr(err, ERR_ID_RANGE);
}

template <int NT, int ITEMS>
__global__ void __launch_bounds__(NT) k_sort_scatter(Tables tb, const int32_t *ids,
                                                     const int32_t *bag_off, int32_t B,
                                                     int64_t nnz, const uint64_t *in,
                                                     uint64_t *out, int q, int passes, int G,
                                                     const uint32_t *thist, const uint32_t *ghist)
{
    constexpr int TILE = NT * ITEMS;
    constexpr int NW = NT / WAVE;
    constexpr int PER = (SORT_BINS + NT - 1) / NT;
    __shared__ SortLay lay;
    __shared__ uint64_t buf[TILE];
    __shared__ uint32_t wc[NW][SORT_BINS];
    __shared__ uint32_t to[SORT_BINS];  // digit's output index less its place in the tile
    __shared__ uint64_t lds[NW];
    __shared__ int32_t t_s;
    const int tid = threadIdx.x, w = wave_id(), lane = lane_id();
    // consecutive tiles (one table's) on one XCD: the runs that neighbouring
    // tiles write to one digit share its L2
    const int64_t tile = xcd_block(blockIdx.x, gridDim.x);
    if (tid < WAVE) {
        sort_layout(lay, bag_off, tb.T, B, nnz, TILE, G);
        const int t = sort_table(lay.tile0, tile);
        if (tid == 0) t_s = t;
    }
    for (int i = tid; i < NW * SORT_BINS; i += NT) (&wc[0][0])[i] = 0;
    __syncthreads();
    const int t = t_s;
    if (t >= tb.T) return;  // past the last tile (uniform)
    const int64_t rows = tb.rows[t];
    int shift, dbits;
    bool first, bad = false;
    if (!sort_digit(rows, q, passes, shift, dbits, first)) return;
    const int bins = 1 << dbits;
    const uint32_t mask = (uint32_t)bins - 1u;
    const int64_t beg = lay.beg[t], end = lay.beg[t + 1];
    const int64_t base = beg + (tile - lay.tile0[t]) * TILE;
    const int n = (int)(end - base < TILE ? end - base : TILE);
    // wave w holds its own contiguous share of the tile, 64 entries at a time
    uint64_t e[ITEMS];
    sort_entries(e, first, ids, in, t, tb.row_bits, rows,
                 [&](int r) {
                     const int i = w * (ITEMS * WAVE) + r * WAVE + lane;
                     return base + (i < n ? i : n - 1);
                 },
                 bad);
    // thread tid owns digits tid * PER ..: the table's entries of each digit,
    // and those in tiles before this one
    uint32_t total[PER] = {}, before[PER] = {};
    {
        const int g0 = lay.group0[t], g1 = lay.group0[t + 1];
        const int lt = (int)(tile - lay.tile0[t]);
        const int mine = g0 + lt / G;
        const int d0 = tid * PER;
        if (d0 < bins) {
#pragma unroll 8
            for (int g = g0; g < g1; ++g)
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const uint32_t x = ghist[(int64_t)g * SORT_BINS + d0 + k];
                    total[k] += x;
                    before[k] += g < mine ? x : 0u;
                }
#pragma unroll 8
            for (int64_t u = tile - lt % G; u < tile; ++u)
#pragma unroll
                for (int k = 0; k < PER; ++k) before[k] += thist[u * SORT_BINS + d0 + k];
        }
    }
    // rank of each entry among the wave's entries with its digit
    const uint64_t lt_mask = lanemask_lt();
    uint32_t rk[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = w * (ITEMS * WAVE) + r * WAVE + lane;
        const bool valid = i < n;
        const uint32_t d = (uint32_t)(e[r] >> (32 + shift)) & mask;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < dbits; ++b) {
            const uint32_t bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const int leader = valid ? __ffsll((unsigned long long)peers) - 1 : lane;
        uint32_t prior = 0;
        if (valid && leader == lane) {
            prior = wc[w][d];
            wc[w][d] = prior + (uint32_t)__popcll(peers);
        }
        prior = __shfl(prior, leader, WAVE);
        rk[r] = prior + (uint32_t)__popcll(peers & lt_mask);
    }
    __syncthreads();
    // digits: where each starts in the table and in the tile, in one scan
    uint32_t cnt[PER], tsum = 0, csum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = tid * PER + k;
        cnt[k] = 0;
        if (d < bins)
            for (int x = 0; x < NW; ++x) cnt[k] += wc[x][d];
        else
            total[k] = 0;
        tsum += total[k];
        csum += cnt[k];
    }
    uint64_t all;
    uint64_t ex = block_excl_scan_n<NT, uint64_t>((uint64_t)tsum << 32 | csum, lds, all);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = tid * PER + k;
        if (d < bins) {
            uint32_t run = (uint32_t)ex;
            to[d] = (uint32_t)beg + (uint32_t)(ex >> 32) + before[k] - run;
            for (int x = 0; x < NW; ++x) {
                const uint32_t c = wc[x][d];
                wc[x][d] = run;
                run += c;
            }
        }
        ex += (uint64_t)total[k] << 32 | cnt[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = w * (ITEMS * WAVE) + r * WAVE + lane;
        if (i < n) {
            const uint32_t d = (uint32_t)(e[r] >> (32 + shift)) & mask;
            const uint32_t p = wc[w][d] + rk[r];
            buf[p < (uint32_t)n ? p : (uint32_t)(n - 1)] = e[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = r * NT + tid;
        if (i < n) {
            const uint64_t x = buf[i];
            const uint32_t p = to[(uint32_t)(x >> (32 + shift)) & mask] + (uint32_t)i;
            // never write past the batch, whatever the counts say
            out[p < (uint64_t)nnz ? p : (uint64_t)(nnz - 1)] = x;
        }
    }
}

// ---------------------------------------------------------------- general path: runs
//
// The sorted entries fall into runs of equal keys.  k_runs<false> counts, per
// tile of the batch, the runs and the backward chunks (BWD_CHUNK positions of
// one run at most) that start in it and the runs longer than one chunk; its
// last block to finish turns the counts into prefixes and writes the batch's
// totals and error bits.  k_runs<true> finds the same starts again and writes
// everything at its place: unique keys, chunk descriptors, and
// per sorted entry the bag (sbag) and the run of its position (inv).  The
// second reading of the entries (8 bytes each) buys tiles that need no order
// among them, so consecutive tiles stay on one XCD and the scattered stores of
// inv, which stay within a table's span, meet in its L2: 0.10 + 0.38 ms for
// 21M IDs, 0.04 + 0.07 ms for 4.3M (42M scattered 4-byte accesses in L2 bound
// the second).  Before, two single-pass scans did this in 0.9 + 1.2 ms for 21M IDs and 0.22 + 0.70 ms
// for 4.3M: the stores of a line came from all XCDs, every descriptor was
// stored by a serial loop, and every long run took an atomic on one address.
constexpr uint32_t KEY_PAST = 0xFFFFFFFFu;  // after the last entry (keys are below 2^31)

// First index of [0, i] whose run reaches i (sorted keys, i > 0), by one wave:
// steps of 64 times the last one, then back down.
__device__ __forceinline__ int64_t run_start(const uint64_t *e, int64_t i, uint32_t key)
{
    const int lane = lane_id();
    int64_t step = 1;
    // in all indices from `hi` to i the key is the run's
    int64_t hi = i;
    while (true) {
        const int64_t p = hi - (int64_t)(lane + 1) * step;
        const bool same = p >= 0 && (uint32_t)(e[p >= 0 ? p : 0] >> 32) == key;
        const uint64_t bal = __ballot(same);
        const int k = bal == ~0ull ? WAVE : __ffsll((unsigned long long)~bal) - 1;
        hi -= (int64_t)k * step;  // the last probed index that still has the key
        if (k == WAVE) {
            step *= WAVE;
        } else if (step > 1) {
            step /= WAVE;
        } else {
            return hi;
        }
    }
}

// LDS place of index i: threads own eight consecutive entries each, and one
// word of padding per eight puts their accesses on different banks.
constexpr __host__ __device__ int run_lds(int i) { return i + (i >> 3); }

template <int NT, int ITEMS, bool EMIT>
__global__ void __launch_bounds__(NT) k_runs(const uint64_t *e, const int32_t *bag_off, int32_t T,
                                             int32_t B, int64_t nnz, const int32_t *bag_of,
                                             BatchDev b, int64_t n_multi_cap, uint64_t *tcount,
                                             int4 *tpre, int32_t tiles, int32_t *arrived,
                                             int32_t *err)
{
    constexpr int TILE = NT * ITEMS;
    constexpr int HALO = BWD_CHUNK;
    __shared__ uint32_t key[run_lds(1 + TILE + HALO)];  // at run_lds(1 + i): entry i of the tile
    __shared__ uint32_t pos[EMIT ? TILE : 1], seg[EMIT ? run_lds(TILE) : 1];
    __shared__ uint64_t lds[NT / WAVE];
    __shared__ int32_t ldsm[NT / WAVE];
    __shared__ int64_t start_s;
    __shared__ int64_t total_s;
    __shared__ int32_t last_s;
    const int tid = threadIdx.x;
    const int64_t tile = xcd_block(blockIdx.x, tiles);
    const int64_t base = tile * TILE;
    if (tid < WAVE) {  // entries there are: the largest table end (offsets may be malformed)
        int64_t end = tid < T ? bag_off[(int64_t)(tid + 1) * B] : 0;
        end = end < 0 ? 0 : (end > nnz ? nnz : end);
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const int32_t x = __shfl_xor((int32_t)end, o, WAVE);
            if (x > end) end = x;
        }
        if (tid == 0) total_s = end;
    }
    __syncthreads();
    const int64_t total = total_s;
    const int n = (int)(total - base < 0 ? 0 : (total - base < TILE ? total - base : TILE));
    {
        // the tile's entries, the one before it and HALO after, all in flight
        // together (indices clamped, values past the last entry replaced)
        auto entry = [&](int64_t g) {
            const uint64_t x = __builtin_nontemporal_load(
                &e[g < 0 ? 0 : (g < total ? g : (total > 0 ? total - 1 : 0))]);
            return g >= 0 && g < total ? x : (uint64_t)KEY_PAST << 32;
        };
        uint64_t x[ITEMS];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) x[r] = entry(base + r * NT + tid);
        const int hi = tid == 0 ? 0 : TILE + tid;  // entry before the tile, then the halo
        const uint64_t y = entry(base + hi - 1);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            key[run_lds(1 + r * NT + tid)] = (uint32_t)(x[r] >> 32);
            if (EMIT) pos[r * NT + tid] = (uint32_t)x[r];
        }
        if (tid <= HALO) key[run_lds(hi)] = (uint32_t)(y >> 32);
    }
    __syncthreads();
    if (tid < WAVE) {  // where the run that reaches into the tile starts
        int64_t s = base;
        if (n > 0 && base > 0 && key[run_lds(0)] == key[run_lds(1)]) s = run_start(e, base, key[run_lds(1)]);
        if (tid == 0) start_s = s;
    }
    // thread tid owns entries tid * ITEMS ..
    uint32_t heads = 0;
    int32_t last_head = -1;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = tid * ITEMS + k;
        if (i < n && (base + i == 0 || key[run_lds(i)] != key[run_lds(1 + i)])) {
            heads |= 1u << k;
            last_head = i;
        }
    }
    // the last head before this thread's entries
    int32_t incl = last_head;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const int32_t x = __shfl_up(incl, o, WAVE);
        if (lane_id() >= o && x > incl) incl = x;
    }
    if (lane_id() == WAVE - 1) ldsm[wave_id()] = incl;
    __syncthreads();
    int32_t prev = __shfl_up(incl, 1, WAVE);
    if (lane_id() == 0) prev = -1;
    for (int x = 0; x < wave_id(); ++x) prev = ldsm[x] > prev ? ldsm[x] : prev;
    int64_t run0 = prev >= 0 ? base + prev : start_s;
    uint32_t starts = 0, longs = 0;  // chunk starts; heads of runs longer than a chunk
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = tid * ITEMS + k;
        if (i >= n) continue;
        const bool head = (heads >> k) & 1u;
        if (head) run0 = base + i;
        if ((base + i - run0) % BWD_CHUNK == 0) starts |= 1u << k;
        if (head && key[run_lds(1 + i + BWD_CHUNK)] == key[run_lds(1 + i)]) longs |= 1u << k;
    }
    // three counts below 2^13 in one word
    static_assert(TILE <= 4096, "counts of a tile take 20 bits each");
    const uint64_t mine = (uint64_t)__popc(heads) | (uint64_t)__popc(starts) << 20 |
                          (uint64_t)__popc(longs) << 40;
    uint64_t all;
    const uint64_t ex = block_excl_scan_n<NT, uint64_t>(mine, lds, all);
    constexpr uint64_t M20 = (1ull << 20) - 1;
    if (!EMIT) {
        if (tid == 0) {
            // the old value is tested before the arrival below, so the word is
            // in memory by then (cleared words never read all ones)
            const uint64_t old = atomicExch((unsigned long long *)&tcount[tile], all);
            last_s = atomicAdd(arrived, old == ~0ull ? 2 : 1) == tiles - 1;
        }
        __syncthreads();
        if (!last_s) return;  // uniform per block
        // ---- the last block: exclusive prefixes of the tiles, batch totals
        const int per = (tiles + NT - 1) / NT;
        const int a = tid * per, z = a + per < tiles ? a + per : tiles;
        uint32_t u = 0, c = 0, m = 0;
#pragma unroll 4
        for (int x = a; x < z; ++x) {
            const uint64_t v = __hip_atomic_load(&tcount[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            u += (uint32_t)(v & M20);
            c += (uint32_t)(v >> 20 & M20);
            m += (uint32_t)(v >> 40);
        }
        uint64_t tot_uc, tot_m;
        const uint64_t uc = block_excl_scan_n<NT, uint64_t>((uint64_t)c << 32 | u, lds, tot_uc);
        uint32_t m0 = (uint32_t)block_excl_scan_n<NT, uint64_t>((uint64_t)m, lds, tot_m);
        uint32_t u0 = (uint32_t)uc, c0 = (uint32_t)(uc >> 32);
#pragma unroll 4
        for (int x = a; x < z; ++x) {
            const uint64_t v = __hip_atomic_load(&tcount[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            tpre[x] = make_int4((int)u0, (int)c0, (int)m0, 0);
            u0 += (uint32_t)(v & M20);
            c0 += (uint32_t)(v >> 20 & M20);
            m0 += (uint32_t)(v >> 40);
        }
        if (tid == 0) {
            const int32_t U = (int32_t)(uint32_t)tot_uc, C = (int32_t)(tot_uc >> 32);
            b.scal[0] = U;
            b.scal[1] = C;
            const int32_t found = atomicExch(err, 0);
            b.scal[2] = found & ~BATCH_LONG_BAG;
            b.scal[3] = (int32_t)tot_m;
            b.scal[4] = (found & BATCH_LONG_BAG) != 0;
            b.seg_chunk0[U] = C;
            __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }
    if (n == 0) return;  // uniform per block
    const int4 pre = tpre[tile];
    int32_t u = pre.x + (int32_t)(ex & M20);   // runs that started before this thread's entries
    int32_t c = pre.y + (int32_t)(ex >> 20 & M20);
    int32_t m = pre.z + (int32_t)(ex >> 40);
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = tid * ITEMS + k;
        if (i >= n) continue;
        const bool head = (heads >> k) & 1u, lng = (longs >> k) & 1u;
        const uint32_t kk = key[run_lds(1 + i)];
        if (head) {
            b.ukeys[u] = kk;
            b.seg_chunk0[u] = c;
            if (lng && m < n_multi_cap) b.multi[m] = u;
            m += lng;
            ++u;
        }
        seg[run_lds(i)] = (uint32_t)(u - 1);
        if ((starts >> k) & 1u) {
            int len = 1;  // of the chunk: the keys are sorted, so equal ends mean equal all through
#pragma unroll
            for (int o = BWD_CHUNK / 2; o > 0; o >>= 1)
                if (key[run_lds(1 + i + len + o - 1)] == kk) len += o;
            const int32_t p0 = (int32_t)(base + i);
            b.chunk_desc[c++] = make_int4(p0, p0 + len, u - 1, head && !lng ? 1 : 2);
        }
    }
    __syncthreads();
    uint32_t p[ITEMS];
    int32_t bag[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = k * NT + tid;
        p[k] = pos[i < n ? i : 0];
        p[k] = p[k] < (uint64_t)nnz ? p[k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) bag[k] = bag_of[p[k]];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int i = k * NT + tid;
        if (i < n) {
            __builtin_nontemporal_store(bag[k], &b.sbag[base + i]);
            b.inv[p[k]] = (int32_t)seg[run_lds(i)];
        }
    }
}

// ---------------------------------------------------------------- LSD radix sort
//
// Stable.  Per pass: tile histograms (digit-major), one scan of the histogram
// table, then a scatter in which every tile ranks its keys per digit with wave
// ballots, round by round (BLOCK keys per round), so equal digits keep input
// order.  Digits are up to RS_MAXBITS wide; a key of b bits takes
// ceil(b / 11) passes of ceil(b / passes) bits each.  A tile is `items`
// rounds: small inputs get short tiles so that more blocks share the work.
constexpr int RS_ITEMS = 8;                 // most rounds per tile
constexpr int RS_TILE = BLOCK * RS_ITEMS;   // longest tile
constexpr int RS_MAXBITS = 11;
constexpr int RS_MAXBINS = 1 << RS_MAXBITS;
// One-launch passes when every block can afford to read the whole
// (bins x tiles) histogram table.
constexpr int64_t RS_FUSED_TABLE = 16384;

int radix_passes(int64_t n, int bits)
{
    return (n <= 1 || bits <= 0) ? 0 : (bits + RS_MAXBITS - 1) / RS_MAXBITS;
}

RadixPlan radix_plan(int64_t n, int bits)
{
    RadixPlan p{};
    p.passes = radix_passes(n, bits);
    if (p.passes == 0) return p;
    p.dbits = (bits + p.passes - 1) / p.passes;
    const int64_t bins = (int64_t)1 << p.dbits;
    auto tiles_for = [n](int r) { return (n + (int64_t)BLOCK * r - 1) / ((int64_t)BLOCK * r); };
    p.items = RS_ITEMS;
    while (p.items > 1 && tiles_for(p.items) < 128 && bins * tiles_for(p.items / 2) <= RS_FUSED_TABLE)
        p.items /= 2;
    p.tiles = tiles_for(p.items);
    p.table = bins * p.tiles;
    p.fused = p.table <= RS_FUSED_TABLE;
    return p;
}

int64_t radix_hist_entries(int64_t n)
{
    const int64_t tiles = (n + RS_TILE - 1) / RS_TILE + 1;
    const int64_t big = (int64_t)RS_MAXBINS * tiles;
    return big > 4 * RS_FUSED_TABLE ? big : 4 * RS_FUSED_TABLE;
}

// hist[d * tiles + tile] = keys of the tile with digit d.  With zero_from /
// zero_n, also clears a range (the histograms later passes accumulate into).
__global__ void __launch_bounds__(BLOCK) k_radix_hist(const uint32_t *keys, int64_t n, int shift,
                                                      int dbits, int items, uint32_t *hist,
                                                      int tiles, uint32_t *zero_from,
                                                      int64_t zero_n)
{
    __shared__ uint32_t h[RS_MAXBINS];
    const int bins = 1 << dbits;
    const uint32_t mask = (uint32_t)bins - 1u;
    for (int d = threadIdx.x; d < bins; d += BLOCK) h[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * BLOCK * items;
    for (int r = 0; r < items; ++r) {
        const int64_t i = base + (int64_t)r * BLOCK + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += BLOCK) hist[(int64_t)d * tiles + blockIdx.x] = h[d];
    for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < zero_n;
         i += (int64_t)gridDim.x * BLOCK)
        zero_from[i] = 0;
}

// Stable scatter of one tile by one digit.  Keys are ranked round by round
// (256 keys per round, in input order): lanes of a wave with the same digit
// find each other with one ballot per digit bit; the lowest of them records
// the wave's count for that digit, stamped with the round, so stale counts of
// earlier rounds read as zero and nothing has to be cleared between rounds.
// base[d] is where the tile's next key of digit d goes.
//  FUSED: base comes from the raw per-tile histogram table (this block sums
//  its column prefix and the digit totals), and the scatter adds each key to
//  the next pass's histogram at its output tile, so a pass is one launch.
//  Otherwise base comes from a scanned (exclusive, digit-major) table.
template <bool FUSED>
__global__ void __launch_bounds__(BLOCK) k_radix_scatter(const uint32_t *kin, const uint32_t *vin,
                                                         int64_t n, int shift, int dbits,
                                                         int items, const uint32_t *table,
                                                         int tiles, uint32_t *kout,
                                                         uint32_t *vout, uint32_t *hist_next,
                                                         int shift_next, int dbits_next)
{
    __shared__ uint32_t base[RS_MAXBINS];
    __shared__ uint32_t wc[BLOCK / WAVE][RS_MAXBINS];
    __shared__ uint32_t lds[BLOCK / WAVE];
    const int tid = threadIdx.x, w = wave_id(), lane = lane_id();
    const int bins = 1 << dbits;
    const uint32_t mask = (uint32_t)bins - 1u;
    const int tile = blockIdx.x;
    const int tile_len = BLOCK * items;
    const int64_t tbase = (int64_t)tile * tile_len;
    // the tile's keys and values, all loads in flight at once
    uint32_t kr[RS_ITEMS], vr[RS_ITEMS];
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        const int64_t i = tbase + (int64_t)r * BLOCK + tid;
        const bool in = r < items && i < n;
        kr[r] = in ? kin[i] : 0u;
        vr[r] = in ? vin[i] : 0u;
    }
    if (FUSED) {
        // digit totals into wc[0], this tile's column prefix into base
        for (int d = tid; d < bins; d += BLOCK) {
            const uint32_t *row = table + (int64_t)d * tiles;
            uint32_t before = 0, total = 0;
#pragma unroll 8
            for (int t = 0; t < tiles; ++t) {
                const uint32_t x = row[t];
                before += t < tile ? x : 0u;
                total += x;
            }
            base[d] = before;
            wc[0][d] = total;
        }
        __syncthreads();
        // exclusive scan of the digit totals: thread tid owns bins/BLOCK
        // consecutive digits (or one digit when bins < BLOCK)
        const int per = bins >= BLOCK ? bins / BLOCK : 1;
        const int d0 = tid * per;
        uint32_t mine = 0;
        for (int q = 0; q < per; ++q)
            if (d0 + q < bins) mine += wc[0][d0 + q];
        uint32_t total;
        uint32_t run = block_excl_scan(mine, lds, total);
        for (int q = 0; q < per; ++q)
            if (d0 + q < bins) {
                const uint32_t x = wc[0][d0 + q];
                base[d0 + q] += run;
                run += x;
            }
    } else {
        for (int d = tid; d < bins; d += BLOCK) base[d] = table[(int64_t)d * tiles + tile];
    }
    __syncthreads();
    for (int q = 0; q < BLOCK / WAVE; ++q)
        for (int d = tid; d < bins; d += BLOCK) wc[q][d] = 0;
    __syncthreads();

    const uint64_t lt = lanemask_lt();
    const uint32_t mask_next = (1u << dbits_next) - 1u;
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
        if (r >= items) break;  // uniform
        const uint32_t stamp = (uint32_t)(r + 1) << 16;
        const int64_t i = tbase + (int64_t)r * BLOCK + tid;
        const bool valid = i < n;
        const uint32_t k = kr[r];
        const uint32_t v = vr[r];
        const uint32_t d = (k >> shift) & mask;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < dbits; ++b) {
            const uint32_t bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
        const int leader = valid ? __ffsll((unsigned long long)peers) - 1 : lane;
        const bool is_leader = valid && leader == lane;
        if (is_leader) wc[w][d] = stamp | (uint32_t)__popcll(peers);
        __syncthreads();
        uint32_t start = 0;
        bool last_wave = false;
        uint32_t total = 0;
        if (is_leader) {
            uint32_t before = 0;
            last_wave = true;
            for (int q = 0; q < BLOCK / WAVE; ++q) {
                const uint32_t e = wc[q][d];
                const uint32_t c = (e & 0xFFFF0000u) == stamp ? (e & 0xFFFFu) : 0u;
                if (q < w) before += c;
                if (q > w && c) last_wave = false;
                total += c;
            }
            start = base[d] + before;
        }
        start = __shfl(start, leader, WAVE);
        __syncthreads();  // every leader has read base[d]
        if (is_leader && last_wave) base[d] += total;
        if (valid) {
            uint32_t p = start + (uint32_t)__popcll(peers & lt);
            p = p < (uint64_t)n ? p : (uint32_t)(n - 1);  // never write past the output
            kout[p] = k;
            vout[p] = v;
            if (FUSED && hist_next)
                atomicAdd(&hist_next[(int64_t)((k >> shift_next) & mask_next) * tiles +
                                     p / (uint32_t)tile_len],
                          1u);
        }
        __syncthreads();
    }
}

struct ValU32 {
    const uint32_t *p;
    __device__ uint32_t operator()(int64_t i, int) const { return p[i]; }
};
struct OutU32 {
    uint32_t *p;
    __device__ void operator()(int64_t i, uint32_t e, uint32_t, int) const { p[i] = e; }
};

// Sorts (k0, v0) by key (LSD, stable); k1/v1 are scratch of the same size.
// The result is in k1/v1 when radix_passes(n, bits) is odd (*in_k1).  With
// prehist (one-launch passes only), the caller has already filled the first
// pass's table (tile t = keys [t * BLOCK * items, ...)) and zeroed the other
// passes' tables (radix_plan gives the layout).
void launch_radix_sort(uint32_t *k0, uint32_t *v0, uint32_t *k1, uint32_t *v1, int64_t n,
                       int bits, uint32_t *hist, ScanWs &ws, bool *in_k1, hipStream_t s,
                       bool prehist)
{
    *in_k1 = false;
    const RadixPlan rp = radix_plan(n, bits);
    const int passes = rp.passes;
    if (passes == 0) return;
    const int dbits = rp.dbits, items = rp.items;
    const int tiles = (int)rp.tiles;
    const int64_t table = rp.table;
    uint32_t *ki = k0, *vi = v0, *ko = k1, *vo = v1;
    if (rp.fused) {
        // hist + P one-launch passes; pass p reads table p and fills table p+1
        if (!prehist)
            hipLaunchKernelGGL(k_radix_hist, dim3(tiles), dim3(BLOCK), 0, s, ki, n, 0, dbits, items,
                               hist, tiles, hist + table, table * (passes - 1));
        for (int p = 0; p < passes; ++p) {
            uint32_t *next = p + 1 < passes ? hist + table * (p + 1) : nullptr;
            hipLaunchKernelGGL(k_radix_scatter<true>, dim3(tiles), dim3(BLOCK), 0, s, ki, vi, n,
                               dbits * p, dbits, items, hist + table * p, tiles, ko, vo, next,
                               dbits * (p + 1), dbits);
            uint32_t *t;
            t = ki, ki = ko, ko = t;
            t = vi, vi = vo, vo = t;
        }
    } else {
        for (int p = 0; p < passes; ++p) {
            const int shift = dbits * p;
            hipLaunchKernelGGL(k_radix_hist, dim3(tiles), dim3(BLOCK), 0, s, ki, n, shift, dbits,
                               items, hist, tiles, (uint32_t *)nullptr, (int64_t)0);
            seg_scan<uint32_t>(SegN{table}, 1, table, ValU32{hist}, OutU32{hist}, ws, s);
            hipLaunchKernelGGL(k_radix_scatter<false>, dim3(tiles), dim3(BLOCK), 0, s, ki, vi, n,
                               shift, dbits, items, hist, tiles, ko, vo, (uint32_t *)nullptr, 0,
                               dbits);
            uint32_t *t;
            t = ki, ki = ko, ko = t;
            t = vi, vi = vo, vo = t;
        }
    }
    *in_k1 = (ki == k1);
}

// ---------------------------------------------------------------- tables in LDS, split by rows
//
// When every table of a batch has at most IG_MAX IDs and the batch at most
// IG_MAX bags per table, one launch does all of the above.  Each table is
// handled by S workgroups, each owning one contiguous range of its rows
// (workgroups take (table, range) pairs in the order they start, from an
// atomic counter).  A workgroup reads the table's offsets and IDs, keeps the
// entries whose row falls in its range in position order (entry = row offset
// << 26 | bag << 13 | position, positions and bags local to the table), sorts
// them by row in LDS, finds the runs of equal rows and their backward chunks,
// then publishes its entry, unique-key, chunk and long-run counts and its
// error bits (epoch-tagged, as the single-pass scan does).  It adds up the
// counts of every workgroup that started before it to place its outputs.
// Keys are table-major and the ranges ascend, so this is the order of the
// general path: a workgroup's sorted entries follow those of the ranges
// before it within the table's span of the batch.  Once a workgroup has read
// all of its inputs it counts itself in *cons; the one that completes the
// count (cons_target) writes cons_seq to the host-coherent word cons_word,
// which tells the host that the caller's arrays are no longer needed, long
// before the kernel ends.  A workgroup can hold a whole table, so any
// distribution of rows over the ranges is handled; an even one spreads the
// sort over S compute units.
constexpr int IG_THREADS = 1024;
constexpr int IG_WAVES = IG_THREADS / WAVE;
constexpr int IG_ITEMS = 8;
constexpr int IG_SHIFT_BAG = 13, IG_SHIFT_ROW = 26;
constexpr uint32_t IG_LOW = (1u << IG_SHIFT_BAG) - 1u;
static_assert(IG_THREADS * IG_ITEMS == IG_MAX, "one item per thread per round");
static_assert(MAX_TABLES * IG_SPLIT_MAX <= IG_THREADS, "one earlier workgroup per thread");

__global__ void __launch_bounds__(IG_THREADS) k_ingest_table(Tables tb, const int32_t *ids,
                                                             const int32_t *bag_off,
                                                             int32_t *bag_off_copy, int32_t B,
                                                             int64_t nnz, int32_t chunk,
                                                             int64_t max_table_ids, BatchDev b,
                                                             int64_t cap_u, int64_t cap_c,
                                                             ScanDev d, int32_t S, uint32_t *cons,
                                                             uint32_t cons_target,
                                                             uint64_t *cons_word, uint32_t cons_seq)
{
    __shared__ uint64_t buf[2][IG_MAX];
    __shared__ uint32_t wc[IG_WAVES][256];
    __shared__ uint32_t lds[IG_WAVES];
    __shared__ uint32_t id_s, multi_s, m_s;
    __shared__ int32_t err_s;
    __shared__ uint32_t before_s[5];
    const int tid = threadIdx.x, w = wave_id(), lane = lane_id();
    if (tid == 0) {
        id_s = atomicAdd(d.counter, 1u) - d.base;
        multi_s = 0;
        err_s = 0;
    }
    __syncthreads();
    const uint32_t id = id_s;
    const int t = (int)(id / (uint32_t)S), sub = (int)(id % (uint32_t)S);
    auto inputs_read = [&]() {  // thread 0, after every read of ids and bag_off
        if (atomicAdd(cons, 1u) + 1u == cons_target)
            __hip_atomic_store(cons_word, (uint64_t)cons_seq, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
    };
    if (t >= tb.T) {  // the counter and the host disagree: give up loudly
        if (tid == 0) {
            atomicOr(d.err, ERR_PLAN);
            inputs_read();
        }
        return;
    }
    const int64_t nbags = (int64_t)tb.T * B;
    // ---- the table's span of the batch, then its IDs and offsets, all loads
    // in flight together
    int64_t j0 = bag_off[(int64_t)t * B], j1 = bag_off[(int64_t)(t + 1) * B];
    j0 = j0 < 0 ? 0 : (j0 > nnz ? nnz : j0);
    j1 = j1 < j0 ? j0 : (j1 > nnz ? nnz : j1);
    const int n = (int)(j1 - j0 < IG_MAX ? j1 - j0 : IG_MAX);
    // a table past the configured bound: the rest is left out and the plan fails
    int32_t err = j1 - j0 > max_table_ids ? ERR_TABLE_IDS : 0;
    int32_t rv[IG_ITEMS];
#pragma unroll
    for (int r = 0; r < IG_ITEMS; ++r) {
        const int i = r * IG_THREADS + tid;
        rv[r] = n > 0 ? ids[j0 + (i < n ? i : n - 1)] : 0;
    }
    // offsets: validate, mark the bag of every position; the first range's
    // workgroup copies them into the ring
    uint32_t *bag_at = reinterpret_cast<uint32_t *>(buf[1]);
    for (int lb = tid; lb < B; lb += IG_THREADS) {
        const int64_t g = (int64_t)t * B + lb;
        const int64_t lo = bag_off[g], hi = bag_off[g + 1];
        if (sub == 0 && bag_off_copy != bag_off) {
            bag_off_copy[g] = (int32_t)lo;
            if (g == nbags - 1) bag_off_copy[g + 1] = (int32_t)hi;
        }
        if (lo > hi || lo < 0 || hi > nnz || (g == 0 && lo != 0) || (g == nbags - 1 && hi != nnz))
            err |= ERR_OFFSETS;
        if (hi - lo > FWD_LONG) err |= BATCH_LONG_BAG;
        const int64_t a = lo - j0 < 0 ? 0 : lo - j0, e = hi - j0 > n ? n : hi - j0;
        for (int64_t i = a; i < e; ++i) bag_at[i] = (uint32_t)lb;
    }
    // this workgroup's rows
    const int64_t rows_t = tb.rows[t];
    const int64_t span = (rows_t + S - 1) / S;
    const int64_t r0 = (int64_t)sub * span;
    const int64_t r1 = r0 + span < rows_t ? r0 + span : rows_t;
    int rbits = 0;
    while ((int64_t)1 << rbits < span) ++rbits;
    __syncthreads();
    // ---- keep the entries of this range, in position order: per round r the
    // waves' counts are laid out (r, wave) and scanned by wave 0
    const uint64_t lt = lanemask_lt();
    uint32_t kept = 0, rank[IG_ITEMS];
    uint32_t *cnt = &wc[0][0];
#pragma unroll
    for (int r = 0; r < IG_ITEMS; ++r) {
        const int i = r * IG_THREADS + tid;
        int32_t row = rv[r];
        if (i < n && (row < 0 || (int64_t)row >= rows_t)) {
            err |= ERR_ID_RANGE;
            row = 0;
        }
        rv[r] = row;
        const bool keep = i < n && row >= r0 && row < r1;
        const uint64_t bal = __ballot(keep);
        kept |= (uint32_t)keep << r;
        rank[r] = (uint32_t)__popcll(bal & lt);
        if (lane == 0) cnt[r * IG_WAVES + w] = (uint32_t)__popcll(bal);
    }
    if (err) atomicOr(&err_s, err);
    __syncthreads();
    if (tid == 0) inputs_read();
    if (w == 0) {
        static_assert(IG_ITEMS * IG_WAVES == 2 * WAVE, "two counts per lane");
        const uint32_t c0 = cnt[2 * lane], c1 = cnt[2 * lane + 1];
        const uint32_t incl = wave_incl_scan(c0 + c1);
        cnt[2 * lane] = incl - c0 - c1;
        cnt[2 * lane + 1] = incl - c1;
        if (lane == WAVE - 1) m_s = incl;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IG_ITEMS; ++r) {
        if ((kept >> r) & 1u) {
            const int i = r * IG_THREADS + tid;
            uint32_t bag = bag_at[i];
            bag = bag < (uint32_t)B ? bag : 0u;  // positions no bag covers: flagged above
            buf[0][cnt[r * IG_WAVES + w] + rank[r]] =
                ((uint64_t)(rv[r] - r0) << IG_SHIFT_ROW) | ((uint64_t)bag << IG_SHIFT_BAG) |
                (uint64_t)i;
        }
    }
    const int m = (int)m_s;
    __syncthreads();
    uint64_t *srt = lds_radix_sort<IG_THREADS, IG_ITEMS>(buf[0], buf[1], m, IG_SHIFT_ROW, rbits,
                                                         wc, lds);
    // the other buffer holds each run's first sorted index and its first chunk
    uint32_t *run0 = reinterpret_cast<uint32_t *>(srt == buf[0] ? buf[1] : buf[0]);
    uint32_t *chunk0 = run0 + IG_MAX;

    // ---- runs of equal rows (blocked: thread tid owns items tid*K .. tid*K+K-1)
    const int K = (m + IG_THREADS - 1) / IG_THREADS;
    const int i0 = tid * K;
    uint32_t heads = 0;
    uint64_t e[IG_ITEMS];
#pragma unroll
    for (int q = 0; q < IG_ITEMS; ++q) {
        const int i = i0 + q;
        const bool in = q < K && i < m;
        e[q] = in ? srt[i] : 0ull;
        const bool h = in && (i == 0 || (srt[i - 1] >> IG_SHIFT_ROW) != (e[q] >> IG_SHIFT_ROW));
        heads |= (uint32_t)h << q;
    }
    uint32_t nU;
    const uint32_t seg_first = block_excl_scan_n<IG_THREADS>((uint32_t)__popc(heads), lds, nU);
    {
        uint32_t sg = seg_first;
#pragma unroll
        for (int q = 0; q < IG_ITEMS; ++q)
            if ((heads >> q) & 1u) run0[sg++] = (uint32_t)(i0 + q);
    }
    __syncthreads();
    // chunks per run (blocked over runs the same way)
    uint32_t nch[IG_ITEMS], csum = 0, msum = 0;
#pragma unroll
    for (int q = 0; q < IG_ITEMS; ++q) {
        const uint32_t sr = (uint32_t)(i0 + q);
        nch[q] = 0;
        if (q < K && sr < nU) {
            const uint32_t len = (sr + 1 < nU ? run0[sr + 1] : (uint32_t)m) - run0[sr];
            nch[q] = (len + (uint32_t)chunk - 1) / (uint32_t)chunk;
            csum += nch[q];
            msum += nch[q] > 1;
        }
    }
    uint32_t nC;
    uint32_t cb = block_excl_scan_n<IG_THREADS>(csum, lds, nC);
    uint32_t nM;
    (void)block_excl_scan_n<IG_THREADS>(msum, lds, nM);
#pragma unroll
    for (int q = 0; q < IG_ITEMS; ++q) {
        const uint32_t sr = (uint32_t)(i0 + q);
        if (q < K && sr < nU) chunk0[sr] = cb;
        cb += nch[q];
    }

    // ---- publish this workgroup's counts, add up those of every earlier one
    uint64_t *st = d.status + (int64_t)id * LB_WORDS;
    if (tid == 0) {
        const uint32_t mine[4] = {nU, nC, nM, (uint32_t)err_s << 16 | (uint32_t)m};
#pragma unroll
        for (int c = 0; c < 4; ++c) lb_publish<uint32_t>(st + c, d.epoch, mine[c]);
    }
    uint32_t v[4] = {0, 0, 0, 0};
    if (tid < (int)id) {  // one thread per earlier workgroup
        const uint64_t *wd = d.status + (int64_t)tid * LB_WORDS;
        int spins = 0;
        bool ok = false;
        while (!ok) {
            ok = true;
#pragma unroll
            for (int c = 0; c < 4; ++c) ok = lb_read<uint32_t>(wd + c, d.epoch, v[c]) && ok;
            if (!ok && ++spins > LB_SPIN) {  // counted as zero; result flagged wrong
                atomicOr(d.err, ERR_PLAN);
                v[0] = v[1] = v[2] = v[3] = 0;
                break;
            }
            if (!ok) __builtin_amdgcn_s_sleep(1);
        }
    }
    {
        // entries before this range within the table; error bits of them all
        const uint32_t ent = tid >= t * S ? (v[3] & 0xFFFFu) : 0u;
        uint32_t eo = v[3] >> 16;
#pragma unroll
        for (int o = WAVE / 2; o > 0; o >>= 1) eo |= __shfl_xor(eo, o, WAVE);
        const uint32_t part[5] = {wave_sum(v[0]), wave_sum(v[1]), wave_sum(v[2]), eo,
                                  wave_sum(ent)};
        if (lane == 0)
#pragma unroll
            for (int c = 0; c < 5; ++c) wc[c][w] = part[c];
        __syncthreads();
        if (tid < 5) {
            uint32_t acc = 0;
            for (int q = 0; q < IG_WAVES; ++q) acc = tid == 3 ? (acc | wc[tid][q]) : acc + wc[tid][q];
            before_s[tid] = acc;
        }
        __syncthreads();
    }
    const uint32_t U0 = before_s[0], C0 = before_s[1], M0 = before_s[2];
    const int64_t jb = j0 + (int64_t)before_s[4];  // this range's first sorted position
    const int rb = tb.row_bits;
    const int64_t n_multi = multi_capacity(cap_u, chunk);

    // ---- outputs: positions
    uint32_t sg = seg_first;
#pragma unroll
    for (int q = 0; q < IG_ITEMS; ++q) {
        const int i = i0 + q;
        if (q >= K || i >= m) break;
        const uint32_t row = (uint32_t)((e[q] >> IG_SHIFT_ROW) + (uint64_t)r0);
        const int32_t bag = (int32_t)((e[q] >> IG_SHIFT_BAG) & IG_LOW);
        const int64_t pos = j0 + (int64_t)(e[q] & IG_LOW);
        const int64_t gi = jb + i;
        if ((heads >> q) & 1u) {
            if ((int64_t)U0 + sg < cap_u) b.ukeys[U0 + sg] = ((uint32_t)t << rb) | row;
            ++sg;
        }
        b.sbag[gi] = (int32_t)((int64_t)t * B + bag);
        b.inv[pos] = (int32_t)(U0 + sg - 1);
    }
    // ---- outputs: runs and their backward chunks
#pragma unroll
    for (int q = 0; q < IG_ITEMS; ++q) {
        const uint32_t sr = (uint32_t)(i0 + q);
        if (q >= K || sr >= nU) break;
        const int64_t gs = (int64_t)U0 + sr;
        const int64_t c0 = (int64_t)C0 + chunk0[sr];
        if (gs >= cap_u) break;
        b.seg_chunk0[gs] = (int32_t)c0;
        const int32_t s0 = (int32_t)(jb + run0[sr]);
        const int32_t s1 = (int32_t)(jb + (sr + 1 < nU ? run0[sr + 1] : (uint32_t)m));
        for (uint32_t c = 0; c < nch[q] && c0 + c < cap_c; ++c) {
            const int32_t p0 = s0 + (int32_t)c * chunk;
            b.chunk_desc[c0 + c] = make_int4(p0, p0 + chunk < s1 ? p0 + chunk : s1, (int32_t)gs,
                                             (int32_t)nch[q]);
        }
        if (nch[q] > 1) {
            const uint32_t mi = M0 + atomicAdd(&multi_s, 1u);  // list order is irrelevant
            if ((int64_t)mi < n_multi) b.multi[mi] = (int32_t)gs;
        }
    }
    if (id == (uint32_t)(tb.T * S - 1) && tid == 0) {  // the batch totals
        const uint32_t U = U0 + nU;
        if ((int64_t)U < cap_u + 1) b.seg_chunk0[U] = (int32_t)(C0 + nC);
        b.scal[0] = (int32_t)U;
        b.scal[1] = (int32_t)(C0 + nC);
        const int32_t found = (int32_t)(before_s[3] | (uint32_t)err_s);
        b.scal[2] = found & ~BATCH_LONG_BAG;
        b.scal[3] = (int32_t)(M0 + nM);
        b.scal[4] = (found & BATCH_LONG_BAG) != 0;
    }
}

// ---------------------------------------------------------------- general path: launches

constexpr int64_t SORT_LARGE = 512 << 10;  // IDs from which the tiles are the long ones
constexpr int SORT_TILE_MIN = 1024;

SortWsSize sort_ws_size(int64_t n)
{
    // tiles (and at most as many groups, and one) of all tables: each table's
    // last one may be short
    const int64_t tiles = (n + SORT_TILE_MIN - 1) / SORT_TILE_MIN + MAX_TABLES + 1;
    return {2 * n, 2 * tiles * SORT_BINS, tiles};
}

// Tiles per group: a power of two up to the square root of a table's mean tiles,
// so that a scatter block adds few group counts, but at least 256 groups in all,
// one k_sort_hist block for each compute unit.  An ingest's time in us with 1024
// and with 256 groups at least: one table of 4.2M IDs 425 and 350, of 21M 1780
// and 1325 (a block adds 641 and 161 group counts); two of 10.5M 1450 and 1270;
// four of 1M 331 and 280; 26 of 160k 205 and 196; 64 of 330k 750 and 750.  Groups
// past the root cost: eight tables of 2.6M, 16 tiles each 1170 and 32 tiles 1205.
static int sort_group(int64_t tiles, int T)
{
    int G = 1;
    while ((int64_t)4 * G * G * T <= tiles && tiles / G > 256) G *= 2;
    return G;
}

template <int NT, int ITEMS>
static void launch_general(const Tables &tb, const BatchDev &b, const int32_t *ids,
                           const int32_t *bag_off, int32_t B, int64_t nnz, int64_t max_table_ids,
                           int64_t cap_u, const SortWs &sw, hipEvent_t consumed, hipStream_t s)
{
    constexpr int TILE = NT * ITEMS;
    const int64_t nbags = (int64_t)tb.T * B;
    int passes = 1;
    for (int t = 0; t < tb.T; ++t) {
        int bits = 1;
        while (bits < 25 && (int64_t)1 << bits < tb.rows[t]) ++bits;
        const int np = (bits + SORT_BITS - 1) / SORT_BITS;
        passes = passes > np ? passes : np;
    }
    const int64_t flat = (nnz + TILE - 1) / TILE;
    const int64_t tiles = flat + tb.T;  // at least those of all tables, whatever their spans
    const int G = sort_group(flat, tb.T);
    const int64_t groups = flat / G + tb.T + 1;
    uint32_t *const thist = sw.hist, *const ghist = sw.hist + tiles * SORT_BINS;
    const int parts = bag_parts(nnz, nbags);
    const int64_t bag_blocks = ((nbags + WAVE - 1) / WAVE * parts + NT / WAVE - 1) / (NT / WAVE);
    for (int q = 0; q < passes; ++q) {
        const uint64_t *const in = sw.e[(passes - q) & 1];  // the last pass writes e[0]
        uint64_t *const out = sw.e[(passes - 1 - q) & 1];
        hipLaunchKernelGGL((k_sort_hist<NT, ITEMS>),
                           dim3((unsigned)(groups + (q == 0 ? bag_blocks : 0))), dim3(NT), 0, s, tb,
                           ids, bag_off, b.bag_off, B, nnz, nbags, max_table_ids, b.bag_of,
                           parts, (int32_t)groups, in, q, passes, G, thist, ghist, sw.err);
        hipLaunchKernelGGL((k_sort_scatter<NT, ITEMS>), dim3((unsigned)tiles), dim3(NT), 0, s, tb,
                           ids, bag_off, B, nnz, in, out, q, passes, G, (const uint32_t *)thist,
                           (const uint32_t *)ghist);
    }
    // the later launches need the offsets only, from the ring's copy
    if (consumed) (void)hipEventRecord(consumed, s);
    const int64_t cap_m = multi_capacity(cap_u, BWD_CHUNK);
    hipLaunchKernelGGL((k_runs<NT, ITEMS, false>), dim3((unsigned)flat), dim3(NT), 0, s,
                       (const uint64_t *)sw.e[0], (const int32_t *)b.bag_off, tb.T, B, nnz,
                       (const int32_t *)b.bag_of, b, cap_m, sw.tcount, sw.tpre, (int32_t)flat,
                       sw.arrived, sw.err);
    hipLaunchKernelGGL((k_runs<NT, ITEMS, true>), dim3((unsigned)flat), dim3(NT), 0, s,
                       (const uint64_t *)sw.e[0], (const int32_t *)b.bag_off, tb.T, B, nnz,
                       (const int32_t *)b.bag_of, b, cap_m, sw.tcount, sw.tpre, (int32_t)flat,
                       sw.arrived, sw.err);
}

// Sort, deduplicate and split into backward chunks one batch of the window.
// ids / bag_off may be the caller's device arrays (read once, here) or the
// ring's own copies; the ring always ends up with the offsets.  Input errors
// are recorded in the batch's own scal[2].
void launch_ingest(const Tables &tb, const BatchDev &b, const int32_t *ids, const int32_t *bag_off,
                   int32_t B, int64_t nnz, int chunk, int64_t max_table_ids,
                   int64_t cap_u, int64_t cap_c, const SortWs &sw, ScanWs &ws,
                   hipEvent_t consumed, const IngestCons &ic, hipStream_t s)
{
    const int64_t nbags = (int64_t)tb.T * B;
    if (nnz > 0 && ingest_in_lds(max_table_ids, B)) {
        const int S = ingest_splits(tb.T);
        const int64_t grid = (int64_t)tb.T * S;
        if (grid > ws.max_tiles) {
            ws.overflow = true;
            return;
        }
        if (ws.epoch == 0xFFFFFFFFu) {  // epochs wrapped: forget every published word
            (void)hipMemsetAsync(ws.status, 0, sizeof(uint64_t) * LB_WORDS * ws.max_tiles, s);
            ws.epoch = 0;
        }
        ScanDev d{ws.status, ws.counter, ws.err, ws.issued, ++ws.epoch, (uint32_t)grid, 1};
        ws.issued += (uint32_t)grid;
        hipLaunchKernelGGL(k_ingest_table, dim3((unsigned)grid), dim3(IG_THREADS), 0, s, tb, ids,
                           bag_off, b.bag_off, B, nnz, chunk, max_table_ids, b, cap_u, cap_c, d,
                           S, ic.counter, ic.target, ic.word, ic.seq);
        return;
    }
    if (nnz == 0) {  // only the offsets to validate and copy
        launch_zero_i32(b.scal, 5, s);
        if (nbags > 0)
            hipLaunchKernelGGL(k_bags, dim3((unsigned)((nbags + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0,
                               s, bag_off, b.bag_off, B, nnz, nbags, max_table_ids, b.bag_of,
                               b.scal + 2);
        else if (bag_off != b.bag_off)
            (void)hipMemcpyAsync(b.bag_off, bag_off, sizeof(int32_t), hipMemcpyDeviceToDevice, s);
        if (consumed) (void)hipEventRecord(consumed, s);
        return;
    }
    // tiles of 4096 entries, or of 1024 where a batch of them would leave most
    // compute units idle
    if (nnz >= SORT_LARGE)
        launch_general<512, 8>(tb, b, ids, bag_off, B, nnz, max_table_ids, cap_u, sw, consumed, s);
    else
        launch_general<256, 4>(tb, b, ids, bag_off, B, nnz, max_table_ids, cap_u, sw, consumed, s);
}

}  // namespace sp
