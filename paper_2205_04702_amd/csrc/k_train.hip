// Data movement and training kernels over the scratchpad Storage.
//
// Row layout: Storage is fp32 [slots][D] in HBM; a row is D/4 float4 words
// and LPR = D/4 lanes cover one row, so one wave64 touches 64/LPR rows per
// pass with fully coalesced 16-byte loads.
#include <hip/hip_ext.h>

#include <type_traits>

#include "sp_device.h"
#include "sp_internal.h"

namespace sp {

struct HostRows {
    const float4 *p[MAX_TABLES];  // device-visible pointers to the pinned host tables
};

// Loads and stores that do not keep the line in the caches: the update reads
// and writes each Storage row once, and streamed rows would otherwise evict
// the bag gradients it reads again for every chunk that uses them.
typedef float nv4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 nt_load(const float4 *p)
{
    const nv4f v = __builtin_nontemporal_load(reinterpret_cast<const nv4f *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void nt_store(float4 *p, float4 x)
{
    nv4f v;
    v.x = x.x;
    v.y = x.y;
    v.z = x.z;
    v.w = x.w;
    __builtin_nontemporal_store(v, reinterpret_cast<nv4f *>(p));
}

__device__ __forceinline__ float4 f4_add(float4 a, float4 b)
{
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// Sum of N values (a power of two), in a tree.
template <int N>
__device__ __forceinline__ float4 f4_tree(const float4 (&v)[N])
{
    float4 t[N];
#pragma unroll
    for (int k = 0; k < N; ++k) t[k] = v[k];
#pragma unroll
    for (int o = N / 2; o > 0; o >>= 1)
#pragma unroll
        for (int k = 0; k < o; ++k) t[k] = f4_add(t[2 * k], t[2 * k + 1]);
    return t[0];
}

__device__ __forceinline__ float4 f4_xor(float4 a, int o)
{
    return make_float4(__shfl_xor(a.x, o, WAVE), __shfl_xor(a.y, o, WAVE), __shfl_xor(a.z, o, WAVE),
                       __shfl_xor(a.w, o, WAVE));
}

// Sum the per-subgroup partial rows of a wave (lane groups of LPR lanes).
template <int LPR>
__device__ __forceinline__ float4 reduce_rows(float4 acc)
{
#pragma unroll
    for (int o = LPR; o < WAVE; o <<= 1) acc = f4_add(acc, f4_xor(acc, o));
    return acc;
}

// ---------------------------------------------------------------- forward

// out[g] = sum of Storage[slot_u[inv[j]]] over the positions j of bag g
// (Sec. II-B, gather then element-wise reduction per table).  Reading each
// position's slot through its unique key costs one more round trip per block
// of positions, hidden behind the other waves, and spares the plan a pass that
// writes a slot per position (it was most of a large commit).
//
// A group of GW lanes adds one bag.  A bag is a chain of dependent loads
// (offsets, unique keys, slots, rows), which is what bounds this kernel where the
// rows come from L2.  With many bags, a group is as many lanes as a row has
// words, eight at least (then several rows at a time), so that a wave works on
// several bags at once: with one wave per bag, 53k bags of four rows of 64 floats
// took 19 us, 12 so; 53k bags of one row of 16 floats 18 us, 7 so.  Large batches
// of long bags are bound by their rows either way: 524k bags of 40 rows of 64
// floats 0.43 ms and 0.40 (13.7 TB/s of requests); 106k bags of 40 rows of 128
// floats 0.195 ms (11.2 TB/s of requests, a quarter of them distinct rows).
// With few or long bags a group is a whole wave (fwd_whole_wave), and where a
// batch has single bags above FWD_LONG positions among shorter ones (SKEW) the
// waves of a block share these, a whole wave for each.
constexpr int FWD_ROWS = 8;
constexpr int FWD_ACC = FWD_ROWS / 2;
constexpr int fwd_lanes(int lpr) { return lpr < 8 ? 8 : lpr; }

// The sum of the rows of one bag per group of GW lanes, in every lane of the
// group with that word: positions beg .. beg + len; all groups of the wave walk
// as far as its longest (in 32 bits: fewer registers, more waves).  The group reads IB positions' slots at a time (the
// next ones while this block's rows arrive) and broadcasts them by shuffles,
// FWD_ROWS row loads in flight per lane.  Sums run over FWD_ACC partial sums
// in position order, two rows added to one another before each (rows one by
// one on 4 partial sums are further from 64 bits than a wave per bag was: bags of 90
// rows of 32 floats 9.7e-8, 8.0e-8 then).
template <int LPR, int GW>
__device__ __forceinline__ float4 bag_sum(const float4 *__restrict__ storage,
                                          const int32_t *__restrict__ inv,
                                          const int32_t *__restrict__ slot_u, int64_t n_unique,
                                          int64_t nslots, int64_t beg, int32_t len, int32_t longest)
{
    constexpr int RPG = GW / LPR;                     // rows per load of a group
    constexpr int BATCH = RPG * FWD_ROWS;             // positions per batch of loads
    constexpr int IPL = BATCH > GW ? BATCH / GW : 1;  // positions held per lane
    constexpr int IB = IPL * GW;                      // positions per block
    const int lane = lane_id(), gl = lane % GW, g0 = lane - gl;
    const int sub = gl / LPR, c = gl % LPR;
    float4 acc[FWD_ACC];
#pragma unroll
    for (int k = 0; k < FWD_ACC; ++k) acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    int32_t ui[IPL], slot[IPL];
    auto load_unique = [&](int32_t base) {  // lane gl holds positions base + l * GW + gl
#pragma unroll
        for (int l = 0; l < IPL; ++l) {
            const int32_t k = base + l * GW + gl;
            ui[l] = k < len ? inv[beg + k] : 0;
        }
    };
    auto load_slots = [&](int32_t base) {
#pragma unroll
        for (int l = 0; l < IPL; ++l) {
            const int32_t k = base + l * GW + gl;
            const int32_t r = k < len ? slot_u[(uint32_t)ui[l] < (uint64_t)n_unique ? ui[l] : 0] : 0;
            slot[l] = (uint32_t)r < (uint64_t)nslots ? r : 0;  // never leave the array
        }
    };
    load_unique(0);
    load_slots(0);
    for (int32_t base = 0; base < longest; base += IB) {
        const int n = len - base < IB ? (len - base < 0 ? 0 : len - base) : IB;
        const int most = longest - base < IB ? longest - base : IB;
        int32_t cur[IPL];
#pragma unroll
        for (int l = 0; l < IPL; ++l) cur[l] = slot[l];
        const bool more = base + IB < longest;
        if (more) load_unique(base + IB);
#pragma unroll
        for (int k0 = 0; k0 < IB; k0 += BATCH) {
            if (k0 >= most) break;  // uniform over the wave
            float4 v[FWD_ROWS];
#pragma unroll
            for (int q = 0; q < FWD_ROWS; ++q) {
                v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (q * RPG + k0 >= most) continue;  // uniform
                const int k = k0 + q * RPG + sub;
                // position k is held by lane k % GW of the group; with several rows
                // per load, k / GW is the same for all of them
                const int32_t r = __shfl(cur[(k0 + q * RPG) / GW], g0 + k % GW, WAVE);
                if (k < n) v[q] = storage[(int64_t)r * LPR + c];
            }
            if (k0 == 0 && more) load_slots(base + IB);  // behind this batch's rows
#pragma unroll
            for (int q = 0; q < FWD_ACC; ++q) acc[q] = f4_add(acc[q], f4_add(v[2 * q], v[2 * q + 1]));
        }
    }
#pragma unroll
    for (int o = 1; o < FWD_ACC; o <<= 1)
#pragma unroll
        for (int k = 0; k < FWD_ACC; k += 2 * o) acc[k] = f4_add(acc[k], acc[k + o]);
#pragma unroll
    for (int o = LPR; o < GW; o <<= 1) acc[0] = f4_add(acc[0], f4_xor(acc[0], o));
    return acc[0];
}

// The sum of one bag's rows by a whole wave, in few registers: it is the rare
// part of a kernel whose other part they bound.
template <int LPR>
__device__ __forceinline__ float4 long_sum(const float4 *__restrict__ storage,
                                           const int32_t *__restrict__ inv,
                                           const int32_t *__restrict__ slot_u, int64_t n_unique,
                                           int64_t nslots, int64_t beg, int64_t end)
{
    constexpr int RPW = WAVE / LPR;  // rows per load
    constexpr int ROWS = RPW * FWD_ROWS < WAVE ? FWD_ROWS : WAVE / RPW;
    const int lane = lane_id(), sub = lane / LPR, c = lane % LPR;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    auto slot_at = [&](int64_t k) {
        const int32_t u = inv[k < end ? k : end - 1];
        const int32_t r = slot_u[(uint32_t)u < (uint64_t)n_unique ? u : 0];
        return (uint32_t)r < (uint64_t)nslots ? r : 0;  // never leave the array
    };
    int32_t next = slot_at(beg + lane);
    for (int64_t base = beg; base < end; base += WAVE) {
        const int32_t cur = next;
        const int n = (int)(end - base < WAVE ? end - base : WAVE);
        next = slot_at(base + WAVE + lane);
        for (int k0 = 0; k0 < n; k0 += RPW * ROWS) {
            float4 v[ROWS];
#pragma unroll
            for (int q = 0; q < ROWS; ++q) {
                const int k = k0 + q * RPW + sub;
                const int32_t r = __shfl(cur, k % WAVE, WAVE);
                v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (k < n) v[q] = storage[(int64_t)r * LPR + c];
            }
            acc = f4_add(acc, f4_tree(v));
        }
    }
    return reduce_rows<LPR>(acc);
}

// SKEW: for batches with bags above FWD_LONG positions.  A block whose long bags
// are few enough leaves them out of its groups' walk and its waves then take them
// in turn.  It decides by the rows that the longest chain adds one after another,
// in rows of one group, a bag's start (offsets, unique key, slot) being worth
// three batches of loads.  53k bags, one in 200 of them of 1000 positions: rows of
// 16 floats 95 us without, 26 so, 38 with a wave per bag; 128 floats 129, 82 and 91.
// The barrier costs short bags 10 to 25% (53k bags of one row of 64 floats 7.7
// us, 8.5 so), so batches without such bags go without.
template <int LPR, int GW, bool SKEW>
__global__ void __launch_bounds__(BLOCK) k_forward(const float4 *__restrict__ storage,
                                                   const int32_t *__restrict__ inv,
                                                   const int32_t *__restrict__ slot_u,
                                                   int64_t n_unique,
                                                   const int32_t *__restrict__ bag_off,
                                                   int64_t nbags, int64_t nslots,
                                                   float4 *__restrict__ out)
{
    constexpr int WAVES = BLOCK / WAVE, NG = WAVE / GW;
    // consecutive bags (one table's) on one XCD: the table's hot rows share its L2
    const int64_t first = xcd_block(blockIdx.x, gridDim.x) * (BLOCK / GW);
    const int64_t g = first + threadIdx.x / GW;
    const int lane = lane_id(), gl = lane % GW;
    int64_t beg = 0, end = 0;
    if (g < nbags) {
        beg = bag_off[g];
        end = bag_off[g + 1];
    }
    int32_t len = end - beg > 0 ? (int32_t)(end - beg) : 0;
    // the wave's longest bag
    int32_t longest = len;
#pragma unroll
    for (int o = GW; o < WAVE; o <<= 1) {
        const int32_t x = __shfl_xor(longest, o, WAVE);
        longest = x > longest ? x : longest;
    }
    if constexpr (!SKEW) {
        const float4 x = bag_sum<LPR, GW>(storage, inv, slot_u, n_unique, nslots, beg, len, longest);
        if (g < nbags && gl < LPR) out[g * LPR + gl] = x;
    } else {
        __shared__ int32_t n_s[WAVES], total_s[WAVES], longest_s[WAVES];
        __shared__ int32_t bag_s[WAVES][NG];  // the long bags of each wave, in the block
        const int w = wave_id();
        const bool lng = len > FWD_LONG;
        const uint64_t heads = __ballot(lng && gl == 0);
        if (lane == 0) n_s[w] = __popcll(heads);
        if (heads) {  // uniform over the wave
            const int32_t t = wave_sum(lng && gl == 0 ? len : 0);
            if (lane == 0) {
                total_s[w] = t;
                longest_s[w] = longest;
            }
            if (lng && gl == 0) bag_s[w][__popcll(heads & lanemask_lt())] = threadIdx.x / GW;
        }
        __syncthreads();
        int n_long = 0;
        int64_t total = 0, most = 0;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            const int c = n_s[k];
            n_long += c;
            if (c) {
                total += total_s[k];
                most = longest_s[k] > most ? longest_s[k] : most;
            }
        }
        bool apart = false;  // uniform over the block
        if (n_long) {
            constexpr int START = 3 * FWD_ROWS * GW / LPR;
            const int64_t share = total / WAVES > most ? total / WAVES : most;
            apart = share / NG + START * ((n_long + WAVES - 1) / WAVES) < most;
        }
        if (apart) {
            len = lng ? 0 : len;
            longest = longest > FWD_LONG ? FWD_LONG : longest;
        }
        const float4 x = bag_sum<LPR, GW>(storage, inv, slot_u, n_unique, nslots, beg, len, longest);
        if (g < nbags && !(apart && lng) && gl < LPR) out[g * LPR + gl] = x;
        if (!apart) return;
        for (int i = w; i < n_long; i += WAVES) {
            int k = 0, j = i;
            while (j >= n_s[k]) j -= n_s[k++];
            const int64_t h = first + bag_s[k][j];
            const float4 y =
                long_sum<LPR>(storage, inv, slot_u, n_unique, nslots, bag_off[h], bag_off[h + 1]);
            if (lane < LPR) out[h * LPR + lane] = y;
        }
    }
}

// ---------------------------------------------------------------- backward + SGD

__device__ __forceinline__ float4 sgd_step(float4 x, float4 g, float lr)
{
    x.x = fmaf(-lr, g.x, x.x);
    x.y = fmaf(-lr, g.y, x.y);
    x.z = fmaf(-lr, g.z, x.z);
    x.w = fmaf(-lr, g.w, x.w);
    return x;
}


// Gradient coalescing and SGD (Sec. II-B "Backpropagation").  The sorted
// positions of one batch form runs of equal keys; each run is cut into chunks
// of at most `chunk` positions.  One group of G = LPR / VPL lanes takes one
// chunk, each lane VPL of the row's LPR 16-byte words (word j * G + c for lane
// c), so a wave works on 64 / G chunks at once and each lane keeps VPL loads
// of every row in flight: more rows per memory round trip than one word per
// lane would give, which is what bounds this kernel (each chunk is a short
// chain of dependent loads: descriptor, then slot and bag indices, then the
// Storage row and gradient rows).  It sums the gradient rows of the bags at
// its positions in ascending position order.
//  * a run of one chunk updates its Storage row directly: W -= lr * g;
//  * a longer run stores per-chunk partial sums, which k_bwd_combine adds in
//    chunk order before updating the row (the kernel boundary orders the two).
constexpr int BWD_INFLIGHT = 8;  // gradient words in flight per lane (rows x VPL)

// Words per lane for rows of LPR words (the launch's grid follows it): two
// from rows of 64 floats up.  Measured alone on the 26x10M workload's update
// (128 floats): 0.80 ms with one word per lane, 0.69 ms with four (fewer
// waves fit: 97 registers), 0.63 ms with two (71 registers, 7 waves per SIMD).
constexpr int bwd_vpl(int lpr) { return lpr >= 16 ? 2 : 1; }

template <int LPR>
__global__ void __launch_bounds__(BLOCK) k_backward(float4 *__restrict__ storage,
                                                    const int4 *__restrict__ chunk_desc,
                                                    const int32_t *__restrict__ sbag,
                                                    const int32_t *__restrict__ slot_u,
                                                    int64_t n_chunks,
                                                    const float4 *__restrict__ grad,
                                                    int64_t nbags, int64_t nslots, float lr,
                                                    float4 *__restrict__ partial)
{
    constexpr int VPL = bwd_vpl(LPR);
    constexpr int G = LPR / VPL;                // lanes per chunk
    constexpr int INFL = BWD_INFLIGHT / VPL;    // gradient rows in flight per lane
    // consecutive chunks (one table's) on one XCD: the table's bag gradients
    // share its L2
    const int64_t t = xcd_block(blockIdx.x, gridDim.x) * BLOCK + threadIdx.x;
    const int64_t ch = t / G;
    const int c = (int)(t % G);
    if (ch >= n_chunks) return;  // whole lane groups leave together
    const int4 d = chunk_desc[ch];  // first position, end position, run, above 1: it has more
    const int64_t p0 = d.x, p1 = d.y;
    const int32_t slot = slot_u[d.z];
    const int64_t nch = d.w;
    // a one-chunk run reads its Storage row beside its gradient rows rather
    // than after them: one memory round trip less on the lane's path
    const bool direct = nch == 1 && (uint32_t)slot < (uint64_t)nslots;
    float4 *const w = storage + (direct ? (int64_t)slot * LPR + c : 0);
    float4 w0[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) w0[j] = direct ? nt_load(w + j * G) : make_float4(0.f, 0.f, 0.f, 0.f);
    // A chunk's bag indices arrive in one coalesced load (lane c of the group
    // holds positions c, c+G, ...) and are broadcast by shuffles, so its
    // gradient rows are requested INFL at a time without waiting on further
    // index loads.  Sums stay in position order.
    constexpr int PER_LANE = BWD_CHUNK / G > 0 ? BWD_CHUNK / G : 1;
    const int gbase = lane_id() - c;
    // 32-bit byte offsets from the uniform base (the gradient array is far
    // below 4 GiB): one address register per load in flight
    const char *__restrict__ gbytes = reinterpret_cast<const char *>(grad);
    float4 acc[VPL];
#pragma unroll
    for (int j = 0; j < VPL; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t base = p0; base < p1; base += BWD_CHUNK) {
        const int n = (int)(p1 - base < BWD_CHUNK ? p1 - base : BWD_CHUNK);
        int32_t mine[PER_LANE];
#pragma unroll
        for (int l = 0; l < PER_LANE; ++l) {
            const int k = l * G + c;
            const int32_t b = k < n ? sbag[base + k] : 0;
            mine[l] = (uint32_t)b < (uint64_t)nbags ? b : 0;
        }
#pragma unroll
        for (int k0 = 0; k0 < BWD_CHUNK; k0 += INFL) {
            if (k0 >= n) break;  // uniform within the lane group
            float4 v[INFL][VPL];
#pragma unroll
            for (int q = 0; q < INFL; ++q) {
                const int k = k0 + q;
                // every lane of the group takes part in the shuffle; only the load is predicated
                const int32_t b = __shfl(mine[k / G], gbase + k % G, WAVE);
                const uint32_t off = (uint32_t)b * (uint32_t)(LPR * 16) + (uint32_t)c * 16u;
#pragma unroll
                for (int j = 0; j < VPL; ++j)
                    v[q][j] = k < n ? *reinterpret_cast<const float4 *>(gbytes + off + j * G * 16)
                                    : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int q = 0; q < INFL; ++q)
#pragma unroll
                for (int j = 0; j < VPL; ++j) acc[j] = f4_add(acc[j], v[q][j]);
        }
    }
    if (nch > 1) {
#pragma unroll
        for (int j = 0; j < VPL; ++j) partial[ch * LPR + j * G + c] = acc[j];
    } else if (direct) {
#pragma unroll
        for (int j = 0; j < VPL; ++j) nt_store(w + j * G, sgd_step(w0[j], acc[j], lr));
    }
}

// Runs longer than one chunk (listed in `multi`, any order): adds a run's chunk
// partials in a fixed strided order (group g of the lane groups that work on
// it takes chunks g, g + groups, ...; then the groups' sums, in a fixed order
// too) and updates the row.  With few runs a block takes each (k_bwd_combine_few), so that
// long ones, a hot row has thousands of chunks, are added side by side.  With many
// most lanes of such blocks would add nothing: one wave takes a run, and the few
// runs above COMBINE_WAVE chunks are left to the whole block, with eight partials
// in flight per lane, one after another.  In us, few and many, rows of 16 / 64 /
// 256 floats:
//        8 runs of 3750 chunks   7 29 / 20 84 /  75 318
//      520 runs of  512          5 15 / 13 22 /  56  96
//     2.6k runs of  102          6 10 / 12 14 /  51  52
//     4.8k runs of   26          6  4 /  8  7 /  20  21
//     5.4k, Zipf                 9  8 / 14 13 /  35  45
//      10k runs of   26         11  6 / 13 12 /  51  54
//      14k, Zipf                20 13 / 27 23 /  85 125
//      52k runs of    5         44 17 / 40 20 /  87  66
// (COMBINE_WAVE at 256: 8 runs of 190 chunks of 256 floats 18 instead of 25 us, one
// such run 16 instead of 8.)
static bool few_runs(int64_t n_multi, int lpr) { return n_multi <= (lpr < 16 ? 4096 : 256 * lpr); }
constexpr int COMBINE_WAVE = 64;

// The partials p[q], q = g, g + groups, ..., UNROLL of them in flight and added in a
// tree before the sum (one by one, the last ones each after the other, 19k runs of
// 50 chunks of 256 floats were 5.2e-8 from 64 bits, with a block per run 4.2e-8).
template <int LPR, int UNROLL>
__device__ __forceinline__ float4 sum_partials(const float4 *__restrict__ p, int64_t nch,
                                               int64_t g, int64_t groups)
{
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t q = g; q < nch; q += UNROLL * groups) {
        float4 v[UNROLL];
#pragma unroll
        for (int k = 0; k < UNROLL; ++k) {
            v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (q + k * groups < nch) v[k] = p[(q + k * groups) * LPR];
        }
        acc = f4_add(acc, f4_tree(v));
    }
    return acc;
}

// One run by the whole block: groups' sums by shuffles, then the waves' in pairs.
template <int LPR>
__device__ __forceinline__ void combine_by_block(float4 *__restrict__ storage,
                                                 const float4 *__restrict__ partial, int64_t c0,
                                                 int64_t nch, int32_t slot, int64_t nslots,
                                                 float lr, float4 (&red)[BLOCK / WAVE][LPR])
{
    static_assert(BLOCK / WAVE == 4, "the waves' sums are added in pairs");
    const int g = threadIdx.x / LPR, c = threadIdx.x % LPR;
    const float4 acc = reduce_rows<LPR>(
        sum_partials<LPR, 8>(partial + c0 * LPR + c, nch, g, BLOCK / LPR));
    if (lane_id() < LPR) red[wave_id()][c] = acc;
    __syncthreads();
    if (g != 0 || (uint32_t)slot >= (uint64_t)nslots) return;
    float4 *const row = storage + (int64_t)slot * LPR + c;
    const float4 sum = f4_add(f4_add(red[0][c], red[1][c]), f4_add(red[2][c], red[3][c]));
    nt_store(row, sgd_step(nt_load(row), sum, lr));
}

template <int LPR>
__global__ void __launch_bounds__(BLOCK) k_bwd_combine(float4 *__restrict__ storage,
                                                       const int32_t *__restrict__ multi,
                                                       int64_t n_multi,
                                                       const int32_t *__restrict__ seg_chunk0,
                                                       const int32_t *__restrict__ slot_u,
                                                       const float4 *__restrict__ partial,
                                                       int64_t nslots, float lr)
{
    constexpr int WAVES = BLOCK / WAVE;
    constexpr int UNROLL = LPR == WAVE ? 8 : 4;  // a single group's chain is the longest
    __shared__ float4 red[WAVES][LPR];
    __shared__ int32_t left[WAVES];  // each wave's run, if the block is to add it
    const int w = wave_id(), lane = lane_id();
    const int64_t m = (int64_t)blockIdx.x * WAVES + w;
    const int32_t s = m < n_multi ? multi[m] : -1;
    int64_t c0 = 0, nch = 0;
    if (s >= 0) {
        c0 = seg_chunk0[s];
        nch = seg_chunk0[s + 1] - c0;
    }
    if (lane == 0) left[w] = nch > COMBINE_WAVE ? s : -1;
    if (nch > 0 && nch <= COMBINE_WAVE) {  // uniform over the wave
        const int c = lane % LPR;
        const int32_t slot = slot_u[s];
        const bool ok = (uint32_t)slot < (uint64_t)nslots;
        float4 *const row = storage + (ok ? (int64_t)slot * LPR : 0) + c;
        const float4 x = nt_load(row);
        const float4 acc = reduce_rows<LPR>(sum_partials<LPR, UNROLL>(
            partial + c0 * LPR + c, nch, lane / LPR, WAVE / LPR));
        if (ok && lane < LPR) nt_store(row, sgd_step(x, acc, lr));
    }
    __syncthreads();
    for (int k = 0; k < WAVES; ++k) {
        const int32_t run = left[k];
        if (run < 0) continue;  // uniform over the block
        const int64_t b0 = seg_chunk0[run], n = seg_chunk0[run + 1] - b0;
        combine_by_block<LPR>(storage, partial, b0, n, slot_u[run], nslots, lr, red);
        __syncthreads();
    }
}

template <int LPR>
__global__ void __launch_bounds__(BLOCK) k_bwd_combine_few(float4 *__restrict__ storage,
                                                           const int32_t *__restrict__ multi,
                                                           const int32_t *__restrict__ seg_chunk0,
                                                           const int32_t *__restrict__ slot_u,
                                                           const float4 *__restrict__ partial,
                                                           int64_t nslots, float lr)
{
    __shared__ float4 red[BLOCK / WAVE][LPR];
    const int32_t s = multi[blockIdx.x];
    const int64_t c0 = seg_chunk0[s], nch = seg_chunk0[s + 1] - c0;
    combine_by_block<LPR>(storage, partial, c0, nch, slot_u[s], nslots, lr, red);
}

// ---------------------------------------------------------------- evict / fill

// Victim i: copy the row its slot held (if any) to staging row i for the
// write-back, then fill the slot with the missing row m_key[i]: read straight
// from the pinned host table (zero-copy over the host link), or, with the
// staged fill, from row i of the rows already copied to the device.  The same
// lanes read the old row before writing the new one.  Every victim's previous
// key is stored after the n staging rows.  With the zero-copy fill the staging
// is pinned host memory too: the old rows cross the link in the other
// direction while the missing ones are read, and the write-back needs no copy
// of its own.  (Such a copy ran beside the forward that waits for this kernel
// and held it: 8 tables of 1M rows of 64 floats, 10.4k misses a step: 55 us
// here, then a forward of 50 us; now 82 and 6.)  With the staged fill it is
// device memory, copied later: there the link is busy with the gathered rows.
// For the zero-copy fill the grid is kept small and each lane
// group keeps MOVE_ROWS victims in flight: some four thousand 64-byte reads
// fill the link's latency, and more only queue up in front of every other
// kernel's misses.  89k rows of 32 bytes: 0.30 ms with 4096 reads in flight
// and the next plan's query beside it 0.026 ms; 0.27 ms with 32k reads, and
// the query 0.26 ms (a step 0.40 and 0.48 ms).  10.4k rows of 256 bytes: 94 us
// with 4096 reads of 64 bytes, 82 us with 8192 and 80 us with 16384.  The
// staged fill only moves rows within HBM and takes a full grid.
// Every row the move reads or writes is touched once, so none of its accesses
// keeps the line in the caches: cached stores of a large fill left the caches
// full of dirty lines, whose write-back then slowed the forward that follows
// (26x10M forward 0.350 ms after a cached fill, 0.317 ms after this one).
__device__ __forceinline__ nv4f nt_row(const float4 *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const nv4f *>(p));
}
__device__ __forceinline__ void nt_row_store(float4 *p, nv4f x)
{
    __builtin_nontemporal_store(x, reinterpret_cast<nv4f *>(p));
}

constexpr int MOVE_MAX_BLOCKS = 32;
constexpr int MOVE_ROWS = 4;
// blocks of the zero-copy fill: a lane reads 16 bytes, and rows below 64 bytes
// take a read each
constexpr int move_blocks(int lpr) { return 4 * lpr < MOVE_MAX_BLOCKS ? 4 * lpr : MOVE_MAX_BLOCKS; }

template <int LPR>
__global__ void __launch_bounds__(BLOCK) k_move(float4 *__restrict__ storage, Tables tb,
                                                HostRows hr, TicketDev tk, int64_t n,
                                                int64_t nslots, float4 *__restrict__ stage,
                                                const float4 *__restrict__ staged)
{
    const int c = (int)(threadIdx.x % LPR);
    const int64_t groups = (int64_t)gridDim.x * (BLOCK / LPR);
    const int64_t g = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) / LPR;
    const uint32_t row_mask = (1u << tb.row_bits) - 1u;
    int32_t *const old_keys = reinterpret_cast<int32_t *>(stage + n * LPR);
    // whole lines at a time: the staging may be host memory
    for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * BLOCK)
        old_keys[i] = tk.v_old_key[i];
    for (int64_t i0 = g; i0 < n; i0 += groups * MOVE_ROWS) {
        // Straight-line code over the pass's MOVE_ROWS victims, with no branch
        // around a load: an entry past n reads entry i0's indices, and one
        // with nothing to read reads row 0 of the scratchpad and drops it.
        // Each round of loads is then in flight together and the values stay
        // in registers until the stores.
        bool in[MOVE_ROWS];
        int32_t old[MOVE_ROWS], v[MOVE_ROWS];
        uint32_t key[MOVE_ROWS];
#pragma unroll
        for (int q = 0; q < MOVE_ROWS; ++q) {
            const int64_t i = i0 + q * groups;
            in[q] = i < n;
            const int64_t ic = in[q] ? i : i0;
            old[q] = tk.v_old_key[ic];
            v[q] = tk.v_slot[ic];
            key[q] = tk.m_key[ic];
        }
        const float4 *src[MOVE_ROWS];
        if (staged) {
#pragma unroll
            for (int q = 0; q < MOVE_ROWS; ++q) src[q] = staged + (i0 + q * groups) * LPR + c;
        } else {
            int tab[MOVE_ROWS];
            int64_t nrows[MOVE_ROWS];
            const float4 *base[MOVE_ROWS];
#pragma unroll
            for (int q = 0; q < MOVE_ROWS; ++q) {
                tab[q] = (int)(key[q] >> tb.row_bits);
                const int tc = tab[q] < tb.T ? tab[q] : 0;
                nrows[q] = tb.rows[tc];
                base[q] = hr.p[tc];
            }
#pragma unroll
            for (int q = 0; q < MOVE_ROWS; ++q) {
                const int64_t row = key[q] & row_mask;
                src[q] = tab[q] < tb.T && row < nrows[q] ? base[q] + row * LPR + c : nullptr;
            }
        }
#pragma unroll
        for (int q = 0; q < MOVE_ROWS; ++q) {
            if (!in[q] || (uint32_t)v[q] >= (uint64_t)nslots) v[q] = -1;
            if (v[q] < 0) src[q] = nullptr;
        }
        nv4f prev[MOVE_ROWS], next[MOVE_ROWS];
#pragma unroll
        for (int q = 0; q < MOVE_ROWS; ++q) {
            prev[q] = nt_row(storage + (v[q] >= 0 && old[q] >= 0 ? (int64_t)v[q] * LPR : 0) + c);
            next[q] = nt_row(src[q] ? src[q] : storage + c);
        }
#pragma unroll
        for (int q = 0; q < MOVE_ROWS; ++q) {
            const int64_t i = i0 + q * groups;
            if (v[q] >= 0 && old[q] >= 0) nt_row_store(stage + i * LPR + c, prev[q]);
            if (src[q]) nt_row_store(storage + (int64_t)v[q] * LPR + c, next[q]);
        }
    }
}

// The write-back's copy to pinned host memory, by a few blocks of one XCD
// (block b runs on XCD b % 8; the others leave at once).  The host link takes
// 56 GB/s, which four blocks already reach; stores beyond that only wait, and
// they wait in the XCD's path to memory in front of every other kernel's
// accesses there.  Measured beside an update-like kernel (scattered rows of 512
// bytes, 224 us alone) with 66 MB on the way: 8 blocks over all XCDs hold it to
// 663 us and 256 blocks to 1182 us, as the runtime's copy kernel did (an update
// of 0.15 ms took 1.4 ms in the 8x400k x 128 workload, all of the copy's
// length); 8 blocks on one XCD leave it at 245 us and reach 55 GB/s alone.
constexpr int PUSH_BLOCKS = 8;
constexpr int PUSH_WORDS = 4;

__global__ void __launch_bounds__(BLOCK) k_push(const float4 *__restrict__ src,
                                                float4 *__restrict__ dst, int64_t words)
{
    if (blockIdx.x % XCDS) return;
    constexpr int64_t stride = (int64_t)PUSH_BLOCKS * BLOCK;
    for (int64_t i0 = (int64_t)(blockIdx.x / XCDS) * BLOCK + threadIdx.x; i0 < words;
         i0 += stride * PUSH_WORDS) {
        nv4f v[PUSH_WORDS];
#pragma unroll
        for (int q = 0; q < PUSH_WORDS; ++q) {
            const int64_t i = i0 + q * stride;
            v[q] = nt_row(src + (i < words ? i : i0));
        }
#pragma unroll
        for (int q = 0; q < PUSH_WORDS; ++q) {
            const int64_t i = i0 + q * stride;
            if (i < words) nt_row_store(dst + i, v[q]);
        }
    }
}

void launch_push(const void *src, void *dst, int64_t bytes, hipStream_t s)
{
    const int64_t words = (bytes + 15) / 16;
    if (words <= 0) return;
    hipLaunchKernelGGL(k_push, dim3(PUSH_BLOCKS * XCDS), dim3(BLOCK), 0, s, (const float4 *)src,
                       (float4 *)dst, words);
}

// ---------------------------------------------------------------- fixed scratch

// Partial sums of split runs for callers that cannot allocate: a fixed array
// per GPU, held until the process ends.  Host code never uses its name as an
// address; it takes the address hipGetSymbolAddress gives on each device.
static __device__ __align__(256) float4 scratch[STATIC_PARTIAL_BYTES / sizeof(float4)];

hipError_t static_partial_address(void **ptr)
{
    return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
}

// ---------------------------------------------------------------- dispatch

#define SP_DISPATCH_LPR(D4, KERNEL, GRID, ...)                                                   \
    switch (D4) {                                                                                \
    case 1: hipLaunchKernelGGL(KERNEL<1>, GRID, dim3(BLOCK), 0, s, __VA_ARGS__); break;          \
    case 2: hipLaunchKernelGGL(KERNEL<2>, GRID, dim3(BLOCK), 0, s, __VA_ARGS__); break;          \
    case 4: hipLaunchKernelGGL(KERNEL<4>, GRID, dim3(BLOCK), 0, s, __VA_ARGS__); break;          \
    case 8: hipLaunchKernelGGL(KERNEL<8>, GRID, dim3(BLOCK), 0, s, __VA_ARGS__); break;          \
    case 16: hipLaunchKernelGGL(KERNEL<16>, GRID, dim3(BLOCK), 0, s, __VA_ARGS__); break;        \
    case 32: hipLaunchKernelGGL(KERNEL<32>, GRID, dim3(BLOCK), 0, s, __VA_ARGS__); break;        \
    default: hipLaunchKernelGGL(KERNEL<64>, GRID, dim3(BLOCK), 0, s, __VA_ARGS__); break;        \
    }

static dim3 grid_rows(int64_t n, int D4)
{
    int64_t threads = n * D4;
    return dim3((unsigned)((threads + BLOCK - 1) / BLOCK));
}

static dim3 grid_waves(int64_t n)
{
    return dim3((unsigned)((n + BLOCK / WAVE - 1) / (BLOCK / WAVE)));
}

void launch_move(float *storage, int dim, const Tables &tb, float *const *host_dev, TicketDev tk,
                 int64_t n_miss, float *stage, const float *staged, hipStream_t s)
{
    if (n_miss <= 0) return;
    const int D4 = dim / 4;
    HostRows hr{};
    for (int t = 0; t < tb.T; ++t) hr.p[t] = (const float4 *)host_dev[t];
    // each lane group places MOVE_ROWS victims per pass
    dim3 grid = grid_rows((n_miss + MOVE_ROWS - 1) / MOVE_ROWS, D4);
    if (!staged) grid.x = grid.x < (unsigned)move_blocks(D4) ? grid.x : (unsigned)move_blocks(D4);
    SP_DISPATCH_LPR(D4, k_move, grid, (float4 *)storage, tb, hr, tk, n_miss,
                    tb.slot_base[tb.T], (float4 *)stage, (const float4 *)staged);
}

// Launches that may carry start/stop events: the events then time the kernel's
// own execution on stream s (null events = plain launch).
#define SP_DISPATCH_LPR_EV(D4, KERNEL, GRID, E0, E1, ...)                                        \
    switch (D4) {                                                                                \
    case 1: hipExtLaunchKernelGGL(KERNEL<1>, GRID, dim3(BLOCK), 0, s, E0, E1, 0, __VA_ARGS__); break;   \
    case 2: hipExtLaunchKernelGGL(KERNEL<2>, GRID, dim3(BLOCK), 0, s, E0, E1, 0, __VA_ARGS__); break;   \
    case 4: hipExtLaunchKernelGGL(KERNEL<4>, GRID, dim3(BLOCK), 0, s, E0, E1, 0, __VA_ARGS__); break;   \
    case 8: hipExtLaunchKernelGGL(KERNEL<8>, GRID, dim3(BLOCK), 0, s, E0, E1, 0, __VA_ARGS__); break;   \
    case 16: hipExtLaunchKernelGGL(KERNEL<16>, GRID, dim3(BLOCK), 0, s, E0, E1, 0, __VA_ARGS__); break; \
    case 32: hipExtLaunchKernelGGL(KERNEL<32>, GRID, dim3(BLOCK), 0, s, E0, E1, 0, __VA_ARGS__); break; \
    default: hipExtLaunchKernelGGL(KERNEL<64>, GRID, dim3(BLOCK), 0, s, E0, E1, 0, __VA_ARGS__); break; \
    }

// Whether a whole wave takes each bag: with few bags, of which groups of lanes
// would leave most of the chip idle, unless they are a few rows each; and with
// bags long enough that a wave's start does not show.  In us, groups and whole
// waves, rows of 16 / 64 floats:
//   2048 bags of   4   3.5 3.7 /  3.5 3.6     4096 bags of  10   3.7 4.0 /  4.1 3.9
//   2048 bags of  40   5.4 3.8 /  7.9 4.8     4096 bags of  20   4.4 4.0 /  5.9 4.5
//    512 bags of 300    31 6.9 /   41  13     4096 bags of 100    15  10 /   19  18
//   8192 bags of  20   5.4 6.4 /  8.6 9.4     8192 bags of  40   9.1 9.4 /   14  15
//   8192 bags of 300    47  43 /   92  89    32768 bags of 100    58  54 /  122 116
//  16384 bags of  40    15  15 /   26  26    32768 bags of  20    15  19 /   26  27
constexpr int64_t FWD_FEW_BAGS = 4096, FWD_FEW_MEAN = 16, FWD_MEAN = 100;
static bool fwd_whole_wave(int64_t nbags, int64_t nnz)
{
    return nnz >= FWD_MEAN * nbags || (nbags <= FWD_FEW_BAGS && nnz >= FWD_FEW_MEAN * nbags);
}

template <int LPR, int GW, bool SKEW>
static void forward_launch(const float4 *storage, int64_t nslots, const int32_t *inv,
                           const int32_t *slot_u, int64_t n_unique, const int32_t *bag_off,
                           int64_t nbags, float4 *out, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    hipExtLaunchKernelGGL((k_forward<LPR, GW, SKEW>), grid_rows(nbags, GW), dim3(BLOCK), 0, s, e0,
                          e1, 0, storage, inv, slot_u, n_unique, bag_off, nbags, nslots, out);
}

void launch_forward(const float *storage, int dim, int64_t nslots, const int32_t *inv,
                    const int32_t *slot_u, int64_t n_unique, const int32_t *bag_off, int64_t nbags,
                    int64_t nnz, bool long_bags, float *out, hipStream_t s, hipEvent_t e0,
                    hipEvent_t e1)
{
    if (nbags <= 0) return;
    const bool wave = fwd_whole_wave(nbags, nnz);
    auto launch = [&](auto lpr) {
        constexpr int LPR = decltype(lpr)::value, GW = fwd_lanes(LPR);
        auto *f = wave          ? forward_launch<LPR, WAVE, false>
                  : long_bags   ? forward_launch<LPR, GW, (GW < WAVE)>
                                : forward_launch<LPR, GW, false>;
        f((const float4 *)storage, nslots, inv, slot_u, n_unique, bag_off, nbags, (float4 *)out, s,
          e0, e1);
    };
    switch (dim / 4) {
    case 1: launch(std::integral_constant<int, 1>()); break;
    case 2: launch(std::integral_constant<int, 2>()); break;
    case 4: launch(std::integral_constant<int, 4>()); break;
    case 8: launch(std::integral_constant<int, 8>()); break;
    case 16: launch(std::integral_constant<int, 16>()); break;
    case 32: launch(std::integral_constant<int, 32>()); break;
    default: launch(std::integral_constant<int, 64>()); break;
    }
}

void launch_backward(float *storage, int dim, int64_t nslots, const BatchDev &b,
                     const int32_t *slot_u, int64_t n_chunks, int64_t n_multi,
                     const float *grad, int64_t nbags, float lr, float *partial, hipStream_t s,
                     hipEvent_t ev[4])
{
    if (n_chunks <= 0) return;
    const int D4 = dim / 4;
    // one lane group of D4 / VPL lanes per chunk
    SP_DISPATCH_LPR_EV(D4, k_backward, grid_rows(n_chunks, D4 / bwd_vpl(D4)), ev[0], ev[1],
                       (float4 *)storage,
                       (const int4 *)b.chunk_desc, (const int32_t *)b.sbag, slot_u, n_chunks,
                       (const float4 *)grad, nbags, nslots, lr, (float4 *)partial);
    if (n_multi <= 0) return;
    if (few_runs(n_multi, D4))
        SP_DISPATCH_LPR_EV(D4, k_bwd_combine_few, dim3((unsigned)n_multi), ev[2], ev[3],
                           (float4 *)storage, (const int32_t *)b.multi,
                           (const int32_t *)b.seg_chunk0, slot_u, (const float4 *)partial, nslots,
                           lr)
    else
        SP_DISPATCH_LPR_EV(D4, k_bwd_combine, grid_waves(n_multi), ev[2], ev[3],
                           (float4 *)storage, (const int32_t *)b.multi, n_multi,
                           (const int32_t *)b.seg_chunk0, slot_u,
                           (const float4 *)partial, nslots, lr)
}

}  // namespace sp
