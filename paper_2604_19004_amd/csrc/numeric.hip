// Numeric pass: Gustavson's row-wise product (paper Section 2.1) with
// open-addressing hash accumulators (Section 2.2) sized per bin, followed by
// the per-row sort that makes the output CSR-compliant (Section 4.2).  Rows of at
// most 2048 products are sorted instead (sortrow.hip) unless they fall on few
// columns or have more than 64 entries.
//
//   k_numeric_group   several short rows per wave (8 or 16 lanes per row), 32- or 64-slot tables in LDS
//   k_numeric_wave    one wave per row, 256-slot table in LDS
//   k_numeric_wg      one workgroup per row, keys + values + sort buffer in LDS (512..8192 slots)
//   k_numeric_hybrid  32768 keys in LDS, values accumulated in a global slab (Section 3.3,
//                     enhanced hash accumulator); rows leave sorted through an LDS bitmap rank
//   k_numeric_heavy   rows beyond the 4096-slot table (or the 2048-slot one) when B's rows are sorted: column
//                     windows, each accumulated in LDS either densely (Section 2.2 dense accumulator iterated over
//                     the row's column range as in Section 3.2) or, for stretches of several light windows, at the
//                     bitmap rank of the product's column (no hash table); products in tiles of 64
//   k_numeric_heavy_flat  rows beyond the 4096-slot table where the pieces of rows of B are short: the same
//                     windows, products numbered one by one
//   k_numeric_global  whole table in global memory, and k_numeric_hybrid: the path of such rows
//                     when B's rows are unsorted (or the window table would be too large)
//
// A row reports overflow (row_nnz = -1) when its table fills up or when it
// produced more entries than the space reserved for it; such rows are redone
// by the caller with bound-sized tables (Section 3.2, overflow handling).
#include "ocean_internal.hpp"
#include "placed.hpp"
#include "tiles.hpp"
#include "traverse.hpp"

namespace ocean {

// The type values are accumulated in inside LDS.  fp32 products are added up in fp64: the LDS atomic ds_add_f32
// measured about twenty times slower than ds_add_f64 on this GPU (a block-diagonal input, same structure in both
// types: dense accumulation 4.27 ms against 2.40 ms; with plain stores in place of the atomics 1.42 against 2.27 ms),
// so an fp32 row costs the LDS of an fp64 row and is faster for it - and closer to the exact sum.
constexpr int ilog2_const(int x) { return x <= 1 ? 0 : 1 + ilog2_const(x >> 1); }

template <typename V> struct AccOf { using type = V; };
template <> struct AccOf<float> { using type = double; };
template <typename V> using acc_t = typename AccOf<V>::type;

template <typename V>
__device__ __forceinline__ void lds_add(V *p, V v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <typename V>
__device__ __forceinline__ void l2_add(V *p, V v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Slot of a key known to be present.
template <int BITS>
__device__ __forceinline__ int lds_find(const int32_t *keys, int32_t key)
{
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    uint32_t h = table_hash(key, BITS);
    const uint32_t step = table_step(key, BITS);
    for (uint32_t probe = 0; probe <= MASK; ++probe) {
        if (keys[h] == key) return (int)h;
        h = (h + step) & MASK;
    }
    return 0;
}

// Add a batch of products to an LDS hash table (keys / vals of 2^BITS slots).
// A wave waits for its slowest lane, so the cost of inserting is set by the
// longest probe sequence among its lanes, not by the average.  Two measures
// keep that short: probe strides depend on the key (double hashing, no
// clustering), and every lane walks its own U products at its own pace - a
// lane that has placed a product goes on to its next one while other lanes are
// still probing, so the wave-wide loop runs for the largest per-lane SUM of
// probes instead of the sum of per-product maxima.  One compare-and-swap per
// lane and round; the value is added as soon as the slot is known
// (add(slot, value, whether the key is new to the table)).  Valid products come
// first in a batch (cj < 0 ends it).  False when the table is full.
template <int BITS, int U, typename V, typename AddFn>
__device__ __forceinline__ bool lds_insert_batch(int32_t *keys, const int32_t (&cj)[U], const V (&cv)[U], AddFn add)
{
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    int idx = 0;
    int32_t key = cj[0];
    V val = cv[0];
    uint32_t h = table_hash(key, BITS);
    uint32_t step = table_step(key, BITS);
    uint32_t rounds = 0;
    bool ok = true;
    while (key >= 0) {
        const int32_t old = atomicCAS(&keys[h], EMPTY_KEY, key);
        if (old == EMPTY_KEY || old == key) {
            add((int)h, val, old == EMPTY_KEY);
            ++idx;
            key = -1;
#pragma unroll
            for (int u = 1; u < U; ++u)
                if (idx == u) { key = cj[u]; val = cv[u]; }
            h = table_hash(key, BITS);
            step = table_step(key, BITS);
            rounds = 0;
        } else {
            h = (h + step) & MASK;
            if (++rounds > MASK) { ok = false; key = -1; }
        }
    }
    return ok;
}

__device__ __forceinline__ int pow2_ceil_i32(int x)
{
    return x <= 1 ? 1 : 1 << (32 - __clz(x - 1));
}

// ======================================================== group kernel ====
// Several short rows per wave: G lanes per row (16 with 64-slot tables, 8 with
// 32-slot tables), 256/G rows per workgroup; no workgroup barrier anywhere: the
// lanes of a row are part of one wave.  These rows are bound by the latency of
// their chain of dependent loads (row id -> offsets -> entries -> rows of B ->
// products), so what counts is how many rows a CU has in flight.
template <typename V, int G, int BITS>
__global__ void __launch_bounds__(256)
k_numeric_group(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
                const int32_t *__restrict__ rows, int64_t count, const int64_t *__restrict__ out_ptr,
                int32_t *__restrict__ out_col, V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    constexpr int SLOTS = 1 << BITS;
    constexpr int R = 256 / G;
    __shared__ int32_t s_keys[R * SLOTS];
    using AV = acc_t<V>;
    __shared__ AV s_vals[R * SLOTS];
    // per row: the traversal's chunk and, when the traversal is done, the gathered keys of the row's table with
    // the slot each came from, in the same memory
    struct Gathered {
        int32_t key[SLOTS];
        uint8_t slot[SLOTS];
    };
    union RowScratch {
        FlatChunk<V, G> fc;
        Gathered g;
    };
    __shared__ RowScratch s_rs[R];
    const int rl = threadIdx.x / G;
    const int sub = threadIdx.x % G;
    int32_t *keys = s_keys + rl * SLOTS;
    int32_t *sbuf = s_rs[rl].g.key;
    uint8_t *slot_of = s_rs[rl].g.slot;
    AV *vals = s_vals + rl * SLOTS;
    const int group_shift = (lane_id() / G) * G;
    const unsigned long long group_mask = (1ull << G) - 1ull;

    const int64_t r = (int64_t)blockIdx.x * R + rl;
    const bool live = r < count;
    const int64_t row = live ? rows[r] : 0;

    for (int s = sub; s < SLOTS; s += G) { keys[s] = EMPTY_KEY; vals[s] = (AV)0; }
    wave_sync();

    bool ovf = false;
    const int64_t e0 = live ? a_rp[row] : 0;
    const int64_t e1 = live ? a_rp[row + 1] : 0;
    auto f = [&](const auto &cj, const auto &cv) {
        if (!lds_insert_batch<BITS>(keys, cj, cv, [&](int slot, V v, bool) { lds_add(&vals[slot], (AV)v); })) ovf = true;
    };
    // the rows of a wave advance together: same number of G-entry chunks for all of them
    const int chunks = (int)wave_max_u32((uint32_t)((e1 - e0 + G - 1) / G));   // (uniform)
    for (int ch = 0; ch < chunks; ++ch) {
        const int64_t e = e0 + (int64_t)ch * G + sub;
        int64_t p0 = 0;
        uint32_t len = 0;
        V a = V();
        if (e < e1) {
            const int64_t k = a_col[e];
            a = a_val[e];
            p0 = b_rp[k];
            len = (uint32_t)(b_rp[k + 1] - p0);
        }
        group_flat<G, true>(s_rs[rl].fc, p0, len, a, b_col, b_val, f);
    }
    wave_sync();

    // gather the occupied keys of this row's table, and where their values are
    int c = 0;
#pragma unroll
    for (int it = 0; it < SLOTS / G; ++it) {
        const int32_t key = keys[it * G + sub];
        const bool occ = key != EMPTY_KEY;
        const unsigned long long m = (__ballot(occ) >> group_shift) & group_mask;
        if (occ) {
            const int at = c + __popcll(m & ((1ull << sub) - 1ull));
            sbuf[at] = key;
            slot_of[at] = (uint8_t)(it * G + sub);
        }
        c += __popcll(m);
    }
    const bool ovf_any = ((__ballot(ovf) >> group_shift) & group_mask) != 0;
    wave_sync();

    // Column order without a sort (Section 4.2 sorts key-pointer pairs; a row this short is cheaper to rank):
    // the place of a key is the number of smaller keys in the row.  Every lane ranks the keys t = sub, sub + G, ...
    // of the gathered list against all c of them, one broadcast read per step; the rows of a wave go through
    // the loop together, as many steps as the longest of them has keys.
    constexpr int T = SLOTS / G;
    const int cmax = (int)wave_max_u32((uint32_t)c);   // uniform for the wave
    int32_t mk[T];
    int rank[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int t = sub + i * G;
        mk[i] = t < c ? sbuf[t] : SORT_PAD;
        rank[i] = 0;
    }
    // (TT: keys per lane that the longest row of the wave needs ranked)
    auto count_smaller = [&](auto tt) {
        constexpr int TT = decltype(tt)::value;
        for (int j = 0; j < cmax; ++j) {
            const int32_t kr = sbuf[j];                   // (j < SLOTS; beyond the row's keys whatever is there)
            const int32_t kj = j < c ? kr : SORT_PAD;     // nothing is smaller than the pad
#pragma unroll
            for (int i = 0; i < TT; ++i) rank[i] += kj < mk[i];
        }
    };
    if (cmax <= G) count_smaller(std::integral_constant<int, 1>{});
    else if (cmax <= 2 * G) count_smaller(std::integral_constant<int, 2>{});
    else count_smaller(std::integral_constant<int, T>{});

    if (live) {
        const int64_t o = out_ptr[row];
        const int64_t cap = out_ptr[row + 1] - o;
        if (ovf_any || (int64_t)c > cap) {
            if (sub == 0) row_nnz[row] = -1;
        } else {
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const int t = sub + i * G;
                if (t < c) {
                    out_col[o + rank[i]] = mk[i];
                    out_val[o + rank[i]] = (V)vals[slot_of[t]];
                }
            }
            if (sub == 0) row_nnz[row] = c;
        }
    }
}

// =================================================== workgroup helpers ====
// s_wave: one word per wave.  With TRAILING_BARRIER = false the caller keeps s_wave untouched until
// a later barrier of its own.
template <int THREADS, bool TRAILING_BARRIER = true>
__device__ __forceinline__ int block_exclusive_scan_i32(int v, int *s_wave, int &total)
{
    const int inc = (int)wave_inclusive_scan_u32((uint32_t)v);
    const int w = threadIdx.x / WAVE;
    if (lane_id() == WAVE - 1) s_wave[w] = inc;
    __syncthreads();
    uint32_t tot;
    const int wave_off = (int)waves_before_u32<THREADS / WAVE>(reinterpret_cast<const uint32_t *>(s_wave), w, tot);
    if (TRAILING_BARRIER) __syncthreads();
    total = (int)tot;
    return wave_off + inc - v;
}

// Who works on one row: a whole workgroup of THREADS threads, or one wave (THREADS = 64) among several
// in a workgroup that each have a row of their own.  The ordered write-out below is written once for both.
struct WorkgroupScope {
    static __device__ __forceinline__ int tid() { return (int)threadIdx.x; }
    static __device__ __forceinline__ void sync() { __syncthreads(); }
    template <int THREADS>
    static __device__ __forceinline__ int exclusive_scan(int v, int *s_wave, int &total)
    {
        return block_exclusive_scan_i32<THREADS>(v, s_wave, total);
    }
};
struct WaveScope {
    static __device__ __forceinline__ int tid() { return lane_id(); }
    static __device__ __forceinline__ void sync() { wave_sync(); }
    template <int THREADS>
    static __device__ __forceinline__ int exclusive_scan(int v, int *, int &total)
    {
        static_assert(THREADS == WAVE, "one wave");
        const int inc = (int)wave_inclusive_scan_u32((uint32_t)v);
        total = (int)wave_read_lane_u32((uint32_t)inc, WAVE - 1);
        return inc - v;
    }
};

// Write the keys of an LDS hash table to the output in increasing column order
// without sorting them.  Every thread holds PER keys of the table in registers
// (EMPTY_KEY = none; key[q] sits in slot q*THREADS + tid).  The keys are counted
// into NB = THREADS*PER buckets of W = 2^shift columns starting at kmin (all keys
// lie in [kmin, kmin + NB*W)), and a prefix sum over the counts gives every
// bucket its range [start, start + count) of the output, which is also its
// private range of the NB-word array `grouped`.  Inside a bucket the rank of a
// key is found in one of two ways, whichever is cheap for that bucket:
//   * a bucket with fewer keys than the W/32 words of a bitmap over its columns
//     lists its keys in its range (the atomic that counted a key also returned
//     its arrival index) and a key counts the smaller ones among them;
//   * a bucket with at least that many keys (a cluster of columns) has room in
//     its range for that bitmap: the keys set their bits and a key's rank is the
//     number of set bits below its own.
// So clustered and scattered columns cost about the same, a few LDS accesses
// per key.  With BF > 1 there are BF buckets per table slot (NB = THREADS*PER*BF): a
// cluster's bitmap then has fewer words below a key's own, and the threads of a wave
// wait for the longest such count among them.  hist: NB/2 + 1 words, zeroed, two
// 16-bit counts per word.  Returns
// the number of keys; with CHECK, -1 (and nothing written) when some listed
// bucket holds more than `limit` keys, for the caller to sort instead.
// Barriers inside; ends without one.  The table's values are overwritten (the
// keys and values are put in order inside LDS and copied out from there).
// `grouped` may be the table's own key array, provided every thread has read
// its keys before the call (barrier).
template <int THREADS, int PER, bool CHECK, typename Scope = WorkgroupScope, int BF = 1, typename AV, typename V>
__device__ __forceinline__ int bucket_emit(const int32_t (&key)[PER], AV *s_vals, int32_t kmin, int shift,
                                           uint32_t *hist, int32_t *grouped, int *s_wave, int *s_flag, int limit,
                                           int64_t o, int64_t cap, long long done, int32_t *__restrict__ out_col,
                                           V *__restrict__ out_val)
{
    static_assert(PER % 2 == 0, "two buckets per word");
    constexpr int NB = THREADS * PER * BF;   // BF buckets per table slot: narrower buckets, shorter bitmaps to rank in
    constexpr int OWNW = PER * BF / 2;       // words of counts (two buckets each) that a thread owns
    const int tid = Scope::tid();
    const int words = shift > 5 ? 1 << (shift - 5) : 1;   // bitmap words of one bucket
    const uint32_t wmask = (1u << shift) - 1u;
    int arrival[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        arrival[q] = 0;
        if (key[q] != EMPTY_KEY) {
            const uint32_t b = (uint32_t)(key[q] - kmin) >> shift;
            const uint32_t old = atomicAdd(&hist[b >> 1], 1u << ((b & 1u) * 16));
            arrival[q] = (int)((old >> ((b & 1u) * 16)) & 0xffffu);
        }
    }
    Scope::sync();
#pragma unroll
    for (int q = 0; q < PER; ++q) grouped[q * THREADS + tid] = 0;
    // counts -> starts, in place; this thread owns buckets 2*tid*OWNW .. 2*(tid+1)*OWNW - 1
    uint32_t wv[OWNW];
    int sum = 0, kmax = 0;
#pragma unroll
    for (int j = 0; j < OWNW; ++j) {
        wv[j] = hist[tid * OWNW + j];
        const int c0 = (int)(wv[j] & 0xffffu), c1 = (int)(wv[j] >> 16);
        sum += c0 + c1;
        if (c0 < words) kmax = max(kmax, c0);
        if (c1 < words) kmax = max(kmax, c1);
    }
    if (CHECK && kmax > limit) *s_flag = 1;
    int total;
    int base = Scope::template exclusive_scan<THREADS>(sum, s_wave, total);
#pragma unroll
    for (int j = 0; j < OWNW; ++j) {
        const int c0 = (int)(wv[j] & 0xffffu), c1 = (int)(wv[j] >> 16);
        hist[tid * OWNW + j] = (uint32_t)base | ((uint32_t)(base + c0) << 16);
        base += c0 + c1;
    }
    if (tid == THREADS - 1) hist[NB / 2] = (uint32_t)total;
    Scope::sync();
    if (CHECK && *s_flag) return -1;   // uniform
    auto start_of = [&](uint32_t b) { return (int)((hist[b >> 1] >> ((b & 1u) * 16)) & 0xffffu); };
    int lo[PER];
    bool bitmap[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        lo[q] = 0; bitmap[q] = false;
        if (key[q] != EMPTY_KEY) {
            const uint32_t x = (uint32_t)(key[q] - kmin);
            const uint32_t b = x >> shift, d = x & wmask;
            lo[q] = start_of(b);
            bitmap[q] = start_of(b + 1) - lo[q] >= words;
            if (bitmap[q]) atomicOr(reinterpret_cast<uint32_t *>(&grouped[lo[q] + (int)(d >> 5)]), 1u << (d & 31u));
            else grouped[lo[q] + arrival[q]] = key[q];
        }
    }
    Scope::sync();
    int rank[PER];
    AV val[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        rank[q] = 0;
        val[q] = AV();
        if (key[q] != EMPTY_KEY) {
            const uint32_t x = (uint32_t)(key[q] - kmin);
            const uint32_t b = x >> shift, d = x & wmask;
            int r = lo[q];
            if (bitmap[q]) {
                const int dw = (int)(d >> 5);
                for (int j = 0; j < dw; ++j) r += __popc((uint32_t)grouped[lo[q] + j]);
                r += __popc((uint32_t)grouped[lo[q] + dw] & ((1u << (d & 31u)) - 1u));
            } else {
                const int hi = start_of(b + 1);
                for (int i = lo[q]; i < hi; ++i) r += grouped[i] < key[q];
            }
            rank[q] = r;
            val[q] = s_vals[q * THREADS + tid];
        }
    }
    Scope::sync();
    // permute keys and values into place inside LDS (every thread holds its own in registers), so
    // that the row leaves with coalesced stores
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (key[q] != EMPTY_KEY) { grouped[rank[q]] = key[q]; s_vals[rank[q]] = val[q]; }
    Scope::sync();
    const long long room = cap - done;
    const int n_out = (long long)total < room ? total : (room > 0 ? (int)room : 0);
    for (int i = tid; i < n_out; i += THREADS) {
        out_col[o + done + i] = grouped[i];
        out_val[o + done + i] = (V)s_vals[i];
    }
    return total;
}

// ========================================================= wave kernel ====
// One wave per row, R rows per workgroup, a table of 2^BITS slots (256, 512 or 1024) per row.  No
// workgroup barrier anywhere: traversal, insertion and the ordered write-out (column buckets, as in the
// workgroup kernels) are all wave-synchronous, so a row costs one wave's instructions instead of a
// workgroup's, and none of the waiting at barriers.  Rows of these sizes are bound by instruction issue,
// not by memory.
template <typename V, int BITS, int R>
__global__ void __launch_bounds__(WAVE * R)
k_numeric_wave(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
               const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
               const int32_t *__restrict__ rows, int64_t count, const int64_t *__restrict__ out_ptr,
               int32_t *__restrict__ out_col, V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    constexpr int SLOTS = 1 << BITS;
    constexpr int PER = SLOTS / WAVE;
    constexpr int BF = 1;
    constexpr int NBK = SLOTS * BF;
    // the traversal's chunk and, after it, the bucket counts of the ordered write-out share one buffer per row
    constexpr size_t HIST_BYTES = (NBK / 2 + 1) * sizeof(uint32_t);
    constexpr size_t SCRATCH = sizeof(FlatChunk<V, WAVE>) > HIST_BYTES ? sizeof(FlatChunk<V, WAVE>) : HIST_BYTES;
    using AV = acc_t<V>;
    __shared__ int32_t s_keys[R * SLOTS];
    __shared__ AV s_vals[R * SLOTS];
    __shared__ __align__(16) unsigned char s_scratch[R][(SCRATCH + 15) / 16 * 16];
    __shared__ int s_flag[R];
    const int rl = threadIdx.x / WAVE;
    const int sub = lane_id();
    int32_t *keys = s_keys + rl * SLOTS;
    AV *vals = s_vals + rl * SLOTS;
    FlatChunk<V, WAVE> &fc = *reinterpret_cast<FlatChunk<V, WAVE> *>(s_scratch[rl]);
    uint32_t *hist = reinterpret_cast<uint32_t *>(s_scratch[rl]);
    const int64_t r = (int64_t)blockIdx.x * R + rl;
    if (r >= count) return;   // whole wave leaves; no workgroup barrier is used below
    const int64_t row = rows[r];
    for (int s = sub; s < SLOTS; s += WAVE) { keys[s] = EMPTY_KEY; vals[s] = (AV)0; }
    wave_sync();
    bool ovf = false;
    wave_traverse<true>(a_col, a_val, a_rp[row], a_rp[row + 1],
                        [&](int32_t k, int64_t &p0, int64_t &len) { p0 = b_rp[k]; len = b_rp[k + 1] - p0; },
                        b_col, b_val, fc, [&](const auto &cj, const auto &cv) {
                            if (!lds_insert_batch<BITS>(keys, cj, cv, [&](int slot, V v, bool) { lds_add(&vals[slot], (AV)v); })) ovf = true;
                        });
    wave_sync();
    // ---- ordered write-out through column buckets
    int32_t key[PER];
    int lmin = 0x7fffffff, lmax = -1;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        key[q] = keys[q * WAVE + sub];
        if (key[q] != EMPTY_KEY) { lmin = min(lmin, key[q]); lmax = max(lmax, key[q]); }
    }
    for (int j = sub; j < NBK / 2 + 1; j += WAVE) hist[j] = 0u;
    // (column ids are not negative: both extremes as maxima of unsigned numbers)
    const int kmax = (int)wave_max_u32((uint32_t)(lmax + 1)) - 1;
    const int kmin = 0x7fffffff - (int)wave_max_u32((uint32_t)(0x7fffffff - lmin));
    const bool ovf_any = __ballot(ovf) != 0;
    if (kmax < 0) {   // uniform: the row has no entries
        if (sub == 0) row_nnz[row] = 0;
        return;
    }
    wave_sync();   // every lane holds its keys in registers (the key array becomes the buckets' memory), counts are zero
    // smallest shift with (kmax - kmin) >> shift < NBK: the bits of the range beyond those of the bucket count
    static_assert((NBK & (NBK - 1)) == 0, "bucket count is a power of two");
    const int range_bits = 32 - __clz((uint32_t)(kmax - kmin) | 1u);
    const int shift = range_bits > ilog2_const(NBK) ? range_bits - ilog2_const(NBK) : 0;
    const int64_t o = out_ptr[row];
    const int64_t cap = out_ptr[row + 1] - o;
    const int c = bucket_emit<WAVE, PER, false, WaveScope, BF>(key, vals, kmin, shift, hist, keys, nullptr, &s_flag[rl], 0, o, cap, 0,
                                                           out_col, out_val);
    if (sub == 0) row_nnz[row] = (ovf_any || (int64_t)c > cap) ? -1 : c;
}

// ==================================================== workgroup kernel ====
// BF: column buckets per table slot of the ordered write-out (see bucket_emit): 1, or more for inputs with
// clustered columns, up to 2048 buckets.
template <typename V, int BITS, int THREADS, int BF>
__global__ void __launch_bounds__(THREADS)
k_numeric_wg(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
             const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
             const int32_t *__restrict__ rows, int64_t count, const int64_t *__restrict__ out_ptr,
             int32_t *__restrict__ out_col, V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    constexpr int SLOTS = 1 << BITS;
    constexpr int PER = SLOTS / THREADS;
    constexpr int NBK = SLOTS * BF;
    __shared__ int32_t s_keys[SLOTS];
    using AV = acc_t<V>;
    __shared__ int32_t s_sort[SLOTS];
    __shared__ AV s_vals[SLOTS];
    // the traversal's chunk and, after it, the bucket counts of the ordered write-out share one buffer
    constexpr size_t HIST_BYTES = (NBK / 2 + 1) * sizeof(uint32_t);
    constexpr size_t SCRATCH = sizeof(WgChunk<V, THREADS>) > HIST_BYTES ? sizeof(WgChunk<V, THREADS>) : HIST_BYTES;
    __shared__ __align__(16) unsigned char s_scratch[(SCRATCH + 15) / 16 * 16];
    __shared__ int s_wave[THREADS / WAVE];
    __shared__ int s_ovf, s_min, s_max, s_flag;
    WgChunk<V, THREADS> &s_fc = *reinterpret_cast<WgChunk<V, THREADS> *>(s_scratch);
    uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_scratch);
    const int tid = threadIdx.x;
    const int64_t r = blockIdx.x;
    if (r >= count) return;
    const int64_t row = rows[r];

    for (int s = tid; s < SLOTS; s += THREADS) { s_keys[s] = EMPTY_KEY; s_vals[s] = (AV)0; }
    if (tid == 0) { s_ovf = 0; s_min = 0x7fffffff; s_max = -1; s_flag = 0; }
    __syncthreads();

    wg_traverse<THREADS, true>(a_col, a_val, a_rp[row], a_rp[row + 1],
                               [&](int32_t k, int64_t &p0, int64_t &len) { p0 = b_rp[k]; len = b_rp[k + 1] - p0; },
                               b_col, b_val, s_fc, [&](const auto &cj, const auto &cv) {
                                   if (!lds_insert_batch<BITS>(s_keys, cj, cv, [&](int slot, V v, bool) { lds_add(&s_vals[slot], (AV)v); }))
                                       s_ovf = 1;
                               });
    // wg_traverse ends with a barrier

    const int64_t o = out_ptr[row];
    const int64_t cap = out_ptr[row + 1] - o;
    // ---- ordered write-out through column buckets
    int32_t key[PER];
    int lmin = 0x7fffffff, lmax = -1;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        key[q] = s_keys[q * THREADS + tid];
        if (key[q] != EMPTY_KEY) { lmin = min(lmin, key[q]); lmax = max(lmax, key[q]); }
    }
    for (int j = tid; j < NBK / 2 + 1; j += THREADS) s_hist[j] = 0u;
    // (column ids are not negative: both extremes as maxima of unsigned numbers)
    lmax = (int)wave_max_u32((uint32_t)(lmax + 1)) - 1;
    lmin = 0x7fffffff - (int)wave_max_u32((uint32_t)(0x7fffffff - lmin));
    if (lane_id() == 0 && lmax >= 0) { atomicMin(&s_min, lmin); atomicMax(&s_max, lmax); }
    __syncthreads();
    const int kmin = __builtin_amdgcn_readfirstlane(s_min), kmax = __builtin_amdgcn_readfirstlane(s_max);   // (the same in every thread)
    if (kmax < 0) {   // uniform: the row has no entries
        if (tid == 0) row_nnz[row] = 0;
        return;
    }
    // smallest shift with (kmax - kmin) >> shift < NBK: the bits of the range beyond those of the bucket count
    static_assert((NBK & (NBK - 1)) == 0, "bucket count is a power of two");
    const int range_bits = 32 - __clz((uint32_t)(kmax - kmin) | 1u);
    const int shift = range_bits > ilog2_const(NBK) ? range_bits - ilog2_const(NBK) : 0;
    constexpr bool CHECK = SLOTS >= 4096;   // smaller tables: even one bucket with every key is cheap to rank
    int c = bucket_emit<THREADS, PER, CHECK, WorkgroupScope, BF>(key, s_vals, kmin, shift, s_hist, s_sort, s_wave, &s_flag, 1024, o, cap, 0,
                                             out_col, out_val);
    if (c >= 0) {
        if (tid == 0) row_nnz[row] = (s_ovf || (int64_t)c > cap) ? -1 : c;
        return;
    }

    // ---- columns too clustered for the buckets: compact the keys, sort them (bitonic), look the values up
    int mine = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) mine += (key[q] != EMPTY_KEY);
    int pos = block_exclusive_scan_i32<THREADS>(mine, s_wave, c);
#pragma unroll
    for (int q = 0; q < PER; ++q)
        if (key[q] != EMPTY_KEY) s_sort[pos++] = key[q];
    const int N = pow2_ceil_i32(c);
    __syncthreads();
    for (int s = c + tid; s < N; s += THREADS) s_sort[s] = SORT_PAD;
    __syncthreads();

    for (int k = 2; k <= N; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < (N >> 1); i += THREADS) {
                const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                const int hi = lo | j;
                const int32_t x = s_sort[lo], y = s_sort[hi];
                if ((x > y) == ((lo & k) == 0)) { s_sort[lo] = y; s_sort[hi] = x; }
            }
            __syncthreads();
        }
    }

    if (s_ovf || (int64_t)c > cap) {
        if (tid == 0) row_nnz[row] = -1;
    } else {
        for (int t = tid; t < c; t += THREADS) {
            const int32_t k2 = s_sort[t];
            out_col[o + t] = k2;
            out_val[o + t] = (V)s_vals[lds_find<BITS>(s_keys, k2)];
        }
        if (tid == 0) row_nnz[row] = c;
    }
}

// A product as it is added to an accumulator that says by -0 that nothing has been added yet: never -0 itself.  (As a
// multiplication and an addition of their own: contracted, a negative product that underflows would stay -0.)
template <typename V>
__device__ __forceinline__ double dense_addend(V v)
{
#pragma clang fp contract(off)
    return (double)v + 0.0;
}

// Whether something has been added to such an accumulator.
__device__ __forceinline__ bool dense_there(double v) { return __double_as_longlong(v) != (long long)0x8000000000000000ull; }

// ================================================== dense-range kernel ====
// Dense accumulator (Section 2.2) over the row's own column range, for rows whose range [cmin, cmin + DS_MAX_COLS)
// is no larger than the hash table they would get (Section 3.3, accumulator selection): an accumulator per column of
// the range in LDS, no keys, no probing.  As in the dense windows of the heavy rows, -0 says that nothing has been added
// to a column, so a product is one LDS add and nothing else; a ballot per 64 columns numbers the row's entries in
// column order.  A product
// outside the range (B's rows not in column order: the range was a guess) makes the row report overflow, like a
// row with more entries than were reserved for it; the caller redoes such rows with hash tables.
// COLS: columns the range may have (4096, or less where the rows' ranges allow it: what LDS a row takes decides how many
// rows a compute unit works on, and every column is cleared and looked at.  100 000 rows of 2500 products in blocks of
// 1000 columns: 842 us with 4096).
// TILED: products in tiles of 64 entries of a row of B (tiles.hpp) instead of numbered one by one.  dspan_in_tiles says where.
// What bounds it is what its waves issue and wait for, row by row: 60 000 rows in blocks of 1000 columns, rows of B of 50 entries, fp64,
// numeric stage 393 us with presence bits that were read before they were set, 370 without them, 378 in tiles whose next
// steps were loaded ahead (78 registers, 6 waves a SIMD), 342 in tiles loaded when they are used (55 registers, 8 waves): so
// where fp64 values would cost the waves.  Rows of 78 entries 675, 605, 511, 467; blocks of 4000 columns (LDS for four waves),
// 50 entries: 736, 650, 594, 605; fp32, 1000 columns, 50 entries: 347, 318, 289, 289.
// PLACED: all rows in order, a workgroup each, which waits for the row's place in C (placed.hpp; rows, out_ptr and row_nnz are
// not used); a product outside the range ends the attempt.  Workgroup 0 gives the places.
constexpr int DS_THREADS = 256;
template <typename V, bool TILED, int COLS, bool PLACED>
__global__ void __launch_bounds__(DS_THREADS, COLS <= 1024 ? 8 : COLS <= 2048 ? 7 : 4)   // (waves a SIMD that the LDS allows)
k_numeric_dspan(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
                const int32_t *__restrict__ rows, int64_t count, const int32_t *__restrict__ cmin,
                const int64_t *__restrict__ out_ptr, int32_t *__restrict__ out_col, V *__restrict__ out_val,
                int32_t *__restrict__ row_nnz, const Placing<V> p)
{
    constexpr int WAVES = DS_THREADS / WAVE;
    constexpr int PER = COLS / DS_THREADS;   // a wave looks at PER times 64 columns that lie together
    using Chunk = std::conditional_t<TILED, TileChunk<V, uint32_t, DS_THREADS>, WgChunk<V, DS_THREADS>>;
    __shared__ double s_vals[COLS + (TILED ? WAVE : 0)];   // (behind the columns: a place per lane for what is no product)
    __shared__ Chunk s_ch;
    __shared__ uint32_t s_wave[WAVES];
    __shared__ int s_bad;
    __shared__ long long s_place;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    if (PLACED && blockIdx.x == 0) {   // uniform
        static_assert(sizeof(Turn) <= sizeof(s_vals), "the places are given from the accumulators' memory");
        place_units(p.counts, p.places, p.m, p.total, p.flags, p.placer_polls, *reinterpret_cast<Turn *>(s_vals));
        return;
    }
    const int64_t r = (int64_t)blockIdx.x - (PLACED ? 1 : 0);
    if (!PLACED && r >= count) return;
    const int64_t row = PLACED ? r : (int64_t)rows[r];
    const int32_t c0 = cmin[row];
    for (int j = tid; j < COLS; j += DS_THREADS) s_vals[j] = -0.0;
    if (tid == 0) s_bad = 0;
    if constexpr (TILED) {
        const int64_t e0 = a_rp[row], e1 = a_rp[row + 1];
        uint32_t farthest = 0u;   // columns from c0 on, of this lane's products
        for (int64_t base = e0; base < e1; base += DS_THREADS) {
            const int64_t e = base + tid;
            int64_t p0 = 0, len = 0;
            V a = V();
            if (e < e1) {
                const int32_t k = a_col[e];
                a = a_val[e];
                p0 = b_rp[k];
                len = b_rp[k + 1] - p0;
            }
            if (base > e0) __syncthreads();   // (the chunk may still be read)
            const int nent = e1 - base < DS_THREADS ? (int)(e1 - base) : DS_THREADS;
            const uint32_t total = tile_open<DS_THREADS>(s_ch, nent, (uint32_t)p0, (uint32_t)len, a);   // (the accumulators are clear, too)
            if (total == 0u) continue;   // uniform
            Tiles<V, uint32_t> tiles;
            constexpr bool AHEAD = sizeof(V) == 4 || COLS > 2048;
            tile_walk<DS_THREADS, 2, true, AHEAD>(s_ch, nent, total, b_col, b_val, tiles, false, [&](const TileFour<V> (&f)[2], const Tiles<V, uint32_t> &t) {
                const V av[2] = {row_lane<0>(t.a), row_lane<1>(t.a)};
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (f[u].skip >= 4) continue;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t d = (uint32_t)(f[u].col[i] - c0);   // (a column before c0 wraps to a large number)
                        const bool own = i >= f[u].skip && f[u].col[i] >= 0;
                        farthest = own && d > farthest ? d : farthest;
                        lds_add(&s_vals[own && d < (uint32_t)COLS ? d : (uint32_t)(COLS + lane)], dense_addend(av[u] * f[u].val[i]));
                    }
                }
            });
        }
        if (farthest >= (uint32_t)COLS) s_bad = 1;
        __syncthreads();
    } else {
        __syncthreads();
        wg_traverse<DS_THREADS, true>(a_col, a_val, a_rp[row], a_rp[row + 1],
                                      [&](int32_t k, int64_t &p0, int64_t &len) { p0 = b_rp[k]; len = b_rp[k + 1] - p0; },
                                      b_col, b_val, s_ch, [&](const auto &cj, const auto &cv) {
                                          constexpr int U = sizeof(cj) / sizeof(cj[0]);
#pragma unroll
                                          for (int u = 0; u < U; ++u) {
                                              if (cj[u] < 0) continue;
                                              const uint32_t d = (uint32_t)(cj[u] - c0);
                                              if (d < (uint32_t)COLS) lds_add(&s_vals[d], dense_addend(cv[u]));
                                              else s_bad = 1;
                                          }
                                      });
        // (wg_traverse ends with a barrier)
    }
    const int j0 = wave * (COLS / WAVES) + lane;   // the lane's columns: j0, j0 + 64, ...
    double v[PER];
    unsigned long long there[PER];
    uint32_t mine = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = s_vals[j0 + i * WAVE];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        there[i] = __ballot(dense_there(v[i]));
        mine += (uint32_t)__popcll(there[i]);
    }
    if (lane == 0) s_wave[wave] = mine;
    __syncthreads();
    uint32_t total;
    const uint32_t before = waves_before_u32<WAVES>(s_wave, wave, total);
    int64_t o;
    if constexpr (PLACED) {
        if (wave == 0) {
            if (lane == 0) {
                if (s_bad) atomicOr(p.flags, FLAG_GAVE_UP);
                post(p.counts + row, total + 1u);
            }
            const int64_t place = wait_for_place(p.places + row, p.flags, p.unit_polls);
            if (lane == 0) {
                s_place = place;
                if (place >= 0) {
                    p.c_rp[row] = place;
                    if (row == p.m - 1) p.c_rp[p.m] = place + total;
                }
            }
        }
        __syncthreads();
        o = s_place;
        if (o < 0 || o + total > p.slots) return;   // uniform
    } else {
        o = out_ptr[row];
        const int64_t cap = out_ptr[row + 1] - o;
        if (s_bad || (int64_t)total > cap) {   // uniform
            if (tid == 0) row_nnz[row] = -1;
            return;
        }
        if (tid == 0) row_nnz[row] = (int)total;
    }
    int32_t *to_col = out_col + o;
    V *to_val = out_val + o;
    uint32_t at = before;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(there[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)there[i], at));
        if ((there[i] >> lane) & 1ull) {
            to_col[rank] = c0 + j0 + i * WAVE;
            to_val[rank] = (V)v[i];
        }
        at += (uint32_t)__popcll(there[i]);
    }
}

// All rows through the dense accumulator over their ranges, of at most l.span_cols columns, straight to their places.
template <typename V>
static hipError_t dispatch_placed_span(const Csr &A, const Csr &B, const PlacedLaunch &l, hipStream_t s)
{
    const V *av = static_cast<const V *>(A.val);
    const V *bv = static_cast<const V *>(B.val);
    V *ov = static_cast<V *>(l.out_val);
    const Placing<V> p{A.rows, l.c_rp, l.out_col, ov, l.slots, l.counts, l.places, l.total, l.flags, l.placer_polls, l.unit_polls};
    const auto kernel = l.tiled ? (l.span_cols <= 1024   ? k_numeric_dspan<V, true, 1024, true>
                                   : l.span_cols <= 2048 ? k_numeric_dspan<V, true, 2048, true>
                                                         : k_numeric_dspan<V, true, (int)DS_MAX_COLS, true>)
                                : (l.span_cols <= 1024   ? k_numeric_dspan<V, false, 1024, true>
                                   : l.span_cols <= 2048 ? k_numeric_dspan<V, false, 2048, true>
                                                         : k_numeric_dspan<V, false, (int)DS_MAX_COLS, true>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(A.rows + 1)), dim3(DS_THREADS), 0, s, A.rp, A.col, av, B.rp, B.col, bv, nullptr, A.rows,
                       l.cmin, nullptr, l.out_col, ov, nullptr, p);
    return hipGetLastError();
}

hipError_t launch_placed_span(const Csr &A, const Csr &B, int dtype, const PlacedLaunch &l, hipStream_t s)
{
    if (A.rows <= 0) return hipSuccess;
    if (l.cmin == nullptr || l.span_cols > DS_MAX_COLS) return hipErrorInvalidValue;
    return dtype == OCEAN_F64 ? dispatch_placed_span<double>(A, B, l, s) : dispatch_placed_span<float>(A, B, l, s);
}

// ======================================================= hybrid kernel ====
// Keys of a 32768-slot table stay in LDS; values are accumulated with
// fire-and-forget atomics into this workgroup's slab in global memory (it is
// 256 KB, so it lives in the L2 of the XCD the workgroup runs on).  The row is
// emitted in ascending order without a comparison sort: the (key, slot) pairs
// are first dumped to a list in global memory, which frees the 128 KB of keys
// for a bitmap over 512 K columns plus its per-word prefix popcount; a key's
// rank in the row is then the number of set bits below it.
constexpr int HY_BITS = 15;
constexpr int HY_SLOTS = 1 << HY_BITS;
constexpr int HY_THREADS = 1024;
constexpr int HY_WIN = 524288;          // columns per ranking window
constexpr int HY_WORDS = HY_WIN / 32;   // 16384 bitmap words + 16384 prefix words = the key table's 128 KB

template <typename V>
__global__ void __launch_bounds__(HY_THREADS)
k_numeric_hybrid(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                 const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
                 const int32_t *__restrict__ rows, int64_t count, unsigned long long *queue,
                 V *__restrict__ slab_all, uint2 *__restrict__ pairs_all, const int64_t *__restrict__ out_ptr,
                 int32_t *__restrict__ out_col, V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    constexpr int PER = HY_SLOTS / HY_THREADS;   // 32 slots per thread
    constexpr int WPT = HY_WORDS / HY_THREADS;   // 16 bitmap words per thread
    __shared__ int32_t s_keys[HY_SLOTS];
    __shared__ WgChunk<V, HY_THREADS> s_fc;
    __shared__ int s_wave[HY_THREADS / WAVE];
    __shared__ int s_ovf;
    __shared__ int s_min, s_max;
    __shared__ unsigned int s_cnt;
    __shared__ long long s_row;
    uint32_t *s_bm = reinterpret_cast<uint32_t *>(s_keys);   // valid only after the keys were dumped
    uint32_t *s_pre = s_bm + HY_WORDS;
    const int tid = threadIdx.x;
    V *slab = slab_all + (size_t)blockIdx.x * HY_SLOTS;
    uint2 *pairs = pairs_all + (size_t)blockIdx.x * HY_SLOTS;

    for (;;) {
        if (tid == 0) s_row = (long long)atomicAdd(queue, 1ull);
        __syncthreads();
        const int64_t r = s_row;
        if (r >= count) break;   // uniform: every wave of the workgroup leaves here
        const int64_t row = rows[r];
        for (int s = tid; s < HY_SLOTS; s += HY_THREADS) s_keys[s] = EMPTY_KEY;
        if (tid == 0) { s_ovf = 0; s_min = 0x7fffffff; s_max = -1; s_cnt = 0; }
        __syncthreads();

        wg_traverse<HY_THREADS, true>(a_col, a_val, a_rp[row], a_rp[row + 1],
                                      [&](int32_t k, int64_t &p0, int64_t &len) { p0 = b_rp[k]; len = b_rp[k + 1] - p0; },
                                      b_col, b_val, s_fc, [&](const auto &cj, const auto &cv) {
                                          if (!lds_insert_batch<HY_BITS>(s_keys, cj, cv, [&](int slot, V v, bool) { l2_add(&slab[slot], v); }))
                                              s_ovf = 1;
                                      });
        __threadfence();   // the slab additions are in L2 before anyone exchanges them out
        __syncthreads();

        // dump (key, slot) pairs; one LDS atomic per wave and pass
        int kmin = 0x7fffffff, kmax = -1;
        for (int q = 0; q < PER; ++q) {
            const int slot = q * HY_THREADS + tid;
            const int32_t key = s_keys[slot];
            const bool occ = key != EMPTY_KEY;
            const unsigned long long m = __ballot(occ);
            unsigned int base = 0;
            if (lane_id() == 0 && m) base = atomicAdd(&s_cnt, (unsigned int)__popcll(m));
            base = __shfl(base, 0, WAVE);
            if (occ) {
                pairs[base + __popcll(m & ((1ull << lane_id()) - 1ull))] = make_uint2((unsigned)key, (unsigned)slot);
                kmin = key < kmin ? key : kmin;
                kmax = key > kmax ? key : kmax;
            }
        }
        kmin = -group_reduce_max(-kmin, WAVE);
        kmax = group_reduce_max(kmax, WAVE);
        if (lane_id() == 0) { atomicMin(&s_min, kmin); atomicMax(&s_max, kmax); }
        __threadfence();   // the pairs are read back by other waves of this workgroup
        __syncthreads();

        const int64_t o = out_ptr[row];
        const int64_t cap = out_ptr[row + 1] - o;
        const int lo_key = s_min, hi_key = s_max;
        const int c = (int)s_cnt;
        int done = 0;
        for (int64_t w0 = (int64_t)(lo_key >= 0 ? lo_key : 0) & ~(int64_t)(HY_WIN - 1); w0 <= (int64_t)hi_key; w0 += HY_WIN) {
#pragma unroll
            for (int q = 0; q < WPT; ++q) s_bm[q * HY_THREADS + tid] = 0u;
            __syncthreads();
            for (int i = tid; i < c; i += HY_THREADS) {
                const int64_t d = (int64_t)(int32_t)__hip_atomic_load(&pairs[i].x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - w0;
                if (d >= 0 && d < HY_WIN) atomicOr(&s_bm[d >> 5], 1u << (d & 31));
            }
            __syncthreads();
            int cnt[WPT];
            int mine = 0;
#pragma unroll
            for (int q = 0; q < WPT; ++q) { cnt[q] = __popc(s_bm[tid * WPT + q]); mine += cnt[q]; }
            int wtotal;
            int run = block_exclusive_scan_i32<HY_THREADS>(mine, s_wave, wtotal);
#pragma unroll
            for (int q = 0; q < WPT; ++q) { s_pre[tid * WPT + q] = (uint32_t)run; run += cnt[q]; }
            __syncthreads();
            for (int i = tid; i < c; i += HY_THREADS) {
                const int32_t key = (int32_t)__hip_atomic_load(&pairs[i].x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int64_t d = (int64_t)key - w0;
                if (d >= 0 && d < HY_WIN) {
                    const int slot = (int)__hip_atomic_load(&pairs[i].y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const int rank = done + (int)s_pre[d >> 5] + __popc(s_bm[d >> 5] & ((1u << (d & 31)) - 1u));
                    const V val = __hip_atomic_exchange(&slab[slot], (V)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((int64_t)rank < cap) { out_col[o + rank] = key; out_val[o + rank] = val; }
                }
            }
            done += wtotal;
            __syncthreads();
        }
        if (tid == 0) row_nnz[row] = (s_ovf || (int64_t)done > cap) ? -1 : done;
        __threadfence();
        __syncthreads();
    }
}

// ======================================================== heavy kernel ====
// Rows whose output exceeds the 4096-slot LDS table (or the 2048-slot one, see choose_heavy), when B's rows are sorted and the
// pieces that a pass finds of them fill tiles by half (heavy_in_tiles).
// The column range is cut into windows of HV_WIN columns and
// bw[k*(n_win+1)+w] is the position in B's arrays of the first entry of row k
// with column >= w*HV_WIN, so any run of windows can be visited on its own.  One
// workgroup first counts the row's products per window (an upper bound of the
// entries of that window), then walks the windows in order, carrying the
// running output offset.  Both kinds of pass accumulate in LDS only, need no
// hash table, and leave their entries in column order:
//   * a window with more products than a ranked pass may have entries is
//     accumulated densely (Section 2.2 dense accumulator, iterated over the row's
//     column range as in Section 3.2): an accumulator per column, one LDS add per
//     product.  -0 stands for a column without products (no addend is ever -0), so
//     there are no presence bits; the window is read once, a ballot per 64 columns
//     numbers its entries;
//   * consecutive lighter windows (a stretch of up to 16, 262 144 columns) are ranked:
//     a first walk over their products marks the columns in a bitmap, whose prefix
//     popcounts number the entries of C, and a second one adds every product at its
//     column's number - 8192 accumulators a pass, as many windows at a time as have
//     so many entries, however many products they are.  A stretch of few tiles keeps
//     its products in registers between the two.
// The products are walked in tiles of 64 of one piece of a row of B, 16 lanes a tile, four
// consecutive products a lane (one 16-byte load of columns, two of fp64 values), tiles dealt
// out evenly to the waves.  What a tile needs (position, length, A's value) is found by one
// search per 64 tiles and reaches the 16 lanes by DPP moves: no search, LDS read or 64-bit
// prefix per product.  R-MAT scale 18 (68 800 rows, 3.0 G products, most rows 4 to 90 long pieces):
// 11.29 -> 9.98 ms against products numbered one by one, single sparse passes of at most 8192
// products and presence bits (whole
// calls: 14.6 -> 13.1 ms; scale 20 110.1 -> 106.5; scale 14 in fp32 0.74 -> 0.71).  Counters of scale 20 (89.9 ms): 73 vector
// and 9 LDS instructions per 64 products, vector issue 43 % of the cycles, bank conflicts 18 % (3.5 an LDS instruction); a wave
// waits for data or at a barrier in 55 % of its cycles, for its turn to issue in 24 %.  No unit is full: one workgroup fills
// the compute unit, so that its phases do not overlap.
// Two workgroups of 512 threads, windows of half the size: 9.6 ms before the last steps on scale 18, but
// 0.22 against 0.15 on scale 15 and twice the window table; tiles of 64 lanes, 8 products a batch,
// the tile's numbers in scalar registers: the same time with 15 % more vector instructions.
constexpr int HV_THREADS = 1024;
constexpr int HV_WAVES = HV_THREADS / WAVE;
constexpr int HV_WG_PER_CU = 1;
constexpr int HV_WIN = 16384;                      // columns of a window, and accumulators of a dense pass
constexpr int HV_RUN = 16;                         // windows of a stretch, at most
constexpr int HV_CAP = 8192;                       // entries of C that a ranked pass accumulates, products of a light window
constexpr int HV_MAXWIN = 512;                     // windows per row the kernel can plan for
constexpr int HV_CHUNK = 512;                      // entries of A whose pieces of B are laid end to end at a time
constexpr int HV_KEEP = 8;                         // tiles per wave up to which a stretch's products stay in registers
static_assert(HV_RUN <= HV_WAVES && HV_WIN / 32 == 8 * WAVE, "a wave per window and eight words per lane");

// The region's parts in a ranked pass (bytes): accumulators and columns by rank, prefix counts and bitmap by column.
constexpr int HV_AT_COL = (HV_CAP + WAVE) * 8;
constexpr int HV_AT_PRE = HV_AT_COL + (HV_CAP + WAVE) * 4;
constexpr int HV_AT_MAP = HV_AT_PRE + HV_RUN * (HV_WIN / 32) * 2;
constexpr int HV_REGION = HV_AT_MAP + HV_RUN * (HV_WIN / 8) + WAVE * 4;
static_assert(HV_REGION >= (HV_WIN + WAVE) * 8 && HV_AT_PRE % 16 == 0 && HV_AT_MAP % 16 == 0, "a dense pass takes the region from its start");

// x, as a number that the compiler doesn't know: what is computed from it stays inside the loop that it is taken in,
// instead of a register of its own through all of it.
__device__ __forceinline__ int hv_hide(int x)
{
    asm("" : "+v"(x));
    return x;
}

// p[i], the byte offset in 32 bits (an address of one register beside the uniform p).
template <typename T>
__device__ __forceinline__ T *hv_at(T *p, uint32_t i) { return reinterpret_cast<T *>(reinterpret_cast<char *>(p) + i * (uint32_t)sizeof(T)); }

template <typename V>
__global__ void __launch_bounds__(HV_THREADS)
k_numeric_heavy(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                const uint32_t *__restrict__ bw, int n_win, const int32_t *__restrict__ b_col,
                const V *__restrict__ b_val, const int32_t *__restrict__ rows, int64_t count,
                unsigned long long *queue, const int64_t *__restrict__ out_ptr, int32_t *__restrict__ out_col,
                V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    __shared__ __align__(16) unsigned char s_u[HV_REGION];
    __shared__ TileChunk<V, uint32_t, HV_CHUNK> s_ch;
    __shared__ uint32_t s_pw[HV_MAXWIN];                  // products of the row per window
    __shared__ __align__(16) uint32_t s_grp[HV_WIN / WAVE];   // dense pass: entries of C per 64 columns
    __shared__ uint32_t s_win[HV_WAVES];                  // ranked pass: entries of C per window
    __shared__ long long s_row;
    double *s_vals = reinterpret_cast<double *>(s_u);
    int32_t *s_col = reinterpret_cast<int32_t *>(s_u + HV_AT_COL);
    uint16_t *s_pre = reinterpret_cast<uint16_t *>(s_u + HV_AT_PRE);
    uint32_t *s_map = reinterpret_cast<uint32_t *>(s_u + HV_AT_MAP);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const size_t stride = (size_t)n_win + 1;

    for (int j = threadIdx.x; j < HV_WIN; j += HV_THREADS) s_vals[j] = -0.0;
    for (int w = threadIdx.x; w < HV_MAXWIN; w += HV_THREADS) s_pw[w] = 0u;
    // The first row of a workgroup is that of its number, the next ones are drawn from a counter, a row ahead.  (With the first one
    // drawn, too, some workgroups had two of 250 rows and others none: rows of 400 000 products in 2 windows 306 us, 197 now.)
    if (threadIdx.x == 0) s_row = (long long)blockIdx.x;
    bool clean = true;   // every accumulator of the dense window is -0; the first HV_CAP always are between passes
    __syncthreads();

    for (;;) {
        const int tid = hv_hide((int)threadIdx.x), lane = tid & (WAVE - 1);
        // where lanes without a product add and mark, so that none has to be switched off: behind the arrays' own places
        const uint32_t dump = (uint32_t)(HV_WIN + lane), rank_dump = (uint32_t)(HV_CAP + lane), map_dump = (uint32_t)(HV_RUN * (HV_WIN / 32) + lane);
        const long long ticket = wave_first(s_row);
        if (ticket >= count) break;   // uniform exit
        const int64_t row = rows[count - 1 - ticket];   // from the end of the list, where the rows with the largest bounds are
        const int64_t e0 = a_rp[row];
        const int64_t o = out_ptr[row];
        const int64_t cap = out_ptr[row + 1] - o;
        const int64_t ne = a_rp[row + 1] - e0;
        long long done = 0;
        unsigned long long drawn = 0;
        if (tid == 0) drawn = atomicAdd(queue, 1ull);

        // the first HV_CHUNK entries of the row stay in registers over all passes
        const int nent0 = ne < HV_CHUNK ? (int)ne : HV_CHUNK;
        int32_t ek = 0;
        V ea = V();
        if (tid < nent0) { ek = a_col[e0 + tid]; ea = a_val[e0 + tid]; }
        // ---- products of the row per window: one (entry, window) pair per thread and step
        {
            const int de = HV_THREADS / n_win, dw = HV_THREADS % n_win;
            int64_t e = tid / n_win;
            int w = tid % n_win;
            while (e < ne) {
                // four pairs per turn, so that their dependent loads (entry -> boundaries) overlap
                int64_t pe[4];
                int pw[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pe[i] = e; pw[i] = w;
                    e += de;
                    w += dw;
                    if (w >= n_win) { w -= n_win; ++e; }
                }
                int32_t k[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) k[i] = pe[i] < ne ? a_col[e0 + pe[i]] : 0;
                uint32_t d[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t *t = bw + (size_t)k[i] * stride;
                    d[i] = pe[i] < ne ? t[pw[i] + 1] - t[pw[i]] : 0u;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (d[i]) atomicAdd(&s_pw[pw[i]], d[i]);
            }
        }
        __syncthreads();
        if (tid == 0) s_row = (long long)(gridDim.x + drawn);   // (read by all before that barrier; the next row's behind one more)

        // ---- walk the windows, pass by pass.  Next pass from window `from` on: p0 == n_win when nothing is left.
        // Every wave plans for itself, 64 windows at a look, lane l window x + l.
        auto plan = [&](int from, int &p0, int &p1, bool &pdense) {
            p0 = n_win; p1 = n_win; pdense = false;
            for (int x = from; x < n_win; x += WAVE) {   // uniform
                const int wl = x + lane;
                const uint32_t n = wl < n_win ? s_pw[wl] : 0u;
                const unsigned long long some = __ballot(n > 0u);
                if (some == 0ull) continue;
                const int k = __ffsll((long long)some) - 1;   // windows x .. x+k-1 are empty
                const unsigned long long light = __ballot(wl < n_win && n <= (uint32_t)HV_CAP) >> k;
                int run = light == ~0ull ? WAVE : __ffsll((long long)~light) - 1;   // light windows in a row from x + k on
                run = run < WAVE - k ? run : WAVE - k;
                run = run < HV_RUN ? run : HV_RUN;
                p0 = x + k;
                pdense = run == 0;
                p1 = p0 + (run == 0 ? 1 : run);
                return;
            }
        };
        int w, w1;
        bool dense;
        plan(0, w, w1, dense);
        if (w == n_win) __syncthreads();   // (nothing at all: the counts are cleared below)
        // window boundaries of this thread's entry: those of the next pass are fetched one pass ahead
        const bool have0 = tid < nent0;
        const uint32_t *t0 = bw + (size_t)ek * stride;
        uint32_t c_lo = have0 ? t0[w] : 0u, c_hi = have0 ? t0[w1] : 0u;
        while (w < n_win) {
            int nx0, nx1;
            bool nxdense;
            plan(w1, nx0, nx1, nxdense);
            // (no entry has products in the windows skipped between two passes: the next pass starts at c_hi)
            const uint32_t n_hi = have0 ? t0[nx1] : 0u;
            const uint32_t col0 = (uint32_t)w * HV_WIN;
            const int run = w1 - w;
            // opens the pieces of entries base .. base + HV_CHUNK - 1 in windows [from, to) of the stretch
            auto open = [&](int64_t base, int from, int to, int &nent) {
                const int64_t left = ne - base;
                nent = left < HV_CHUNK ? (int)left : HV_CHUNK;
                uint32_t lo = 0u, hi = 0u;
                V a = V();
                if (tid < nent) {
                    if (base == 0) {
                        a = ea;
                        lo = from == w ? c_lo : t0[from];
                        hi = to == w1 ? c_hi : t0[to];
                    } else {
                        const uint32_t *t = bw + (size_t)a_col[e0 + base + tid] * stride;
                        a = a_val[e0 + base + tid];
                        lo = t[from];
                        hi = t[to];
                    }
                }
                return tile_open<HV_THREADS>(s_ch, nent, lo, hi - lo, a);
            };
            if (dense) {
                if (!clean) {   // uniform
                    __syncthreads();   // (the pass before may still be reading its columns there)
                    for (int j = HV_CAP + tid; j < HV_WIN; j += HV_THREADS) s_vals[j] = -0.0;
                    clean = true;
                }
                for (int64_t base = 0; base < ne; base += HV_CHUNK) {
                    int nent;
                    if (base > 0) __syncthreads();
                    const uint32_t total = open(base, w, w1, nent);
                    Tiles<V, uint32_t> tiles;
                    if (total > 0u)
                        tile_walk<HV_THREADS, 2, true>(s_ch, nent, total, b_col, b_val, tiles, false, [&](const TileFour<V> (&f)[2], const Tiles<V, uint32_t> &t) {
                            const V a[2] = {row_lane<0>(t.a), row_lane<1>(t.a)};
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                if (f[u].skip >= 4) continue;
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const uint32_t d = (uint32_t)f[u].col[i] - col0;
                                    lds_add(&s_vals[i >= f[u].skip && d < (uint32_t)HV_WIN ? d : dump], dense_addend(a[u] * f[u].val[i]));   // (d holds for a consistent table)
                                }
                            }
                        });
                }
                __syncthreads();
                // ---- window -> output, in column order: thread t holds columns t, t + 1024, ...
                constexpr int STEPS = HV_WIN / HV_THREADS;
                double v[STEPS];
#pragma unroll
                for (int i = 0; i < STEPS; ++i) v[i] = s_vals[i * HV_THREADS + tid];
                uint32_t count = 0u;   // lane i: entries of C among the wave's 64 columns of step i
#pragma unroll
                for (int i = 0; i < STEPS; ++i) {
                    s_vals[i * HV_THREADS + tid] = -0.0;
                    const uint32_t n = (uint32_t)__popcll(__ballot(dense_there(v[i])));
                    count = lane == i ? n : count;
                }
                if (lane < STEPS) s_grp[lane * HV_WAVES + wave] = count;
                __syncthreads();
                // entries before each group of 64 columns: lane l has groups 4 l .. 4 l + 3
                const uint4 g = reinterpret_cast<const uint4 *>(s_grp)[lane];
                const uint32_t sum = g.x + g.y + g.z + g.w;
                const uint32_t incl = wave_inclusive_scan_u32(sum);
                const uint32_t all = wave_read_lane_u32(incl, WAVE - 1);
                const int q = wave & 3;   // (group i * 16 + wave is number q of lane 4 i + wave / 4)
                const uint32_t before = incl - sum + (q > 0 ? g.x : 0u) + (q > 1 ? g.y : 0u) + (q > 2 ? g.z : 0u);
                const uint32_t room = cap - done < (long long)HV_WIN ? (cap > done ? (uint32_t)(cap - done) : 0u) : (uint32_t)HV_WIN;
                int32_t *to_col = out_col + o + done;
                V *to_val = out_val + o + done;
#pragma unroll
                for (int i = 0; i < STEPS; ++i) {
                    const bool there = dense_there(v[i]);
                    const unsigned long long all_there = __ballot(there);
                    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(all_there >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)all_there, 0u)) +
                                          wave_read_lane_u32(before, 4 * i + (wave >> 2));
                    if (there && rank < room) {
                        __builtin_nontemporal_store((int32_t)(col0 + (uint32_t)(i * HV_THREADS + tid)), hv_at(to_col, rank));
                        __builtin_nontemporal_store((V)v[i], hv_at(to_val, rank));
                    }
                }
                done += all;
            } else {
                clean = false;
                uint4 *map4 = reinterpret_cast<uint4 *>(s_map);
                for (int j = tid; j < run * (HV_WIN / 128); j += HV_THREADS) map4[j] = make_uint4(0u, 0u, 0u, 0u);
                const uint32_t cols = (uint32_t)run * HV_WIN;
                auto mark = [&](const TileFour<V> (&f)[2], const Tiles<V, uint32_t> &) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if (f[u].skip >= 4) continue;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t d = (uint32_t)f[u].col[i] - col0;
                            atomicOr(&s_map[i >= f[u].skip && d < cols ? d >> 5 : map_dump], 1u << (d & 31u));
                        }
                    }
                };
                uint32_t skip = 0u;   // entries of the stretch before the pass's
                auto add = [&](const TileFour<V> (&f)[2], const Tiles<V, uint32_t> &t) {
                    const V a[2] = {row_lane<0>(t.a), row_lane<1>(t.a)};
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        if (f[u].skip >= 4) continue;
                        uint32_t word[4], pre[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t d = (uint32_t)f[u].col[i] - col0;
                            const uint32_t at = d < cols ? d >> 5 : 0u;
                            word[i] = s_map[at];
                            pre[i] = s_pre[at];
                        }
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t d = (uint32_t)f[u].col[i] - col0;
                            const uint32_t rank = (pre[i] + (uint32_t)__popc(word[i] & ((1u << (d & 31u)) - 1u)) - skip) & 0xffffu;
                            const uint32_t at = i >= f[u].skip && d < cols && rank < (uint32_t)HV_CAP ? rank : rank_dump;   // (the last holds by construction)
                            s_col[at] = f[u].col[i];   // products of one column all write the same id
                            lds_add(&s_vals[at], (double)(V)(a[u] * f[u].val[i]));
                        }
                    }
                };
                uint32_t upto = 0u;   // lane l: entries of the stretch up to window l (lanes from `run` on: all)
                // ranks: entries of the stretch before every word of the bitmap (a wave per window, eight words per lane)
                auto count = [&]() {
                    uint4 x0 = make_uint4(0u, 0u, 0u, 0u), x1 = x0;
                    if (wave < run) {
                        x0 = map4[wave * (HV_WIN / 128) + lane * 2];
                        x1 = map4[wave * (HV_WIN / 128) + lane * 2 + 1];
                    }
                    const uint32_t n0 = __popc(x0.x), n1 = n0 + __popc(x0.y), n2 = n1 + __popc(x0.z), n3 = n2 + __popc(x0.w),
                                   n4 = n3 + __popc(x1.x), n5 = n4 + __popc(x1.y), n6 = n5 + __popc(x1.z), n7 = n6 + __popc(x1.w);
                    const uint32_t incl = wave_inclusive_scan_u32(n7);
                    if (lane == WAVE - 1) s_win[wave] = incl;
                    __syncthreads();
                    const uint32_t per_win = lane < HV_WAVES ? s_win[lane] : 0u;
                    upto = wave_inclusive_scan_u32(per_win);
                    if (wave < run) {
                        const uint32_t b = wave_read_lane_u32(upto - per_win, wave) + incl - n7;
                        auto two = [&](uint32_t lo, uint32_t hi) { return ((b + lo) & 0xffffu) | ((b + hi) << 16); };
                        reinterpret_cast<uint4 *>(s_pre)[wave * WAVE + lane] = make_uint4(two(0u, n0), two(n1, n2), two(n3, n4), two(n5, n6));
                    }
                    __syncthreads();
                };
                // the pass's n entries to C
                auto write = [&](uint32_t n) {
                    const uint32_t room = cap - done < (long long)n ? (cap > done ? (uint32_t)(cap - done) : 0u) : n;
                    int32_t *to_col = out_col + o + done;
                    V *to_val = out_val + o + done;
                    for (uint32_t i = (uint32_t)tid; i < n; i += HV_THREADS) {
                        const double v = s_vals[i] + 0.0;
                        s_vals[i] = -0.0;
                        if (i < room) {
                            __builtin_nontemporal_store(s_col[i], hv_at(to_col, i));
                            __builtin_nontemporal_store((V)v, hv_at(to_val, i));
                        }
                    }
                    done += n;
                };
                int nent;
                uint32_t total = open(0, w, w1, nent);
                if (ne <= HV_CHUNK && total <= (uint32_t)(HV_KEEP * HV_WAVES)) {   // uniform
                    // ---- so few tiles that the products stay in registers from the marking to the adding up
                    const uint32_t span = (total + HV_WAVES * TILE_STEP - 1) / (HV_WAVES * TILE_STEP) * TILE_STEP;
                    const uint32_t k0 = (uint32_t)wave * span, k1 = k0 + span < total ? k0 + span : total;
                    TileFour<V> f[2];
                    Tiles<V, uint32_t> t;
                    if (k0 < total) {   // uniform for the wave
                        t.find(s_ch, nent, total, k0, k1);
                        tile_load<0, true>(t, b_col, b_val, f[0]);
                        tile_load<1, true>(t, b_col, b_val, f[1]);
                        mark(f, t);
                    } else {
                        f[0] = f[1] = TileFour<V>{};
                        t = Tiles<V, uint32_t>{};
                    }
                    __syncthreads();
                    count();
                    if (k0 < total) add(f, t);
                    __syncthreads();
                    write(wave_read_lane_u32(upto, WAVE - 1));
                } else {
                    Tiles<V, uint32_t> tiles{};
                    for (int64_t base = 0; base < ne; base += HV_CHUNK) {
                        if (base > 0) {
                            __syncthreads();
                            total = open(base, w, w1, nent);
                        }
                        if (total > 0u) tile_walk<HV_THREADS, 2, false>(s_ch, nent, total, b_col, b_val, tiles, false, mark);
                    }
                    __syncthreads();
                    count();
                    // accumulate and write, as many windows at a time as have HV_CAP entries (all of them, as a rule)
                    for (int g0 = 0; g0 < run;) {   // uniform
                        const unsigned long long fit = __ballot(lane >= g0 && lane < run && upto - skip <= (uint32_t)HV_CAP) >> g0;
                        int g1 = g0 + __ffsll((long long)~fit) - 1;
                        g1 = g1 > g0 ? g1 : g0 + 1;   // (a window of the stretch fits by itself)
                        const uint32_t n = wave_read_lane_u32(upto, g1 - 1) - skip;
                        const bool whole = g0 == 0 && g1 == run;
                        for (int64_t base = 0; base < ne; base += HV_CHUNK) {
                            if (!whole || ne > HV_CHUNK) {   // (else the chunk is still open)
                                __syncthreads();
                                total = open(base, w + g0, w + g1, nent);
                            }
                            if (total > 0u) tile_walk<HV_THREADS, 2, true>(s_ch, nent, total, b_col, b_val, tiles, whole && ne <= HV_CHUNK && total <= (uint32_t)HV_THREADS, add);
                        }
                        __syncthreads();
                        write(n < (uint32_t)HV_CAP ? n : (uint32_t)HV_CAP);
                        skip += n;
                        g0 = g1;
                    }
                }
            }
            c_lo = c_hi; c_hi = n_hi;
            w = nx0; w1 = nx1; dense = nxdense;
        }
        for (int j = tid; j < n_win; j += HV_THREADS) s_pw[j] = 0u;   // (no wave plans behind a pass's barriers)
        if (tid == 0) row_nnz[row] = done > cap ? -1 : (int32_t)done;
        __syncthreads();
    }
}

// ================================ heavy kernel, product by product ====
// The same rows where the pieces of rows of B that a pass finds are short, so that tiles of 64 entries would be mostly empty
// (heavy_in_tiles says where): the products of a pass are numbered one by one, and a lane has one at a time, whatever
// the lengths of the pieces.  Windows and window table are k_numeric_heavy's; a pass is
//   * a window with more products than a sparse pass can stage: HV_WIN accumulators and a presence bitmap in LDS, one
//     LDS add and one LDS or per product; the bitmap's prefix popcount places each present column at its sorted position;
//   * consecutive windows whose products fit the staging memory left beside their bitmap (a sparse stretch: up to 8192
//     products over 10 windows, fewer over more): an expand-sort-compress accumulator whose sort is a bitmap rank.  Every
//     product is written to LDS at its own number (no atomics), or stays in its thread's registers, and marks its
//     column in a bitmap over the stretch; the prefix popcount of the bitmap is the position of each column in the
//     output, so a second sweep over the products adds each value at its column's rank.
// What bounds it is the gather of B's entries, at what the memory system gives for pieces this short, and the search for the
// entry of every product.  2000 rows of 24 000 products on 262 144 columns, fp64, numeric stage in tiles and here: rows of B
// of 2 entries 4493 and 1994 us, of 8 2996 and 1496, of 32 1469 and 1079, of 64 936 and 833, of 512 746 and 819.
constexpr int HF_THREADS = 1024;
constexpr int HF_REGION = 131072;                  // bytes of LDS that hold the accumulator of a pass
constexpr int HF_PPT = 8;                          // products of a sparse pass per thread, at most
constexpr int HF_HCAP = HF_PPT * HF_THREADS;       // products one sparse pass takes at most: 8192
constexpr int HF_RPT = 48;                         // chunks of up to 48 products per thread find their entries by rank
                                                   // (most dense windows then do: 96.8 -> 94.9 ms; 4 KB more LDS)

// QUERY: dense windows read a column's presence bit and set it only when it is clear (Section 4.1).
template <typename V, bool QUERY>
__global__ void __launch_bounds__(HF_THREADS)
k_numeric_heavy_flat(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                const uint32_t *__restrict__ bw, int n_win, const int32_t *__restrict__ b_col,
                const V *__restrict__ b_val, const int32_t *__restrict__ rows, int64_t count,
                unsigned long long *queue, const int64_t *__restrict__ out_ptr, int32_t *__restrict__ out_col,
                V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    constexpr int WIN = HV_WIN;
    constexpr int WORDS = HV_WIN / 32;
    // one 128 KB region, used either as the dense window or as a sparse pass's products, bitmap and prefix counts
    __shared__ __align__(16) unsigned char s_u[HF_REGION];
    __shared__ uint32_t s_dbm[WORDS];
    __shared__ WgChunk<V, HF_THREADS, HF_RPT> s_fc;
    __shared__ int s_wave[HF_THREADS / WAVE];
    __shared__ uint32_t s_pw[HV_MAXWIN + 1];   // s_pw[w]: products of the row in the windows before w
    __shared__ int s_ovf;
    __shared__ unsigned long long s_alloc;   // wg_flat_chunk_keep's
    __shared__ long long s_row;
    static_assert(WORDS <= HF_THREADS, "the prefix counts of a dense window reuse the chunk's array of prefix sums");
    uint32_t *s_dpre = s_fc.excl;   // (free between the traversal of a pass and the next one)
    using AV = acc_t<V>;
    static_assert(sizeof(AV) == 8 && HF_REGION == WIN * 8, "a region full of accumulators is a window");
    AV *s_vals = reinterpret_cast<AV *>(s_u);                                      // dense: WIN accumulators
    // sparse pass: staged products (column, value) by product number; once every thread holds its
    // products in registers the same memory takes the output (columns, accumulated values) by rank
    // Its memory is laid out per pass: the more windows a stretch spans, the more of the region goes to
    // the bitmap (WIN/8 bytes per window) and its prefix counts (WIN/16), the less to staged products
    // (4 + sizeof(AV) bytes each, in multiples of one product per thread).
    constexpr int OV = WIN / 8 + WIN / 16;
    auto sparse_cap = [](int run) {
        const int c = (HF_REGION - run * OV) / (4 + (int)sizeof(AV)) / HF_THREADS * HF_THREADS;
        return c > HF_HCAP ? HF_HCAP : (c < 0 ? 0 : c);
    };
    int32_t *s_scol = reinterpret_cast<int32_t *>(s_u);
    const int tid = threadIdx.x;
    const size_t stride = (size_t)n_win + 1;

    for (int j = tid; j < WIN; j += HF_THREADS) s_vals[j] = (AV)0;
    for (int j = tid; j < WORDS; j += HF_THREADS) s_dbm[j] = 0u;
    bool dense_clean = true;   // the region is an all-zero dense window
    bool chunk_clean = false;  // the traversal's marks are as wg_flat_chunk_keep leaves them

    for (;;) {
        if (tid == 0) {
            s_row = (long long)atomicAdd(queue, 1ull);
            s_ovf = 0;
        }
        for (int w = tid; w <= n_win; w += HF_THREADS) s_pw[w] = 0u;
        __syncthreads();
        if (s_row >= count) break;   // uniform exit
        const int64_t r = count - 1 - s_row;   // from the end of the list, where the rows with the largest bounds are
        const int64_t row = rows[r];
        const int64_t e0 = a_rp[row], e1 = a_rp[row + 1];
        const int64_t o = out_ptr[row];
        const int64_t cap = out_ptr[row + 1] - o;
        const int64_t ne = e1 - e0;
        long long done = 0;

        // the first HF_THREADS entries of the row stay in registers over all passes
        int32_t ek = 0;
        V ea = V();
        if (tid < ne) { ek = a_col[e0 + tid]; ea = a_val[e0 + tid]; }
        // ---- products of the row per window: one (entry, window) pair per thread and step
        {
            const int de = HF_THREADS / n_win, dw = HF_THREADS % n_win;
            int64_t e = tid / n_win;
            int w = tid % n_win;
            while (e < ne) {
                // four pairs per turn, so that their dependent loads (entry -> boundaries) overlap
                int64_t pe[4];
                int pw[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pe[i] = e; pw[i] = w;
                    e += de;
                    w += dw;
                    if (w >= n_win) { w -= n_win; ++e; }
                }
                int32_t k[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) k[i] = pe[i] < ne ? a_col[e0 + pe[i]] : 0;
                uint32_t d[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t *t = bw + (size_t)k[i] * stride;
                    d[i] = pe[i] < ne ? t[pw[i] + 1] - t[pw[i]] : 0u;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (d[i]) atomicAdd(&s_pw[pw[i] + 1], d[i]);
            }
        }
        __syncthreads();
        {   // counts -> running sums (n_win <= HV_MAXWIN <= HF_THREADS: one window per thread)
            const int mine = tid < n_win ? (int)s_pw[tid + 1] : 0;
            int all;
            const int before = block_exclusive_scan_i32<HF_THREADS>(mine, s_wave, all);
            if (tid < n_win) s_pw[tid + 1] = (uint32_t)(before + mine);
        }
        __syncthreads();

        // ---- walk the windows, pass by pass
        // next pass from window `from` on: a window with more products than a sparse pass can stage (dense),
        // or a run of windows whose products fit the staging memory that is left beside the run's bitmap
        // (sparse); p0 == n_win when nothing is left
        // Every wave plans for itself, 64 windows at a look: lane l holds the running sum behind window
        // from + l, a ballot finds the first window with products, and since the products of a stretch
        // grow with its length while its capacity shrinks, a second ballot finds how far the stretch goes.
        const int lane = tid & (WAVE - 1);
        auto plan = [&](int from, int &p0, int &p1, bool &pdense) {
            p0 = n_win; p1 = n_win; pdense = false;
            for (int x = from; x < n_win; x += WAVE) {   // uniform
                const uint32_t before = s_pw[x];
                const int wl = x + lane;   // this lane's window
                const uint32_t upto = s_pw[(wl < n_win ? wl : n_win - 1) + 1] - before;   // products of [x, wl]
                const unsigned long long some = __ballot(wl < n_win && upto > 0u);
                if (some == 0ull) continue;
                const int k = __ffsll((long long)some) - 1;   // windows x .. x+k-1 are empty
                const unsigned long long fits = __ballot(lane >= k && wl < n_win && upto <= (uint32_t)sparse_cap(lane - k + 1));
                // lanes k, k+1, ... that fit in a row: the stretch
                const unsigned long long stop = ~(fits >> k);
                const int run = stop ? __ffsll((long long)stop) - 1 : WAVE - k;
                p0 = x + k;
                pdense = run == 0;
                p1 = p0 + (run == 0 ? 1 : run);
                return;
            }
        };
        int w, w1;
        bool dense;
        plan(0, w, w1, dense);
        // window boundaries of this thread's entry: those of the next pass are fetched one pass ahead
        const bool have0 = tid < ne;
        const uint32_t *t0 = bw + (size_t)ek * stride;
        uint32_t c_lo = have0 ? t0[w] : 0u, c_hi = have0 ? t0[w1] : 0u;
        while (w < n_win) {
            int nx0, nx1;
            bool nxdense;
            plan(w1, nx0, nx1, nxdense);
            // (no entry has products in the windows skipped between two passes: the next pass starts at c_hi)
            const uint32_t n_hi = have0 ? t0[nx1] : 0u;
            // memory of a sparse pass (see above)
            const int scap = sparse_cap(w1 - w);
            AV *s_sval = reinterpret_cast<AV *>(s_u + (size_t)scap * 4);
            uint16_t *s_hpre = reinterpret_cast<uint16_t *>(s_u + (size_t)scap * (4 + sizeof(AV)));
            uint32_t *s_hbm = reinterpret_cast<uint32_t *>(s_u + (size_t)scap * (4 + sizeof(AV)) + (size_t)(w1 - w) * (WIN / 16));
            const int hwords = (w1 - w) * (WIN / 32);
            // accumulator of this pass
            if (dense) {
                if (!dense_clean) {
                    for (int j = tid; j < WIN; j += HF_THREADS) s_vals[j] = (AV)0;
                    dense_clean = true;
                }
            } else {
                for (int j = tid; j < (w1 - w) * (WIN / 32); j += HF_THREADS) s_hbm[j] = 0u;
                dense_clean = false;
            }
            // (no barrier: the traversal below has barriers of its own before the first product arrives)
            // products of windows [w, w1)
            const int32_t col0 = w * WIN;
            uint32_t staged = 0;   // products of this pass staged so far (sparse pass, uniform)
            auto f = [&](const auto &cj, const auto &cv, uint32_t q0) {
                constexpr int U = sizeof(cj) / sizeof(cj[0]);
                if (dense) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const unsigned d = (unsigned)(cj[u] - col0);
                        if (cj[u] >= 0 && d < (unsigned)WIN) {   // d is in range for a consistent window table
                            lds_add(&s_vals[d], (AV)cv[u]);
                            // Section 4.1: with many products per output entry most presence bits are set already;
                            // reading the bit first then saves the write (a stale read only costs a redundant OR)
                            const uint32_t bit = 1u << (d & 31);
                            if (!QUERY || !(s_dbm[d >> 5] & bit)) atomicOr(&s_dbm[d >> 5], bit);
                        }
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t at = staged + q0 + (uint32_t)u * WAVE + (uint32_t)(tid & (WAVE - 1));
                        const uint32_t d = (uint32_t)(cj[u] - col0);
                        if (cj[u] >= 0 && at < (uint32_t)scap && d < (uint32_t)hwords * 32u) {   // both hold by construction
                            s_scol[at] = cj[u];
                            s_sval[at] = (AV)cv[u];
                            atomicOr(&s_hbm[d >> 5], 1u << (d & 31u));
                        }
                    }
                }
            };
            if (!dense && ne <= HF_THREADS) {
                // ---- sparse pass of a row whose entries fit one chunk: no staging, every product stays in the
                // registers of the thread that fetched it, from the sweep that marks the columns to the sweep
                // that adds the values at their ranks
                constexpr int NBATCH = HF_PPT / FLAT_U;
                static_assert(HF_PPT % FLAT_U == 0, "whole batches");
                int32_t kc[HF_PPT];
                V kv[HF_PPT];
                auto mark = [&](int32_t col) {
                    const uint32_t d = (uint32_t)(col - col0);
                    if (d < (uint32_t)hwords * 32u) atomicOr(&s_hbm[d >> 5], 1u << (d & 31u));   // holds by construction
                };
                bool fits;
                wg_flat_chunk_keep<HF_THREADS, NBATCH>(s_fc, (int)ne, (int64_t)c_lo, c_hi - c_lo, ea, b_col, b_val, kc, kv,
                                                       mark, fits, chunk_clean, s_alloc);
                chunk_clean = true;
                if (!fits && tid == 0) s_ovf = 1;   // cannot happen: passes are planned from the counts
                const int wpt = (hwords + HF_THREADS - 1) / HF_THREADS;   // bitmap words per thread (consecutive)
                int mine = 0;
                for (int q = 0; q < wpt; ++q) {
                    const int j = tid * wpt + q;
                    if (j < hwords) mine += __popc(s_hbm[j]);
                }
                int htotal;
                int run = block_exclusive_scan_i32<HF_THREADS, false>(mine, s_wave, htotal);   // (barrier below)
                for (int q = 0; q < wpt; ++q) {
                    const int j = tid * wpt + q;
                    if (j < hwords) { s_hpre[j] = (uint16_t)run; run += __popc(s_hbm[j]); }
                }
                for (int i = tid; i < htotal; i += HF_THREADS) s_sval[i] = (AV)0;   // (htotal <= products <= scap)
                __syncthreads();
#pragma unroll
                for (int i = 0; i < HF_PPT; ++i) {
                    const uint32_t d = (uint32_t)(kc[i] - col0);
                    if (kc[i] >= 0 && d < (uint32_t)hwords * 32u) {
                        const int rank = (int)s_hpre[d >> 5] + __popc(s_hbm[d >> 5] & ((1u << (d & 31u)) - 1u));
                        s_scol[rank] = kc[i];           // products of one column all write the same id
                        lds_add(&s_sval[rank], (AV)kv[i]);
                    }
                }
                __syncthreads();
                const long long room = cap - done;
                const int n_out = (long long)htotal < room ? htotal : (room > 0 ? (int)room : 0);
                for (int i = tid; i < n_out; i += HF_THREADS) {
                    __builtin_nontemporal_store(s_scol[i], &out_col[o + done + i]);
                    __builtin_nontemporal_store((V)s_sval[i], &out_val[o + done + i]);
                }
                done += htotal;
                __syncthreads();
            } else {
                for (int64_t base = 0; base < ne; base += HF_THREADS) {
                    int32_t k = ek;
                    V a = ea;
                    const bool have = base + tid < ne;
                    if (base > 0 && have) { k = a_col[e0 + base + tid]; a = a_val[e0 + base + tid]; }
                    uint32_t c0 = c_lo, c1 = c_hi;
                    if (base > 0) {
                        c0 = c1 = 0;
                        if (have) {
                            const uint32_t *t = bw + (size_t)k * stride;
                            c0 = t[w];
                            c1 = t[w1];
                        }
                    }
                    const int64_t left = ne - base;
                    staged += wg_flat_chunk<HF_THREADS, true>(s_fc, left < HF_THREADS ? (int)left : HF_THREADS, (int64_t)c0,
                                                              c1 - c0, a, b_col, b_val, f);
                    chunk_clean = false;
                }
                if (dense) {
                    // ---- dense window -> output, in column order
                    const uint32_t word = tid < WORDS ? s_dbm[tid] : 0u;
                    int wtotal;
                    const int ex = block_exclusive_scan_i32<HF_THREADS>(__popc(word), s_wave, wtotal);
                    if (tid < WORDS) s_dpre[tid] = (uint32_t)ex;
                    __syncthreads();
                    // Thread t looks at columns t, t + 1024, ...: in every step the lanes of a wave read
                    // consecutive values (no LDS bank conflicts) and the present ones among them go to
                    // consecutive places of the output (coalesced stores).
                    constexpr int STEPS = WIN / HF_THREADS;
#pragma unroll 4
                    for (int i = 0; i < STEPS; ++i) {
                        const int j = i * HF_THREADS + tid;
                        const uint32_t wbits = s_dbm[j >> 5];
                        if ((wbits >> (j & 31)) & 1u) {
                            const long long rank = done + (long long)s_dpre[j >> 5] + __popc(wbits & ((1u << (j & 31)) - 1u));
                            const V val = (V)s_vals[j];
                            s_vals[j] = (AV)0;
                            if (rank < cap) { __builtin_nontemporal_store((int32_t)(col0 + j), &out_col[o + rank]); __builtin_nontemporal_store(val, &out_val[o + rank]); }
                        }
                    }
                    __syncthreads();
                    if (tid < WORDS) s_dbm[tid] = 0u;
                    done += wtotal;
                    __syncthreads();
                } else {
                    // ---- sparse pass: rank of every column = set bits below it in the bitmap of the stretch
                    const int wpt = (hwords + HF_THREADS - 1) / HF_THREADS;   // bitmap words per thread (consecutive)
                    int mine = 0;
                    for (int q = 0; q < wpt; ++q) {
                        const int j = tid * wpt + q;
                        if (j < hwords) mine += __popc(s_hbm[j]);
                    }
                    int htotal;
                    int run = block_exclusive_scan_i32<HF_THREADS, false>(mine, s_wave, htotal);   // (barrier below)
                    for (int q = 0; q < wpt; ++q) {
                        const int j = tid * wpt + q;
                        if (j < hwords) { s_hpre[j] = (uint16_t)run; run += __popc(s_hbm[j]); }
                    }
                    __syncthreads();
                    // every thread takes its share of the staged products into registers, with their ranks
                    if (staged > (uint32_t)scap) staged = scap;   // cannot happen: passes are planned from the counts
                    int32_t pc[HF_PPT];
                    AV pv[HF_PPT];
                    int pr[HF_PPT];
#pragma unroll
                    for (int i = 0; i < HF_PPT; ++i) {
                        const uint32_t at = (uint32_t)i * HF_THREADS + tid;
                        pc[i] = -1; pv[i] = AV(); pr[i] = 0;
                        if (at < staged) {
                            pc[i] = s_scol[at];
                            pv[i] = s_sval[at];
                            s_sval[at] = (AV)0;   // (htotal <= staged: the values of the output start from zero)
                            const uint32_t d = (uint32_t)(pc[i] - col0);
                            pr[i] = (int)s_hpre[d >> 5] + __popc(s_hbm[d >> 5] & ((1u << (d & 31u)) - 1u));
                        }
                    }
                    __syncthreads();
                    // the staging memory becomes the output of the pass: columns and values by rank
#pragma unroll
                    for (int i = 0; i < HF_PPT; ++i) {
                        if (pc[i] >= 0) {
                            s_scol[pr[i]] = pc[i];          // products of one column all write the same id
                            lds_add(&s_sval[pr[i]], pv[i]);
                        }
                    }
                    __syncthreads();
                    const long long room = cap - done;
                    const int n_out = (long long)htotal < room ? htotal : (room > 0 ? (int)room : 0);
                    for (int i = tid; i < n_out; i += HF_THREADS) {
                        __builtin_nontemporal_store(s_scol[i], &out_col[o + done + i]);
                        __builtin_nontemporal_store((V)s_sval[i], &out_val[o + done + i]);
                    }
                    done += htotal;
                    __syncthreads();
                }
            }
            c_lo = c_hi; c_hi = n_hi;
            w = nx0; w1 = nx1; dense = nxdense;
        }
        if (tid == 0) row_nnz[row] = (s_ovf || done > cap) ? -1 : (int32_t)done;
        __syncthreads();
    }
}

// Positions of the column-window boundaries inside every row of B:
// bw[k*(n_win+1)+w] = first position p in row k with col[p] >= w*win (row end if none).
// One 16-lane group per row; a row of WT_LONG or more entries is left to the whole workgroup (every entry is
// looked at on its own, together with its predecessor), which takes the long rows of its 16 one after the other:
// the longest row of a power-law matrix, walked by 16 lanes, was most of the kernel's time.
// flags |= 8 when a row is not sorted ascending.  spread: some 256 workgroups, every step-th, add the entries of their rows, and
// these times the windows from the row's first to its last.
constexpr int WT_LONG = 1024;
__global__ void __launch_bounds__(256)
k_window_table(const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, int64_t rows, int win_log2,
               int n_win, int64_t long_from, uint32_t *__restrict__ bw, int32_t *flags, unsigned long long *spread, int step)
{
    __shared__ long long s_long[16];
    __shared__ int s_nlong;
    __shared__ unsigned long long s_spread[2];
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t k = gt >> 4;
    const int sub = (int)(gt & 15);
    if (threadIdx.x == 0) s_nlong = 0;
    if (threadIdx.x < 2) s_spread[threadIdx.x] = 0ull;
    __syncthreads();
    bool unsorted = false;
    const bool sampled = blockIdx.x % (unsigned)step == 0u;   // uniform
    // entries first, first + step, ... of row r (positions p0 .. p1 - 1, p0 < p1), four per lane and turn
    // (unconditional reads, index clamped), so that a long row is not bound by the latency of one load after the other
    auto walk = [&](int64_t r, int64_t p0, int64_t p1, int first, int step) {
        uint32_t *t = bw + (size_t)r * ((size_t)n_win + 1);
        for (int64_t q = p0 + first; q < p1; q += 4 * (int64_t)step) {
            int32_t c[4], cp[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t p = q + (int64_t)step * i;
                const int64_t pc = p < p1 ? p : p1 - 1;
                c[i] = b_col[pc];
                cp[i] = b_col[pc > p0 ? pc - 1 : p0];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t p = q + (int64_t)step * i;
                if (p >= p1) break;
                const int wc = c[i] >> win_log2;
                int wprev = -1;
                if (p > p0) {
                    unsorted |= cp[i] > c[i];
                    wprev = cp[i] >> win_log2;
                }
                for (int w = wprev + 1; w <= wc; ++w) t[w] = (uint32_t)p;
                if (p == p1 - 1)
                    for (int w = wc + 1; w <= n_win; ++w) t[w] = (uint32_t)p1;
            }
        }
    };
    if (k < rows) {
        const int64_t p0 = b_rp[k], p1 = b_rp[k + 1];
        if (sampled && sub == 0 && p1 > p0) {
            const int64_t windows = (int64_t)(b_col[p1 - 1] >> win_log2) - (b_col[p0] >> win_log2);
            atomicAdd(&s_spread[0], (unsigned long long)(p1 - p0));
            atomicAdd(&s_spread[1], (unsigned long long)((p1 - p0) * ((windows < 0 ? -windows : windows) + 1)));
        }
        if (p0 == p1) {
            uint32_t *t = bw + (size_t)k * ((size_t)n_win + 1);
            for (int w = sub; w <= n_win; w += 16) t[w] = (uint32_t)p0;
        } else if (p1 - p0 >= long_from) {
            if (sub == 0) s_long[atomicAdd(&s_nlong, 1)] = k;
        } else {
            walk(k, p0, p1, sub, 16);
        }
    }
    __syncthreads();
    if (sampled && threadIdx.x < 2) atomicAdd(&spread[threadIdx.x], s_spread[threadIdx.x]);
    const int nlong = s_nlong;
    for (int i = 0; i < nlong; ++i) {   // uniform
        const int64_t r = s_long[i];
        walk(r, b_rp[r], b_rp[r + 1], (int)threadIdx.x, 256);
    }
    if (unsorted) atomicOr(flags, 8);
}

hipError_t launch_window_table(const Csr &B, int dtype, uint32_t *bw, int *n_win_out, int32_t *flags, unsigned long long *spread, hipStream_t s)
{
    (void)dtype;
    const int win_log2 = ilog2_const(HV_WIN);
    const int n_win = (int)((B.cols + (1ll << win_log2) - 1) >> win_log2);
    *n_win_out = n_win;
    if (B.rows == 0) return hipSuccess;
    // ("long" is relative: 1024 entries or eight times the average row, whichever is more)
    const double avg = (double)B.nnz / (double)B.rows;
    const int64_t long_from = 8.0 * avg > (double)WT_LONG ? (int64_t)(8.0 * avg) : (int64_t)WT_LONG;
    const int step = (int)(B.rows / (16 * 256)) | 1;   // (odd: the long rows of a power-law matrix are powers of two apart)
    launch_in_pieces(B.rows, 16, 256, [&](int64_t first, int64_t n) {
        hipLaunchKernelGGL(k_window_table, dim3((unsigned)((n + 15) / 16)), dim3(256), 0, s, B.rp + first, B.col, n, win_log2,
                           n_win, long_from, bw + (size_t)first * ((size_t)n_win + 1), flags, spread, step);
    });
    return hipGetLastError();
}

int heavy_workgroups_per_cu() { return HV_WG_PER_CU; }

int dense_window_count(int64_t n_cols, int dtype)
{
    (void)dtype;
    const int win_log2 = ilog2_const(HV_WIN);
    return (int)((n_cols + (1ll << win_log2) - 1) >> win_log2);
}

// ======================================================= global kernel ====
// The table of a row lives in this workgroup's region of global memory
// (tables are EMPTY / zero between rows).  Rows are emitted in order through
// an LDS bitmap over windows of 512 K columns, which also restores the table.
constexpr int GL_THREADS = 1024;
constexpr int GL_WIN = 524288;
constexpr int GL_WORDS = GL_WIN / 32;   // 16384

template <typename V>
__global__ void __launch_bounds__(GL_THREADS)
k_numeric_global(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                 const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
                 const int32_t *__restrict__ rows, int64_t count, unsigned long long *queue,
                 int32_t *__restrict__ gkeys_all, V *__restrict__ gvals_all, int gbits_max, double coef,
                 const int64_t *__restrict__ out_ptr, int32_t *__restrict__ out_col, V *__restrict__ out_val,
                 int32_t *__restrict__ row_nnz)
{
    constexpr int WPT = GL_WORDS / GL_THREADS;   // 16 words per thread
    __shared__ uint32_t s_bm[GL_WORDS];
    __shared__ uint32_t s_pre[GL_WORDS];
    __shared__ WgChunk<V, GL_THREADS> s_fc;
    __shared__ int s_wave[GL_THREADS / WAVE];
    __shared__ int s_ovf;
    __shared__ int s_min, s_max;
    __shared__ long long s_row;
    const int tid = threadIdx.x;
    int32_t *gk = gkeys_all + ((size_t)blockIdx.x << gbits_max);
    V *gv = gvals_all + ((size_t)blockIdx.x << gbits_max);

    for (;;) {
        if (tid == 0) s_row = (long long)atomicAdd(queue, 1ull);
        __syncthreads();
        const int64_t r = s_row;
        if (r >= count) break;
        const int64_t row = rows[r];
        const int64_t o = out_ptr[row];
        const int64_t cap = out_ptr[row + 1] - o;
        // table size of this row: a power of two holding coef * capacity, at most the region
        int bits = 10;
        {
            const double want = coef * (double)cap;
            while (bits < gbits_max && (double)(1ll << bits) < want) ++bits;
        }
        const int64_t slots = 1ll << bits;
        if (tid == 0) { s_ovf = 0; s_min = 0x7fffffff; s_max = -1; }
        __syncthreads();

        int kmin = 0x7fffffff, kmax = -1;
        wg_traverse<GL_THREADS, true>(a_col, a_val, a_rp[row], a_rp[row + 1],
                                      [&](int32_t k, int64_t &p0, int64_t &len) { p0 = b_rp[k]; len = b_rp[k + 1] - p0; },
                                      b_col, b_val, s_fc, [&](const auto &cj, const auto &cv) {
                                          constexpr int U = sizeof(cj) / sizeof(cj[0]);
                                          const uint32_t mask = (1u << bits) - 1u;
                                          uint32_t h[U], st[U];
                                          bool pend[U];
                                          bool any = false;
#pragma unroll
                                          for (int u = 0; u < U; ++u) {
                                              pend[u] = cj[u] >= 0;
                                              h[u] = table_hash(cj[u], bits);
                                              st[u] = table_step(cj[u], bits);
                                              any |= pend[u];
                                              if (pend[u]) {
                                                  kmin = cj[u] < kmin ? cj[u] : kmin;
                                                  kmax = cj[u] > kmax ? cj[u] : kmax;
                                              }
                                          }
                                          uint32_t rounds = 0;
                                          while (any) {   // all unresolved products probe together: their L2 round trips overlap
                                              int32_t old[U];
#pragma unroll
                                              for (int u = 0; u < U; ++u)
                                                  if (pend[u]) old[u] = atomicCAS(&gk[h[u]], EMPTY_KEY, cj[u]);
                                              any = false;
#pragma unroll
                                              for (int u = 0; u < U; ++u) {
                                                  if (pend[u]) {
                                                      if (old[u] == EMPTY_KEY || old[u] == cj[u]) {
                                                          pend[u] = false;
                                                          l2_add(&gv[h[u]], cv[u]);
                                                      } else {
                                                          h[u] = (h[u] + st[u]) & mask;
                                                          any = true;
                                                      }
                                                  }
                                              }
                                              if (any && ++rounds > mask) { s_ovf = 1; break; }
                                          }
                                      });
        kmin = -group_reduce_max(-kmin, WAVE);
        kmax = group_reduce_max(kmax, WAVE);
        if (lane_id() == 0) { atomicMin(&s_min, kmin); atomicMax(&s_max, kmax); }
        __threadfence();
        __syncthreads();

        const int lo_key = s_min, hi_key = s_max;
        long long done = 0;
        for (int64_t w0 = (int64_t)(lo_key >= 0 ? lo_key : 0) & ~(int64_t)(GL_WIN - 1); w0 <= (int64_t)hi_key; w0 += GL_WIN) {
#pragma unroll
            for (int q = 0; q < WPT; ++q) s_bm[tid * WPT + q] = 0u;
            __syncthreads();
            for (int64_t s = tid; s < slots; s += GL_THREADS) {
                const int32_t key = __hip_atomic_load(&gk[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int64_t d = (int64_t)key - w0;
                if (key != EMPTY_KEY && d >= 0 && d < GL_WIN) atomicOr(&s_bm[d >> 5], 1u << (d & 31));
            }
            __syncthreads();
            int cnt[WPT];
            int mine = 0;
#pragma unroll
            for (int q = 0; q < WPT; ++q) { cnt[q] = __popc(s_bm[tid * WPT + q]); mine += cnt[q]; }
            int wtotal;
            int run = block_exclusive_scan_i32<GL_THREADS>(mine, s_wave, wtotal);
#pragma unroll
            for (int q = 0; q < WPT; ++q) { s_pre[tid * WPT + q] = (uint32_t)run; run += cnt[q]; }
            __syncthreads();
            for (int64_t s = tid; s < slots; s += GL_THREADS) {
                const int32_t key = __hip_atomic_load(&gk[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int64_t d = (int64_t)key - w0;
                if (key != EMPTY_KEY && d >= 0 && d < GL_WIN) {
                    const long long rank = done + (long long)s_pre[d >> 5] + __popc(s_bm[d >> 5] & ((1u << (d & 31)) - 1u));
                    const V val = __hip_atomic_exchange(&gv[s], (V)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&gk[s], EMPTY_KEY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (rank < cap) { out_col[o + rank] = key; out_val[o + rank] = val; }
                }
            }
            done += wtotal;
            __syncthreads();
        }
        if (tid == 0) row_nnz[row] = (s_ovf || done > cap) ? -1 : (int32_t)done;
        __threadfence();
        __syncthreads();
    }
}

// ============================================================ dispatch ====
template <typename V>
static hipError_t dispatch(const Csr &A, const Csr &B, const NumLaunch &l, int /*gb_log2*/, hipStream_t s)
{
    if (l.count <= 0) return hipSuccess;
    const V *av = static_cast<const V *>(A.val);
    const V *bv = static_cast<const V *>(B.val);
    V *ov = static_cast<V *>(l.out_val);
#define OCEAN_WG_BF(BITS, THREADS, BF)                                                                              \
    launch_in_pieces(l.count, 1, THREADS, [&](int64_t first, int64_t n) {                                           \
        hipLaunchKernelGGL((k_numeric_wg<V, BITS, THREADS, BF>), dim3((unsigned)n), dim3(THREADS), 0, s, A.rp, A.col,   \
                           av, B.rp, B.col, bv, l.rows + first, n, l.out_ptr, l.out_col, ov, l.row_nnz);            \
    })
#define OCEAN_WG(BITS, THREADS) OCEAN_WG_BF(BITS, THREADS, 1)
    switch (l.bin) {
    case NB_E16:
    case NB_G8:
        launch_in_pieces(l.count, 32, 256, [&](int64_t first, int64_t n) {
            hipLaunchKernelGGL((k_numeric_group<V, 8, 5>), dim3((unsigned)((n + 31) / 32)), dim3(256), 0, s, A.rp, A.col, av,
                               B.rp, B.col, bv, l.rows + first, n, l.out_ptr, l.out_col, ov, l.row_nnz);
        });
        break;
    case NB_G16:
        launch_in_pieces(l.count, 16, 256, [&](int64_t first, int64_t n) {
            hipLaunchKernelGGL((k_numeric_group<V, 16, 6>), dim3((unsigned)((n + 15) / 16)), dim3(256), 0, s, A.rp, A.col, av,
                               B.rp, B.col, bv, l.rows + first, n, l.out_ptr, l.out_col, ov, l.row_nnz);
        });
        break;
#define OCEAN_WAVE(BITS, R)                                                                                        \
    launch_in_pieces(l.count, R, WAVE * (R), [&](int64_t first, int64_t n) {                                         \
        hipLaunchKernelGGL((k_numeric_wave<V, BITS, R>), dim3((unsigned)((n + (R) - 1) / (R))), dim3(WAVE * (R)), 0, s,  \
                           A.rp, A.col, av, B.rp, B.col, bv, l.rows + first, n, l.out_ptr, l.out_col, ov, l.row_nnz); \
    })
    case NB_W64: OCEAN_WAVE(8, 4); break;
    // a wave per row while the rows of the bin are light; a workgroup per row when they hold many products each
    // (a wave per row was measured for the 512- and 1024-slot bins too: 1.3 - 1.6 x slower than a workgroup per row)
    case NB_S512:
        if (l.fine_buckets) OCEAN_WG_BF(9, 128, 4);
        else OCEAN_WG(9, 128);
        break;
    case NB_S1K:
        if (l.fine_buckets) OCEAN_WG_BF(10, 256, 2);
        else OCEAN_WG(10, 256);
        break;
    case NB_S2K: OCEAN_WG(11, 512); break;
    case NB_S4K: OCEAN_WG(12, 512); break;
    case NB_S8K: OCEAN_WG(13, 1024); break;
    case NB_DSPAN:
        if (l.cmin == nullptr) return hipErrorInvalidValue;
#define OCEAN_DSPAN(TILED, COLS)                                                                                          \
    launch_in_pieces(l.count, 1, DS_THREADS, [&](int64_t first, int64_t n) {                                              \
        hipLaunchKernelGGL((k_numeric_dspan<V, TILED, COLS, false>), dim3((unsigned)n), dim3(DS_THREADS), 0, s, A.rp, A.col,   \
                           av, B.rp, B.col, bv, l.rows + first, n, l.cmin, l.out_ptr, l.out_col, ov, l.row_nnz,           \
                           Placing<V>{});                                                                                 \
    })
#define OCEAN_DSPAN_COLS(TILED)                                                                                           \
    do {                                                                                                                  \
        if (l.span_cols <= 1024) OCEAN_DSPAN(TILED, 1024);                                                                \
        else if (l.span_cols <= 2048) OCEAN_DSPAN(TILED, 2048);                                                           \
        else OCEAN_DSPAN(TILED, (int)DS_MAX_COLS);                                                                        \
    } while (0)
        if (l.tiled) OCEAN_DSPAN_COLS(true);
        else OCEAN_DSPAN_COLS(false);
#undef OCEAN_DSPAN_COLS
#undef OCEAN_DSPAN
        break;
    case NB_HYBRID:
        if (l.bw != nullptr) return hipErrorInvalidValue;   // such rows go with the last bin
        else
            hipLaunchKernelGGL((k_numeric_hybrid<V>), dim3((unsigned)l.n_wg), dim3(HY_THREADS), 0, s, A.rp, A.col, av,
                               B.rp, B.col, bv, l.rows, l.count, l.queue, static_cast<V *>(l.slab),
                               static_cast<uint2 *>(l.pairs), l.out_ptr, l.out_col, ov, l.row_nnz);
        break;
    case NB_GLOBAL:
        if (l.bw != nullptr && !l.tiled) {
            const auto kernel = l.query_bitmap ? k_numeric_heavy_flat<V, true> : k_numeric_heavy_flat<V, false>;
            hipLaunchKernelGGL(kernel, dim3((unsigned)l.n_wg), dim3(HF_THREADS), 0, s, A.rp, A.col, av, l.bw,
                               l.n_win, B.col, bv, l.rows, l.count, l.queue, l.out_ptr, l.out_col, ov, l.row_nnz);
        } else if (l.bw != nullptr)
            hipLaunchKernelGGL((k_numeric_heavy<V>), dim3((unsigned)l.n_wg), dim3(HV_THREADS), 0, s, A.rp, A.col, av, l.bw,
                               l.n_win, B.col, bv, l.rows, l.count, l.queue, l.out_ptr, l.out_col, ov, l.row_nnz);
        else
            hipLaunchKernelGGL((k_numeric_global<V>), dim3((unsigned)l.n_wg), dim3(GL_THREADS), 0, s, A.rp, A.col, av,
                               B.rp, B.col, bv, l.rows, l.count, l.queue, l.gkeys, static_cast<V *>(l.gvals), l.gbits,
                               l.coef, l.out_ptr, l.out_col, ov, l.row_nnz);
        break;
    default: return hipErrorInvalidValue;
    }
#undef OCEAN_WG
#undef OCEAN_WG_BF
#undef OCEAN_WAVE
    return hipGetLastError();
}

hipError_t launch_numeric_bin(const Csr &A, const Csr &B, int dtype, const NumLaunch &l, int gb_log2, hipStream_t s)
{
    return dtype == OCEAN_F64 ? dispatch<double>(A, B, l, gb_log2, s) : dispatch<float>(A, B, l, gb_log2, s);
}

}  // namespace ocean
