// Binning (paper Sections 2.3, 3.2, 5.3): turn a per-row size prediction into a
// hash-table size, a kernel configuration ("bin") and an output capacity,
// group row ids per bin, and the prefix sums that place rows in memory.
#include "ocean_internal.hpp"

namespace ocean {

constexpr int TPB = 256;
// Rows a workgroup of the kernels below handles, 1, 4 or 8 per thread: a tile.  The kernel that fixes the rows' capacities
// also sums them per tile, so that one more launch, which adds up the sums of the tiles before its own, places the rows.
// Workgroups add to the same few global counters, 12 ns apart, so large matrices have larger tiles: 1 M rows in 512 instead
// of 1024 workgroups.
// Small ones have small tiles: 4096 rows are a handful of workgroups either way, and a thread's rows are one latency
// after the other (classification of 4096 rows 9 us with four rows per thread).
static int row_items(int64_t m) { return m > 262144 ? 8 : m > 65536 ? 4 : 1; }
constexpr int64_t DIRECT_TILES = 4096;   // up to here every workgroup adds up the tiles before it (8.4 M rows: 16 loads a thread)

static int64_t row_tiles(int64_t m) { return (m + TPB * row_items(m) - 1) / (TPB * row_items(m)); }
int64_t scan_tmp_elems(int64_t n) { return row_tiles(n) + 1; }

// Sum over the workgroup, in every thread.  s_part: one word per wave; barriers inside, s_part may be reused after.
__device__ __forceinline__ long long block_sum(long long v, long long *s_part)
{
    v = group_reduce_sum(v, WAVE);
    if (lane_id() == 0) s_part[threadIdx.x / WAVE] = v;
    __syncthreads();
    long long t = 0;
    for (int w = 0; w < TPB / WAVE; ++w) t += s_part[w];
    __syncthreads();
    return t;
}

struct BinTable {
    int n;
    int32_t slots[OCEAN_MAX_BINS];
};

// Sort class of a row (products pr, entries ne, hash bin `bin`): the smallest class that holds it, or 0 (hash table).
// Sorting costs what the products cost, a hash table what its slots and the products cost, so a row whose many
// products fall on few columns is left to its small table.  Measured, ns per row, fp64, whole numeric stage of 200 000
// equal rows: no merging (table of 1.15 slots per product) 49 products 0.6 sorted / 0.7 hashed, 225 1.6 / 2.7, 484 2.9 /
// 5.3, 961 5.3 / 13.0, 1444 7.9 / 17, 1936 12.1 / 26; 408 products on 103 columns 1.8 / 2.8, 707 on 180 3.1 / 4.1; tables
// of 512 slots: 800 products on 205 columns 3.3 / 3.0, 896 on 286 3.3 / 3.3, 1024 on 294 3.4 / 3.4, but 1090 on 129 (256
// slots) 5.1 / 4.3 and 1682 on 281 (512 slots) 8.5 / 6.4: with up to 512 slots the line lies at 1024 products.
// Rows of at most 1024 products in small tables are cheaper hashed as well; whether they are is decided for the class,
// from the bins of its rows (see run_numeric).
__device__ __forceinline__ int sort_class(long long pr, long long ne, int bin, unsigned mask)
{
    const int most = bin <= NB_S512 ? 1024 : 2048;
    for (int c = 1; c < SORT_CLASSES; ++c)
        if (pr <= kSortClass[c].cap && ne <= kSortClass[c].entries)
            return kSortClass[c].cap <= most && ((mask >> c) & 1u) ? c : 0;
    return 0;
}

// need = table slots the row asks for, cap = output entries reserved for it.
//   mode 0  upper bound: cap = ub = min(prod, n), need = ceil(bound_coef * ub)   (Section 3.2, upper-bound workflow)
//   (in modes 1 and 2 the table is limited to ceil(bound_coef * ub) slots as well: more cannot be of use)
//   mode 1  estimate:    cap = ceil(coef * scale * est), need = ceil(table_coef * scale * est), both limited to ub
//                        (Section 5.3: estimate x coefficient; table_coef <= coef)
//   mode 2  exact:       cap = nnz, need = ceil(coef * nnz) limited to ub   (two-pass workflow)
//   mode 3  symbolic:    need = ceil(1.25 * e), no capacity; e = ub, or with assisted binning (coef > 1,
//                        Section 4.1) ceil(prod / coef) kept inside [longest referenced row of B, ub]
// max_cap receives the largest capacity among the rows of the last (global-memory) bin.
// sort_mask: bit c set = sort class c may be used (modes 0, 1, 2; see kSortClass); a_rp: row offsets of A.
// bin_of_row receives the row's key, class * OCEAN_MAX_BINS + bin, which is the bin itself for rows that are not
// sorted; bin_count and bin_prod have one counter per key.
template <int ROW_ITEMS>
__global__ void __launch_bounds__(TPB)
k_classify(int64_t m, int mode, double coef, double table_coef, double bound_coef, double scale, BinTable bt, int64_t n_cols, int64_t few_products,
           const int64_t *__restrict__ prod, const double *__restrict__ est, const int32_t *__restrict__ nnz_exact,
           const int32_t *__restrict__ row_mask, const int32_t *__restrict__ lower_bound,
           const int32_t *__restrict__ cmin, const int32_t *__restrict__ cmax, int vbytes, unsigned sort_mask,
           const int64_t *__restrict__ a_rp, uint8_t *__restrict__ bin_of_row, int32_t *__restrict__ cap,
           int64_t *__restrict__ tile_cap, int32_t *zero, unsigned long long *bin_count, unsigned long long *bin_prod,
           unsigned long long *max_cap, unsigned long long *uncounted, unsigned long long *work)
{
    constexpr int ROW_TILE = TPB * ROW_ITEMS;
    __shared__ unsigned int s_cnt[ROW_KEYS];
    __shared__ unsigned long long s_prod[ROW_KEYS];
    __shared__ unsigned int s_maxcap, s_uncounted;
    static_assert(ROW_KEYS <= TPB && ROW_KEYS <= BIN_NONE, "one thread per key, keys in a byte");
    if (threadIdx.x < ROW_KEYS) { s_cnt[threadIdx.x] = 0; s_prod[threadIdx.x] = 0ull; }
    // (2048 rows of fewer than 2^20 entries: below 2^31; longer rows are added to the totals one by one)
    __shared__ unsigned int s_nnz_a[OCEAN_MAX_BINS], s_nnz_c[OCEAN_MAX_BINS];
    __shared__ long long s_part[TPB / WAVE];
    if (threadIdx.x < OCEAN_MAX_BINS) { s_nnz_a[threadIdx.x] = 0u; s_nnz_c[threadIdx.x] = 0u; }
    if (threadIdx.x == 0) s_maxcap = s_uncounted = 0;
    __syncthreads();
    long long caps = 0;
#pragma unroll
    for (int q = 0; q < ROW_ITEMS; ++q) {
        const int64_t i = (int64_t)blockIdx.x * ROW_TILE + q * TPB + threadIdx.x;
        if (i >= m) break;
        int bin = BIN_NONE;
        long long c = 0;
        const bool active = (row_mask == nullptr) || (row_mask[i] < 0);
        const long long pr = prod[i];
        const long long ub = pr < n_cols ? pr : n_cols;
        if (active && ub > 0) {
            long long need;
            // the most slots a row can make use of: its bound with the load factor of bound-sized tables
            const long long ub_slots = bound_coef > 1.0 ? (long long)ceil(bound_coef * (double)ub) : ub;
            if (mode == 0) {
                c = ub;
                need = ub_slots;
            } else if (mode == 1) {
                double want = ceil(coef * scale * est[i]);
                c = want >= (double)ub ? ub : (long long)want;
                if (c < 1) c = 1;
                double slots = ceil(table_coef * scale * est[i]);
                need = slots >= (double)ub_slots ? ub_slots : (long long)slots;
                if (need < 1) need = 1;
            } else if (mode == 2) {
                c = nnz_exact[i];
                if (c < 0) {
                    c = 0;
                    atomicAdd(&s_uncounted, 1u);
                }
                double want = ceil(coef * (double)c);
                need = want >= (double)ub_slots ? ub_slots : (long long)want;
                if (need < c) need = c;
            } else {
                long long e = ub;
                if (coef > 1.0) {
                    const double q = ceil((double)pr / coef);
                    e = q >= (double)ub ? ub : (long long)q;
                    if (lower_bound != nullptr && e < (long long)lower_bound[i]) e = lower_bound[i];
                    if (e > ub) e = ub;
                    if (e < 1) e = 1;
                }
                need = e + (e + 3) / 4;
            }
            int span_class = 0;
            bin = bt.n - 1;
            for (int b = 0; b < bt.n; ++b)
                if ((long long)bt.slots[b] >= need) { bin = b; break; }
            // (by what the row's work is: its bound stops at the columns, or is divided)
            if (few_products > 0 && bin >= SB_S16K) bin = pr > few_products ? SB_BITMAP : bin == SB_BITMAP ? SB_S32K : bin;
            if (cmin != nullptr) {
                // Section 3.3, accumulator selection: the dense accumulator over the row's own column range where
                // it needs no more memory than the hash table the row would get
                const long long span = (long long)cmax[i] - (long long)cmin[i] + 1;
                if (mode == 3) {
                    // A bitmap of 4096 columns costs a workgroup per row whatever the row, so rows of few products are
                    // cheaper in a key table (see run_symbolic for what becomes of them).  Predict stage of 200 000 rows, us,
                    // bitmap / keys: 512 products on 800 columns 321 / 215, 768 330 / 289, 800 334 / 324, 832 (4096 keys)
                    // 332 / 376, 2500 547 / 707; on 1500 columns 640 328 / 299, 768 331 / 334; on 400 columns, 1024 keys,
                    // 1280 399 / 381, 1536 408 / 436.
                    if (span > 0 && span <= DS_MAX_COLS && bin > SB_W64)
                        bin = bin == SB_S1K && pr <= (span > 512 ? 768 : 1280) ? SB_SPAN_FEW : SB_SPAN;
                } else if (dense_span_pays(span, (long long)bt.slots[bin], vbytes)) {
                    bin = NB_DSPAN;
                    for (int d = DSPAN_CLASSES - 1; d >= 0; --d)
                        if (span <= kDspanCols[d]) span_class = SORT_CLASSES + d;
                    if (c > span) c = span;
                }
            }
            if (mode != 3 && bin == bt.n - 1 && c > 0) atomicMax(&s_maxcap, (unsigned int)c);
            const long long ne = a_rp != nullptr ? a_rp[i + 1] - a_rp[i] : 0;
            if (work != nullptr) {
                if (ne < (1 << 20)) atomicAdd(&s_nnz_a[bin], (unsigned int)ne);
                else atomicAdd(&work[bin], (unsigned long long)ne);
                if (mode == 2) {
                    if (c < (1 << 20)) atomicAdd(&s_nnz_c[bin], (unsigned int)c);
                    else atomicAdd(&work[OCEAN_MAX_BINS + bin], (unsigned long long)c);
                }
            }
            if (sort_mask != 0u && bin < NB_COUNT && pr <= kSortClass[SORT_CLASSES - 1].cap)
                bin += sort_class(pr, ne, bin, sort_mask) * OCEAN_MAX_BINS;
            bin += span_class * OCEAN_MAX_BINS;
            atomicAdd(&s_cnt[bin], 1u);
            if (bin_prod != nullptr) atomicAdd(&s_prod[bin], (unsigned long long)pr);
        }
        bin_of_row[i] = (uint8_t)bin;
        if (cap != nullptr) cap[i] = (int32_t)c;
        if (zero != nullptr) zero[i] = 0;
        caps += c;
    }
    if (tile_cap != nullptr) {
        const long long sum = block_sum(caps, s_part);
        if (threadIdx.x == 0) tile_cap[blockIdx.x] = sum;
    }
    __syncthreads();
    if (work != nullptr && threadIdx.x < OCEAN_MAX_BINS) {
        if (s_nnz_a[threadIdx.x]) atomicAdd(&work[threadIdx.x], (unsigned long long)s_nnz_a[threadIdx.x]);
        if (s_nnz_c[threadIdx.x]) atomicAdd(&work[OCEAN_MAX_BINS + threadIdx.x], (unsigned long long)s_nnz_c[threadIdx.x]);
    }
    if (threadIdx.x < ROW_KEYS && s_cnt[threadIdx.x]) atomicAdd(&bin_count[threadIdx.x], (unsigned long long)s_cnt[threadIdx.x]);
    if (bin_prod != nullptr && threadIdx.x < ROW_KEYS && s_prod[threadIdx.x]) atomicAdd(&bin_prod[threadIdx.x], s_prod[threadIdx.x]);
    if (threadIdx.x == 0 && s_maxcap && max_cap != nullptr) atomicMax(max_cap, (unsigned long long)s_maxcap);
    if (threadIdx.x == 0 && s_uncounted && uncounted != nullptr) atomicAdd(uncounted, (unsigned long long)s_uncounted);
}

// tile_cap (may be null): receives the sum of the capacities of every tile of rows (scan_tmp_elems(m) words).
// zero (may be null): an array of m words to clear.  work (may be null): [0 .. bins) += entries of A, [bins .. 2 bins) +=
// exact entries of C (mode 2) of the rows of each bin.  uncounted (may be null): += rows without an exact number (mode 2, below 0).
hipError_t launch_classify(int64_t m, const BinParams &p, double scale, const int64_t *prod, const double *est,
                           const int32_t *nnz_exact, const int32_t *row_mask, const int32_t *lower_bound,
                           uint8_t *bin_of_row, int32_t *cap, int64_t *tile_cap, int32_t *zero, unsigned long long *bin_count,
                           unsigned long long *bin_prod, unsigned long long *max_cap, unsigned long long *uncounted,
                           unsigned long long *work, hipStream_t s)
{
    static_assert(NB_ALL <= OCEAN_MAX_BINS, "the dense-range bin has a place in the per-bin arrays");
    if (m == 0) return hipSuccess;
    BinTable bt;
    bt.n = p.n_bins;
    for (int b = 0; b < OCEAN_MAX_BINS; ++b) bt.slots[b] = b < p.n_bins ? p.slots[b] : 0;
    const int64_t tiles = row_tiles(m);
    const double table_coef = (p.table_coef > 0.0 && p.table_coef < p.coef) ? p.table_coef : p.coef;
    const auto kernel = row_items(m) == 1 ? k_classify<1> : row_items(m) == 4 ? k_classify<4> : k_classify<8>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(TPB), 0, s, m, p.mode, p.coef, table_coef, p.bound_coef, scale, bt,
                       p.n_cols, p.few_products, prod, est, nnz_exact, row_mask, lower_bound, p.cmin, p.cmax, p.vbytes,
                       p.sort_mask, p.a_rp, bin_of_row, cap, tile_cap, zero, bin_count, bin_prod, max_cap, uncounted, work);
    return hipGetLastError();
}

// Where the rows go, from the tiles' sums and the keys' counts, in one launch:
//   out (may be null)       exclusive prefix sum of in[0 .. m) with m + 1 elements; total_out receives the last one
//   bin_rows (may be null)  row ids grouped by key: key b occupies bin_rows[prefix(b) .. prefix(b) + count(b)).  A
//                           workgroup counts its rows per key in LDS, claims one contiguous range per key, then fills it
// tile_sum: sums of in over the tiles, or, with `scanned`, their exclusive prefix sums.  It replaced a three-launch scan
// (one workgroup for up to 65 536 rows: 39 us for 32 768) and a scatter: 5 us a launch.
template <int ROW_ITEMS>
__global__ void __launch_bounds__(TPB)
k_place(int64_t m, const int32_t *__restrict__ in, const int64_t *__restrict__ tile_sum, bool scanned,
        int64_t *__restrict__ out, unsigned long long *total_out, int n_keys, const uint8_t *__restrict__ bin_of_row,
        const unsigned long long *__restrict__ bin_count, unsigned long long *bin_cursor, int32_t *__restrict__ bin_rows)
{
    constexpr int ROW_TILE = TPB * ROW_ITEMS;
    __shared__ unsigned int s_cnt[ROW_KEYS];
    __shared__ unsigned int s_base[ROW_KEYS];
    __shared__ unsigned int s_wave[TPB / WAVE];
    __shared__ long long s_part[TPB / WAVE];
    const int tid = threadIdx.x;
    const int64_t tile = blockIdx.x;
    // every thread: ROW_ITEMS rows in a stretch
    const int64_t first = tile * ROW_TILE + (int64_t)tid * ROW_ITEMS;
    if (out != nullptr) {
        long long before = 0;
        if (!scanned)
            for (int64_t t = tid; t < tile; t += TPB) before += tile_sum[t];
        else if (tid == 0) before = tile_sum[tile];
        before = block_sum(before, s_part);
        int32_t item[ROW_ITEMS];
        long long mine = 0;
#pragma unroll
        for (int q = 0; q < ROW_ITEMS; ++q) {
            item[q] = first + q < m ? in[first + q] : 0;
            mine += item[q];
        }
        long long inc = mine;
        for (int off = 1; off < WAVE; off <<= 1) {
            const long long o = __shfl_up(inc, off, WAVE);
            if (lane_id() >= off) inc += o;
        }
        if (lane_id() == WAVE - 1) s_part[tid / WAVE] = inc;
        __syncthreads();
        long long run = before + inc - mine;
        for (int w = 0; w < tid / WAVE; ++w) run += s_part[w];
#pragma unroll
        for (int q = 0; q < ROW_ITEMS; ++q) {
            if (first + q < m) {
                out[first + q] = run;
                run += item[q];
                if (first + q == m - 1) {
                    out[m] = run;
                    if (total_out != nullptr) *total_out = (unsigned long long)run;
                }
            }
        }
    }
    if (bin_rows == nullptr) return;   // uniform
    if (tid < ROW_KEYS) s_cnt[tid] = 0u;
    // first place of every key: prefix sum of the counts (fewer than 2^31 rows in all)
    const unsigned int total = tid < n_keys ? (unsigned int)bin_count[tid] : 0u;
    const unsigned int upto = wave_inclusive_scan_u32(total);
    if (lane_id() == WAVE - 1) s_wave[tid / WAVE] = upto;
    __syncthreads();
    // (here a thread takes rows TPB apart: the rows of a list then stay nearly in order, and the kernels that read the list
    // find the offsets and entries of neighbouring rows together - 4 neighbouring rows per thread cost the Laplacian's
    // numeric kernel a sixth: 147 -> 172 us)
    const int64_t row0 = tile * ROW_TILE + tid;
    int key[ROW_ITEMS];
    unsigned int rank[ROW_ITEMS];
#pragma unroll
    for (int q = 0; q < ROW_ITEMS; ++q) {
        key[q] = row0 + q * TPB < m ? (int)bin_of_row[row0 + q * TPB] : BIN_NONE;
        rank[q] = key[q] != BIN_NONE ? atomicAdd(&s_cnt[key[q]], 1u) : 0u;
    }
    __syncthreads();
    if (tid < n_keys) {
        unsigned int start = upto - total;
        for (int w = 0; w < tid / WAVE; ++w) start += s_wave[w];
        s_base[tid] = start + (s_cnt[tid] ? (unsigned int)atomicAdd(&bin_cursor[tid], (unsigned long long)s_cnt[tid]) : 0u);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ROW_ITEMS; ++q)
        if (key[q] != BIN_NONE) bin_rows[s_base[key[q]] + rank[q]] = (int32_t)(row0 + q * TPB);
}

// Exclusive prefix sums of the tiles' sums, in place, by one workgroup (more than DIRECT_TILES tiles).
__global__ void __launch_bounds__(TPB)
k_scan_tiles(int64_t *tile_sum, int64_t tiles)
{
    __shared__ long long s_part[TPB / WAVE];
    long long carry = 0;
    for (int64_t base = 0; base < tiles; base += TPB) {
        const int64_t i = base + threadIdx.x;
        const long long v = i < tiles ? tile_sum[i] : 0;
        long long inc = v;
        for (int off = 1; off < WAVE; off <<= 1) {
            const long long o = __shfl_up(inc, off, WAVE);
            if (lane_id() >= off) inc += o;
        }
        if (lane_id() == WAVE - 1) s_part[threadIdx.x / WAVE] = inc;
        __syncthreads();
        long long before = carry;
        for (int w = 0; w < (int)threadIdx.x / WAVE; ++w) before += s_part[w];
        if (i < tiles) tile_sum[i] = before + inc - v;
        for (int w = 0; w < TPB / WAVE; ++w) carry += s_part[w];
        __syncthreads();
    }
}

// in / tile_sum / out: see k_place, out null: no prefix sum.  bin_rows null: no grouping.
hipError_t launch_place(int64_t m, const int32_t *in, int64_t *tile_sum, int64_t *out, unsigned long long *total_out,
                        int n_keys, const uint8_t *bin_of_row, const unsigned long long *bin_count,
                        unsigned long long *bin_cursor, int32_t *bin_rows, hipStream_t s)
{
    if (m == 0) return hipSuccess;
    const int64_t tiles = row_tiles(m);
    const bool scan_first = out != nullptr && tiles > DIRECT_TILES;
    if (scan_first) hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(TPB), 0, s, tile_sum, tiles);
    const auto kernel = row_items(m) == 1 ? k_place<1> : row_items(m) == 4 ? k_place<4> : k_place<8>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(TPB), 0, s, m, in, tile_sum, scan_first, out, total_out, n_keys,
                       bin_of_row, bin_count, bin_cursor, bin_rows);
    return hipGetLastError();
}

// Produced entries per row: their sums per tile (for launch_place), the rows that overflowed (< 0), and, with work, the
// entries of C per bin of the other rows.  nnz2 (may be null): a row's entries where the first attempt overflowed; then
// final_nnz receives what counts and that is what is summed.
template <int ROW_ITEMS>
__global__ void __launch_bounds__(TPB)
k_count_rows(int64_t m, const int32_t *__restrict__ nnz1, const int32_t *__restrict__ nnz2, int32_t *__restrict__ final_nnz,
             int64_t *__restrict__ tile_sum, unsigned long long *overflowed, const uint8_t *__restrict__ bin_of_row,
             unsigned long long *work)
{
    constexpr int ROW_TILE = TPB * ROW_ITEMS;
    __shared__ unsigned int s_nnz_c[OCEAN_MAX_BINS];
    __shared__ long long s_part[TPB / WAVE];
    if (threadIdx.x < OCEAN_MAX_BINS) s_nnz_c[threadIdx.x] = 0u;
    __syncthreads();
    long long sum = 0;
    int bad = 0;
#pragma unroll
    for (int q = 0; q < ROW_ITEMS; ++q) {
        const int64_t i = (int64_t)blockIdx.x * ROW_TILE + q * TPB + threadIdx.x;
        if (i >= m) break;
        int32_t c = nnz1[i];
        bad += c < 0;
        if (work != nullptr && c > 0) {
            const int b = (int)bin_of_row[i] % OCEAN_MAX_BINS;
            if (c < (1 << 20)) atomicAdd(&s_nnz_c[b], (unsigned int)c);   // (2048 rows: below 2^31)
            else atomicAdd(&work[OCEAN_MAX_BINS + b], (unsigned long long)c);
        }
        if (nnz2 != nullptr) {
            c = c >= 0 ? c : nnz2[i];
            final_nnz[i] = c;
        }
        sum += c;
    }
    const unsigned long long rows = (unsigned long long)block_sum(bad, s_part);
    sum = block_sum(sum, s_part);
    if (threadIdx.x == 0) {
        if (tile_sum != nullptr) tile_sum[blockIdx.x] = sum;
        if (rows != 0 && overflowed != nullptr) atomicAdd(overflowed, rows);
    }
    if (work != nullptr && threadIdx.x < OCEAN_MAX_BINS && s_nnz_c[threadIdx.x])
        atomicAdd(&work[OCEAN_MAX_BINS + threadIdx.x], (unsigned long long)s_nnz_c[threadIdx.x]);
}

hipError_t launch_count_rows(int64_t m, const int32_t *nnz1, const int32_t *nnz2, int32_t *final_nnz, int64_t *tile_sum,
                             unsigned long long *overflowed, const uint8_t *bin_of_row, unsigned long long *work, hipStream_t s)
{
    if (m == 0) return hipSuccess;
    const auto kernel = row_items(m) == 1 ? k_count_rows<1> : row_items(m) == 4 ? k_count_rows<4> : k_count_rows<8>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)row_tiles(m)), dim3(TPB), 0, s, m, nnz1, nnz2, final_nnz,
                       tile_sum, overflowed, bin_of_row, work);
    return hipGetLastError();
}

// Rows, products, entries of A and entries of C per bin where rows were placed without being binned: the hash bin is the
// one that k_classify gives a row by its bound (mode 0) or its exact size (mode 2); fixed_bin >= 0: that one.  A thread adds up
// rows of one bin in registers until it meets another (1 M rows that all add to the same counters in LDS: 19 us).
__global__ void __launch_bounds__(TPB)
k_row_stats(int64_t m, int mode, int fixed_bin, double coef, double bound_coef, int64_t n_cols, const int64_t *__restrict__ prod,
            const int64_t *__restrict__ a_rp, const int64_t *__restrict__ c_rp, unsigned long long *bin_count,
            unsigned long long *bin_prod, unsigned long long *work)
{
    __shared__ unsigned long long s_sum[4][OCEAN_MAX_BINS];
    const int tid = threadIdx.x;
    if (tid < 4 * OCEAN_MAX_BINS) s_sum[tid / OCEAN_MAX_BINS][tid % OCEAN_MAX_BINS] = 0ull;
    __syncthreads();
    unsigned long long mine[4] = {0ull, 0ull, 0ull, 0ull};
    int of = -1;
    auto flush = [&]() {
        if (of >= 0 && mine[0] != 0ull)
            for (int i = 0; i < 4; ++i) atomicAdd(&s_sum[i][of], mine[i]);
    };
    // two rows per thread and turn, their loads issued together
    const int64_t stride = (int64_t)gridDim.x * TPB;
    for (int64_t i0 = (int64_t)blockIdx.x * TPB + tid; i0 < m; i0 += 2 * stride) {
        long long pr[2], ne[2], nc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t i = i0 + u * stride < m ? i0 + u * stride : i0;
            pr[u] = i0 + u * stride < m ? prod[i] : 0;
            ne[u] = a_rp[i + 1] - a_rp[i];
            nc[u] = c_rp[i + 1] - c_rp[i];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (pr[u] == 0) continue;
            int bin = fixed_bin;
            if (bin < 0) {   // uniform
                const long long ub = pr[u] < n_cols ? pr[u] : n_cols;
                long long need = bound_coef > 1.0 ? (long long)ceil(bound_coef * (double)ub) : ub;
                if (mode == 2) {
                    const double want = ceil(coef * (double)nc[u]);
                    need = want >= (double)need ? need : (long long)want;
                    if (need < nc[u]) need = nc[u];
                }
                bin = NB_COUNT - 1;
#pragma unroll
                for (int b = NB_COUNT - 2; b >= 0; --b)
                    if ((long long)kNumericSlots[b] >= need) bin = b;
            }
            if (bin != of) {
                flush();
                of = bin;
                mine[0] = mine[1] = mine[2] = mine[3] = 0ull;
            }
            mine[0] += 1ull;
            mine[1] += (unsigned long long)pr[u];
            mine[2] += (unsigned long long)ne[u];
            mine[3] += (unsigned long long)nc[u];
        }
    }
    // (what is left is of one bin in most waves: one set of atomics for the wave)
    const int first = __builtin_amdgcn_readfirstlane(of);
    if (first >= 0 && __ballot(of != first) == 0ull) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned long long all = group_reduce_sum(mine[i], WAVE);
            if (lane_id() == 0) atomicAdd(&s_sum[i][first], all);
        }
    } else {
        flush();
    }
    __syncthreads();
    if (tid < 4 * OCEAN_MAX_BINS) {
        const int what = tid / OCEAN_MAX_BINS, bin = tid % OCEAN_MAX_BINS;
        unsigned long long *to = what == 0 ? bin_count + bin : what == 1 ? bin_prod + bin : work + (what - 2) * OCEAN_MAX_BINS + bin;
        if (s_sum[what][bin]) atomicAdd(to, s_sum[what][bin]);
    }
}

hipError_t launch_row_stats(int64_t m, int mode, int fixed_bin, double coef, double bound_coef, int64_t n_cols, const int64_t *prod,
                            const int64_t *a_rp, const int64_t *c_rp, unsigned long long *bin_count,
                            unsigned long long *bin_prod, unsigned long long *work, hipStream_t s)
{
    if (m == 0) return hipSuccess;
    const int64_t want = (m + TPB * 4 - 1) / (TPB * 4);
    hipLaunchKernelGGL(k_row_stats, dim3((unsigned)(want < 512 ? want : 512)), dim3(TPB), 0, s, m, mode, fixed_bin, coef, bound_coef, n_cols,
                       prod, a_rp, c_rp, bin_count, bin_prod, work);
    return hipGetLastError();
}

// ------------------------------------------------------------ small fills
template <typename T>
__global__ void k_fill(T *p, int64_t n, T v)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

template <typename T>
static hipError_t fill(T *p, int64_t n, T v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + TPB * 4 - 1) / (TPB * 4);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(TPB), 0, s, p, n, v);
    return hipGetLastError();
}
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s) { return fill<unsigned long long>(p, n, v, s); }

}  // namespace ocean
