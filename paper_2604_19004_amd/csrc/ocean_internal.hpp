// Internal declarations shared by the HIP translation units of the library.
// gfx950 only: wave64, 160 KB LDS per workgroup, native LDS/global fp64 atomic add.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ocean_spgemm.h"
#include "rules.hpp"

namespace ocean {

constexpr int WAVE = 64;
constexpr int32_t EMPTY_KEY = -1;          // column ids are >= 0
constexpr int32_t SORT_PAD = 0x7fffffff;   // sorts after every valid column id

// ---------------------------------------------------------------- bins ----
// Numeric bins (Section 4.3 uses five halving configurations plus a
// multi-short-row and a long-row one; the sizes here are re-derived for 160 KB
// of LDS and 64-wide waves).  slots = hash-table entries of the bin.
enum NumericBin {
    NB_E16 = 0,   // 16 slots: with sizes from the product bound, expand-sort-compress, 16 lanes per row (else as NB_G8)
    NB_G8,        // 8 lanes per row, 8 rows per wave, 32 slots (product bound: expand-sort-compress, 32 lanes per row)
    NB_G16,       // 16 lanes per row, 4 rows per wave, 64 slots
    NB_W64,       // one wave per row, 256 slots
    NB_S512,      // one workgroup per row from here on
    NB_S1K,
    NB_S2K,
    NB_S4K,
    NB_S8K,       // largest table with keys and values both in LDS
    NB_HYBRID,    // 32768 keys in LDS, values in a global slab (Section 3.3, enhanced hash accumulator)
    NB_GLOBAL,    // whole table in global memory
    NB_COUNT
};
constexpr int32_t kNumericSlots[NB_COUNT] = {16, 32, 64, 256, 512, 1024, 2048, 4096, 8192, 32768, 0x7fffffff};

enum SymbolicBin {
    SB_G16 = 0,   // 64 keys
    SB_W64,       // 256 keys
    SB_S1K,
    SB_S4K,
    SB_S16K,
    SB_S32K,      // 128 KB of keys
    SB_BITMAP,    // LDS bitmap over column windows
    SB_COUNT
};
// (after the bins of ocean_bin_layout) rows whose column range is known and at most DS_MAX_COLS columns: a bitmap over it;
// then those of them with so few products that a table of 1024 keys is cheaper
constexpr int SB_SPAN = SB_COUNT;
constexpr int SB_SPAN_FEW = SB_COUNT + 1;
constexpr int SB_ALL = SB_COUNT + 2;
constexpr int32_t kSymbolicSlots[SB_COUNT] = {64, 256, 1024, 4096, 16384, 32768, 0x7fffffff};

constexpr int32_t BIN_NONE = 255;          // row takes no part in this launch set

// Dense accumulator over a row's own column range (Section 3.3, accumulator selection: the kind that needs fewer
// resources, dense when both need the same).  Rows of the 512-slot bin and beyond are candidates; the range must fit the
// kernel's LDS window.  The line is that of values of the type's own size and a presence bit per column against keys and values of
// a hash table, where it was measured.  The accumulators hold 8 bytes a column in either type now, and no bits, and the kernel takes
// 0.4 to 1.0 of its time of then, so rows at the line are on its better side (not measured again: more rows might be).
constexpr int NB_DSPAN = NB_COUNT;          // index of that bin in the per-bin arrays (after the hash bins)
constexpr int NB_ALL = NB_COUNT + 1;
constexpr int64_t DS_MAX_COLS = 4096;
__host__ __device__ inline bool dense_span_pays(long long span, long long slots, int vbytes)
{
    return span > 0 && span <= DS_MAX_COLS && slots >= 512 && span * (8 * vbytes + 1) <= slots * 8 * (4 + vbytes);
}

// Rows of few products are accumulated by sorting them (sortrow.hip) instead of through their bin's hash table.  A
// sort class takes rows of at most `cap` intermediate products and `entries` entries of A.  (64 entries: each has a place in
// LDS; with 256 places the rows of 65 to 256 entries take 0.53 to 0.88 of their time in the hash kernels, but the rows of
// fewer, which share the kernel, 1.08 to 1.12 in the classes of 512 and 1024 products, where LDS decides how many rows a
// compute unit works on.  Numeric stage of 200 000 rows: 100 entries x 10 2.40 and 1.27 ms, 32 x 32 0.92 and 1.03 ms.)
// ps: picoseconds a row of the class costs where there are many (fp64, one MI355X; see sort_class).
// table_bin, table_ps: the largest hash bin whose table takes a row of the class in less time than sorting it (0: none), and
// the picoseconds it saves: rows whose products fall on few columns (see run_numeric).
struct SortClass { int cap, entries, ps, table_bin, table_ps; };
constexpr int SORT_CLASSES = 13;            // class 0: not sorted, the bin's own kernel
constexpr SortClass kSortClass[SORT_CLASSES] = {
    {0, 0, 0, 0, 0}, {32, 32, 400, 0, 0}, {64, 64, 600, NB_G8, 40}, {96, 64, 800, NB_G8, 50}, {128, 64, 1000, NB_G8, 70},
    {192, 64, 1300, NB_G8, 150}, {256, 64, 1600, NB_G8, 200}, {384, 64, 2300, NB_G16, 300}, {512, 64, 2900, NB_G16, 400},
    {768, 64, 4100, NB_W64, 500}, {1024, 64, 5300, NB_W64, 900}, {1536, 64, 7900, NB_S1K, 600}, {2048, 64, 12100, NB_S1K, 2500}};
// Rows of the dense-range bin (NB_DSPAN below) whose range is at most kDspanCols[d] columns form a class of their own.
constexpr int DSPAN_CLASSES = 2;
constexpr int kDspanCols[DSPAN_CLASSES] = {1024, 2048};
// Rows are grouped by (class, bin): key = class * OCEAN_MAX_BINS + bin, so that the rows of a class are adjacent.
constexpr int ROW_KEYS = (SORT_CLASSES + DSPAN_CLASSES) * OCEAN_MAX_BINS;

// ------------------------------------------------------------- CSR view ----
struct Csr {
    const int64_t *rp;
    const int32_t *col;
    const void *val;
    int64_t rows, cols, nnz;
};

// ------------------------------------------------------ device helpers ----
#if defined(__HIPCC__)
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (WAVE - 1)); }

// Orders this wave's LDS/global accesses for the compiler; the hardware runs a
// wave's LDS instructions in issue order, so lanes of one wave see each
// other's earlier writes after this point.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t fmix32(uint32_t h)
{
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

// Hash used by the HLL sketches (the same function must build every sketch
// that is merged, Section 3.1).
__device__ __forceinline__ uint32_t hll_hash(int32_t col) { return fmix32((uint32_t)col + 0x9E3779B9u); }

// Fibonacci hashing for the accumulator tables: top `bits` bits of key * golden ratio.
__device__ __forceinline__ uint32_t table_hash(int32_t key, int bits)
{
    return ((uint32_t)key * 0x9E3779B1u) >> (32 - bits);
}

// Probe stride of a key (double hashing): odd, so it visits every slot of a
// power-of-two table.  A wave waits for its slowest lane, so what matters is
// the longest probe sequence among 64 concurrent insertions; linear probing's
// clustering makes that several times longer than with independent strides,
// and LDS has no locality that would reward neighbouring slots.
__device__ __forceinline__ uint32_t table_step(int32_t key, int bits)
{
    return ((((uint32_t)key * 0x85EBCA6Bu) >> (32 - bits)) << 1) | 1u;
}

// Inclusive prefix sum over the 64 lanes of a wave with data-parallel-primitive moves, which
// cost a vector instruction each and no trip to LDS: shifts by 1, 2, 4 and 8 lanes inside the
// rows of 16 lanes, then lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into the upper
// half.  A lane without a source adds 0.  Every lane of the wave must be active.
__device__ __forceinline__ uint32_t wave_inclusive_scan_u32(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15, rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31, rows 2 and 3
    return v;
}
// The same inside every group of G = 8 or 16 consecutive lanes (sub = lane inside the group).
template <int G>
__device__ __forceinline__ uint32_t group_inclusive_scan_u32(uint32_t v, int sub)
{
    static_assert(G == 8 || G == 16, "groups inside one row of 16 lanes");
    uint32_t o;
    o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false); v += sub >= 1 ? o : 0u;
    o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false); v += sub >= 2 ? o : 0u;
    o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false); v += sub >= 4 ? o : 0u;
    if (G == 16) { o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false); v += sub >= 8 ? o : 0u; }
    return v;
}
// Sum over every group of G = 8 or 16 consecutive lanes, in each of its lanes (butterfly of
// lane swaps: neighbours, pairs, mirrored halves of 8, mirrored rows of 16).
template <int G>
__device__ __forceinline__ uint32_t group_sum_u32(uint32_t v)
{
    static_assert(G == 8 || G == 16, "groups inside one row of 16 lanes");
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);    // quad_perm [1,0,3,2]
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);    // quad_perm [2,3,0,1]
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, false);   // row_half_mirror
    if (G == 16) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, false);   // row_mirror
    return v;
}
// Value of lane `l` (the same number in every lane) of v.
__device__ __forceinline__ uint32_t wave_read_lane_u32(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, __builtin_amdgcn_readfirstlane(l));
}
// The first lane's value, as a wave-uniform number.
__device__ __forceinline__ long long wave_first(long long v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((unsigned long long)v >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}
// Sum over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v)
{
    return wave_read_lane_u32(wave_inclusive_scan_u32(v), WAVE - 1);
}
// Largest value over the wave, as a wave-uniform number: the moves of the prefix sum with max in place of
// add (a lane without a source keeps its own value), read from the last lane.  Every lane must be active.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    auto larger = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    v = larger(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = larger(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = larger(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = larger(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = larger(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15, rows 1 and 3
    v = larger(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31, rows 2 and 3
    return wave_read_lane_u32(v, WAVE - 1);
}
// Workgroup level of a two-level prefix sum: part[w] holds the sum of wave w (NW <= 64 waves).
// Returns the sum of the waves before `wave`; total = sum of all.  Every lane must be active.
template <int NW>
__device__ __forceinline__ uint32_t waves_before_u32(const uint32_t *part, int wave, uint32_t &total)
{
    static_assert(NW <= WAVE, "one lane per wave");
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    const uint32_t inc = wave_inclusive_scan_u32(lane < NW ? part[lane] : 0u);
    total = wave_read_lane_u32(inc, NW - 1);
    const uint32_t upto = wave_read_lane_u32(inc, wave > 0 ? wave - 1 : 0);
    return wave > 0 ? upto : 0u;
}

template <typename T>
__device__ __forceinline__ T group_reduce_sum(T v, int width)
{
    for (int off = width >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}
template <typename T>
__device__ __forceinline__ T group_reduce_max(T v, int width)
{
    for (int off = width >> 1; off > 0; off >>= 1) {
        T o = __shfl_xor(v, off, WAVE);
        v = o > v ? o : v;
    }
    return v;
}
#endif

// LDS of a row of pr products that a wave sorts (a SortRow of 64 lanes, the fewest products per lane there is a sort for, and
// 64 entries, cut off behind the row's own places).
__host__ __device__ constexpr int sort_row_bytes(int pr, int vbytes)
{
    const int ppt = pr <= 128 ? 2 : pr <= 192 ? 3 : pr <= 256 ? 4 : pr <= 384 ? 6 : pr <= 512 ? 8 : pr <= 768 ? 12 : pr <= 1024 ? 16 : pr <= 1536 ? 24 : 32;
    const int places = pr + (pr >> (ppt >= 12 ? 4 : 3)) + 1;
    return (64 * (4 + vbytes) + 8 * ppt + vbytes * places + 7) & ~7;
}

// Totals of the row-products pass are kept in ROW_TOTAL_SLOTS slots of ROW_TOTAL_STRIDE 64-bit words each (256
// bytes apart): [0] sum of products, [1] largest row, [2] products of the heavy rows, [3] rows of A without a product,
// [4 + c] rows of sort class c (the smallest that holds the row; 0: none does), then the most LDS that four rows from
// a multiple of four on take where a wave sorts a row (sort_row_bytes; no less than that), then products, different
// columns and number of the rows whose columns were counted (MERGE_SAMPLE of them, where asked for); see analysis.hip.
constexpr int ROW_TOTAL_SLOTS = 32;
constexpr int ROW_TOTAL_STRIDE = 32;
constexpr int ROW_TOTAL_CLASS = 4;
constexpr int ROW_TOTAL_LDS = ROW_TOTAL_CLASS + SORT_CLASSES;
constexpr int ROW_TOTAL_MERGE = ROW_TOTAL_LDS + 1, ROW_TOTALS = ROW_TOTAL_MERGE + 3;
static_assert(ROW_TOTALS <= ROW_TOTAL_STRIDE, "a word per class");
constexpr int MERGE_SAMPLE = 512;        // rows
constexpr int MERGE_PRODUCTS = 256;      // of a row whose columns are counted, at most
constexpr int MERGE_LENGTH = 32;         // of the rows of B that it names: a lane walks one

// Rows of the sample whose columns are counted, the products and entries of A from which on they count as all different, and
// where the sums over them are (count_columns).
constexpr int COUNT_ROWS = 512, COUNT_PRODUCTS = 8192, COUNT_ENTRIES = 256;
constexpr int COUNT_SUMS = 5, COUNT_SLOTS = 16, COUNT_STRIDE = 8;
inline int count_rows(int64_t n_sample) { return (int)(n_sample < COUNT_ROWS ? n_sample : COUNT_ROWS); }

constexpr int SPAN_TOTALS = 5, SPAN_SLOTS = 8, SPAN_STRIDE = 16;   // see k_row_spans (a slot has a line of its own)

// Most workgroups of `threads` threads in one launch.  The runtime takes a grid's size in threads modulo 2^32 and reports
// nothing (16 778 240 workgroups of 256 threads ran as 1024), so longer lists of rows go in several launches.
constexpr int64_t most_blocks(int threads) { return 0xffffffffLL / threads; }

// go(first, n): one launch for rows first .. first + n - 1 of a list of count rows, rows_per_block of them a workgroup.
template <typename Go>
inline void launch_in_pieces(int64_t count, int rows_per_block, int threads, Go go)
{
    const int64_t most = most_blocks(threads) * rows_per_block;
    for (int64_t first = 0; first < count; first += most) go(first, count - first < most ? count - first : most);
}

// --------------------------------------------------- launcher prototypes ----
// analysis.hip
hipError_t launch_validate(const Csr &B, int32_t *flags, unsigned long long *near_pairs, hipStream_t s);
hipError_t launch_row_products(const Csr &A, const int64_t *b_rp, int64_t b_rows, int64_t *prod, int32_t *maxb,
                               unsigned long long *totals, int32_t *flags, bool validate, unsigned long long *near_pairs,
                               unsigned long long *zero, int64_t zero_words, int vbytes, const Csr *merge_sample, hipStream_t s);
hipError_t launch_publish_totals(const unsigned long long *totals, const int32_t *flags, int64_t *out, hipStream_t s);
hipError_t launch_hll_sketch(const Csr &B, int m, uint8_t *sketches, int lanes_div, hipStream_t s);
hipError_t launch_hll_merge(const Csr &A, const uint8_t *sketches, int m, const int64_t *rows, int64_t n_rows,
                            const int64_t *prod, const int32_t *maxb, const int64_t *b_rp, int64_t b_cols,
                            double *est, uint8_t *merged, int lanes_div, hipStream_t s);
hipError_t launch_sample(const Csr &A, const Csr *reach /*B; null: reach not asked for*/, const Csr *count /*B; null: nothing counted*/,
                         int64_t b_cols, const uint8_t *sketches, int m, int64_t ns, uint32_t seed, const int64_t *prod,
                         const int32_t *maxb, double *est, int64_t *prod_out, int32_t *span_out,
                         unsigned long long *count_totals, int lanes_div, hipStream_t s);
hipError_t launch_count(const Csr &A, const Csr &B, int64_t ns, uint32_t seed, const int64_t *prod, const int32_t *flags,
                        unsigned long long *count_totals, hipStream_t s);
hipError_t launch_row_spans(const Csr &A, const Csr &B, const int64_t *ends, const int64_t *prod, int vbytes, double bound_coef,
                                int32_t *cmin, int32_t *cmax, unsigned long long *totals, hipStream_t s);
hipError_t launch_check_sorted(const Csr &B, int32_t *flags, int64_t *ends /*a word per row of B*/, hipStream_t s);
hipError_t launch_sample_reduce(int64_t n_rows, const int64_t *prod, const double *est, const int32_t *span, int64_t n_cols, int vbytes,
                                double bound_coef,
                                double *out /*[6]: sum prod, sum est, sum cr, sum cr^2, rows, rows a dense range pays for*/,
                                hipStream_t s);

// binning.hip
struct BinParams {
    int mode;            // 0 upper bound, 1 estimate, 2 exact nnz, 3 symbolic pass (see k_classify)
    double coef;         // table slots per predicted entry; mode 3: the compression ratio the product counts
                         // are divided by (assisted symbolic binning, Section 4.1), 1.0 = plain product counts
    double table_coef;   // mode 1: table slots per estimated entry when smaller than coef (0: coef itself); the
                         // reserved output stays coef x estimate
    double bound_coef;   // table slots per intermediate product beyond which a table is of no use (modes 0, 1, 2;
                         // at most 1.0 = the product bound itself)
    const int32_t *cmin; // per row: first and last column the row can reach (k_row_spans), or null: rows whose range
    const int32_t *cmax; // pays for it go to the dense-range bin NB_DSPAN (modes 0, 1, 2), rows whose range is at most
                         // DS_MAX_COLS columns and that need more than 256 keys to SB_SPAN or SB_SPAN_FEW (mode 3)
    int vbytes;          // bytes of a value (with cmin)
    unsigned sort_mask;  // sort classes that may be used (bit c; modes 0, 1, 2), 0: none
    const int64_t *a_rp; // row offsets of A (with sort_mask or work sums)
    int n_bins;
    int32_t slots[OCEAN_MAX_BINS];
    int64_t n_cols;
    int64_t few_products; // mode 3, 0: none: rows beyond the 4096-slot bin go to SB_S32K with at most so many products, to SB_BITMAP with more
};
hipError_t launch_classify(int64_t m, const BinParams &p, double scale, const int64_t *prod, const double *est,
                           const int32_t *nnz_exact, const int32_t *row_mask, const int32_t *lower_bound,
                           uint8_t *bin_of_row, int32_t *cap, int64_t *tile_cap, int32_t *zero, unsigned long long *bin_count,
                           unsigned long long *bin_prod /*products per key, may be null*/, unsigned long long *max_cap,
                           unsigned long long *uncounted, unsigned long long *work, hipStream_t s);
hipError_t launch_place(int64_t m, const int32_t *in, int64_t *tile_sum, int64_t *out, unsigned long long *total_out,
                        int n_keys, const uint8_t *bin_of_row, const unsigned long long *bin_count,
                        unsigned long long *bin_cursor, int32_t *bin_rows, hipStream_t s);
hipError_t launch_count_rows(int64_t m, const int32_t *nnz1, const int32_t *nnz2, int32_t *final_nnz, int64_t *tile_sum,
                             unsigned long long *overflowed, const uint8_t *bin_of_row, unsigned long long *work, hipStream_t s);
hipError_t launch_row_stats(int64_t m, int mode, int fixed_bin, double coef, double bound_coef, int64_t n_cols, const int64_t *prod,
                            const int64_t *a_rp, const int64_t *c_rp, unsigned long long *bin_count,
                            unsigned long long *bin_prod, unsigned long long *work, hipStream_t s);
int64_t scan_tmp_elems(int64_t n);   // words of tile sums for n rows
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s);

// symbolic.hip
constexpr int64_t SYMBOLIC_FEW_COLS = 1 << 18;
struct SymLaunch {
    const int32_t *rows;   // row ids of this bin
    int64_t count;
    int bin;
    bool query_bitmap;     // bitmap kernel: read a column's bit before setting it (Section 4.1)
    const int32_t *cmin;   // SB_SPAN: first column each row can reach
    bool tiled;            // SB_BITMAP: symbolic_in_tiles
    bool few;              // SB_BITMAP: rows of at most symbolic_few_products, by smaller workgroups
    bool may_overflow;     // tables were sized from a guess (assisted binning): a row whose table fills up
                           // reports -1 instead of a count and probing gives up early
};
hipError_t launch_symbolic_bin(const Csr &A, const Csr &B, const SymLaunch &l, int gb_log2, int32_t *nnz_out,
                               int n_wg, unsigned long long *queue, hipStream_t s);

// order.hip
size_t sort_rows_scratch_bytes(int64_t count);
hipError_t launch_sort_b_rows(const Csr &B, int dtype, int32_t *col_out, void *val_out, int32_t *flags, hipStream_t s);
hipError_t launch_sort_rows_by_products(const int64_t *prod, int32_t *rows, int64_t count, void *scratch, hipStream_t s);

// numeric.hip
struct NumLaunch {
    const int32_t *rows;
    int64_t count;
    int bin;
    const int64_t *out_ptr;   // [m+1]: start of each row's output region; capacity = out_ptr[i+1]-out_ptr[i]
    int32_t *out_col;
    void *out_val;
    int32_t *row_nnz;         // written per row: entries produced, or -1 on overflow
    // scratch of NB_HYBRID / NB_GLOBAL
    void *slab;               // hybrid: n_wg slabs of 32768 values, all zero on entry and on exit
    void *pairs;              // hybrid: n_wg lists of 32768 (key, slot) pairs, scratch
    int32_t *gkeys;           // global: n_wg tables of 2^gbits keys, all EMPTY on entry and on exit
    void *gvals;              // global: n_wg tables of 2^gbits values, all zero on entry and on exit
    int gbits;
    int n_wg;                 // persistent workgroups of the hybrid / global kernels
    unsigned long long *queue; // their shared row counter, zero on entry
    double coef;              // global: table slots per reserved output entry
    const uint32_t *bw;       // dense kernel: window boundary table of B, or null to use the global-table kernel
    int n_win;
    bool tiled;               // dense-range bin: dspan_in_tiles; rows in column windows: heavy_in_tiles
    bool query_bitmap;        // rows in column windows, not in tiles: read a column's presence bit before setting it (Section 4.1)
    bool fine_buckets;        // 512- and 1024-slot bins: order the row through 2048 column buckets (clustered columns)
    const int32_t *cmin;      // dense-range bin: first column each row can reach
    int span_cols;            // dense-range bin: the rows' ranges are at most so many columns (kDspanCols or DS_MAX_COLS)
};
hipError_t launch_window_table(const Csr &B, int dtype, uint32_t *bw, int *n_win_out, int32_t *flags, unsigned long long *spread /*2 words, += entries of sampled rows, entries times windows*/, hipStream_t s);
int heavy_workgroups_per_cu();   // workgroups of the column-window kernel that one compute unit holds
int dense_window_count(int64_t n_cols, int dtype);
hipError_t launch_numeric_bin(const Csr &A, const Csr &B, int dtype, const NumLaunch &l, int gb_log2, hipStream_t s);

// esc.hip
struct EscLaunch {
    const int32_t *rows;      // row ids, each with at most `lanes` intermediate products
    int64_t count;
    int lanes;                // 16 or 32 lanes (= products) per row
    const int64_t *out_ptr;
    int32_t *out_col;
    void *out_val;
    int32_t *row_nnz;
};
constexpr int64_t ESC_MAX_COLS = (1ll << 26) - 1;   // column id and lane number share one 32-bit sort key
hipError_t launch_numeric_esc(const Csr &A, const Csr &B, int dtype, const EscLaunch &l, hipStream_t s);

// sortrow.hip
struct SortLaunch {
    const int32_t *rows;      // row ids of one sort class
    int64_t count;
    int cls;
    const int64_t *out_ptr;
    int32_t *out_col;
    void *out_val;
    int32_t *row_nnz;
};
hipError_t launch_numeric_sort(const Csr &A, const Csr &B, int dtype, const SortLaunch &l, hipStream_t s);

// placed.hip
// Rows of a unit where all rows are placed as rows of a class: 256 / G for the classes below a wave, else the four of a
// workgroup.
constexpr int kPlacedRows[SORT_CLASSES] = {0, 32, 16, 16, 16, 8, 8, 4, 4, 4, 4, 4, 4};
inline int64_t placed_units(int64_t m, int cls) { return (m + kPlacedRows[cls] - 1) / kPlacedRows[cls]; }
struct PlacedLaunch {
    int cls;                  // every row has at most this class's products and entries
    const int64_t *prod;      // products per row
    const int32_t *cmin;      // dense ranges: first column each row can reach
    int span_cols;            // and the most columns in a row's range
    bool tiled;               // and NumLaunch's
    int pool;                 // LDS of a workgroup: the most that four rows from a multiple of four on take (classes of whole waves)
    int64_t *c_rp;            // receives the row offsets of C
    int32_t *out_col;
    void *out_val;
    int64_t slots;            // entries that fit into out_col / out_val
    uint32_t *counts;         // placed_units words, zero
    unsigned long long *places;   // the same
    unsigned long long *total;    // receives the entries of C
    int32_t *flags;           // |= 32: a wait ran out and the result is not complete
    int placer_polls, unit_polls;   // polls, about a microsecond each, after which waits run out
    bool by_xcd;              // units_by_xcd of the device (units.hpp)
};
hipError_t launch_placed(const Csr &A, const Csr &B, int dtype, const PlacedLaunch &l, hipStream_t s);
hipError_t launch_placed_span(const Csr &A, const Csr &B, int dtype, const PlacedLaunch &l, hipStream_t s);   // numeric.hip; units of a row
hipError_t launch_trim(int dtype, const int32_t *col, const void *val, int64_t n, int32_t *c_col, void *c_val, hipStream_t s);

// compact.hip
hipError_t launch_compact(int64_t m, int dtype, const int64_t *c_rp, const int32_t *nnz1, const int64_t *ptr1,
                          const int32_t *col1, const void *val1, const int64_t *ptr2, const int32_t *col2,
                          const void *val2, int32_t *c_col, void *c_val, int g_log2, int64_t nnz_c, hipStream_t s);

hipError_t launch_compact_range(int64_t m, int dtype, const int64_t *c_rp, const int32_t *nnz1, const int64_t *ptr1,
                                const int32_t *col1, const void *val1, const int64_t *ptr2, const int32_t *col2,
                                const void *val2, int32_t *dst_col, void *dst_val, int64_t first, int64_t last,
                                int64_t dst_off, hipStream_t s);

}  // namespace ocean
