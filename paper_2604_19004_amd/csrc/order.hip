// Order of the rows inside the launch of the heavy-row kernel.  Its persistent
// workgroups take rows one by one from the end of the list; a row of a
// power-law matrix can hold a hundred times the work of the median row of its
// bin, and one that is handed out late keeps a single CU busy long after all
// others have finished.  Handing out the longest rows first needs no exact
// sort: rows are ordered by a coarse key of their product count (its binary
// exponent and the three bits below the leading one, i.e. classes 12 % wide)
// with one counting pass - count per class, prefix sum, scatter.  The order
// inside a class is whatever the atomics give; it has no effect on the result.
#include "ocean_internal.hpp"

namespace ocean {

namespace {
constexpr int OB_CLASSES = 512;   // 64 exponents x 8
constexpr int OB_THREADS = 256;
constexpr int OB_ITEMS = 8;       // rows per thread of the scatter
constexpr size_t SORT_ALIGN = 256;
inline size_t sort_up(size_t b) { return (b + SORT_ALIGN - 1) / SORT_ALIGN * SORT_ALIGN; }

__device__ __forceinline__ int product_class(int64_t p)
{
    if (p <= 0) return 0;
    const int e = 63 - __clzll((long long)p);
    const int m = e >= 3 ? (int)((p >> (e - 3)) & 7) : (int)((p << (3 - e)) & 7);
    return e * 8 + m;   // < 512, monotone in p
}

__global__ void __launch_bounds__(OB_THREADS)
k_order_count(const int64_t *__restrict__ prod, const int32_t *__restrict__ rows, int64_t count, unsigned int *hist)
{
    __shared__ unsigned int s_hist[OB_CLASSES];
    for (int j = threadIdx.x; j < OB_CLASSES; j += OB_THREADS) s_hist[j] = 0u;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * OB_THREADS + threadIdx.x; i < count; i += (int64_t)gridDim.x * OB_THREADS)
        atomicAdd(&s_hist[product_class(prod[rows[i]])], 1u);
    __syncthreads();
    for (int j = threadIdx.x; j < OB_CLASSES; j += OB_THREADS)
        if (s_hist[j]) atomicAdd(&hist[j], s_hist[j]);
}

// counts -> first position of every class (exclusive prefix sum), in place; one workgroup of OB_CLASSES threads
__global__ void __launch_bounds__(OB_CLASSES)
k_order_scan(unsigned int *hist)
{
    __shared__ unsigned int s_part[OB_CLASSES / WAVE];
    const unsigned int v = hist[threadIdx.x];
    const unsigned int inc = wave_inclusive_scan_u32(v);
    if (lane_id() == WAVE - 1) s_part[threadIdx.x / WAVE] = inc;
    __syncthreads();
    uint32_t total;
    const uint32_t before = waves_before_u32<OB_CLASSES / WAVE>(s_part, (int)threadIdx.x / WAVE, total);
    hist[threadIdx.x] = before + inc - v;
}

// A workgroup ranks its tile of rows per class in LDS, claims one range per class, and writes its rows there.
__global__ void __launch_bounds__(OB_THREADS)
k_order_scatter(const int64_t *__restrict__ prod, const int32_t *__restrict__ rows, int64_t count,
                unsigned int *cursor, int32_t *__restrict__ out)
{
    __shared__ unsigned int s_cnt[OB_CLASSES];
    __shared__ unsigned int s_base[OB_CLASSES];
    for (int j = threadIdx.x; j < OB_CLASSES; j += OB_THREADS) s_cnt[j] = 0u;
    __syncthreads();
    const int64_t tile = (int64_t)blockIdx.x * OB_THREADS * OB_ITEMS;
    int32_t row[OB_ITEMS];
    int cls[OB_ITEMS];
    unsigned int rank[OB_ITEMS];
#pragma unroll
    for (int q = 0; q < OB_ITEMS; ++q) {
        const int64_t i = tile + (int64_t)q * OB_THREADS + threadIdx.x;
        cls[q] = -1; row[q] = 0; rank[q] = 0;
        if (i < count) {
            row[q] = rows[i];
            cls[q] = product_class(prod[row[q]]);
            rank[q] = atomicAdd(&s_cnt[cls[q]], 1u);
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < OB_CLASSES; j += OB_THREADS)
        s_base[j] = s_cnt[j] ? atomicAdd(&cursor[j], s_cnt[j]) : 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < OB_ITEMS; ++q)
        if (cls[q] >= 0) out[s_base[cls[q]] + rank[q]] = row[q];
}
}  // namespace

// ---- a copy of B with every row's entries in column order -------------------------------------------
// Needed when B's rows come unsorted and so much work sits in heavy rows that the kernels which accumulate
// in global memory would be bound by atomic throughput (the case Section 5.4 reports for the enhanced hash
// accumulator): the column-window kernel needs sorted rows.
// Rows of up to SB_SHORT entries: a wave per row, up to two entries a lane, and every entry's place is the number of entries
// before it - each key is read from its lane once and compared with all, so the values go straight to their places.
// Rows of fewer than sort_bitmap_from entries: a workgroup of 256 threads per row, a bitonic network orders (column id, position) in
// LDS and the values follow their positions (indirect sort, Section 4.2).
// Longer rows: a workgroup of 1024 per row.  A bitmap over the columns, 262 144 at a time, numbers them (prefix popcounts), and every
// entry goes to its column's number; where a column comes twice, a network orders the row instead, whose steps of at most
// 64 places stay within a wave and need no barrier.  Rows longer than SB_MAX are copied unsorted: flags |= 16 and the caller keeps B
// as it is.
// R-MAT of scale 15, 216 000 entries in 32768 rows, of which a few hold thousands, fp64: 100 us with a network for every row, 36 as it
// is (20 + 16).  6 M entries in rows of equal length, stage with the copy in us, network and bitmap: 131 072 columns, rows of 200 249
// and 386, of 300 260 and 284, of 1000 148 and 121, of 3000 459 and 210; 2^20 columns, four turns, of 200 255 and 1927, of 1000
// 152 and 286, of 3000 463 and 395; 32 768 columns, of 130 350 and 463, of 300 258 and 244, of 600 281 and 168.
namespace {
constexpr int SB_GROUPS = 2;
constexpr int SB_SHORT = SB_GROUPS * WAVE;
constexpr int SB_WAVES = 4;
constexpr int SB_THREADS = 1024;
constexpr int SB_MAX = SORT_BITMAP_NONE - 1;
constexpr int SB_WORDS = SB_MAX * 2;          // of the bitmap, in the pairs' memory
constexpr int SB_NET_THREADS = 256;

template <typename V>
__global__ void __launch_bounds__(WAVE * SB_WAVES)
k_sort_b_short(const int64_t *__restrict__ rp, const int32_t *__restrict__ col, const V *__restrict__ val, int64_t rows,
               int32_t *__restrict__ col_out, V *__restrict__ val_out)
{
    const int lane = lane_id();
    const int64_t stride = (int64_t)gridDim.x * SB_WAVES;
    for (int64_t row = (int64_t)blockIdx.x * SB_WAVES + __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE); row < rows; row += stride) {
        const int64_t p0 = rp[row];
        const int64_t full = rp[row + 1] - p0;
        if (full > SB_SHORT) continue;   // uniform for the wave
        const int len = (int)full;
        const int groups = (len + WAVE - 1) / WAVE;
        uint32_t key[SB_GROUPS];   // (the lane's entries: number lane and 64 + lane; the largest number where there is none)
        int32_t place[SB_GROUPS] = {};
#pragma unroll
        for (int q = 0; q < SB_GROUPS; ++q) key[q] = q * WAVE + lane < len ? (uint32_t)col[p0 + q * WAVE + lane] : ~0u;
#pragma unroll
        for (int g = 0; g < SB_GROUPS; ++g) {
            if (g >= groups) break;   // uniform
            const int n = len - g * WAVE < WAVE ? len - g * WAVE : WAVE;
            for (int j = 0; j < n; ++j) {
                const uint32_t k = wave_read_lane_u32(key[g], j);
#pragma unroll
                for (int q = 0; q < SB_GROUPS; ++q) {   // (equal columns stay in their order)
                    if (q >= groups) break;
                    const bool before = q == g ? k < key[q] || (k == key[q] && j < lane) : q > g ? k <= key[q] : k < key[q];
                    place[q] += before;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < SB_GROUPS; ++q) {
            if (q * WAVE + lane < len) {
                col_out[p0 + place[q]] = (int32_t)key[q];
                val_out[p0 + place[q]] = val[p0 + q * WAVE + lane];
            }
        }
    }
}

// Workgroup b has rows b, b + gridDim.x, ... of SB_SHORT + 1 .. CAP entries that are fewer than `below`.
template <typename V, int CAP>
__global__ void __launch_bounds__(SB_NET_THREADS)
k_sort_b_middle(const int64_t *__restrict__ rp, const int32_t *__restrict__ col, const V *__restrict__ val, int64_t rows,
                int below, int32_t *__restrict__ col_out, V *__restrict__ val_out)
{
    __shared__ int32_t s_key[CAP];
    __shared__ uint16_t s_pos[CAP];
    __shared__ unsigned long long s_mine[SB_NET_THREADS / WAVE];
    const int tid = threadIdx.x;
    for (int64_t from = blockIdx.x; from < rows; from += (int64_t)gridDim.x * SB_NET_THREADS) {
        const int64_t r = from + (int64_t)tid * gridDim.x;
        const int64_t entries = r < rows ? rp[r + 1] - rp[r] : 0;
        const unsigned long long there = __ballot(entries > SB_SHORT && entries < below);
        if (lane_id() == 0) s_mine[tid / WAVE] = there;
        __syncthreads();
        for (int w = 0; w < SB_NET_THREADS / WAVE; ++w) {
            for (unsigned long long left = s_mine[w]; left != 0ull; left &= left - 1ull) {   // uniform
                const int64_t row = from + (int64_t)(w * WAVE + __ffsll(left) - 1) * gridDim.x;
                const int64_t p0 = rp[row];
                const int len = (int)(rp[row + 1] - p0);
                int n = 2 * SB_SHORT;
                while (n < len) n <<= 1;
                for (int i = tid; i < n; i += SB_NET_THREADS) {
                    s_key[i] = i < len ? col[p0 + i] : SORT_PAD;
                    s_pos[i] = (uint16_t)i;
                }
                __syncthreads();
                for (int k = 2; k <= n; k <<= 1) {
                    for (int j = k >> 1; j > 0; j >>= 1) {
                        for (int i = tid; i < (n >> 1); i += SB_NET_THREADS) {
                            const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                            const int hi = lo | j;
                            const int32_t x = s_key[lo], y = s_key[hi];
                            if ((x > y) == ((lo & k) == 0)) {
                                s_key[lo] = y; s_key[hi] = x;
                                const uint16_t t = s_pos[lo]; s_pos[lo] = s_pos[hi]; s_pos[hi] = t;
                            }
                        }
                        __syncthreads();
                    }
                }
                for (int i = tid; i < len; i += SB_NET_THREADS) {
                    col_out[p0 + i] = s_key[i];
                    val_out[p0 + i] = val[p0 + s_pos[i]];
                }
                __syncthreads();   // the arrays are rewritten for the next row
            }
        }
        __syncthreads();
    }
}

// Workgroup b has rows b, b + gridDim.x, ... of `least` entries or more.
template <typename V>
__global__ void __launch_bounds__(SB_THREADS)
k_sort_b_long(const int64_t *__restrict__ rp, const int32_t *__restrict__ col, const V *__restrict__ val, int64_t rows,
              int64_t cols, int least, int32_t *__restrict__ col_out, V *__restrict__ val_out, int32_t *flags)
{
    __shared__ unsigned long long s_key[SB_MAX];   // column id, position
    __shared__ uint16_t s_pre[SB_WORDS];           // entries before each word of the bitmap
    __shared__ uint32_t s_sum[SB_THREADS / WAVE];
    uint32_t *const s_bits = reinterpret_cast<uint32_t *>(s_key);
    __shared__ unsigned long long s_long[SB_THREADS / WAVE];
    const int tid = threadIdx.x;
    for (int64_t from = blockIdx.x; from < rows; from += (int64_t)gridDim.x * SB_THREADS) {
        const int64_t mine = from + (int64_t)tid * gridDim.x;
        const unsigned long long there = __ballot(mine < rows && rp[mine < rows ? mine + 1 : 0] - rp[mine < rows ? mine : 0] >= least);
        if (lane_id() == 0) s_long[tid / WAVE] = there;
        __syncthreads();
        for (int w = 0; w < SB_THREADS / WAVE; ++w) {
            for (unsigned long long left = s_long[w]; left != 0ull; left &= left - 1ull) {   // uniform
                const int64_t row = from + (int64_t)(w * WAVE + __ffsll(left) - 1) * gridDim.x;
                const int64_t p0 = rp[row];
                const int64_t full = rp[row + 1] - p0;
                if (full > SB_MAX) {   // uniform: copied as it is, so that the copy stays a valid matrix (its column ids are in range)
                    if (tid == 0) atomicOr(flags, 16);
                    for (int64_t i = tid; i < full; i += SB_THREADS) { col_out[p0 + i] = col[p0 + i]; val_out[p0 + i] = val[p0 + i]; }
                    continue;
                }
                const int len = (int)full;
                bool done = true;
                uint32_t before = 0u;   // entries with columns of the turns before
                for (int64_t c0 = 0; done && c0 < cols; c0 += 32 * SB_WORDS) {   // (all uniform)
                    const int words = (int)(cols - c0 < 32 * SB_WORDS ? (cols - c0 + 31) / 32 : SB_WORDS);
                    const int per = (words + SB_THREADS - 1) / SB_THREADS;
                    for (int i = tid; i < words; i += SB_THREADS) s_bits[i] = 0u;
                    __syncthreads();
                    bool twice = false;
                    for (int i = tid; i < len; i += SB_THREADS) {
                        const int64_t d = (int64_t)col[p0 + i] - c0;
                        if (d < 0 || d >= 32 * (int64_t)words) continue;
                        const uint32_t bit = 1u << (d & 31);
                        twice |= (atomicOr(&s_bits[d >> 5], bit) & bit) != 0u;
                    }
                    if (__syncthreads_or(twice)) {
                        done = false;
                        break;
                    }
                    uint32_t mine = 0u;
                    for (int i = tid * per; i < (tid + 1) * per && i < words; ++i) mine += (uint32_t)__popc(s_bits[i]);
                    const uint32_t incl = wave_inclusive_scan_u32(mine);
                    if (lane_id() == WAVE - 1) s_sum[tid / WAVE] = incl;
                    __syncthreads();
                    uint32_t all;
                    uint32_t run = waves_before_u32<SB_THREADS / WAVE>(s_sum, tid / WAVE, all) + incl - mine;
                    for (int i = tid * per; i < (tid + 1) * per && i < words; ++i) {
                        s_pre[i] = (uint16_t)run;
                        run += (uint32_t)__popc(s_bits[i]);
                    }
                    __syncthreads();
                    for (int i = tid; i < len; i += SB_THREADS) {
                        const int32_t c = col[p0 + i];
                        const int64_t d = (int64_t)c - c0;
                        if (d < 0 || d >= 32 * (int64_t)words) continue;
                        const uint32_t at = before + s_pre[d >> 5] + (uint32_t)__popc(s_bits[d >> 5] & ((1u << (d & 31)) - 1u));
                        col_out[p0 + at] = c;
                        val_out[p0 + at] = val[p0 + i];
                    }
                    before += all;
                    __syncthreads();   // the bitmap is cleared for the next turn or row
                }
                if (done && before == (uint32_t)len) continue;
                __syncthreads();
                int n = 512;
                while (n < len) n <<= 1;
                for (int i = tid; i < n; i += SB_THREADS)
                    s_key[i] = i < len ? ((unsigned long long)(uint32_t)col[p0 + i] << 32) | (uint32_t)i : ~0ull;
                __syncthreads();
                for (int k = 2; k <= n; k <<= 1) {
                    for (int j = k >> 1; j > 0; j >>= 1) {
                        for (int i = tid; i < (n >> 1); i += SB_THREADS) {
                            const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                            const int hi = lo | j;
                            const unsigned long long x = s_key[lo], y = s_key[hi];
                            if ((x > y) == ((lo & k) == 0)) { s_key[lo] = y; s_key[hi] = x; }
                        }
                        // pairs i .. i + 63 of a wave lie in 128 places of its own while j <= 64
                        if (j > WAVE || (j == 1 && k >= 2 * WAVE)) {
                            __syncthreads();
                        } else {
                            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                            __builtin_amdgcn_wave_barrier();
                        }
                    }
                }
                __syncthreads();
                for (int i = tid; i < len; i += SB_THREADS) {
                    const unsigned long long x = s_key[i];
                    col_out[p0 + i] = (int32_t)(x >> 32);
                    val_out[p0 + i] = val[p0 + (uint32_t)x];
                }
                __syncthreads();   // the places are rewritten for the next row
            }
        }
        __syncthreads();
    }
}
}  // namespace

hipError_t launch_sort_b_rows(const Csr &B, int dtype, int32_t *col_out, void *val_out, int32_t *flags, hipStream_t s)
{
    if (B.rows == 0 || B.nnz == 0) return hipSuccess;
    const int64_t waves = (B.rows + SB_WAVES - 1) / SB_WAVES;
    const dim3 short_grid((unsigned)(waves < 65536 ? waves : 65536));
    // (primes of which two is no small root: long rows of a power-law matrix are sums of few powers of two)
    auto grid = [&](int64_t most) { return dim3((unsigned)(B.rows < most ? B.rows : most)); };
    const dim3 long_grid = grid(1019);
    auto launch = [&](auto zero) {
        using V = decltype(zero);
        const V *val = static_cast<const V *>(B.val);
        V *out = static_cast<V *>(val_out);
        hipLaunchKernelGGL(k_sort_b_short<V>, short_grid, dim3(WAVE * SB_WAVES), 0, s, B.rp, B.col, val, B.rows, col_out, out);
        const int bitmap_from = sort_bitmap_from(B.cols);
        static_assert(SB_SHORT < SORT_BITMAP_LEAST, "rows of a wave come first");
        const auto middle = bitmap_from <= 512 ? k_sort_b_middle<V, 512> : bitmap_from <= 1024 ? k_sort_b_middle<V, 1024>
                            : bitmap_from <= 2048 ? k_sort_b_middle<V, 2048> : k_sort_b_middle<V, SB_MAX>;
        if (bitmap_from > SORT_BITMAP_LEAST)
            hipLaunchKernelGGL(middle, grid(bitmap_from <= 2048 ? 2039 : 1531 /* that the LDS leaves room for */), dim3(SB_NET_THREADS), 0, s, B.rp, B.col, val, B.rows, bitmap_from, col_out, out);
        hipLaunchKernelGGL(k_sort_b_long<V>, long_grid, dim3(SB_THREADS), 0, s, B.rp, B.col, val, B.rows, B.cols, bitmap_from,
                           col_out, out, flags);
    };
    if (dtype == OCEAN_F64) launch(0.0);
    else launch(0.0f);
    return hipGetLastError();
}

size_t sort_rows_scratch_bytes(int64_t count)
{
    if (count <= 1 || count > 0x7fffffffLL) return 0;
    return sort_up((size_t)OB_CLASSES * sizeof(unsigned int)) + sort_up((size_t)count * 4);
}

// rows[0..count) reordered in place by ascending class of their product counts.  scratch:
// sort_rows_scratch_bytes(count) bytes.
hipError_t launch_sort_rows_by_products(const int64_t *prod, int32_t *rows, int64_t count, void *scratch, hipStream_t s)
{
    if (count <= 1 || count > 0x7fffffffLL) return hipSuccess;
    char *base = static_cast<char *>(scratch);
    unsigned int *hist = reinterpret_cast<unsigned int *>(base);
    int32_t *rows_out = reinterpret_cast<int32_t *>(base + sort_up((size_t)OB_CLASSES * sizeof(unsigned int)));
    hipError_t e = hipMemsetAsync(hist, 0, (size_t)OB_CLASSES * sizeof(unsigned int), s);
    if (e != hipSuccess) return e;
    int64_t blocks = (count + OB_THREADS * OB_ITEMS - 1) / (OB_THREADS * OB_ITEMS);
    const int64_t count_blocks = blocks < 512 ? blocks : 512;
    hipLaunchKernelGGL(k_order_count, dim3((unsigned)count_blocks), dim3(OB_THREADS), 0, s, prod, rows, count, hist);
    hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(OB_CLASSES), 0, s, hist);
    hipLaunchKernelGGL(k_order_scatter, dim3((unsigned)blocks), dim3(OB_THREADS), 0, s, prod, rows, count, hist, rows_out);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return hipMemcpyAsync(rows, rows_out, (size_t)count * 4, hipMemcpyDeviceToDevice, s);
}

}  // namespace ocean
