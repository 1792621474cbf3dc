// Analysis step and HyperLogLog size prediction (paper Sections 2.4, 3.1, 3.2).
//
//   k_validate        input check (row offsets ascending, column ids in range)
//   k_row_products    input check of A; prod[i] = sum_{k in A_i} nnz(B_k); P and the largest row; longest B row per A row
//   k_hll_sketch      construct: one m-register sketch per row of B, registers live in LDS per lane group
//   k_hll_merge       merge along each row of A (byte-wise max of 8 registers per lane) + estimate
//   k_sample_reduce   sums over the sampled rows for the sampled compression ratio
//
// All kernels are HBM/L2-bound gathers; rows are mapped to groups of G lanes
// (G a power of two <= 64 chosen from the average row length) so that short
// rows do not leave most of a 64-wide wave idle.
#include <type_traits>

#include "ocean_internal.hpp"

namespace ocean {

constexpr int TPB = 256;

static inline int ilog2_ceil(double x, int lo, int hi)
{
    int l = lo;
    while (l < hi && (double)(1 << l) < x) ++l;
    return l;
}

// ---------------------------------------------------------------- validate
// near_pairs (may be null): a measure of how clustered the columns of the matrix are, taken on a sample (for a B that is A
// itself by k_row_products, from the rows that are not long) - every 16th workgroup adds the number of entries it looked at to near_pairs[0] and the number of those whose
// successor's column id is 1 .. 4 larger to near_pairs[1] (pairs across a row boundary count too; they are few).
// One pair of atomics per sampling workgroup: same-address atomics serialise at about 12 ns each.
__global__ void k_validate(const int64_t *rp, const int32_t *col, int64_t rows, int64_t cols, int64_t nnz,
                           int32_t *flags, int bit, unsigned long long *near_pairs)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    const bool sampling = near_pairs != nullptr && (blockIdx.x & 15u) == 0u;   // uniform
    unsigned int near = 0, seen = 0;
    for (int64_t i = t0; i < rows; i += stride) {
        int64_t a = rp[i], b = rp[i + 1];
        bad |= (b < a) | (a < 0) | (b > nnz);
    }
    if (t0 == 0) bad |= (rp[0] != 0) | (rp[rows] != nnz);
    for (int64_t e = t0; e < nnz; e += stride) {
        int32_t c = col[e];
        bad |= ((uint32_t)c >= (uint64_t)cols);
        if (sampling && e + 1 < nnz) { near += (uint32_t)(col[e + 1] - c - 1) < 4u; ++seen; }
    }
    if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(flags, bit);
    if (sampling) {
        __shared__ unsigned int s_near, s_seen;
        if (threadIdx.x == 0) { s_near = 0u; s_seen = 0u; }
        __syncthreads();
        const unsigned int wave_near = wave_sum_u32(near), wave_seen = wave_sum_u32(seen);
        if (lane_id() == 0) { atomicAdd(&s_near, wave_near); atomicAdd(&s_seen, wave_seen); }
        __syncthreads();
        if (threadIdx.x == 0 && s_seen) {
            atomicAdd(&near_pairs[0], (unsigned long long)s_seen);
            atomicAdd(&near_pairs[1], (unsigned long long)s_near);
        }
    }
}

// Input check of B, bit 2 of flags.  near_pairs: two zeroed device counters (see k_validate).  A is checked by the kernel
// that counts its products; where B is the same matrix that kernel takes the sample as well.
hipError_t launch_validate(const Csr &B, int32_t *flags, unsigned long long *near_pairs, hipStream_t s)
{
    int64_t work = B.nnz > B.rows ? B.nnz : B.rows;
    int blocks = (int)((work + TPB * 4 - 1) / (TPB * 4));
    if (blocks < 1) blocks = 1;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_validate, dim3(blocks), dim3(TPB), 0, s, B.rp, B.col, B.rows, B.cols, B.nnz, flags, 2, near_pairs);
    return hipGetLastError();
}

// ---------------------------------------------------------------- long rows
// The long rows of a power-law matrix sit side by side (their numbers share bit patterns), so the workgroup that meets
// them in its stretch of rows is the whole kernel's time.  The kernels below therefore leave them to workgroups of their
// own, the first n_long of the same launch: workgroup b of them looks at rows 4 b .. 4 b + 3 of every stretch of 4 n_long
// rows and takes the long ones among them.  n_long is a prime and not near a power of two: the long rows of a power-law matrix
// have few one bits in their numbers, and of the 3981 rows of 256 entries and more of R-MAT scale 18 one workgroup of 1023 had
// 35, one of 997 has 12.  A second launch for them cost matrices without any 5 us.  One for every 16 rows, rounded down by an eighth
// at most: where every row is long (4000 rows of 3000 entries, row products) 127 workgroups took 155 us, 241 take 111.
constexpr int LONG_ROWS = 4;        // neighbouring rows that such a workgroup looks at together
constexpr int WAVE_ROW = 2048;      // up to here a wave takes a long row of k_row_products, four turns of eight entries a lane

static int long_row_blocks(int64_t rows)
{
    for (int n : {997, 881, 787, 691, 613, 547, 487, 431, 383, 347, 307, 277, 241, 211, 191, 167, 149, 137, 113, 101, 89, 79, 71, 59, 53,
                  47, 41, 37, 29, 23, 19, 17, 13, 11, 7, 5, 3})
        if ((int64_t)n * 16 <= rows) return n;
    return 1;
}

// take(row) for every row of 0 .. rows - 1 for which size(row) is 2, by the whole workgroup of THREADS threads (uniform,
// barriers allowed), and take_wave(row) for those where it is 1, by one wave (0: not a long row).  s_list: THREADS words,
// s_n: one.
template <int THREADS = TPB, typename Size, typename TakeWave, typename Take>
__device__ __forceinline__ void for_long_rows(int64_t rows, int n_long, int32_t *s_list, int *s_n, Size size, TakeWave take_wave,
                                              Take take)
{
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int64_t stretch = (int64_t)n_long * LONG_ROWS;
    const int64_t first = (int64_t)blockIdx.x * LONG_ROWS + tid % LONG_ROWS + (int64_t)(tid / LONG_ROWS) * stretch;
    for (int64_t base = 0; base < rows; base += stretch * (THREADS / LONG_ROWS)) {   // uniform
        if (tid == 0) *s_n = 0;
        __syncthreads();
        const int64_t r = base + first;
        const int of = r < rows ? size(r) : 0;
        if (of != 0) s_list[atomicAdd(s_n, 1)] = of == 1 ? (int32_t)r : ~(int32_t)r;
        __syncthreads();
        const int n = *s_n;
        for (int i = 0, seen = 0; i < n; ++i) {   // uniform
            const int32_t of_wave = __builtin_amdgcn_readfirstlane(s_list[i]);
            if (of_wave >= 0 && seen++ % (THREADS / WAVE) == wave) take_wave((int64_t)of_wave);
        }
        for (int i = 0; i < n; ++i) {
            const int32_t of_all = s_list[i];
            if (of_all < 0) take((int64_t)~of_all);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------ row products
// One group of 2^g_log2 lanes per row, a fixed number of workgroups striding
// over the rows: the totals cost one atomic per workgroup, not one per row tile
// (same-address atomics from all XCDs serialise in the memory fabric).  A row
// far longer than the average would keep its few lanes busy for a long time:
// it is left to the workgroups for long rows.
// Totals of the row-products pass.  Same-address atomics from all over the chip serialise in the L2 at about 12
// ns each, and there is one set per workgroup: they are spread over ROW_TOTAL_SLOTS slots of 256 bytes (two
// cache lines each) by workgroup index and added up by whoever reads them (sum_row_totals on the host).
// slot[0] += products, slot[1] = max(products of a row), slot[2] += products of the rows whose product count
// exceeds heavy_from (the rows that outgrow the LDS hash tables), slot[3] += rows without products, then the rows of each
// sort class, the most LDS of four sorted rows and the sums of sampled rows (ROW_TOTAL_CLASS, _LDS, _MERGE).  s_tot: the workgroup's own, summed in
// LDS, so that its sums leave in one instruction.
__device__ __forceinline__ void block_totals(long long tsum, long long tmax, long long theavy, int lds_most,
                                             unsigned long long *s_tot, unsigned long long *totals)
{
    const long long wsum = group_reduce_sum(tsum, WAVE);
    const long long wmax = group_reduce_max(tmax, WAVE);
    const long long wheavy = group_reduce_sum(theavy, WAVE);
    const int most = (int)wave_max_u32((uint32_t)lds_most);
    if (lane_id() == 0) {
        atomicAdd(&s_tot[0], (unsigned long long)wsum);
        atomicMax(&s_tot[1], (unsigned long long)wmax);
        atomicAdd(&s_tot[2], (unsigned long long)wheavy);
        atomicMax(&s_tot[ROW_TOTAL_LDS], (unsigned long long)most);
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < ROW_TOTALS && s_tot[t] != 0ull) {
        unsigned long long *slot = totals + (size_t)(blockIdx.x % ROW_TOTAL_SLOTS) * ROW_TOTAL_STRIDE;
        if (t == 1 || t == ROW_TOTAL_LDS) atomicMax(&slot[t], s_tot[t]);
        else atomicAdd(&slot[t], s_tot[t]);
    }
}

// Smallest sort class that holds a row of pr products from ne entries, 0: none.
__device__ __forceinline__ int smallest_sort_class(int pr, int ne)
{
    static_assert(kSortClass[2].entries == kSortClass[SORT_CLASSES - 1].entries, "classes differ in entries below the second only");
    int cls = 1;
#pragma unroll
    for (int c = 1; c < SORT_CLASSES; ++c) cls += pr > kSortClass[c].cap;
    if (cls == 1 && ne > kSortClass[1].entries) cls = 2;
    return cls < SORT_CLASSES && ne <= kSortClass[2].entries ? cls : 0;
}

// Sum and maximum over every group of 2^GL lanes, in each of its lanes: swaps of neighbours, pairs, mirrored halves and rows
// (data-parallel moves, no trip to LDS) up to 16 lanes.
template <int GL>
__device__ __forceinline__ void group_totals(unsigned long long &sum, uint32_t &most)
{
    auto step = [&](auto ctrl) {
        constexpr int CTRL = decltype(ctrl)::value;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)sum, CTRL, 0xf, 0xf, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(sum >> 32), CTRL, 0xf, 0xf, false);
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)most, CTRL, 0xf, 0xf, false);
        sum += ((unsigned long long)hi << 32) | lo;
        most = o > most ? o : most;
    };
    if constexpr (GL >= 1) step(std::integral_constant<int, 0xB1>());    // quad_perm [1,0,3,2]
    if constexpr (GL >= 2) step(std::integral_constant<int, 0x4E>());    // quad_perm [2,3,0,1]
    if constexpr (GL >= 3) step(std::integral_constant<int, 0x141>());   // row_half_mirror
    if constexpr (GL >= 4) step(std::integral_constant<int, 0x140>());   // row_mirror
    for (int off = 16; off < (1 << GL); off <<= 1) {
        sum += __shfl_xor(sum, off, WAVE);
        const uint32_t o = __shfl_xor(most, off, WAVE);
        most = o > most ? o : most;
    }
}

// Two neighbouring row offsets, in one load.
typedef uint32_t RowEnds __attribute__((ext_vector_type(4), aligned(8)));
__device__ __forceinline__ unsigned long long row_length(RowEnds e)
{
    return (((unsigned long long)e.w << 32) | e.z) - (((unsigned long long)e.y << 32) | e.x);
}

// bad_bit: bit of flags that any fault of A sets besides its own (0: none, and A's ends are not looked at).
// near_pairs (given where B is the same matrix): see k_validate; the sample is every 16th workgroup of those for rows that
// are not long, so the long rows of a power-law matrix are not in it.  It decides nothing but which of two orderings of a
// small hash table is used and, by a descending pair of columns in a sampled row, which sets bit 8, whether B's window
// table is tried: never the result.
//
// What bounds it: a gather of two row offsets of B per entry of A, one line a lane, which the address unit takes one a cycle,
// and for rows of few entries the instructions per row.  Offsets come in one 16-byte load instead of two of 8, totals of a row go
// through lane moves instead of LDS, and a row's class is found in 32 bits.
// MERGE: n_merge workgroups, after those for long rows, count the different columns of MERGE_SAMPLE rows of C.  It is bound by
// a chain of four to eleven loads, which ends before the other workgroups do; with rows of B of any length it did not (R-MAT
// scale 15: 29 us instead of 17).
template <int GL, bool MERGE>
__global__ void __launch_bounds__(TPB, 8)
k_row_products(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, int64_t m, int64_t a_nnz,
               const int64_t *__restrict__ b_rp, int64_t b_rows, int64_t long_from, int n_long,
               int64_t *__restrict__ prod, int32_t *__restrict__ maxb, unsigned long long *totals, int32_t *flags,
               int64_t heavy_from, int bad_bit, unsigned long long *near_pairs, unsigned long long *zero, int64_t zero_words,
               int vbytes, const int32_t *__restrict__ b_col, int64_t b_nnz, int n_merge)
{
    constexpr int G = 1 << GL;
    constexpr int R = TPB >> GL;
    __shared__ unsigned int s_near, s_seen;
    __shared__ unsigned long long s_tot[ROW_TOTALS];
    __shared__ uint32_t s_seen_col[MERGE ? TPB / WAVE : 1][MERGE ? 2 * MERGE_PRODUCTS : 1];
    __shared__ unsigned long long s_sum[TPB / WAVE];
    __shared__ uint32_t s_max[TPB / WAVE];
    __shared__ int32_t s_list[TPB];
    __shared__ int s_n;
    const int tid = threadIdx.x;
    const int rl = tid >> GL;
    const int sub = tid & (G - 1);
    const bool for_long = (int)blockIdx.x < n_long;   // uniform
    if (!MERGE) n_merge = 0;
    const int64_t block = (int64_t)blockIdx.x - n_long - n_merge, blocks = (int64_t)gridDim.x - n_long - n_merge;
    const bool for_merge = MERGE && !for_long && block < 0;        // uniform
    const bool sampling = near_pairs != nullptr && block >= 0 && (block & 15) == 0;   // uniform
    unsigned int near = 0, seen = 0;
    long long tsum = 0, tmax = 0, theavy = 0;
    bool unsorted = false;
    int lds_most = 0;
    if (tid < ROW_TOTALS) s_tot[tid] = 0ull;
    for (int64_t i = (int64_t)blockIdx.x * TPB + tid; i < zero_words; i += (int64_t)gridDim.x * TPB) zero[i] = 0ull;
    __syncthreads();
    bool bad = false, bad_rp = bad_bit != 0 && blockIdx.x == 0 && tid == 0 && (a_rp[0] != 0 || a_rp[m] != a_nnz);
    // entries first, first + step, ... below e1: U independent chains (entry -> row offsets of B) in flight per lane;
    // reads are unconditional (index clamped) so that they are issued together
    auto walk = [&](auto depth, int64_t first, int64_t e1, int step, unsigned long long &p, uint32_t &mx) {
        constexpr int U = decltype(depth)::value;
        for (int64_t e = first; e < e1; e += U * (int64_t)step) {
            int32_t k[U];
            bool ok[U];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int64_t idx = e + (int64_t)i * step;
                ok[i] = idx < e1;
                k[i] = a_col[ok[i] ? idx : e];
            }
            if (sampling) {
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    const int64_t idx = e + (int64_t)i * step;
                    if (ok[i] && idx + 1 < a_nnz) {
                        const int32_t next = a_col[idx + 1];
                        near += (uint32_t)(next - k[i] - 1) < 4u;
                        ++seen;
                        unsorted |= idx + 1 < e1 && next < k[i];
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < U; ++i)
                if ((uint32_t)k[i] >= (uint64_t)b_rows) { bad = true; k[i] = 0; ok[i] = false; }
            if (b_rows == 0) continue;   // uniform
            RowEnds ends[U];
#pragma unroll
            for (int i = 0; i < U; ++i) ends[i] = *reinterpret_cast<const RowEnds *>(b_rp + k[i]);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const unsigned long long len = ok[i] ? row_length(ends[i]) : 0ull;
                p += len;
                const uint32_t most = len > 0x7fffffffull ? 0x7fffffffu : (uint32_t)len;
                mx = most > mx ? most : mx;
            }
        }
    };
    auto store = [&](int64_t row, int64_t ne, unsigned long long p, uint32_t mx) {
        prod[row] = (int64_t)p;
        maxb[row] = (int32_t)mx;
        tsum += (long long)p;
        tmax = (long long)p > tmax ? (long long)p : tmax;
        theavy += (long long)p > heavy_from ? (long long)p : 0;
        const int cls = p == 0 ? -1 : smallest_sort_class(p < (1u << 20) ? (int)p : 1 << 20, ne < (1 << 20) ? (int)ne : 1 << 20);
        atomicAdd(&s_tot[ROW_TOTAL_CLASS + cls], 1ull);
    };
    if (for_long) {
        for_long_rows(m, n_long, s_list, &s_n,
                      [&](int64_t r) {
                          const int64_t e0 = a_rp[r], e1 = a_rp[r + 1];
                          if (e0 < 0 || e1 > a_nnz || e1 - e0 < long_from) return 0;   // (bad ones are reported below)
                          return e1 - e0 < WAVE_ROW ? 1 : 2;
                      },
                      [&](int64_t row) {
                          const int64_t e0 = a_rp[row], e1 = a_rp[row + 1];
                          unsigned long long p = 0;
                          uint32_t mx = 0;
                          walk(std::integral_constant<int, 8>(), e0 + lane_id(), e1, WAVE, p, mx);
                          group_totals<6>(p, mx);
                          if (lane_id() == 0) store(row, e1 - e0, p, mx);
                      },
                      [&](int64_t row) {
                          unsigned long long p = 0;
                          uint32_t mx = 0;
                          walk(std::integral_constant<int, 8>(), a_rp[row] + tid, a_rp[row + 1], TPB, p, mx);
                          group_totals<6>(p, mx);
                          if (lane_id() == 0) { s_sum[tid / WAVE] = p; s_max[tid / WAVE] = mx; }
                          __syncthreads();
                          if (tid == 0) {
                              p = mx = 0;
                              for (int j = 0; j < TPB / WAVE; ++j) { p += s_sum[j]; mx = s_max[j] > mx ? s_max[j] : mx; }
                              store(row, a_rp[row + 1] - a_rp[row], p, mx);
                          }
                          __syncthreads();
                      });
    } else if (for_merge) {   // (never without MERGE)
        // The different columns among a row's products, by a wave: the offsets of B are not checked yet, nor are A's.
        const int64_t turn = (int64_t)((int)blockIdx.x - n_long) * (TPB / WAVE) + tid / WAVE;
        const int64_t part = m / MERGE_SAMPLE;   // (at least one row)
        const int64_t row = turn * part + (int64_t)((uint32_t)turn * 2654435769u >> 8) % part;
        uint32_t *seen_col = s_seen_col[tid / WAVE];
        for (int i = lane_id(); i < 2 * MERGE_PRODUCTS; i += WAVE) seen_col[i] = 0xffffffffu;
        wave_sync();
        const int64_t e0 = a_rp[row], e1 = a_rp[row + 1];
        bool fits = e0 >= 0 && e1 >= e0 && e1 <= a_nnz && e1 - e0 <= WAVE;   // uniform for the wave
        int64_t p0 = 0;
        uint32_t len = 0;
        if (fits && e0 + lane_id() < e1) {
            const int32_t k = a_col[e0 + lane_id()];
            if ((uint32_t)k < (uint64_t)b_rows) {
                const int64_t first = b_rp[k], end = b_rp[k + 1];
                if (first >= 0 && end >= first && end <= b_nnz) {
                    p0 = first;
                    len = end - first > MERGE_LENGTH ? MERGE_PRODUCTS + 1 : (uint32_t)(end - first);
                }
            }
        }
        const uint32_t products = wave_sum_u32(len);
        fits = fits && products <= (uint32_t)MERGE_PRODUCTS;
        if (!fits) len = 0;
        uint32_t fresh = 0;
        for (uint32_t i = 0; i < len; i += 4) {
            uint32_t col[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) col[u] = (uint32_t)b_col[p0 + (i + u < len ? i + u : i)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i + u >= len) continue;
                uint32_t at = col[u] * 2654435769u >> 23;   // (at most half of the 512 places are taken: a free one is met)
                static_assert(MERGE_PRODUCTS == 256, "nine bits");
                for (;;) {
                    const uint32_t was = atomicCAS(&seen_col[at], 0xffffffffu, col[u]);
                    fresh += was == 0xffffffffu;
                    if (was == 0xffffffffu || was == col[u]) break;
                    at = (at + 1) & (2 * MERGE_PRODUCTS - 1);
                }
            }
        }
        fresh = wave_sum_u32(fresh);
        if (lane_id() == 0 && fits) {
            atomicAdd(&s_tot[ROW_TOTAL_MERGE], (unsigned long long)products);
            atomicAdd(&s_tot[ROW_TOTAL_MERGE + 1], (unsigned long long)fresh);
            atomicAdd(&s_tot[ROW_TOTAL_MERGE + 2], 1ull);
        }
    } else {
        for (int64_t base = block * R; base < m; base += blocks * R) {
            const int64_t row = base + rl;
            unsigned long long p = 0;
            uint32_t mx = 0;
            bool mine = row < m;
            int64_t ne = 0;
            if (mine) {
                // offsets outside [0, nnz] or descending are reported and never used as they stand: this kernel
                // runs before the host has seen the verdict of the input check
                int64_t e0 = a_rp[row], e1 = a_rp[row + 1];
                if (e0 < 0 || e1 < e0 || e1 > a_nnz) { bad_rp = true; e0 = 0; e1 = 0; }
                ne = e1 - e0;
                mine = n_long == 0 || ne < long_from;   // uniform for the group
                if (mine) walk(std::integral_constant<int, 4>(), e0 + sub, e1, G, p, mx);
            }
            group_totals<GL>(p, mx);
            if (mine && sub == 0) store(row, ne, p, mx);
            // (with more lanes a wave has fewer than four rows: four times the row that takes most.  Where no row of the wave
            // has more than 256 products, four rows take the least there is, which the host knows)
            if (__ballot(p > 256ull) != 0ull) {
                int lds = sort_row_bytes(p < 2048ull ? (int)p : 2048, vbytes);
                if constexpr (GL <= 4) {
                    lds += __shfl_xor(lds, G, WAVE);
                    lds += __shfl_xor(lds, 2 * G, WAVE);
                } else {
                    lds *= 4;
                }
                lds_most = lds > lds_most ? lds : lds_most;
            }
        }
    }
    block_totals(tsum, tmax, theavy, lds_most, s_tot, totals);
    if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(flags, 4 | bad_bit);
    if (__ballot(bad_rp) != 0 && lane_id() == 0) atomicOr(flags, 1);
    if (__ballot(unsorted) != 0 && lane_id() == 0) atomicOr(flags, 8);
    if (sampling) {
        if (tid == 0) { s_near = 0u; s_seen = 0u; }
        __syncthreads();
        const unsigned int wave_near = wave_sum_u32(near), wave_seen = wave_sum_u32(seen);
        if (lane_id() == 0) { atomicAdd(&s_near, wave_near); atomicAdd(&s_seen, wave_seen); }
        __syncthreads();
        if (tid == 0 && s_seen) {
            atomicAdd(&near_pairs[0], (unsigned long long)s_seen);
            atomicAdd(&near_pairs[1], (unsigned long long)s_near);
        }
    }
}

// validate: A's offsets must begin at 0 and end at its number of entries as well, and any fault of A sets bit 1 of flags
// (offsets that descend or leave [0, nnz] always do, column ids outside [0, b_rows) always set bit 4).  near_pairs (may
// be null): see k_validate.  zero: zero_words words that the kernel clears on the way, for a later one.  vbytes:
// bytes of a value, for the LDS that sorted rows take.  merge_sample (may be null): B, to count the different columns of
// MERGE_SAMPLE rows of C on the way, see run_placed.
hipError_t launch_row_products(const Csr &A, const int64_t *b_rp, int64_t b_rows, int64_t *prod, int32_t *maxb,
                               unsigned long long *totals, int32_t *flags, bool validate, unsigned long long *near_pairs,
                               unsigned long long *zero, int64_t zero_words, int vbytes, const Csr *merge_sample, hipStream_t s)
{
    const int64_t heavy_from = kNumericSlots[NB_S4K];   // beyond the largest LDS hash table that sorted inputs use
    if (A.rows == 0) return hipSuccess;
    const double avg = (double)A.nnz / (double)A.rows;
    const int g_log2 = ilog2_ceil(avg / 4.0, 1, 6);   // (a lane keeps four entries in flight)
    // Long: eight turns of the group, and more entries than any sort class takes, as the LDS of four sorted rows is summed up
    // where the rows that are not long are (with two lanes a row eight turns are 64 entries, which can be sorted).
    const int64_t turns = (int64_t)32 << g_log2, unsorted_from = kSortClass[SORT_CLASSES - 1].entries + 1;
    const int64_t long_from = turns > unsorted_from ? turns : unsorted_from;
    const int R = TPB >> g_log2;
    int64_t blocks = (A.rows + R - 1) / R;
    if (blocks > 2048) blocks = 2048;
    const int n_long = A.nnz >= long_from ? long_row_blocks(A.rows) : 0;
    const int n_merge = merge_sample != nullptr && A.rows >= MERGE_SAMPLE && g_log2 <= 4 ? MERGE_SAMPLE / (TPB / WAVE) : 0;
    const auto kernel = n_merge != 0 ? (g_log2 == 1 ? k_row_products<1, true> : g_log2 == 2 ? k_row_products<2, true>
                                        : g_log2 == 3 ? k_row_products<3, true> : k_row_products<4, true>)
                        : g_log2 == 1 ? k_row_products<1, false> : g_log2 == 2 ? k_row_products<2, false>
                        : g_log2 == 3 ? k_row_products<3, false> : g_log2 == 4 ? k_row_products<4, false>
                        : g_log2 == 5 ? k_row_products<5, false> : k_row_products<6, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(blocks + n_long + n_merge)), dim3(TPB), 0, s, A.rp, A.col, A.rows, A.nnz,
                       b_rp, b_rows, long_from, n_long, prod, maxb, totals, flags, heavy_from, validate ? 1 : 0, near_pairs, zero,
                       zero_words, vbytes, n_merge != 0 ? merge_sample->col : nullptr, n_merge != 0 ? merge_sample->nnz : 0, n_merge);
    return hipGetLastError();
}

// Totals of a finished row-products pass, handed to a caller-owned device array: {P, largest row, flags}.
__global__ void k_publish_totals(const unsigned long long *totals, const int32_t *flags, int64_t *out)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        unsigned long long sum = 0, mx = 0;
        for (int i = 0; i < ROW_TOTAL_SLOTS; ++i) {
            sum += totals[(size_t)i * ROW_TOTAL_STRIDE];
            const unsigned long long v = totals[(size_t)i * ROW_TOTAL_STRIDE + 1];
            mx = v > mx ? v : mx;
        }
        out[0] = (int64_t)sum;
        out[1] = (int64_t)mx;
        out[2] = (int64_t)*flags;
    }
}

hipError_t launch_publish_totals(const unsigned long long *totals, const int32_t *flags, int64_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_publish_totals, dim3(1), dim3(WAVE), 0, s, totals, flags, out);
    return hipGetLastError();
}

// ------------------------------------------------------------- HLL sketch
// Registers of the rows in flight sit in LDS as 32-bit words (LDS has a
// 32-bit atomic max, Section 3.1 "parallel updates ... atomicMax"); they are
// packed to one byte per register (Section 4.3) when the sketch is stored.
// A row of SK_LONG or more entries is left to the whole workgroup, which takes the long rows of a turn one
// after the other once the lane groups are through with the short ones: on a power-law matrix the longest
// row, walked by one group of 16 lanes, was most of the kernel's time (R-MAT: 0.77 ms).  "Long" is relative: a row
// of long_from entries or more, which the launcher sets to 1024 or eight times the average row, whichever is more
// (where every row is long, sixteen groups side by side are 6 - 12 % faster than the workgroup on one row at a time).
// Where the rows are known or suspected to be skewed, the rows of LONG_SKEWED entries or more go to the workgroups for
// long rows (see for_long_rows): R-MAT scale 18, 64 registers: 72 us with the long rows by the workgroup that met them.
constexpr int SK_LONG = 1024;
constexpr int LONG_SKEWED = 256;

template <int M>
__device__ __forceinline__ void hll_add(uint32_t *regs, int32_t c)
{
    constexpr int P = (M == 32) ? 5 : (M == 64) ? 6 : 7;
    const uint32_t h = hll_hash(c);
    const uint32_t w = h >> P;
    const uint32_t rank = w ? (uint32_t)(__clz((int)w) - P + 1) : (uint32_t)(32 - P + 1);
    atomicMax(&regs[h & (M - 1)], rank);
}

template <int M>
__global__ void __launch_bounds__(TPB)
k_hll_sketch(const int64_t *__restrict__ rp, const int32_t *__restrict__ col, int64_t rows, int g_log2,
             int64_t long_from, int n_long, uint8_t *__restrict__ out)
{
    extern __shared__ uint32_t s_regs[];  // [TPB >> g_log2][M]
    __shared__ uint32_t s_big[M];
    __shared__ int32_t s_long[TPB];   // (at most TPB / 8 rows per turn of the groups, which have 8 lanes or more)
    __shared__ int s_nlong;
    const int G = 1 << g_log2;
    const int sub = threadIdx.x & (G - 1);
    const int rl = threadIdx.x >> g_log2;
    const int R = TPB >> g_log2;
    uint32_t *my = s_regs + rl * M;
    auto store = [&](const uint32_t *regs, int64_t row, int first, int step) {
        uint32_t *dst = reinterpret_cast<uint32_t *>(out + row * M);
        for (int j = first; j < M / 4; j += step)
            dst[j] = regs[4 * j] | (regs[4 * j + 1] << 8) | (regs[4 * j + 2] << 16) | (regs[4 * j + 3] << 24);
    };
    // a long row, by the whole workgroup
    auto take = [&](int64_t lrow) {
        for (int j = threadIdx.x; j < M; j += TPB) s_big[j] = 0;
        __syncthreads();
        const int64_t p1 = rp[lrow + 1];
        for (int64_t p = rp[lrow] + threadIdx.x; p < p1; p += 8 * (int64_t)TPB) {
            int32_t c[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int64_t q = p + (int64_t)k * TPB;
                c[k] = col[q < p1 ? q : p1 - 1];
            }
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (p + (int64_t)k * TPB < p1) hll_add<M>(s_big, c[k]);
        }
        __syncthreads();
        store(s_big, lrow, (int)threadIdx.x, TPB);
        __syncthreads();
    };
    if ((int)blockIdx.x < n_long) {   // uniform
        for_long_rows(rows, n_long, s_long, &s_nlong, [&](int64_t r) { return rp[r + 1] - rp[r] >= long_from ? 2 : 0; },
                      [](int64_t) {}, take);
        return;
    }
    for (int64_t base = ((int64_t)blockIdx.x - n_long) * R; base < rows; base += ((int64_t)gridDim.x - n_long) * R) {   // uniform
        const int64_t row = base + rl;
        if (threadIdx.x == 0) s_nlong = 0;
        for (int j = sub; j < M; j += G) my[j] = 0;
        __syncthreads();
        bool mine = false;
        if (row < rows) {
            const int64_t p0 = rp[row], p1 = rp[row + 1];
            mine = p1 - p0 < long_from;
            if (!mine && n_long == 0 && sub == 0) s_long[atomicAdd(&s_nlong, 1)] = (int32_t)row;
            // four column ids per lane and turn (unconditional reads, index clamped): a long row is bound by
            // the latency of one load after the other otherwise
            for (int64_t p = p0 + sub; mine && p < p1; p += 4 * (int64_t)G) {
                int32_t c[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t q = p + (int64_t)i * G;
                    c[i] = col[q < p1 ? q : p1 - 1];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (p + (int64_t)i * G < p1) hll_add<M>(my, c[i]);
            }
        }
        wave_sync();
        if (mine) store(my, row, sub, G);
        __syncthreads();
        const int nlong = s_nlong;
        for (int i = 0; i < nlong; ++i) take((int64_t)s_long[i]);   // uniform
        __syncthreads();   // (everyone has read s_nlong before the next turn clears it)
    }
}

// lanes_div: 1, or 4 when the rows are known to be of similar lengths - a lane keeps four entries in flight, so a
// quarter of the lanes per row puts four times the rows in flight (short rows are bound by the latency of their
// chain of loads); with skewed lengths the long rows then keep their few lanes busy long after the others.
hipError_t launch_hll_sketch(const Csr &B, int m, uint8_t *sketches, int lanes_div, hipStream_t s)
{
    if (B.rows == 0) return hipSuccess;
    const double avg = (double)B.nnz / (double)B.rows;
    const int g_log2 = ilog2_ceil(avg / (double)lanes_div, 3, 6);
    const int R = TPB >> g_log2;
    int64_t blocks = (B.rows + R - 1) / R;
    if (blocks > 256 * 64) blocks = 256 * 64;
    const size_t lds = (size_t)R * m * sizeof(uint32_t);
    const int64_t least = lanes_div == 1 ? LONG_SKEWED : SK_LONG;
    const int64_t long_from = 8.0 * avg > (double)least ? (int64_t)(8.0 * avg) : least;
    const int n_long = lanes_div == 1 && B.nnz >= long_from ? long_row_blocks(B.rows) : 0;
    blocks += n_long;
    switch (m) {
    case 32: hipLaunchKernelGGL(k_hll_sketch<32>, dim3((unsigned)blocks), dim3(TPB), lds, s, B.rp, B.col, B.rows, g_log2, long_from, n_long, sketches); break;
    case 64: hipLaunchKernelGGL(k_hll_sketch<64>, dim3((unsigned)blocks), dim3(TPB), lds, s, B.rp, B.col, B.rows, g_log2, long_from, n_long, sketches); break;
    case 128: hipLaunchKernelGGL(k_hll_sketch<128>, dim3((unsigned)blocks), dim3(TPB), lds, s, B.rp, B.col, B.rows, g_log2, long_from, n_long, sketches); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// -------------------------------------------------------------- HLL merge
// Sixteen registers of a sketch, as they are loaded and stored (sketches may come from a caller: 8-byte alignment), and the
// maxima of many such: the packed 16-bit maximum orders by the upper byte, so one of the words as they are gives the odd
// registers' maxima and one of the words without the upper bytes the even registers', three instructions for four registers.
typedef uint32_t Regs16 __attribute__((ext_vector_type(4), aligned(8)));
typedef unsigned short Pair16 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t max16x2(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(Pair16, a), __builtin_bit_cast(Pair16, b)));
}
struct RegMax {
    uint32_t odd[4] = {0u, 0u, 0u, 0u}, even[4] = {0u, 0u, 0u, 0u};
    __device__ __forceinline__ void add(Regs16 r)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            odd[i] = max16x2(odd[i], r[i]);
            even[i] = max16x2(even[i], r[i] & 0x00ff00ffu);
        }
    }
    __device__ __forceinline__ Regs16 get() const
    {
        Regs16 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (odd[i] & 0xff00ff00u) | even[i];
        return r;
    }
};
__device__ __forceinline__ Regs16 max_regs(Regs16 a, Regs16 b)
{
    RegMax m;
    m.add(a);
    m.add(b);
    return m.get();
}
// Maxima over lanes first, first + step, .. up to `lanes` (powers of two) that hold the same registers, in each of them.
__device__ __forceinline__ Regs16 lanes_max(Regs16 r, int step, int lanes)
{
    for (int off = step; off < lanes; off <<= 1) {
        Regs16 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (uint32_t)__shfl_xor((int)r[i], off, WAVE);
        r = max_regs(r, o);
    }
    return r;
}

__device__ __forceinline__ double hll_alpha(int m)
{
    return m == 32 ? 0.697 : m == 64 ? 0.709 : 0.7213 / (1.0 + 1.079 / (double)m);
}

// One group of G lanes per selected row of A; L = M/16 lanes cover one sketch (16 registers per lane) so G/L entries of the
// row are merged at once.  Each 64-byte sketch of B is read as one coalesced line.  What bounds it is the latency of the
// chain offsets -> entries -> sketches and the part of the sketches that misses the L2 (with 8 registers a lane and the
// maximum in 64-bit arithmetic it was instructions as well: all rows of R-MAT scale 18 with 64 registers, 4 M sketches,
// 304 us, now 150 in both launches).
// Long rows: long_from entries or more.  Where all rows of a matrix that is or may be skewed are merged, n_long workgroups
// at the front of the grid take them, a wave each up to huge_from entries and by all threads from there on, or those are
// left to k_hll_merge_long (huge_here false).  With n_long = 0 the workgroup that meets a long row takes it.
constexpr int MG_LONG = 2048;
constexpr int MG_SKEWED = 64;
constexpr int MG_WAVE = 1024;    // a wave takes up to 64 entries a turn with 64 registers, and 16 turns are 20 us

// Entries first, first + step, ... of a row, for one slice (16 registers) of the sketch: U per lane and turn
// (unconditional reads, index clamped; merging a sketch twice is harmless), so that the dependent loads entry ->
// sketch of U entries overlap.
// spans: what else the sample wants to know of the row, the first and last column it can reach.
struct Reach {
    const int32_t *b_col = nullptr;   // null: not asked for
    int first = 0x7fffffff, last = -1;
};
template <int L, int U, bool SAMPLE = false>
__device__ __forceinline__ void hll_walk(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col,
                                         const uint64_t *__restrict__ sk, const int64_t *__restrict__ b_rp, int64_t row,
                                         int slice, int first, int step, RegMax &acc, long long &blen_max,
                                         Reach *reach = nullptr)
{
    const int64_t e1 = a_rp[row + 1];
    for (int64_t e = a_rp[row] + first; e < e1; e += U * (int64_t)step) {
        int32_t k[U];
        Regs16 regs[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int64_t q = e + (int64_t)i * step;
            k[i] = a_col[q < e1 ? q : e1 - 1];
        }
#pragma unroll
        for (int i = 0; i < U; ++i) regs[i] = *reinterpret_cast<const Regs16 *>(sk + ((int64_t)k[i] * L + slice) * 2);
#pragma unroll
        for (int i = 0; i < U; ++i) acc.add(regs[i]);
        if (SAMPLE && reach->b_col != nullptr && slice == 0) {
            RowEnds ends[U];
#pragma unroll
            for (int i = 0; i < U; ++i) ends[i] = *reinterpret_cast<const RowEnds *>(b_rp + k[i]);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int64_t p0 = (int64_t)(((unsigned long long)ends[i].y << 32) | ends[i].x);
                const int64_t len = (int64_t)row_length(ends[i]);
                if (len > 0) {
                    const int32_t c0 = reach->b_col[p0], c1 = reach->b_col[p0 + len - 1];
                    reach->first = c0 < reach->first ? c0 : reach->first;
                    reach->last = c1 > reach->last ? c1 : reach->last;
                }
            }
        }
        if (!SAMPLE && b_rp != nullptr && slice == 0) {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const long long len = b_rp[k[i] + 1] - b_rp[k[i]];
                blen_max = len > blen_max ? len : blen_max;
            }
        }
    }
}

// Row t of the stratified sample of Section 3.2, one row out of each of ns equal strata of `rows` rows (both below 2^31), chosen
// by a hash of the stratum's number and the seed: the same rows as the host helper behind ocean_sample_rows gives.
struct SampleOf {
    int64_t rows, ns;
    int64_t first;                  // number of the launch's first sampled row
    uint32_t seed;
    int64_t whole_from;             // rows of so many entries count as reaching everywhere
    const int32_t *b_col;           // null: reach not asked for
    int64_t *prod_out;              // products of the sampled rows
    int32_t *span_out;              // columns they can reach, 0: none, the largest number: everywhere
    const int32_t *count_col;       // B's columns, for the rows whose columns are counted
    unsigned long long *count_totals;   // and the sums over them
    __device__ __forceinline__ int64_t row(int64_t slot) const
    {
        const int64_t t = first + slot;
        const uint64_t lo = (uint64_t)t * (uint64_t)rows / (uint64_t)ns;
        const uint64_t hi = (uint64_t)(t + 1) * (uint64_t)rows / (uint64_t)ns;
        return (int64_t)(lo + fmix32(seed + 0x9E3779B9u * (uint32_t)(t + 1)) % (hi - lo));
    }
};

// L consecutive lanes hold the merged sketch of slot t (row `row`), 16 registers each: estimate and store.  (Sums of up to
// 128 powers of two from 2^-33 on are exact, in whatever order.)
template <int M>
__device__ __forceinline__ void hll_finish(Regs16 acc, long long blen_max, int64_t t, int64_t row, int slice, bool write,
                                           const int64_t *__restrict__ prod, const int32_t *__restrict__ maxb,
                                           int64_t b_cols, double *__restrict__ est, uint64_t *__restrict__ merged)
{
    constexpr int L = M / 16;
    double ssum = 0.0;
    int zeros = 0;
#pragma unroll
    for (int b = 0; b < 16; ++b) {
        const unsigned r = (acc[b / 4] >> (8 * (b % 4))) & 0xFFu;
        ssum += __longlong_as_double((long long)(1023 - (int)r) << 52);  // 2^-r, exact
        zeros += (r == 0);
    }
    for (int off = L >> 1; off > 0; off >>= 1) {
        ssum += __shfl_xor(ssum, off, WAVE);
        zeros += __shfl_xor(zeros, off, WAVE);
    }
    if (write) {
        if (merged != nullptr) *reinterpret_cast<Regs16 *>(merged + (t * L + slice) * 2) = acc;
        if (slice == 0) {
            const double dm = (double)M;
            double e = hll_alpha(M) * dm * dm / ssum;
            if (e <= 2.5 * dm && zeros > 0) e = dm * log(dm / (double)zeros);
            if (prod != nullptr) {
                const long long pr = prod[row];
                const double hi = (double)(pr < b_cols ? pr : b_cols);
                const double lo = (double)(maxb != nullptr ? (long long)maxb[row] : blen_max);
                e = e < lo ? lo : e;
                e = e > hi ? hi : e;
            }
            est[t] = e;
        }
    }
}

// A row by a whole workgroup of THREADS threads.  s_regs: 4 words per lane of a sketch and wave, s_blen: one word per wave.
template <int M, int THREADS, int U>
__device__ __forceinline__ void hll_row_by_all(Regs16 (*s_regs)[M / 16], long long *s_blen, const int64_t *__restrict__ a_rp,
                                               const int32_t *__restrict__ a_col, const uint64_t *__restrict__ sk, int64_t t,
                                               int64_t row, const int64_t *__restrict__ prod, const int32_t *__restrict__ maxb,
                                               const int64_t *__restrict__ b_rp, int64_t b_cols, double *__restrict__ est,
                                               uint64_t *__restrict__ merged)
{
    constexpr int L = M / 16, NW = THREADS / WAVE;
    const int tid = threadIdx.x, slice = tid & (L - 1), wave = tid / WAVE;
    RegMax acc;
    long long blen = 0;
    hll_walk<L, U>(a_rp, a_col, sk, b_rp, row, slice, tid / L, THREADS / L, acc, blen);
    const Regs16 mine = lanes_max(acc.get(), L, WAVE);
    blen = group_reduce_max(blen, WAVE);
    if (lane_id() < L) s_regs[wave][lane_id()] = mine;
    if (lane_id() == 0) s_blen[wave] = blen;
    __syncthreads();
    if (tid < WAVE) {   // (the whole first wave: lane swaps)
        RegMax all;
        long long longest = 0;
        for (int w = 0; w < NW; ++w) {
            all.add(s_regs[w][slice]);
            longest = s_blen[w] > longest ? s_blen[w] : longest;
        }
        hll_finish<M>(all.get(), longest, t, row, slice, tid < L, prod, maxb, b_cols, est, merged);
    }
    __syncthreads();
}

// The different columns of a row of C, by a workgroup: a bit for each by 17 bits of its hash, and what that many places with
// so many taken stand for (linear counting: of up to 8192 columns some 0.2 % off at one standard deviation; sketches of 64
// registers are 13 %, and rows over the same columns all err alike).  A wave takes an entry of A, four in flight: the chain
// offsets -> entries -> offsets of B -> columns, up to four times over, ends before the merge of the sample that runs
// beside it.  A row with more than COUNT_ENTRIES entries would not; its products count as so many columns.
// totals: COUNT_SLOTS slots of COUNT_STRIDE words, where the sums over the rows of products, columns (to the nearest whole one),
// products squared, columns squared and products times columns are spread.
constexpr int COUNT_LOG2 = 17;
__device__ __forceinline__ void count_columns(uint32_t *s_bits, int *s_n, const int64_t *__restrict__ a_rp,
                                              const int32_t *__restrict__ a_col, const int64_t *__restrict__ b_rp,
                                              const int32_t *__restrict__ b_col, int64_t row, int64_t products,
                                              unsigned long long *totals)
{
    constexpr int WORDS = 1 << (COUNT_LOG2 - 5), U = 4, NW = TPB / WAVE;
    const int tid = threadIdx.x;
    for (int i = tid; i < WORDS; i += TPB) s_bits[i] = 0u;
    if (tid == 0) *s_n = 0;
    __syncthreads();
    const int64_t e0 = a_rp[row], e1 = a_rp[row + 1];
    const bool walked = products <= COUNT_PRODUCTS && e1 - e0 <= COUNT_ENTRIES;   // uniform
    for (int64_t e = e0 + tid / WAVE; walked && e < e1; e += U * NW) {
        int32_t k[U];
        RowEnds ends[U];
#pragma unroll
        for (int i = 0; i < U; ++i) k[i] = a_col[e + i * NW < e1 ? e + i * NW : e];
#pragma unroll
        for (int i = 0; i < U; ++i) ends[i] = *reinterpret_cast<const RowEnds *>(b_rp + k[i]);
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int64_t p0 = (int64_t)(((unsigned long long)ends[i].y << 32) | ends[i].x);
            const int len = e + i * NW < e1 ? (int)row_length(ends[i]) : 0;
            for (int q0 = lane_id(); q0 < len; q0 += U * WAVE) {
                int32_t c[U];
#pragma unroll
                for (int j = 0; j < U; ++j) c[j] = b_col[p0 + (q0 + j * WAVE < len ? q0 + j * WAVE : q0)];
#pragma unroll
                for (int j = 0; j < U; ++j) {   // (a column twice is no harm)
                    const uint32_t h = hll_hash(c[j]) >> (32 - COUNT_LOG2);
                    atomicOr(&s_bits[h >> 5], 1u << (h & 31u));
                }
            }
        }
    }
    __syncthreads();
    int ones = 0;
    for (int i = tid; i < WORDS; i += TPB) ones += __popc(s_bits[i]);
    ones = group_reduce_sum(ones, WAVE);
    if (lane_id() == 0) atomicAdd(s_n, ones);
    __syncthreads();
    if (tid < COUNT_SUMS) {
        const double places = (double)(1 << COUNT_LOG2);
        const unsigned long long p = (unsigned long long)products, of = (unsigned long long)llrint(-places * log1p(-(double)*s_n / places));
        const unsigned long long n = walked && of < p ? of : p;
        const unsigned long long sum = tid == 0 ? p : tid == 1 ? n : tid == 2 ? p * p : tid == 3 ? n * n : p * n;
        atomicAdd(totals + (size_t)(blockIdx.x % COUNT_SLOTS) * COUNT_STRIDE + tid, sum);
    }
}

// (8: with the code for long rows beside it the compiler would take 96 registers and leave 5 waves per SIMD; 10 % slower
// on 256 000 rows of 34 entries)
// SAMPLE: the rows are the sample's, whose products and reach are written beside their estimates; n_long workgroups at the front
// count the columns of rows of it.
template <int M, bool SAMPLE>
__global__ void __launch_bounds__(TPB, 8)
k_hll_merge(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col,
            const uint64_t *__restrict__ sk, const int64_t *__restrict__ rows, int64_t n_rows, int g_log2,
            int64_t long_from, int64_t huge_from, bool huge_here, int n_long, const int64_t *__restrict__ prod,
            const int32_t *__restrict__ maxb, const int64_t *__restrict__ b_rp,
            int64_t b_cols, double *__restrict__ est, uint64_t *__restrict__ merged, const SampleOf sample)
{
    constexpr int L = M / 16;
    auto row_of = [&](int64_t t) { return SAMPLE ? sample.row(t) : rows ? rows[t] : t; };
    __shared__ int32_t s_long[TPB];   // (slot of the row, i.e. its position among the selected rows)
    __shared__ int s_nlong;
    __shared__ Regs16 s_regs[TPB / WAVE][L];
    __shared__ long long s_blen[TPB / WAVE];
    __shared__ uint32_t s_bits[SAMPLE ? 1 << (COUNT_LOG2 - 5) : 1];
    const int G = 1 << g_log2;  // >= L
    if (SAMPLE && (int)blockIdx.x < n_long) {   // uniform
        const int64_t row = sample.row((int64_t)blockIdx.x * sample.ns / n_long);
        count_columns(s_bits, &s_nlong, a_rp, a_col, b_rp, sample.count_col, row, prod[row], sample.count_totals);
        return;
    }
    auto take = [&](int64_t t2) {
        hll_row_by_all<M, TPB, 4>(s_regs, s_blen, a_rp, a_col, sk, t2, row_of(t2), prod, maxb, b_rp, b_cols, est, merged);
    };
    if (!SAMPLE && (int)blockIdx.x < n_long) {   // uniform (all rows, no row list)
        for_long_rows(n_rows, n_long, s_long, &s_nlong,
                      [&](int64_t r) {
                          const int64_t ne = a_rp[r + 1] - a_rp[r];
                          return ne < long_from ? 0 : ne < huge_from ? 1 : huge_here ? 2 : 0;
                      },
                      [&](int64_t row) {
                          const int lane = lane_id();
                          RegMax acc;
                          long long blen = 0;
                          hll_walk<L, 4>(a_rp, a_col, sk, b_rp, row, lane & (L - 1), lane / L, WAVE / L, acc, blen);
                          const Regs16 all = lanes_max(acc.get(), L, WAVE);
                          if (b_rp != nullptr) blen = group_reduce_max(blen, WAVE);
                          hll_finish<M>(all, blen, row, row, lane & (L - 1), lane < L, prod, maxb, b_cols, est, merged);
                      },
                      take);
        return;
    }
    const int64_t gt = ((int64_t)blockIdx.x - n_long) * blockDim.x + threadIdx.x;
    const int64_t t = gt >> g_log2;
    const int sub = (int)(gt & (G - 1));
    if (threadIdx.x == 0) s_nlong = 0;
    __syncthreads();
    const int slice = sub & (L - 1);
    const int part = sub / L;
    const int parts = G / L;
    RegMax acc;
    long long blen_max = 0;
    int64_t row = -1;
    bool mine = false;
    Reach reach;
    int64_t ne = 0;
    if (t < n_rows) {
        row = row_of(t);
        ne = a_rp[row + 1] - a_rp[row];
        mine = ne < long_from;
        if (SAMPLE && ne < sample.whole_from) reach.b_col = sample.b_col;
        if (mine) hll_walk<L, 4, SAMPLE>(a_rp, a_col, sk, b_rp, row, slice, part, parts, acc, blen_max, &reach);
        else if ((SAMPLE || n_long == 0) && sub == 0) s_long[atomicAdd(&s_nlong, 1)] = (int32_t)t;
    }
    const Regs16 all = lanes_max(acc.get(), L, G);
    if (SAMPLE) {
        reach.first = -group_reduce_max(-reach.first, G);
        reach.last = group_reduce_max(reach.last, G);
        if (t < n_rows && sub == 0) {
            sample.prod_out[t] = prod[row];
            sample.span_out[t] = ne >= sample.whole_from ? 0x7fffffff : reach.last < reach.first ? 0 : reach.last - reach.first + 1;
        }
    } else if (b_rp != nullptr) {
        blen_max = group_reduce_max(blen_max, G);
    }
    hll_finish<M>(all, blen_max, t, row, slice, mine && part == 0, prod, maxb, b_cols, est, merged);
    __syncthreads();
    const int nlong = s_nlong;
    for (int i = 0; i < nlong; ++i) take((int64_t)s_long[i]);   // uniform
}

// The rows of huge_from entries and more in a merge over all rows of a large matrix, a workgroup of 1024 threads on one after
// the other: a row of 28 000 entries, four in flight per lane, takes a workgroup of 256 threads 100 us, and a launch is
// 5.  Rows are spread over the workgroups as in for_long_rows.
constexpr int LONG_THREADS = 1024;
template <int M>
__global__ void __launch_bounds__(LONG_THREADS)
k_hll_merge_long(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const uint64_t *__restrict__ sk,
                 int64_t n_rows, int64_t huge_from, const int64_t *__restrict__ prod, const int32_t *__restrict__ maxb,
                 const int64_t *__restrict__ b_rp, int64_t b_cols, double *__restrict__ est, uint64_t *__restrict__ merged)
{
    __shared__ Regs16 s_regs[LONG_THREADS / WAVE][M / 16];
    __shared__ long long s_blen[LONG_THREADS / WAVE];
    __shared__ int32_t s_list[LONG_THREADS];
    __shared__ int s_n;
    for_long_rows<LONG_THREADS>(
        n_rows, (int)gridDim.x, s_list, &s_n, [&](int64_t r) { return a_rp[r + 1] - a_rp[r] >= huge_from ? 2 : 0; }, [](int64_t) {},
        [&](int64_t row) {
            hll_row_by_all<M, LONG_THREADS, 4>(s_regs, s_blen, a_rp, a_col, sk, row, row, prod, maxb, b_rp, b_cols, est, merged);
        });
}

hipError_t launch_hll_merge(const Csr &A, const uint8_t *sketches, int m, const int64_t *rows, int64_t n_rows,
                            const int64_t *prod, const int32_t *maxb, const int64_t *b_rp, int64_t b_cols,
                            double *est, uint8_t *merged, int lanes_div, hipStream_t s)
{
    if (n_rows == 0) return hipSuccess;
    const int L = m / 16;
    const double avg = A.rows ? (double)A.nnz / (double)A.rows : 1.0;
    // All rows of a matrix that is or may be skewed: the long rows go to waves and workgroups of their own, so the others can
    // have a twelfth of the lanes (four entries in flight per lane, and three times the rows).  Workgroups for long rows that find
    // none keep others waiting: one for every 64 rows.  With an eighth, and one for every 16, up to 15 % slower than before rows of
    // one length had such workgroups (20 000 to 50 000 rows of 36 to 130 entries); 306 inputs of 20 000 to 260 000 rows of 10 to 300
    // entries, equal and skewed, in units of that time: 0.79 then, 0.75 now.
    const bool spread = lanes_div == 1 && rows == nullptr;
    int g_log2 = ilog2_ceil(avg * L / (double)(spread ? 12 : lanes_div), 0, 6);   // (lanes_div: see launch_hll_sketch)
    while ((1 << g_log2) < L) ++g_log2;
    const uint64_t *sk = reinterpret_cast<const uint64_t *>(sketches);
    uint64_t *mg = reinterpret_cast<uint64_t *>(merged);
    // (R-MAT scale 18, 64 registers, both launches: long from 8 times the average row on 160 us, from 4 times 150, from twice 155)
    const double times = spread ? 4.0 : 8.0;
    const int64_t least = spread ? MG_SKEWED : MG_LONG;
    const int64_t long_from = times * avg > (double)least ? (int64_t)(times * avg) : least;
    const int64_t huge_from = long_from > MG_WAVE ? long_from : MG_WAVE;
    const bool own_launch = spread && A.nnz >= (1 << 20);
    const int rows_per_block = TPB >> g_log2;
    const auto kernel = m == 32 ? k_hll_merge<32, false> : m == 64 ? k_hll_merge<64, false> : k_hll_merge<128, false>;
    if (m != 32 && m != 64 && m != 128) return hipErrorInvalidValue;
    // (pieces that leave room for the workgroups for long rows: see most_blocks)
    const int64_t most = (most_blocks(TPB) - 1024) * rows_per_block;
    for (int64_t t0 = 0; t0 < n_rows; t0 += most) {
        const int64_t n = n_rows - t0 < most ? n_rows - t0 : most;
        const int n_long = spread && A.nnz >= long_from ? long_row_blocks(n / 4) : 0;
        const int64_t blocks = (n + rows_per_block - 1) / rows_per_block + n_long;
        const int64_t r0 = rows ? 0 : t0;   // (without a list, slot t is row t: the rows' own arrays move along)
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(TPB), 0, s, A.rp + r0, A.col, sk, rows ? rows + t0 : nullptr, n,
                           g_log2, long_from, huge_from, !own_launch, n_long, prod ? prod + r0 : nullptr, maxb ? maxb + r0 : nullptr,
                           b_rp, b_cols, est + t0, mg ? mg + t0 * L * 2 : nullptr, SampleOf{});
    }
    if (own_launch) {
        const int n = long_row_blocks(n_rows);
        const auto huge = m == 32 ? k_hll_merge_long<32> : m == 64 ? k_hll_merge_long<64> : k_hll_merge_long<128>;
        hipLaunchKernelGGL(huge, dim3(n), dim3(LONG_THREADS), 0, s, A.rp, A.col, sk, n_rows, huge_from, prod, maxb, b_rp, b_cols,
                           est, mg);
    }
    return hipGetLastError();
}

// Estimates, products and, with `reach` (B) given, reach of the ns sampled rows, and, with `count` (B) given, the sums of
// count_columns over count_rows(ns) of them: one launch for what the sample looks at.
hipError_t launch_sample(const Csr &A, const Csr *reach, const Csr *count, int64_t b_cols, const uint8_t *sketches, int m, int64_t ns,
                         uint32_t seed, const int64_t *prod, const int32_t *maxb, double *est, int64_t *prod_out, int32_t *span_out,
                         unsigned long long *count_totals, int lanes_div, hipStream_t s)
{
    if (ns <= 0) return hipSuccess;
    const int L = m / 16;
    const double avg = A.rows ? (double)A.nnz / (double)A.rows : 1.0;
    int g_log2 = ilog2_ceil(avg * L / (double)lanes_div, 0, 6);
    while ((1 << g_log2) < L) ++g_log2;
    const int64_t long_from = 8.0 * avg > (double)MG_LONG ? (int64_t)(8.0 * avg) : MG_LONG;
    const int64_t whole_from = ((int64_t)64 << ilog2_ceil(avg / 4.0, 1, 6)) + 1;   // (as k_row_spans)
    const int64_t whole = whole_from < long_from ? whole_from : long_from;
    const auto kernel = m == 32 ? k_hll_merge<32, true> : m == 64 ? k_hll_merge<64, true> : k_hll_merge<128, true>;
    const int64_t *b_rp = reach ? reach->rp : count ? count->rp : nullptr;
    const int rows_per_block = TPB >> g_log2;
    const int64_t most = (most_blocks(TPB) - COUNT_ROWS) * rows_per_block;
    for (int64_t first = 0; first < ns; first += most) {
        const int64_t n = ns - first < most ? ns - first : most;
        const int n_count = first == 0 && count ? count_rows(ns) : 0;
        const SampleOf sample{A.rows, ns, first, seed, whole, reach ? reach->col : nullptr, prod_out + first, span_out + first,
                              count ? count->col : nullptr, count_totals};
        const int64_t blocks = (n + rows_per_block - 1) / rows_per_block + n_count;
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(TPB), 0, s, A.rp, A.col, reinterpret_cast<const uint64_t *>(sketches),
                           nullptr, n, g_log2, long_from, long_from, true, n_count, prod, maxb, b_rp, b_cols, est + first, nullptr, sample);
    }
    return hipGetLastError();
}

// The sums of count_columns over count_rows(ns) of ns sampled rows, without the sample; nothing where flags say that the inputs
// are not valid.
__global__ void __launch_bounds__(TPB)
k_count_columns(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const int64_t *__restrict__ b_rp,
                const int64_t *__restrict__ prod, const int32_t *__restrict__ flags, const SampleOf sample)
{
    __shared__ uint32_t s_bits[1 << (COUNT_LOG2 - 5)];
    __shared__ int s_n;
    if (*flags & 7) return;   // uniform
    const int64_t row = sample.row((int64_t)blockIdx.x * sample.ns / gridDim.x);
    count_columns(s_bits, &s_n, a_rp, a_col, b_rp, sample.count_col, row, prod[row], sample.count_totals);
}

hipError_t launch_count(const Csr &A, const Csr &B, int64_t ns, uint32_t seed, const int64_t *prod, const int32_t *flags,
                        unsigned long long *count_totals, hipStream_t s)
{
    const int n = count_rows(ns);
    if (n <= 0) return hipSuccess;
    const SampleOf sample{A.rows, ns, 0, seed, 0, nullptr, nullptr, nullptr, B.col, count_totals};
    hipLaunchKernelGGL(k_count_columns, dim3((unsigned)n), dim3(TPB), 0, s, A.rp, A.col, B.rp, prod, flags, sample);
    return hipGetLastError();
}

// ------------------------------------------------------------- row spans
// Column range that a row of C can reach: from the first entry of the rows of B it references to their last
// entry (B's rows in column order; where they are not, the range is only a guess, and the kernel that relies
// on it checks every product against it).  Used to choose the dense accumulator for rows whose range fits it
// (Section 3.3, accumulator selection).  One lane group per row as in k_row_products; rows of A with more than
// 64 entries per lane of the group are left with the full range (they are heavy rows, which have a
// dense accumulator of their own).
// ends: first and last column of every row of B in one word of 8 bytes (k_check_sorted writes them in passing), which is a
// gather per entry instead of three.  The rows' ranges are summed up in totals, SPAN_SLOTS slots of SPAN_STRIDE words: rows
// with products, those of them whose range is longer than DS_MAX_COLS, the longest range of the others, the sum of the lesser
// of range and products (which bounds C), and the rows that a dense accumulator over their range pays for, with tables sized
// by the product bound.
__global__ void __launch_bounds__(TPB)
k_row_spans(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const int2 *__restrict__ ends, int64_t n, int g_log2,
            int32_t *__restrict__ cmin, int32_t *__restrict__ cmax, const int64_t *__restrict__ prod, int64_t n_cols, int vbytes,
            double bound_coef, unsigned long long *totals)
{
    __shared__ unsigned long long s_tot[SPAN_TOTALS];
    const int G = 1 << g_log2;
    const int R = TPB >> g_log2;
    const int rl = threadIdx.x >> g_log2;
    const int sub = threadIdx.x & (G - 1);
    if (threadIdx.x < SPAN_TOTALS) s_tot[threadIdx.x] = 0ull;
    __syncthreads();
    unsigned long long with = 0, beyond = 0, longest = 0, most = 0, pay = 0;
    for (int64_t base = (int64_t)blockIdx.x * R; base < n; base += (int64_t)gridDim.x * R) {
        const int64_t row = base + rl;
        int lo = 0x7fffffff, hi = -1;
        bool whole = false;
        if (row < n) {
            const int64_t e0 = a_rp[row], e1 = a_rp[row + 1];
            whole = e1 - e0 > (int64_t)G * 64;
            for (int64_t e = e0 + sub; !whole && e < e1; e += 4 * G) {
                int32_t k[4];
                int2 of[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t idx = e + (int64_t)i * G;
                    k[i] = a_col[idx < e1 ? idx : e];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) of[i] = ends[k[i]];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    lo = of[i].x < lo ? of[i].x : lo;
                    hi = of[i].y > hi ? of[i].y : hi;
                }
            }
        }
        lo = -group_reduce_max(-lo, G);
        hi = group_reduce_max(hi, G);
        if (row < n && sub == 0) {
            cmin[row] = whole ? 0 : lo;
            cmax[row] = whole ? 0x7fffffff : hi;   // (hi < lo: a row without products)
            const long long pr = prod[row];
            if (pr > 0) {
                const unsigned long long span = whole ? 0x80000000ull : (unsigned long long)((long long)hi - lo + 1);
                const double ub = pr < n_cols ? (double)pr : (double)n_cols;
                long long slots = 16;
                while ((double)slots < bound_coef * ub && slots < (1ll << 40)) slots <<= 1;
                ++with;
                beyond += span > (unsigned long long)DS_MAX_COLS;
                longest = span <= (unsigned long long)DS_MAX_COLS && span > longest ? span : longest;
                most += span < (unsigned long long)pr ? span : (unsigned long long)pr;
                pay += dense_span_pays((long long)span, slots, vbytes);
            }
        }
    }
    const unsigned long long mine[SPAN_TOTALS] = {with, beyond, longest, most, pay};
#pragma unroll
    for (int i = 0; i < SPAN_TOTALS; ++i) {
        const unsigned long long wave = i == 2 ? group_reduce_max(mine[i], WAVE) : group_reduce_sum(mine[i], WAVE);
        if (lane_id() == 0 && wave != 0ull) {
            if (i == 2) atomicMax(&s_tot[i], wave);
            else atomicAdd(&s_tot[i], wave);
        }
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < SPAN_TOTALS && s_tot[t] != 0ull) {
        unsigned long long *slot = totals + (size_t)(blockIdx.x % SPAN_SLOTS) * SPAN_STRIDE;
        if (t == 2) atomicMax(&slot[2], s_tot[2]);
        else atomicAdd(&slot[t], s_tot[t]);
    }
}

hipError_t launch_row_spans(const Csr &A, const Csr &B, const int64_t *ends, const int64_t *prod, int vbytes, double bound_coef,
                            int32_t *cmin, int32_t *cmax, unsigned long long *totals, hipStream_t s)
{
    if (A.rows <= 0) return hipSuccess;
    const double avg = (double)A.nnz / (double)A.rows;
    const int g_log2 = ilog2_ceil(avg / 4.0, 1, 6);
    const int R = TPB >> g_log2;
    int64_t blocks = (A.rows + R - 1) / R;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_row_spans, dim3((unsigned)blocks), dim3(TPB), 0, s, A.rp, A.col, reinterpret_cast<const int2 *>(ends), A.rows,
                       g_log2, cmin, cmax, prod, B.cols, vbytes, bound_coef, totals);
    return hipGetLastError();
}

// flags |= 8 when some row of B is not in ascending column order (then the ranges of k_row_spans are guesses).  Eight
// lanes per row.  ends: receives every row's first and last column (the largest number and -1 for an empty row).
__global__ void __launch_bounds__(TPB)
k_check_sorted(const int64_t *__restrict__ rp, const int32_t *__restrict__ col, int64_t rows, int32_t *flags, int2 *__restrict__ ends)
{
    constexpr int G = 8;
    const int sub = threadIdx.x & (G - 1);
    bool bad = false;
    for (int64_t r = ((int64_t)blockIdx.x * TPB + threadIdx.x) / G; r < rows; r += (int64_t)gridDim.x * (TPB / G)) {
        const int64_t first = rp[r], last = rp[r + 1] - 1;
        if (sub == 0) ends[r] = first <= last ? make_int2(col[first], col[last]) : make_int2(0x7fffffff, -1);
        for (int64_t p = first + sub; p < last; p += 4 * G) {
            int32_t a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t q = p + i * G < last ? p + i * G : p;   // (p < last)
                a[i] = col[q];
                b[i] = col[q + 1];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) bad |= a[i] > b[i];
        }
    }
    if (__ballot(bad) != 0 && lane_id() == 0) atomicOr(flags, 8);
}

hipError_t launch_check_sorted(const Csr &B, int32_t *flags, int64_t *ends, hipStream_t s)
{
    if (B.rows == 0) return hipSuccess;
    int64_t blocks = (B.rows * 8 + TPB - 1) / TPB;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_check_sorted, dim3((unsigned)blocks), dim3(TPB), 0, s, B.rp, B.col, B.rows, flags, reinterpret_cast<int2 *>(ends));
    return hipGetLastError();
}

// --------------------------------------------------------- sample reduce
// Sums over the sampled rows in a fixed order (one workgroup, strided partial sums, butterflies over lanes, then the waves in
// turn), so the sampled CR is the same on every run.
// out[0] = sum of products, out[1] = sum of estimates (their ratio is the sampled CR, Section 3.2);
// out[2], out[3] = sum and sum of squares of the per-row ratios products / estimate, out[4] = rows counted
// (mean and standard deviation of the compression ratio over the sample, Section 4.1); out[5] = sampled rows
// whose column range is narrow enough for the dense accumulator to pay.
constexpr int SR_THREADS = 1024;
constexpr int SR_SUMS = 6;
__global__ void __launch_bounds__(SR_THREADS)
k_sample_reduce(int64_t n_rows, const int64_t *__restrict__ prod, const double *__restrict__ est, const int32_t *__restrict__ span,
                int64_t n_cols, int vbytes, double bound_coef, double *out)
{
    __shared__ double s_acc[SR_THREADS / WAVE][SR_SUMS];
    double acc[SR_SUMS] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    // four sampled rows per thread and turn, their loads issued together
    for (int64_t t0 = threadIdx.x; t0 < n_rows; t0 += 4 * SR_THREADS) {
        double e[4], p[4];
        int32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t t = t0 + (int64_t)i * SR_THREADS;
            const int64_t q = t < n_rows ? t : t0;
            e[i] = t < n_rows ? est[q] : 0.0;
            p[i] = (double)prod[q];
            w[i] = span[q];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (e[i] > 0.0) {
                const double q = p[i] / e[i];
                acc[0] += p[i]; acc[1] += e[i]; acc[2] += q; acc[3] += q * q; acc[4] += 1.0;
                const double ub = p[i] < (double)n_cols ? p[i] : (double)n_cols;
                long long slots = 16;
                while ((double)slots < bound_coef * ub && slots < (1ll << 40)) slots <<= 1;   // table from the bound
                if (dense_span_pays((long long)w[i], slots, vbytes)) acc[5] += 1.0;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < SR_SUMS; ++k) {
        const double wave = group_reduce_sum(acc[k], WAVE);
        if (lane_id() == 0) s_acc[threadIdx.x / WAVE][k] = wave;
    }
    __syncthreads();
    if (threadIdx.x < SR_SUMS) {
        double sum = 0.0;
        for (int w = 0; w < SR_THREADS / WAVE; ++w) sum += s_acc[w][threadIdx.x];
        out[threadIdx.x] = sum;
    }
}

hipError_t launch_sample_reduce(int64_t n_rows, const int64_t *prod, const double *est, const int32_t *span, int64_t n_cols, int vbytes,
                                double bound_coef, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sample_reduce, dim3(1), dim3(SR_THREADS), 0, s, n_rows, prod, est, span, n_cols, vbytes, bound_coef, out);
    return hipGetLastError();
}

}  // namespace ocean
