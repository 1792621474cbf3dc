// Short rows by expand-sort-compress with several products per lane (paper Section 2.2, "ESC"; Section 4.2 for the
// packed keys): the numeric kernel of rows with at most 2048 intermediate products.
//
// G consecutive lanes of a wave own one row and hold PPT products each (G * PPT = CAP products at most), 64 / G
// rows per wave.  No hash table, no probing and no workgroup barrier:
//   expand    the row's entries are read G at a time, their rows of B laid end to end; every product finds its entry
//             by the number of segment starts at or before it (a bitmap and a population count); the column id and
//             the product's number share one 32-bit key, the value a * b waits in LDS at that number;
//   sort      a bitonic network over the CAP keys.  Lane l holds elements l * PPT .. l * PPT + PPT - 1, so steps
//             over less than PPT elements are a minimum and a maximum inside the lane, and the others one lane move
//             (a DPP modifier where there is one) and a median-of-three against 0 or ~0 that keeps the smaller or
//             the larger key.  Every merge starts with a mirrored step, so all comparisons go the same way;
//   compress  a key whose column differs from its predecessor's opens an entry of C; a prefix sum numbers them, the
//             openers store their value at the entry's place in LDS, the others add theirs, and the row leaves with
//             coalesced stores, in column order.
// What bounds it is vector issue: 880 vector instructions per row of the 512-product class, of which the sort is 530, are
// 489 us for 341 000 rows (of the rectangular input, before there was a class of 384) at one per four cycles and SIMD,
// 541 us measured.  The work
// does not depend on where the columns lie or how many products merge.  Sizes of 3 * 2^i products cost a third less
// per row than the next power of two (see settle).  Against the hash kernels (one MI355X, fp64 unless said): numeric
// stage of the rectangular input (264 products a row) 1.50 -> 0.94 ms, clustered fp32 (762 products, 234 columns) 2.55 ->
// 1.50 ms, 100 003 uniform rows of 1023 products fp32 1.29 -> 0.40 ms, Laplacian (25 products) 0.22 -> 0.19 ms.
#include <type_traits>

#include "ocean_internal.hpp"

namespace ocean {

namespace {

constexpr uint32_t SR_PAD = 0xffffffffu;   // key of a slot without a product: sorts last

// Value of the lane `MASK` away (lane index xor MASK).
template <int MASK>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane)
{
    const int x = (int)v;
    if constexpr (MASK == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true);    // quad_perm [1,0,3,2]
    else if constexpr (MASK == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
    else if constexpr (MASK == 3) return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x1B, 0xf, 0xf, true);   // quad_perm [3,2,1,0]
    else if constexpr (MASK == 7) return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true);  // row_half_mirror
    else if constexpr (MASK == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true);  // row_ror:8
    else if constexpr (MASK == 15) return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, true); // row_mirror
    else if constexpr (MASK == 63) return (uint32_t)__builtin_amdgcn_ds_bpermute((WAVE - 1 - lane) << 2, x);
    else return (uint32_t)__builtin_amdgcn_ds_swizzle(x, (MASK << 10) | 0x1f);   // 4, 16, 31: inside 32 lanes
}

// bound = 0 keeps the smaller, bound = ~0 the larger of two keys (v_med3_u32)
__device__ __forceinline__ uint32_t keep(uint32_t a, uint32_t b, uint32_t bound)
{
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    const uint32_t x = hi < bound ? hi : bound;
    return lo < x ? x : lo;
}

template <int PPT>
__device__ __forceinline__ void exchange(uint32_t (&k)[PPT], int i, int j)
{
    const uint32_t a = k[i], b = k[j];
    k[i] = a < b ? a : b;
    k[j] = a < b ? b : a;
}

// One step between lanes: element (lane, u) with element (lane ^ MASK, MIRROR ? PPT - 1 - u : u).
template <int MASK, bool MIRROR, int PPT>
__device__ __forceinline__ void lane_step(uint32_t (&k)[PPT], int lane)
{
    constexpr int TOP = MASK >= 32 ? 32 : MASK >= 16 ? 16 : MASK >= 8 ? 8 : MASK >= 4 ? 4 : MASK >= 2 ? 2 : 1;
    const uint32_t bound = (lane & TOP) ? 0xffffffffu : 0u;
    uint32_t t[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) t[u] = lane_xor<MASK>(k[MIRROR ? PPT - 1 - u : u], lane);
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        k[u] = keep(k[u], t[u], bound);
        // (nothing at run time: ends the chain of minima and maxima here, which the compiler otherwise follows through
        // the whole network, in a time that doubles with every step)
        asm("" : "+v"(k[u]));
    }
}

// The N keys from OFF on, which rise and then fall (or the reverse), into order: halves compared element by element, then
// each half on its own.  Three keys are one minimum, median and maximum, which makes N = 3 * 2^i the cheaper sizes.
template <int N, int OFF, int PPT>
__device__ __forceinline__ void settle(uint32_t (&k)[PPT])
{
    if constexpr (N == 3) {
        const uint32_t a = k[OFF], b = k[OFF + 1], c = k[OFF + 2];
        const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
        const uint32_t x = hi < c ? hi : c;
        k[OFF] = lo < c ? lo : c;          // v_min3_u32
        k[OFF + 1] = lo < x ? x : lo;      // v_med3_u32
        k[OFF + 2] = hi < c ? c : hi;      // v_max3_u32
    } else if constexpr (N > 1) {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) exchange(k, OFF + i, OFF + N / 2 + i);
        settle<N / 2, OFF>(k);
        settle<N / 2, OFF + N / 2>(k);
    }
}

// The N keys from OFF on, in any order, into order.
template <int N, int OFF, int PPT>
__device__ __forceinline__ void sort_inside(uint32_t (&k)[PPT])
{
    if constexpr (N == 3) {
        settle<3, OFF>(k);
    } else if constexpr (N > 1) {
        sort_inside<N / 2, OFF>(k);
        sort_inside<N / 2, OFF + N / 2>(k);
#pragma unroll
        for (int i = 0; i < N / 2; ++i) exchange(k, OFF + i, OFF + N - 1 - i);
        settle<N / 2, OFF>(k);
        settle<N / 2, OFF + N / 2>(k);
    }
}

// Ascending order over the G * PPT keys of every group of G lanes; element (lane, u) is number lane * PPT + u.
template <int G, int PPT>
__device__ __forceinline__ void sort_keys(uint32_t (&k)[PPT], int lane)
{
    sort_inside<PPT, 0>(k);
    if constexpr (G >= 2) { lane_step<1, true>(k, lane); settle<PPT, 0>(k); }
    if constexpr (G >= 4) { lane_step<3, true>(k, lane); lane_step<1, false>(k, lane); settle<PPT, 0>(k); }
    if constexpr (G >= 8) {
        lane_step<7, true>(k, lane); lane_step<2, false>(k, lane); lane_step<1, false>(k, lane); settle<PPT, 0>(k);
    }
    if constexpr (G >= 16) {
        lane_step<15, true>(k, lane); lane_step<4, false>(k, lane); lane_step<2, false>(k, lane); lane_step<1, false>(k, lane);
        settle<PPT, 0>(k);
    }
    if constexpr (G >= 32) {
        lane_step<31, true>(k, lane); lane_step<8, false>(k, lane); lane_step<4, false>(k, lane); lane_step<2, false>(k, lane);
        lane_step<1, false>(k, lane); settle<PPT, 0>(k);
    }
    if constexpr (G >= 64) {
        lane_step<63, true>(k, lane); lane_step<16, false>(k, lane); lane_step<8, false>(k, lane); lane_step<4, false>(k, lane);
        lane_step<2, false>(k, lane); lane_step<1, false>(k, lane); settle<PPT, 0>(k);
    }
}

// Inclusive prefix sum and total over every group of G lanes.
template <int G>
__device__ __forceinline__ uint32_t group_scan(uint32_t v, int sub, uint32_t &total)
{
    if constexpr (G == 64) {
        const uint32_t inc = wave_inclusive_scan_u32(v);
        total = wave_read_lane_u32(inc, WAVE - 1);
        return inc;
    } else if constexpr (G == 32) {
        uint32_t inc = group_inclusive_scan_u32<16>(v, sub & 15);
        inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, 0x142, 0xa, 0xf, false);   // lane 15 of the row before, into rows 1 and 3
        total = (uint32_t)__shfl((int)inc, (lane_id() & ~31) + 31, WAVE);
        return inc;
    } else {
        total = group_sum_u32<G>(v);
        return group_inclusive_scan_u32<G>(v, sub);
    }
}

constexpr int log2_of(int x) { return x <= 1 ? 0 : 1 + log2_of((x + 1) >> 1); }   // rounded up

}  // namespace

// rows: row ids, each with at most CAP products and ENT entries; column ids below 2^(32 - log2 CAP) - 1, B's arrays
// below 2^32 entries (positions are kept in 32 bits).  The rest as in the hash kernels.
// THREADS: 256, or 64 where a row takes so much LDS that whole workgroups of four would leave some of it unused.
template <typename V, int G, int PPT, int ENT, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_numeric_sort(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
               const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
               const int32_t *__restrict__ rows, int64_t count, const int64_t *__restrict__ out_ptr,
               int32_t *__restrict__ out_col, V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    constexpr int CAP = G * PPT;
    constexpr int LB = log2_of(CAP);
    constexpr int R = THREADS / G;
    constexpr int MW = (CAP + 63) / 64;   // 64-bit words of segment starts
    constexpr int BATCH = PPT % 4 == 0 ? 4 : 3;
    static_assert(PPT % BATCH == 0 && 64 % G == 0, "whole batches");
    // places of the sorted row are spread by one slot in eight or sixteen, so that the lanes' stores, PPT apart, meet
    // different banks
    constexpr int SPREAD = PPT >= 12 ? 4 : 3;
    constexpr int PLACES = CAP + (CAP >> SPREAD);
    auto place = [](int r) { return r + (r >> SPREAD); };
    struct Row {
        // the products' values by number (type V), then the values of the row of C by rank, then its columns: what LDS
        // a row takes decides how many rows a compute unit works on (1024 products: with a place of their own for the
        // columns 2 waves per SIMD and 506 us for 100 003 rows, one place for all three 4 waves and 380 us)
        double acc[PLACES];
        uint32_t pos[ENT];     // position in B of an entry's first product, minus that product's number
        V a[ENT];
        unsigned long long start[MW];
    };
    __shared__ Row s_row[R];
    const int lane = lane_id();
    const int sub = lane & (G - 1);
    const int rl = G == WAVE ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE) : (int)threadIdx.x / G;
    const int shift = lane & ~(G - 1);
    constexpr unsigned long long GMASK = G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull;
    Row &sr = s_row[rl];
    V *s_val = reinterpret_cast<V *>(sr.acc);

    const int64_t r = (int64_t)blockIdx.x * R + rl;
    const bool live = r < count;
    if (G == WAVE && !live) return;   // (a whole wave; there is no workgroup barrier)
    const int64_t row = live ? rows[r] : 0;
    const int64_t e0 = live ? a_rp[row] : 0;
    int ne = live ? (int)(a_rp[row + 1] - e0) : 0;
    ne = ne < ENT ? ne : ENT;   // (holds: the caller lists no other rows)

    // ---- expand
    for (int w = sub; w < MW; w += G) sr.start[w] = 0ull;
    wave_sync();
    uint32_t total = 0;
    int nseg = 0;
    const int chunks = G >= ENT ? 1 : (int)wave_max_u32((uint32_t)((ne + G - 1) / G));   // the rows of a wave advance together
    for (int ch = 0; ch < chunks; ++ch) {
        const int e = ch * G + sub;
        int64_t p0 = 0;
        uint32_t len = 0;
        V a = V();
        if (e < ne) {
            const int64_t k = a_col[e0 + e];
            a = a_val[e0 + e];
            p0 = b_rp[k];
            len = (uint32_t)(b_rp[k + 1] - p0);
        }
        uint32_t sum;
        const uint32_t first = total + group_scan<G>(len, sub, sum) - len;
        const unsigned long long some = (__ballot(len > 0) >> shift) & GMASK;
        if (len > 0 && first < (uint32_t)CAP) {   // (the second holds: at most CAP products)
            const int at = nseg + __popcll(some & ((1ull << sub) - 1ull));
            sr.pos[at] = (uint32_t)p0 - first;
            sr.a[at] = a;
            atomicOr(reinterpret_cast<uint32_t *>(sr.start) + (first >> 5), 1u << (first & 31u));
        }
        total += sum;
        nseg += __popcll(some);
    }
    total = total < (uint32_t)CAP ? total : (uint32_t)CAP;
    wave_sync();

    uint32_t key[PPT];
    {
        int run = 0;   // segments that start in the words before
#pragma unroll
        for (int u0 = 0; u0 < PPT; u0 += BATCH) {
            uint32_t p[BATCH];
            V a[BATCH];
            V b[BATCH];
            int32_t c[BATCH];
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int u = u0 + i;
                const unsigned long long m = sr.start[u * G / 64];
                const uint32_t q = (uint32_t)(u * G + sub);
                const int seg = run + __popcll(m & ((2ull << (u * G % 64 + sub)) - 1ull)) - 1;
                if ((u + 1) * G % 64 == 0) run += __popcll(m);
                const int s = q < total ? seg : 0;
                p[i] = sr.pos[s] + q;
                a[i] = sr.a[s];
            }
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const uint32_t q = (uint32_t)((u0 + i) * G + sub);
                c[i] = 0;
                b[i] = V();
                if (q < total) { c[i] = b_col[p[i]]; b[i] = b_val[p[i]]; }
            }
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const uint32_t q = (uint32_t)((u0 + i) * G + sub);
                key[u0 + i] = q < total ? ((uint32_t)c[i] << LB) | q : SR_PAD;
                s_val[q] = a[i] * b[i];
            }
        }
    }

    // ---- sort
    sort_keys<G, PPT>(key, lane);

    // ---- compress
    const uint32_t before = (uint32_t)__shfl_up((int)key[PPT - 1], 1, WAVE);   // last key of the lane below
    bool head[PPT];
    uint32_t heads = 0;
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const uint32_t prev = u == 0 ? before : key[u - 1];
        head[u] = key[u] != SR_PAD && ((u == 0 && sub == 0) || ((prev ^ key[u]) >> LB) != 0u);
        heads += head[u];
    }
    uint32_t n_out;
    int rank = (int)(group_scan<G>(heads, sub, n_out) - heads) - 1;
    wave_sync();
    V val[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const uint32_t q = key[u] & ((1u << LB) - 1u);
        val[u] = s_val[CAP == 1 << LB || q < (uint32_t)CAP ? q : 0u];   // (a pad's number is the largest there is)
    }
    wave_sync();
    int at[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        rank += head[u];
        at[u] = place(rank < 0 ? 0 : rank);
        if (head[u]) sr.acc[at[u]] = (double)val[u];
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < PPT; ++u)
        if (!head[u] && key[u] != SR_PAD)
            __hip_atomic_fetch_add(&sr.acc[at[u]], (double)val[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    wave_sync();
    const int64_t o = live ? out_ptr[row] : 0;
    const int64_t cap = live ? out_ptr[row + 1] - o : 0;
    const int n_write = (int64_t)n_out <= cap ? (int)n_out : 0;   // (a row that does not fit writes nothing)
    for (int i = sub; i < n_write; i += G) out_val[o + i] = (V)sr.acc[place(i)];
    wave_sync();
    int32_t *s_col = reinterpret_cast<int32_t *>(sr.acc);
#pragma unroll
    for (int u = 0; u < PPT; ++u)
        if (head[u]) s_col[at[u]] = (int32_t)(key[u] >> LB);
    wave_sync();
    for (int i = sub; i < n_write; i += G) out_col[o + i] = s_col[place(i)];
    if (live && sub == 0) row_nnz[row] = (int64_t)n_out <= cap ? (int32_t)n_out : -1;
}

template <typename V>
static hipError_t dispatch_sort(const Csr &A, const Csr &B, const SortLaunch &l, hipStream_t s)
{
    const V *av = static_cast<const V *>(A.val);
    const V *bv = static_cast<const V *>(B.val);
    V *ov = static_cast<V *>(l.out_val);
#define OCEAN_SORT(CLS, G, PPT, THREADS)                                                                              \
    case CLS:                                                                                                        \
        static_assert(kSortClass[CLS].cap == G * PPT, "products of the class");                                       \
        launch_in_pieces(l.count, THREADS / G, THREADS, [&](int64_t first, int64_t n) {                               \
            hipLaunchKernelGGL((k_numeric_sort<V, G, PPT, kSortClass[CLS].entries, THREADS>),                         \
                               dim3((unsigned)((n + THREADS / G - 1) / (THREADS / G))), dim3(THREADS), 0, s, A.rp,      \
                               A.col, av, B.rp, B.col, bv, l.rows + first, n, l.out_ptr, l.out_col, ov, l.row_nnz);     \
        });                                                                                                          \
        break
    switch (l.cls) {
        OCEAN_SORT(1, 8, 4, 256);
        OCEAN_SORT(2, 16, 4, 256);
        OCEAN_SORT(3, 16, 6, 256);
        OCEAN_SORT(4, 16, 8, 256);
        OCEAN_SORT(5, 32, 6, 256);
        OCEAN_SORT(6, 32, 8, 256);
        OCEAN_SORT(7, 64, 6, 256);
        OCEAN_SORT(8, 64, 8, 256);
        OCEAN_SORT(9, 64, 12, 64);
        OCEAN_SORT(10, 64, 16, 64);
        OCEAN_SORT(11, 64, 24, 64);
        OCEAN_SORT(12, 64, 32, 64);
    default: return hipErrorInvalidValue;
    }
#undef OCEAN_SORT
    return hipGetLastError();
}

hipError_t launch_numeric_sort(const Csr &A, const Csr &B, int dtype, const SortLaunch &l, hipStream_t s)
{
    if (l.count <= 0) return hipSuccess;
    return dtype == OCEAN_F64 ? dispatch_sort<double>(A, B, l, s) : dispatch_sort<float>(A, B, l, s);
}

}  // namespace ocean
