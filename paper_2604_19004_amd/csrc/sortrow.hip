// The numeric kernel of rows with few products, from lists of row ids: see sortrow.hpp.
#include "sortrow.hpp"

namespace ocean {

// rows: row ids, each with at most CAP products and ENT entries; column ids below 2^(32 - log2 CAP) - 1, B's arrays
// below 2^32 entries (positions are kept in 32 bits).  The rest as in the hash kernels.
// THREADS: 256, or 64 where a row takes so much LDS that whole workgroups of four would leave some of it unused.
// Values are added up in LDS, in places of 8 bytes, and heads are lane masks of their own: rows placed in C (placed.hip) cannot
// afford the places, rows from lists can, and where many products merge this is faster (clustered rows of 762 products, fp32:
// classes of 768 and 1024 products 609 and 759 us, by sortrow.hpp's steps 684 and 797).
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

// The same for rows of more than 1024 products, by the steps of sortrow.hpp: sums in registers, places of the value's own size.
// 100 000 rows of 1444 and of 2025 products, fp32: 575 and 815 us, by the kernel above 653 and 1085.
template <typename V, int G, int PPT, int ENT, int THREADS>
__global__ void __launch_bounds__(THREADS)
k_numeric_sort_long(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
               const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
               const int32_t *__restrict__ rows, int64_t count, const int64_t *__restrict__ out_ptr,
               int32_t *__restrict__ out_col, V *__restrict__ out_val, int32_t *__restrict__ row_nnz)
{
    constexpr int R = THREADS / G;
    __shared__ SortRow<V, G, PPT, ENT> s_row[R];
    const int lane = lane_id();
    const int sub = lane & (G - 1);
    const int rl = G == WAVE ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE) : (int)threadIdx.x / G;
    SortRow<V, G, PPT, ENT> &sr = s_row[rl];

    const int64_t r = (int64_t)blockIdx.x * R + rl;
    const bool live = r < count;
    if (G == WAVE && !live) return;   // (a whole wave; there is no workgroup barrier)
    const int64_t row = live ? rows[r] : 0;
    const int64_t e0 = live ? a_rp[row] : 0;
    const int ne = live ? (int)(a_rp[row + 1] - e0) : 0;
    SortedRow<V, G, PPT, ENT> row_c;
    row_c.sort(sr, lane, sub, e0, ne, a_col, a_val, b_rp, b_col, b_val);
    row_c.accumulate(sr.acc, sub);
    const int64_t o = live ? out_ptr[row] : 0;
    const int64_t cap = live ? out_ptr[row + 1] - o : 0;
    const bool fits = (int64_t)row_c.n_out <= cap;   // (a row that does not fit writes nothing)
    row_c.write(sr.acc, sub, o, fits ? (int)row_c.n_out : 0, out_col, out_val);
    if (live && sub == 0) row_nnz[row] = fits ? (int32_t)row_c.n_out : -1;
}

template <typename V>
static hipError_t dispatch_sort(const Csr &A, const Csr &B, const SortLaunch &l, hipStream_t s)
{
    const V *av = static_cast<const V *>(A.val);
    const V *bv = static_cast<const V *>(B.val);
    V *ov = static_cast<V *>(l.out_val);
#define OCEAN_SORT(KERNEL, CLS, G, PPT, THREADS)                                                                      \
    case CLS:                                                                                                        \
        static_assert(kSortClass[CLS].cap == G * PPT, "products of the class");                                       \
        launch_in_pieces(l.count, THREADS / G, THREADS, [&](int64_t first, int64_t n) {                               \
            hipLaunchKernelGGL((KERNEL<V, G, PPT, kSortClass[CLS].entries, THREADS>),                                  \
                               dim3((unsigned)((n + THREADS / G - 1) / (THREADS / G))), dim3(THREADS), 0, s, A.rp,      \
                               A.col, av, B.rp, B.col, bv, l.rows + first, n, l.out_ptr, l.out_col, ov, l.row_nnz);     \
        });                                                                                                          \
        break
    switch (l.cls) {
        OCEAN_SORT(k_numeric_sort, 1, 8, 4, 256);
        OCEAN_SORT(k_numeric_sort, 2, 16, 4, 256);
        OCEAN_SORT(k_numeric_sort, 3, 16, 6, 256);
        OCEAN_SORT(k_numeric_sort, 4, 16, 8, 256);
        OCEAN_SORT(k_numeric_sort, 5, 32, 6, 256);
        OCEAN_SORT(k_numeric_sort, 6, 32, 8, 256);
        OCEAN_SORT(k_numeric_sort, 7, 64, 6, 256);
        OCEAN_SORT(k_numeric_sort, 8, 64, 8, 256);
        OCEAN_SORT(k_numeric_sort, 9, 64, 12, 64);
        OCEAN_SORT(k_numeric_sort, 10, 64, 16, 64);
        OCEAN_SORT(k_numeric_sort_long, 11, 64, 24, 64);
        OCEAN_SORT(k_numeric_sort_long, 12, 64, 32, 64);
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
