// The numeric kernel of rows with few products, from lists of row ids: see sortrow.hpp.
#include "sortrow.hpp"

namespace ocean {

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
    row_c.accumulate(sr, sub);
    const int64_t o = live ? out_ptr[row] : 0;
    const int64_t cap = live ? out_ptr[row + 1] - o : 0;
    const bool fits = (int64_t)row_c.n_out <= cap;   // (a row that does not fit writes nothing)
    row_c.write(sr, sub, o, fits ? (int)row_c.n_out : 0, out_col, out_val);
    if (live && sub == 0) row_nnz[row] = fits ? (int32_t)row_c.n_out : -1;
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
