// Rows that are accumulated by sorting (sortrow.hpp) and written straight to their place in C (placed.hpp).
#include "placed.hpp"
#include "sortrow.hpp"

namespace ocean {

// Rows of one class below a wave: 256 / G rows per workgroup, the unit.
template <typename V, int G, int PPT, int ENT>
__global__ void __launch_bounds__(256)
k_placed_group(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
               const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val, Placing<V> p)
{
    constexpr int R = 256 / G;
    static_assert(R <= WAVE, "a lane per row in the prefix sum");
    __shared__ SortRow<V, G, PPT, ENT> s_row[R];
    __shared__ uint32_t s_n[R], s_before[R];
    __shared__ long long s_place;
    const int lane = lane_id();
    const int sub = lane & (G - 1);
    const int rl = (int)threadIdx.x / G;
    const bool first_wave = threadIdx.x < WAVE;
    const int64_t units = (p.m + R - 1) / R;
    if (blockIdx.x == 0) {   // uniform
        place_units(p.counts, p.places, units, p.total, p.flags, p.placer_polls, *reinterpret_cast<Turn *>(s_row));
        return;
    }
    const int64_t unit = (int64_t)blockIdx.x - 1;
    const int64_t row = unit * R + rl;
    const bool live = row < p.m;
    const int64_t e0 = live ? a_rp[row] : 0;
    const int ne = live ? (int)(a_rp[row + 1] - e0) : 0;
    SortRow<V, G, PPT, ENT> &sr = s_row[rl];
    SortedRow<V, G, PPT, ENT> c;
    c.template sort<true>(sr, lane, sub, e0, ne, a_col, a_val, b_rp, b_col, b_val);
    if (sub == 0) s_n[rl] = c.n_out;
    __syncthreads();
    if (first_wave) {
        const uint32_t v = lane < R ? s_n[lane] : 0u;
        const uint32_t inc = wave_inclusive_scan_u32(v);
        if (lane < R) s_before[lane] = inc - v;
        if (lane == WAVE - 1) post(p.counts + unit, inc + 1u);
    }
    c.template accumulate<true>(sr, sub);
    if (first_wave) {
        const int64_t o = wait_for_place(p.places + unit, p.flags, p.unit_polls);
        if (lane == 0) s_place = o;
    }
    __syncthreads();
    if (s_place < 0) return;   // uniform
    const int64_t o = s_place + s_before[rl];
    if (live && sub == 0) {
        p.c_rp[row] = o;
        if (row == p.m - 1) p.c_rp[p.m] = o + c.n_out;
    }
    c.write(sr, sub, o, live && o + c.n_out <= p.slots ? (int)c.n_out : 0, p.out_col, p.out_val);
}

// What the four waves of a workgroup tell each other: no barrier, so that a wave can be anywhere in its own size of sort.
struct FourRows {
    unsigned int arrived;
    uint32_t n[4];                // entries + 1, 0: not known yet
    unsigned long long place;     // of the unit + 1, 0: not known yet
};

__device__ __forceinline__ void publish_row(FourRows &f, int wave, uint32_t n_out, uint32_t *count)
{
    if (lane_id() == 0) {
        __hip_atomic_store(&f.n[wave], n_out + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (__hip_atomic_fetch_add(&f.arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) == 3u) {
            uint32_t sum = 0;
            for (int w = 0; w < 4; ++w) sum += __hip_atomic_load(&f.n[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - 1u;
            post(count, sum + 1u);
        }
    }
    wave_sync();
}

// Where a wave's row goes, or -1.  The first wave asks for the unit's place, the others wait for it (and for the rows before
// theirs) in the LDS.
template <typename V>
__device__ __forceinline__ int64_t place_row(FourRows &f, int wave, int64_t unit, const Placing<V> &p)
{
    if (wave == 0) {
        const int64_t o = wait_for_place(p.places + unit, p.flags, p.unit_polls);
        if (lane_id() == 0)
            __hip_atomic_store(&f.place, o < 0 ? NO_PLACE : (unsigned long long)o + 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return o;
    }
    unsigned long long place;
    while ((place = __hip_atomic_load(&f.place, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0ull) __builtin_amdgcn_s_sleep(4);
    if (place == NO_PLACE) return -1;
    int64_t o = (int64_t)place - 1;
    for (int w = 0; w < wave; ++w) {
        uint32_t n;
        while ((n = __hip_atomic_load(&f.n[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0u) __builtin_amdgcn_s_sleep(1);
        o += n - 1u;
    }
    return o;
}

// sorted(c, sr, lane) for a row of pr products by a whole wave, c and sr of the row's own size.
template <typename V, int MAX, typename Sorted>
__device__ __forceinline__ void sort_by_size(char *lds, int64_t row, int pr, const int64_t *__restrict__ a_rp,
                                             const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                                             const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col,
                                             const V *__restrict__ b_val, Sorted sorted)
{
    const int lane = lane_id();
    const int64_t e0 = a_rp[row];
    const int ne = (int)(a_rp[row + 1] - e0);
#define OCEAN_PLACED(PPT)                                                                                        \
    if constexpr (PPT <= MAX)                                                                                    \
        if (pr <= 64 * PPT) {                                                                                    \
            SortRow<V, WAVE, PPT, 64> &sr = *reinterpret_cast<SortRow<V, WAVE, PPT, 64> *>(lds);                 \
            SortedRow<V, WAVE, PPT, 64> c;                                                                       \
            c.template sort<true>(sr, lane, lane, e0, ne, a_col, a_val, b_rp, b_col, b_val);                                    \
            sorted(c, sr, lane);                                                                                 \
            return;                                                                                              \
        }
    OCEAN_PLACED(2)
    OCEAN_PLACED(3)
    OCEAN_PLACED(4)
    OCEAN_PLACED(6)
    OCEAN_PLACED(8)
    OCEAN_PLACED(12)
    OCEAN_PLACED(16)
    OCEAN_PLACED(24)
    OCEAN_PLACED(32)
#undef OCEAN_PLACED
}

// Rows of at most 64 * MAX products, four neighbouring ones per workgroup and unit, a wave each; the sort's size is the row's
// own, and so is what it takes of the workgroup's LDS, which holds the four rows that need most.
template <typename V, int MAX>
__global__ void __launch_bounds__(256, MAX <= 8 ? 8 : MAX <= 16 ? 7 : MAX <= 24 ? 5 : 4)
k_placed_wave(const int64_t *__restrict__ a_rp, const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
              const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col, const V *__restrict__ b_val,
              const int64_t *__restrict__ prod, Placing<V> p)
{
    extern __shared__ __align__(16) char s_pool[];
    __shared__ FourRows s_four;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    if (blockIdx.x == 0) {   // uniform
        place_units(p.counts, p.places, (p.m + 3) / 4, p.total, p.flags, p.placer_polls, *reinterpret_cast<Turn *>(s_pool));
        return;
    }
    const int64_t unit = (int64_t)blockIdx.x - 1, row = unit * 4 + wave;
    if (threadIdx.x == 0) {
        s_four.arrived = 0u;
        s_four.place = 0ull;
    }
    if (threadIdx.x < 4) s_four.n[threadIdx.x] = 0u;
    int before = 0;   // LDS of the rows before this wave's
    for (int64_t r = unit * 4; r < row; ++r) before += sort_row_bytes(r < p.m ? (int)prod[r] : 0, sizeof(V));
    const int pr = row < p.m ? (int)prod[row] : 0;
    __syncthreads();
    if (row >= p.m) {
        publish_row(s_four, wave, 0u, p.counts + unit);
        return;
    }
    sort_by_size<V, MAX>(s_pool + before, row, pr, a_rp, a_col, a_val, b_rp, b_col, b_val, [&](auto &c, auto &sr, int lane) {
        publish_row(s_four, wave, c.n_out, p.counts + unit);
        c.template accumulate<true>(sr, lane);
        const int64_t o = place_row(s_four, wave, unit, p);
        if (o < 0) return;
        if (lane == 0) {
            p.c_rp[row] = o;
            if (row == p.m - 1) p.c_rp[p.m] = o + c.n_out;
        }
        c.write(sr, lane, o, o + c.n_out <= p.slots ? (int)c.n_out : 0, p.out_col, p.out_val);
    });
}

// The first n entries of one pair of arrays into another.
template <typename V>
__global__ void __launch_bounds__(256)
k_trim(const int32_t *__restrict__ col, const V *__restrict__ val, int64_t n, int32_t *__restrict__ c_col, V *__restrict__ c_val)
{
    struct alignas(16) Four { int32_t c[4]; };
    struct alignas(16) Values { V v[16 / sizeof(V)]; };
    constexpr int PER = 16 / sizeof(V);
    const int64_t stride = (int64_t)gridDim.x * 256, t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t cols4 = n / 4, vals = n / PER;
    for (int64_t i = t; i < cols4; i += stride) reinterpret_cast<Four *>(c_col)[i] = reinterpret_cast<const Four *>(col)[i];
    for (int64_t i = t; i < vals; i += stride) reinterpret_cast<Values *>(c_val)[i] = reinterpret_cast<const Values *>(val)[i];
    if (t < n - cols4 * 4) c_col[cols4 * 4 + t] = col[cols4 * 4 + t];
    if (t < n - vals * PER) c_val[vals * PER + t] = val[vals * PER + t];
}

hipError_t launch_trim(int dtype, const int32_t *col, const void *val, int64_t n, int32_t *c_col, void *c_val, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 256 * 8 - 1) / (256 * 8);
    if (blocks > 8192) blocks = 8192;
    if (dtype == OCEAN_F64)
        hipLaunchKernelGGL(k_trim<double>, dim3((unsigned)blocks), dim3(256), 0, s, col, static_cast<const double *>(val), n,
                           c_col, static_cast<double *>(c_val));
    else
        hipLaunchKernelGGL(k_trim<float>, dim3((unsigned)blocks), dim3(256), 0, s, col, static_cast<const float *>(val), n,
                           c_col, static_cast<float *>(c_val));
    return hipGetLastError();
}

template <typename V>
static hipError_t dispatch_placed(const Csr &A, const Csr &B, const PlacedLaunch &l, hipStream_t s)
{
    const V *av = static_cast<const V *>(A.val);
    const V *bv = static_cast<const V *>(B.val);
    const Placing<V> p{A.rows, l.c_rp, l.out_col, static_cast<V *>(l.out_val), l.slots, l.counts, l.places, l.total, l.flags, l.placer_polls, l.unit_polls};
    const unsigned blocks = (unsigned)(placed_units(A.rows, l.cls) + 1);
#define OCEAN_GROUP(CLS, G, PPT)                                                                                         \
    case CLS:                                                                                                           \
        static_assert(kSortClass[CLS].cap == G * PPT && kPlacedRows[CLS] == 256 / G, "rows of a unit of the class");      \
        hipLaunchKernelGGL((k_placed_group<V, G, PPT, kSortClass[CLS].entries>), dim3(blocks), dim3(256), 0, s, A.rp,    \
                           A.col, av, B.rp, B.col, bv, p);                                                               \
        break
#define OCEAN_WAVE(MAX)                                                                                                  \
    hipLaunchKernelGGL((k_placed_wave<V, MAX>), dim3(blocks), dim3(256), (size_t)l.pool, s, A.rp, A.col, av, B.rp, B.col, \
                       bv, l.prod, p)
    switch (l.cls) {
        OCEAN_GROUP(1, 8, 4);
        OCEAN_GROUP(2, 16, 4);
        OCEAN_GROUP(3, 16, 6);
        OCEAN_GROUP(4, 16, 8);
        OCEAN_GROUP(5, 32, 6);
        OCEAN_GROUP(6, 32, 8);
    case 7: case 8: OCEAN_WAVE(8); break;
    case 9: case 10: OCEAN_WAVE(16); break;
    case 11: OCEAN_WAVE(24); break;
    case 12: OCEAN_WAVE(32); break;
    default: return hipErrorInvalidValue;
    }
#undef OCEAN_GROUP
#undef OCEAN_WAVE
    return hipGetLastError();
}

hipError_t launch_placed(const Csr &A, const Csr &B, int dtype, const PlacedLaunch &l, hipStream_t s)
{
    if (A.rows <= 0) return hipSuccess;
    return dtype == OCEAN_F64 ? dispatch_placed<double>(A, B, l, s) : dispatch_placed<float>(A, B, l, s);
}

}  // namespace ocean
