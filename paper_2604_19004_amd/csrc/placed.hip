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
    c.template accumulate<true>(sr.acc, sub);
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
    c.write(sr.acc, sub, o, live && o + c.n_out <= p.slots ? (int)c.n_out : 0, p.out_col, p.out_val);
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

// ---- rows whose products gather: most of them lie in a window of a few hundred columns.  These are added up in an accumulator
// per column (-0: no product yet, and no addend is -0), and only the others are sorted, in a network of their own number; their
// entries come before and behind the window's.  A row of 762 products of the clustered input, 105 of them outside: 2111 -> 1198 vector
// instructions.  The call 2.22 -> 1.93 ms (with shorter placing turns and neighbouring units on one XCD); the rest is waiting: 1.43
// ms where a row doesn't wait for its place, 1.02 with nothing behind the loads of the products.  Of a row's 18 us 8 are the chain
// of loads before them, 5 the wait for the rows before.  Limits: below 6 products a lane the sort costs no more than the window; from
// more than 24 (8-byte values: 12) on the values of a row need registers that the launch does not have.
// Rows that do not gather pay for five lane reads and a median (rectangular input: within 0.5 %).
template <typename V> constexpr bool gathers(int ppt) { return ppt >= 6 && ppt <= (sizeof(V) == 4 ? 24 : 12); }   // products per lane of the rows that are looked at
struct Gathered {
    int32_t base;                 // first column of the window
    int width;                    // columns, a multiple of the wave
    int rest;                     // products outside
};
// LDS of the products outside the window: their values, spread as SortRow::acc, and their columns.
template <typename V>
__device__ __forceinline__ int rest_places(int rest) { return rest + (rest >> 3) + 1; }

// The window lies around the median column of five products, from rows of B all over the first two thirds of the row's products.  It
// is none where fewer than three of them are in it, as with columns in no order.
template <typename V, int PPT>
__device__ __forceinline__ bool find_window(const SortedRow<V, WAVE, PPT, 64> &c, int bytes, Gathered &g)
{
    int32_t m[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) m[i] = (int32_t)((uint32_t)__builtin_amdgcn_readlane((int)c.key[PPT * 2 * i / 15], 13 * i) >> SortedRow<V, WAVE, PPT, 64>::LB);
    int32_t s[5] = {m[0], m[1], m[2], m[3], m[4]};
    auto order = [&](int i, int j) {
        const int32_t lo = s[i] < s[j] ? s[i] : s[j], hi = s[i] < s[j] ? s[j] : s[i];
        s[i] = lo;
        s[j] = hi;
    };
    order(0, 1); order(3, 4); order(2, 4); order(2, 3); order(1, 4); order(0, 3); order(0, 2); order(1, 3); order(1, 2);
    g.width = bytes >= 8 * 512 + 1024 ? 512 : 256;
    const int32_t half = g.width / 2;
    g.base = s[2] > half ? s[2] - half : 0;
    int in = 0;
#pragma unroll
    for (int i = 0; i < 5; ++i) in += (uint32_t)(m[i] - g.base) < (uint32_t)g.width ? 1 : 0;
    return in >= 3;
}

// The products of c (expanded into sr, bytes of LDS) parted into those of the window, added up, and the rest.  False, and nothing has
// changed, where more than half of them lie outside or the row's LDS does not hold both parts.
template <typename V, int PPT>
__device__ __forceinline__ bool part_products(const SortedRow<V, WAVE, PPT, 64> &c, SortRow<V, WAVE, PPT, 64> &sr, int bytes, int lane, Gathered &g)
{
    using Row = SortedRow<V, WAVE, PPT, 64>;
    constexpr uint32_t NO_COL = SR_PAD >> Row::LB;   // a pad's column, above all others
    const uint32_t base = (uint32_t)g.base;
    const uint32_t width = (uint32_t)g.width < NO_COL - base ? (uint32_t)g.width : NO_COL - base;
    int in = 0;
#pragma unroll
    for (int u = 0; u < PPT; ++u) in += __popcll(__ballot((c.key[u] >> Row::LB) - base < width));
    g.rest = (int)c.total - in;
    if (2 * g.rest > (int)c.total || g.rest > 8 * WAVE ||
        8 * g.width + (int)sizeof(V) * rest_places<V>(g.rest) + 4 * g.rest > bytes) return false;   // uniform
    V val[PPT];
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const uint32_t q = (uint32_t)(u * WAVE + lane);
        val[u] = sr.acc[q < c.total ? q : c.total];
    }
    wave_sync();
    double *win = reinterpret_cast<double *>(&sr);
    V *acc = reinterpret_cast<V *>(win + g.width);
    uint32_t *cols = reinterpret_cast<uint32_t *>(acc + rest_places<V>(g.rest));
    for (int i = lane; i < g.width; i += WAVE) win[i] = -0.0;
    wave_sync();
    int run = 0;
#pragma unroll
    for (int u = 0; u < PPT; ++u) {
        const uint32_t col = c.key[u] >> Row::LB;
        const uint32_t d = col - base;
        const bool inside = d < width, other = !inside && col != NO_COL;
        if (inside) __hip_atomic_fetch_add(&win[d], (double)val[u] + 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const unsigned long long others = __ballot(other);
        if (other) {
            const int at = run + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(others >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)others, 0u));
            cols[at] = col;
            acc[at] = val[u];
        }
        run += __popcll(others);
    }
    wave_sync();
    return true;
}

// What part_products has left of a row, to its end: rest <= 64 * R.
template <typename V, int R, typename Finish>
__device__ __forceinline__ void finish_gathered(const Gathered &g, char *lds, int lane, int32_t *__restrict__ out_col,
                                                V *__restrict__ out_val, Finish finish)
{
    using Row = SortedRow<V, WAVE, R, 64>;
    using Lds = SortRow<V, WAVE, R, 64>;
    const double *win = reinterpret_cast<const double *>(lds);
    V *acc = reinterpret_cast<V *>(lds + 8 * g.width);
    const uint32_t *cols = reinterpret_cast<const uint32_t *>(acc + rest_places<V>(g.rest));
    Row c;
    c.total = (uint32_t)g.rest;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const uint32_t q = (uint32_t)(u * WAVE + lane);
        c.key[u] = q < c.total ? (cols[q] << Row::LB) | q : SR_PAD;
    }
    c.order(lane, lane);
    uint32_t below = 0;   // entries of the rest before the window
#pragma unroll
    for (int u = 0; u < R; ++u) below += ((c.heads >> u) & 1u) && (c.key[u] >> Row::LB) < (uint32_t)g.base ? 1u : 0u;
    below = wave_sum_u32(below);
    auto there = [](double v) { return __double_as_longlong(v) != (long long)0x8000000000000000ull; };
    int inside = 0;
    for (int i = 0; i < g.width; i += WAVE) inside += __popcll(__ballot(there(win[i + lane])));
    const int n_rest = (int)c.n_out;
    finish(c.n_out + (uint32_t)inside, [&]() { c.template accumulate<true>(acc, lane); }, [&](int64_t o) {
        for (int i = lane; i < n_rest; i += WAVE) out_val[o + i + (i >= (int)below ? inside : 0)] = acc[Lds::place(i)];
        int64_t at = o + below;
        for (int i = 0; i < g.width; i += WAVE) {
            const double v = win[i + lane];
            const unsigned long long m = __ballot(there(v));
            if (there(v)) {
                const int64_t to = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                out_val[to] = (V)v;
                out_col[to] = g.base + i + lane;
            }
            at += __popcll(m);
        }
        wave_sync();
        c.columns(acc);
        const int32_t *s_col = reinterpret_cast<const int32_t *>(acc);
        for (int i = lane; i < n_rest; i += WAVE) out_col[o + i + (i >= (int)below ? inside : 0)] = s_col[Lds::place(i)];
    });
}

// A row of pr products by a whole wave, in the size of sort that is the row's own.  finish(n_out, accumulate, write): the row's
// entries are counted; accumulate() adds its values up, write(o) writes it from entry o of C on.
template <typename V, int MAX, typename Finish>
__device__ __forceinline__ void row_by_size(char *lds, int pr, int64_t e0, int ne,
                                            const int32_t *__restrict__ a_col, const V *__restrict__ a_val,
                                            const int64_t *__restrict__ b_rp, const int32_t *__restrict__ b_col,
                                            const V *__restrict__ b_val, int32_t *__restrict__ out_col, V *__restrict__ out_val,
                                            Finish finish)
{
    const int lane = lane_id();
    Gathered g;
    const int bytes = sort_row_bytes(pr, sizeof(V));
    const bool parted = [&]() {
#define OCEAN_PLACED(PPT)                                                                                        \
    if constexpr (PPT <= MAX)                                                                                    \
        if (pr <= 64 * PPT) {                                                                                    \
            SortRow<V, WAVE, PPT, 64> &sr = *reinterpret_cast<SortRow<V, WAVE, PPT, 64> *>(lds);                 \
            SortedRow<V, WAVE, PPT, 64> c;                                                                       \
            bool window = false;                                                                                 \
            if constexpr (!gathers<V>(PPT)) {                                                                    \
                c.template sort<true>(sr, lane, lane, e0, ne, a_col, a_val, b_rp, b_col, b_val);                 \
            } else {                                                                                             \
                c.template expand<true>(sr, lane, lane, e0, ne, a_col, a_val, b_rp, b_col, b_val);               \
                if (find_window<V, PPT>(c, bytes, g) && part_products<V, PPT>(c, sr, bytes, lane, g)) return true; \
                c.order(lane, lane);                                                                             \
            }                                                                                                    \
            finish(c.n_out, [&]() { c.template accumulate<true>(sr.acc, lane); },                                \
                   [&](int64_t o) { c.write(sr.acc, lane, o, (int)c.n_out, out_col, out_val); });                \
            return false;                                                                                        \
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
        return false;
    }();
    if (!parted) return;   // uniform
#define OCEAN_REST(R) if (g.rest <= 64 * R) return finish_gathered<V, R>(g, lds, lane, out_col, out_val, finish)
    OCEAN_REST(1);
    OCEAN_REST(2);
    OCEAN_REST(3);
    OCEAN_REST(4);
    OCEAN_REST(6);
    OCEAN_REST(8);
#undef OCEAN_REST
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
    const int64_t unit = unit_of_workgroup((int64_t)blockIdx.x - 1, (p.m + 3) / 4, p.by_xcd);
    const int64_t row = unit * 4 + wave;
    if (threadIdx.x == 0) {
        s_four.arrived = 0u;
        s_four.place = 0ull;
    }
    if (threadIdx.x < 4) s_four.n[threadIdx.x] = 0u;
    const int64_t own = row < p.m ? row : p.m - 1;
    const int64_t e0 = a_rp[own];
    const int ne = (int)(a_rp[own + 1] - e0);
    int before = 0, pr = 0;   // LDS of the rows before this wave's; its own row's products
    int of[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) of[r] = (int)prod[unit * 4 + r < p.m ? unit * 4 + r : p.m - 1];   // (all four on their way together)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int n = unit * 4 + r < p.m ? of[r] : 0;
        before += r < wave ? sort_row_bytes(n, sizeof(V)) : 0;
        pr = r == wave ? n : pr;
    }
    __syncthreads();
    if (row >= p.m) {
        publish_row(s_four, wave, 0u, p.counts + unit);
        return;
    }
    row_by_size<V, MAX>(s_pool + before, pr, e0, ne, a_col, a_val, b_rp, b_col, b_val, p.out_col, p.out_val,
                        [&](uint32_t n_out, auto accumulate, auto write) {
        publish_row(s_four, wave, n_out, p.counts + unit);
        accumulate();
        const int64_t o = place_row(s_four, wave, unit, p);
        if (o < 0) return;
        if (lane_id() == 0) {
            p.c_rp[row] = o;
            if (row == p.m - 1) p.c_rp[p.m] = o + n_out;
        }
        if (o + n_out <= p.slots) write(o);
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
    const Placing<V> p{A.rows, l.c_rp, l.out_col, static_cast<V *>(l.out_val), l.slots, l.counts, l.places, l.total, l.flags, l.placer_polls, l.unit_polls, l.by_xcd};
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
