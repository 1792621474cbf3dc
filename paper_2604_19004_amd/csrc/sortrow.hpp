// Short rows by expand-sort-compress with several products per lane (paper Section 2.2, "ESC"; Section 4.2 for the
// packed keys): rows with at most 2048 intermediate products, for the kernels of sortrow.hip and placed.hip.
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
//   compress  a key whose column differs from its predecessor's opens an entry of C; a prefix sum numbers them, a lane adds
//             up its keys between one head and the next, what an entry has in lanes before comes by a prefix sum over
//             lanes, and the row leaves through LDS with coalesced stores, in column order.
// The steps below are those of rows placed in C (placed.hip) and of listed rows of more than 1024 products
// (k_numeric_sort_long); k_numeric_sort, for smaller listed rows, takes the network and the scans from here and has its own
// expand and accumulate: the values of 8 bytes that it adds up in LDS are faster where LDS is not short (sortrow.hip).
// What bounds it is vector issue: 880 vector instructions per row of the 512-product class, of which the sort is 530, are
// 489 us for 341 000 rows (of the rectangular input, before there was a class of 384) at one per four cycles and SIMD,
// 541 us measured by k_numeric_sort.  Placed, issue was 87 % of the cycles of 762 products a row (2111 instructions, before rows gathered) and is
// 72 % of those of 264 (906 instructions; a wave waits, for loads above all, in 64 % of its cycles, with 6.8 of them on a SIMD).
// The work does not depend on where the columns lie or how many products merge.  Sizes of 3 * 2^i products cost a third less
// per row than the next power of two (see settle).  Against the hash kernels (one MI355X, fp64 unless said): numeric
// stage of the rectangular input (264 products a row) 1.50 -> 0.94 ms, clustered fp32 (762 products, 234 columns) 2.55 ->
// 1.50 ms, 100 003 uniform rows of 1023 products fp32 1.29 -> 0.40 ms, Laplacian (25 products) 0.22 -> 0.19 ms.
#pragma once

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

// v of the lane that CTRL names (DPP), -0, which changes no sum, where it names none or ROWS leaves the lane's row of 16 out.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v)
{
    const long long x = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)0x80000000u, (int)(uint32_t)((unsigned long long)x >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ void carry_step(double &v, uint32_t &stop, bool there)
{
    const double o = dpp_f64<CTRL, ROWS>(v);
    const uint32_t s = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)stop, CTRL, ROWS, 0xf, false);
    v += stop != 0u || !there ? -0.0 : o;
    stop |= there ? s : 0u;
}
// In every group of G lanes: the sum of v over the lanes before this one, back to the last with `first` set (included).
template <int G>
__device__ __forceinline__ double carried(double v, bool first, int sub)
{
    uint32_t stop = first;
    carry_step<0x111, 0xf>(v, stop, G >= 16 || sub >= 1);                       // row_shr:1
    carry_step<0x112, 0xf>(v, stop, G >= 16 || sub >= 2);                       // row_shr:2
    carry_step<0x114, 0xf>(v, stop, G >= 16 || sub >= 4);                       // row_shr:4
    if constexpr (G >= 16) carry_step<0x118, 0xf>(v, stop, true);               // row_shr:8
    if constexpr (G >= 32) carry_step<0x142, 0xa>(v, stop, true);               // row_bcast:15, rows 1 and 3
    if constexpr (G >= 64) carry_step<0x143, 0xc>(v, stop, true);               // row_bcast:31, rows 2 and 3
    const double before = dpp_f64<0x138, 0xf>(v);                               // wave_shr:1
    return sub == 0 ? -0.0 : before;
}

constexpr int log2_of(int x) { return x <= 1 ? 0 : 1 + log2_of((x + 1) >> 1); }   // rounded up

// What a row takes of the LDS.
template <typename V, int G, int PPT, int ENT>
struct SortRow {
    static constexpr int CAP = G * PPT;
    static constexpr int MW = (CAP + 63) / 64;   // 64-bit words of segment starts
    // places of the sorted row are spread by one slot in eight or sixteen, so that the lanes' stores, PPT apart, meet
    // different banks
    static constexpr int SPREAD = PPT >= 12 ? 4 : 3;
    static constexpr int PLACES = CAP + (CAP >> SPREAD);
    static __device__ __forceinline__ int place(int r) { return r + (r >> SPREAD); }
    uint32_t pos[ENT];     // position in B of an entry's first product, minus that product's number
    V a[ENT];
    unsigned long long start[MW];
    // the products' values by number, then the values of the row of C by rank, then its columns: what LDS a row takes
    // decides how many rows a compute unit works on (1024 products: with a place of their own for the columns 2 waves per
    // SIMD and 506 us for 100 003 rows, one place for all three 4 waves and 380 us).  At the end, as a row of fewer products
    // than the class has may be given less (sort_row_bytes).
    V acc[PLACES];
};

// A row of the sort kernels, in the order in which its steps are called; sub = lane inside the group of G lanes that own it.
template <typename V, int G, int PPT, int ENT>
struct SortedRow {
    using Lds = SortRow<V, G, PPT, ENT>;
    static constexpr int CAP = G * PPT;
    static constexpr int LB = log2_of(CAP);
    static constexpr int MW = Lds::MW;
    static constexpr int BATCH = PPT % 6 == 0 ? 6 : PPT % 4 == 0 ? 4 : PPT % 3 == 0 ? 3 : PPT % 2 == 0 ? 2 : 1;
    static_assert(64 % G == 0, "whole groups");

    uint32_t key[PPT];
    uint32_t total;     // products
    uint32_t n_out;     // entries of the row of C
    uint32_t heads;     // bit u: key u opens an entry of C
    uint32_t tails;     // bit u: key u closes one
    int rank0;          // entries before this lane's keys, minus one

    // Entries e0 .. e0 + ne - 1 of A; ne = 0: a group without a row (the rows of a wave advance together).  CUT: see products.
    template <bool CUT = false>
    __device__ __forceinline__ void sort(Lds &sr, int lane, int sub, int64_t e0, int ne, const int32_t *__restrict__ a_col,
                                         const V *__restrict__ a_val, const int64_t *__restrict__ b_rp,
                                         const int32_t *__restrict__ b_col, const V *__restrict__ b_val)
    {
        expand<CUT>(sr, lane, sub, e0, ne, a_col, a_val, b_rp, b_col, b_val);
        order(lane, sub);
    }

    // The first half of it: the products, keys unsorted.
    template <bool CUT>
    __device__ __forceinline__ void expand(Lds &sr, int lane, int sub, int64_t e0, int ne, const int32_t *__restrict__ a_col,
                                           const V *__restrict__ a_val, const int64_t *__restrict__ b_rp,
                                           const int32_t *__restrict__ b_col, const V *__restrict__ b_val)
    {
        ne = ne < ENT ? ne : ENT;   // (holds: the caller lists no other rows)
        open(sr, sub);
        int nseg = 0;
        total = 0;
        const int chunks = G >= ENT ? 1 : (int)wave_max_u32((uint32_t)((ne + G - 1) / G));
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
            add(sr, lane, sub, (uint32_t)p0, len, a, nseg);
        }
        products<CUT>(sr, sub, b_col, b_val);
    }

    __device__ __forceinline__ void open(Lds &sr, int sub)
    {
        for (int w = sub; w < MW; w += G) sr.start[w] = 0ull;
        wave_sync();
    }

    // An entry of A per lane: a times len entries of B from p0 on; nseg: segments before them.
    __device__ __forceinline__ void add(Lds &sr, int lane, int sub, uint32_t p0, uint32_t len, V a, int &nseg)
    {
        const int shift = lane & ~(G - 1);
        constexpr unsigned long long GMASK = G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull;
        uint32_t sum;
        const uint32_t first = total + group_scan<G>(len, sub, sum) - len;
        const unsigned long long some = (__ballot(len > 0) >> shift) & GMASK;
        if (len > 0 && first < (uint32_t)CAP) {   // (the second holds: at most CAP products)
            const int at = nseg + __popcll(some & ((1ull << sub) - 1ull));
            sr.pos[at] = p0 - first;
            sr.a[at] = a;
            atomicOr(reinterpret_cast<uint32_t *>(sr.start) + (first >> 5), 1u << (first & 31u));
        }
        total += sum;
        nseg += __popcll(some);
    }

    // The products of the entries: keys and, in LDS, values by number.  CUT: the row has no more places than its own
    // products need and one (pads use that), and B has fewer than 2^29 entries (byte offsets in 32 bits, which leaves out an
    // address of two registers per load).
    template <bool CUT>
    __device__ __forceinline__ void products(Lds &sr, int sub, const int32_t *__restrict__ b_col,
                                             const V *__restrict__ b_val)
    {
        total = total < (uint32_t)CAP ? total : (uint32_t)CAP;
        wave_sync();
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
                if (q < total) {
                    if constexpr (CUT) {
                        c[i] = *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(b_col) + p[i] * 4u);
                        b[i] = *reinterpret_cast<const V *>(reinterpret_cast<const char *>(b_val) + p[i] * (uint32_t)sizeof(V));
                    } else {
                        c[i] = b_col[p[i]];
                        b[i] = b_val[p[i]];
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const uint32_t q = (uint32_t)((u0 + i) * G + sub);
                key[u0 + i] = q < total ? ((uint32_t)c[i] << LB) | q : SR_PAD;
                sr.acc[!CUT || q < total ? q : total] = a[i] * b[i];
            }
        }
    }

    // The keys into order, entries of C counted.
    __device__ __forceinline__ void order(int lane, int sub)
    {
        sort_keys<G, PPT>(key, lane);
        // a key whose column differs from its predecessor's
        const uint32_t below = (uint32_t)__shfl_up((int)key[PPT - 1], 1, WAVE);   // last key of the lane below
        uint32_t pads = 0u;
        heads = 0u;
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const uint32_t prev = u == 0 ? below : key[u - 1];
            if (key[u] == SR_PAD) pads |= 1u << u;
            else if ((u == 0 && sub == 0) || ((prev ^ key[u]) >> LB) != 0u) heads |= 1u << u;
        }
        const uint32_t opens = heads | pads;
        const uint32_t above = (uint32_t)__shfl_down((int)opens, 1, WAVE) | (uint32_t)(sub == G - 1);   // (every lane takes part)
        tails = ((opens >> 1) | ((above & 1u) << (PPT - 1))) & ~pads;
        const uint32_t mine = (uint32_t)__popc(heads);
        rank0 = (int)(group_scan<G>(mine, sub, n_out) - mine) - 1;
        wave_sync();
    }

    // Place of key u's entry among the values (by rank) of the row.
    __device__ __forceinline__ int place(int u) const
    {
        return Lds::place(rank0 + __popc(heads & (uint32_t)((2ull << u) - 1ull)));
    }

    // The row's values into acc (that of its SortRow), by rank: sums over the keys between a head and its tail, in 64 bits and in the order of
    // the sort.  A lane's keys before its first head belong to an entry that a lane before has opened: what that lane and
    // those between hold of it comes by a prefix sum that starts anew behind every lane with a head.  (Adding up in LDS, an
    // 8-byte atomic for every key that is no head, took 8 bytes a product also for 4-byte values: 100 000 rows of 1444 and of
    // 2025 products fp32 653 -> 575 and 1085 -> 815 us now that a compute unit holds twice the rows; fp64, and smaller
    // classes, within 2 %.)
    template <bool CUT = false>
    __device__ __forceinline__ void accumulate(V *acc, int sub)
    {
        V val[PPT];
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            const uint32_t q = key[u] & ((1u << LB) - 1u);
            // (a pad's number is the largest there is)
            val[u] = acc[CUT ? (q < total ? q : total) : CAP == 1 << LB || q < (uint32_t)CAP ? q : 0u];
        }
        wave_sync();
        double run = -0.0;
#pragma unroll
        for (int u = 0; u < PPT; ++u) {
            run = (u == 0 || ((heads >> u) & 1u) ? -0.0 : run) + (double)val[u];
            if ((tails >> u) & 1u) acc[place(u)] = (V)run;
        }
        const double carry = carried<G>(run, heads != 0u, sub);
        // the lane's first tail, where it closes an entry that a lane before has opened
        if (!(heads & 1u) && tails != 0u) {
            const int t = __ffs((int)tails) - 1;
            const int at = Lds::place(rank0);
            if constexpr (sizeof(V) == sizeof(double)) {
                acc[at] = acc[at] + carry;
            } else {   // (one rounding: the 64-bit sum again)
                run = carry;
#pragma unroll
                for (int u = 0; u < PPT; ++u) run += u <= t ? (double)val[u] : -0.0;
                acc[at] = (V)run;
            }
        }
        wave_sync();
    }

    // The row's columns into acc, by rank, when its values are no longer needed there.
    __device__ __forceinline__ void columns(V *acc)
    {
        int32_t *s_col = reinterpret_cast<int32_t *>(acc);
#pragma unroll
        for (int u = 0; u < PPT; ++u)
            if ((heads >> u) & 1u) s_col[place(u)] = (int32_t)(key[u] >> LB);
        wave_sync();
    }

    // The row to out_col / out_val from position o on.
    __device__ __forceinline__ void write(V *acc, int sub, int64_t o, int n_write, int32_t *__restrict__ out_col,
                                          V *__restrict__ out_val)
    {
        for (int i = sub; i < n_write; i += G) out_val[o + i] = acc[Lds::place(i)];
        wave_sync();
        columns(acc);
        const int32_t *s_col = reinterpret_cast<const int32_t *>(acc);
        for (int i = sub; i < n_write; i += G) out_col[o + i] = s_col[Lds::place(i)];
    }
};

}  // namespace

}  // namespace ocean
