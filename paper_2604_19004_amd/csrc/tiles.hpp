// Traversal of the products of one row of C by a workgroup, for rows of many products (the column-window kernel and the symbolic
// bitmap): pieces of rows of B are cut into tiles of 64 entries, and the tiles are dealt out evenly to the waves.
//
// A row of 16 lanes walks a tile, four consecutive entries a lane (one 16-byte load of column ids, two of fp64 values), so a wave walks
// four tiles in a step.  What a tile needs (position, length, A's value) is found by one search of the pieces per lane and 64
// tiles, and reaches the 16 lanes by DPP moves: no search, LDS read or prefix per product.  B needs eight entries or more
// (TILE_MIN_ENTRIES): the last lane of a tile reads four entries that end with the tile, which may begin before it.
#pragma once

#include <type_traits>

#include "ocean_internal.hpp"

namespace ocean {

using NoVal = unsigned char;   // column ids only (the symbolic pass)

constexpr int TILE_ROW = 16, TILE_STEP = WAVE / TILE_ROW;

// Pieces (position in B's arrays, entries, A's value) of up to N entries of A, and the tiles before each.
template <typename V, typename P, int N>
struct TileChunk {
    static constexpr int SIZE = N;
    static constexpr bool VALS = !std::is_same_v<V, NoVal>;
    uint32_t first[N], len[N];
    P pos[N];
    V a[VALS ? N : 1];
    uint32_t wsum[N / WAVE];
    uint32_t total;
};

// The pieces that the first nent threads hold (len = 0 in all others) into c; returns their tiles.  Every thread calls
// it; c must be free on entry, and is ready behind the barrier that this ends with.
template <int THREADS, typename V, typename P, int N>
__device__ __forceinline__ uint32_t tile_open(TileChunk<V, P, N> &c, int nent, P p, uint32_t len, V a)
{
    static_assert(N <= THREADS && N % WAVE == 0, "a thread per piece");
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const uint32_t tiles = (len + (WAVE - 1)) / WAVE;
    auto put = [&](uint32_t before) {
        c.first[tid] = before;
        c.len[tid] = len;
        c.pos[tid] = p;
        if constexpr (TileChunk<V, P, N>::VALS) c.a[tid] = a;
    };
    if (nent <= WAVE) {   // uniform
        if (tid < WAVE) {
            const uint32_t incl = wave_inclusive_scan_u32(tiles);
            put(incl - tiles);
            if (lane == WAVE - 1) c.total = incl;
        }
        __syncthreads();
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)c.total);
    }
    uint32_t incl = 0;
    if (tid < N) {
        incl = wave_inclusive_scan_u32(tiles);
        if (lane == WAVE - 1) c.wsum[tid / WAVE] = incl;
    }
    __syncthreads();
    uint32_t total;
    const uint32_t before = waves_before_u32<N / WAVE>(c.wsum, tid < N ? tid / WAVE : 0, total);
    if (tid < N) put(before + incl - tiles);
    __syncthreads();
    return total;
}

// v of lane J of every row of 16 lanes, in all of them.
template <int J>
__device__ __forceinline__ uint32_t row_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + J, 0xf, 0xf, false); }   // row_newbcast
// Every row of 16 lanes moved down by J lanes.
template <int J>
__device__ __forceinline__ uint32_t row_down(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + J, 0xf, 0xf, false); }   // row_shl
#define OCEAN_ROW_MOVE(NAME)                                                                                           \
    template <int J>                                                                                                   \
    __device__ __forceinline__ unsigned long long NAME(unsigned long long v)                                           \
    {                                                                                                                  \
        return ((unsigned long long)NAME<J>((uint32_t)(v >> 32)) << 32) | NAME<J>((uint32_t)v);                        \
    }                                                                                                                  \
    template <int J>                                                                                                   \
    __device__ __forceinline__ float NAME(float v) { return __uint_as_float(NAME<J>(__float_as_uint(v))); }            \
    template <int J>                                                                                                   \
    __device__ __forceinline__ double NAME(double v)                                                                   \
    {                                                                                                                  \
        return __longlong_as_double((long long)NAME<J>((unsigned long long)__double_as_longlong(v)));                  \
    }                                                                                                                  \
    template <int J>                                                                                                   \
    __device__ __forceinline__ NoVal NAME(NoVal v) { return v; }
OCEAN_ROW_MOVE(row_lane)
OCEAN_ROW_MOVE(row_down)
#undef OCEAN_ROW_MOVE

// A tile per lane.  Step j's four are with lanes j, 16 + j, 32 + j and 48 + j.
template <typename V, typename P>
struct Tiles {
    P p;
    int32_t n;    // entries; 0: no tile (with p = 4, so that four entries before p are there to be read)
    V a;
    bool edge;    // (uniform) a tile ends among B's first three entries
    bool small;   // (uniform) a piece has fewer than four entries: a lane's first entries may be of another row of B

    // tiles from..to-1 of the chunk (to - from <= 64, to <= total)
    template <int N>
    __device__ __forceinline__ void find(const TileChunk<V, P, N> &c, int nent, uint32_t total, uint32_t from, uint32_t to)
    {
        const uint32_t mine = from + (uint32_t)(lane_id() % TILE_ROW * TILE_STEP + lane_id() / TILE_ROW);
        const uint32_t t = mine < total ? mine : total - 1u;
        int e = 0;   // the last piece that starts at or before tile t (pieces without entries start where the next one does)
        for (int step = nent > 1 ? 1 << (31 - __clz(nent - 1)) : 0; step > 0; step >>= 1)
            if (c.first[e + step] <= t) e += step;
        const uint32_t off = (t - c.first[e]) * WAVE;
        const uint32_t left = c.len[e] - off;
        p = mine < to ? c.pos[e] + off : (P)4;
        n = mine < to ? (int32_t)(left < WAVE ? left : (uint32_t)WAVE) : 0;
        if constexpr (TileChunk<V, P, N>::VALS) a = c.a[e];
        small = __ballot(mine < to && off == 0u && left < 4u) != 0ull;
        edge = small && __ballot(p + (P)(uint32_t)n < (P)4) != 0ull;
    }
    // step J from now on is the first
    template <int J>
    __device__ __forceinline__ void advance()
    {
        p = row_down<J>(p);
        n = (int32_t)row_down<J>((uint32_t)n);
        a = row_down<J>(a);
    }
};

// A lane's four entries of B in a step.  They are its four of the tile, or the tile's last four where those would
// reach beyond its end: the first `skip` of them are then another lane's (all four: the lane has none).
template <typename V>
struct TileFour {
    int32_t col[4];
    V val[4];
    int32_t skip;
};

template <int J, bool VALS, typename V, typename P>
__device__ __forceinline__ void tile_load(const Tiles<V, P> &t, const int32_t *__restrict__ b_col, const V *__restrict__ b_val, TileFour<V> &f)
{
    struct alignas(4) Cols { int32_t v[4]; };
    struct alignas(sizeof(V)) Vals { V v[4]; };
    const int32_t sub = 4 * (lane_id() % TILE_ROW);
    const P p = row_lane<J>(t.p);
    const int32_t n = (int32_t)row_lane<J>((uint32_t)t.n);
    int32_t at = sub < n - 4 ? sub : n - 4;
    const int32_t least = -(int32_t)(p < (P)4 ? p : (P)4);
    at = at > least ? at : least;   // (a tile that ends among B's first three entries)
    f.skip = sub - at;
    const size_t q = (size_t)(p + (P)(int64_t)at);
    const Cols c = *reinterpret_cast<const Cols *>(b_col + q);
#pragma unroll
    for (int i = 0; i < 4; ++i) f.col[i] = c.v[i];
    if constexpr (VALS) {
        const Vals v = *reinterpret_cast<const Vals *>(b_val + q);
#pragma unroll
        for (int i = 0; i < 4; ++i) f.val[i] = v.v[i];
    }
    if (t.edge) {   // uniform
#pragma unroll
        for (int i = 0; i < 4; ++i) f.col[i] = at + i < n ? f.col[i] : -1;
    }
}

// Every product of the open chunk once: use(fours, t) for the lane's part of U steps at a time, t's first U (2 or 4).
// mine: the wave's tiles (its first 64) where `found` says so, and on return where there are no more.
// AHEAD: the next U steps are on their way while these are used.  That takes the registers of U steps more (13 U with
// fp64 values), worth it where they don't cost waves in flight.
template <int THREADS, int U, bool VALS, bool AHEAD = true, typename V, typename P, int N, typename F>
__device__ __forceinline__ void tile_walk(const TileChunk<V, P, N> &c, int nent, uint32_t total, const int32_t *__restrict__ b_col,
                                          const V *__restrict__ b_val, Tiles<V, P> &mine, bool found, F use)
{
    static_assert(U == 2 || U == 4, "sixteen steps are whole batches");
    constexpr uint32_t WAVES = THREADS / WAVE;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const uint32_t span = (total + WAVES * TILE_STEP - 1) / (WAVES * TILE_STEP) * TILE_STEP;
    const uint32_t t0 = wave * span, t1 = t0 + span < total ? t0 + span : total;
    for (uint32_t from = t0; from < t1; from += WAVE) {   // uniform for the wave
        if (!found || from > t0) mine.find(c, nent, total, from, t1);
        Tiles<V, P> t = mine;
        int left = (int)(t1 - from < WAVE ? t1 - from : WAVE);   // tiles
        TileFour<V> f[U];
        if constexpr (!AHEAD) {
            static_assert(U == 2);
            for (;; left -= U * TILE_STEP) {
                tile_load<0, VALS>(t, b_col, b_val, f[0]);
                tile_load<1, VALS>(t, b_col, b_val, f[1]);
                use(f, t);
                if (left <= U * TILE_STEP) break;
                t.template advance<U>();
            }
            continue;
        }
        TileFour<V> g[U];
        tile_load<0, VALS>(t, b_col, b_val, f[0]);
        tile_load<1, VALS>(t, b_col, b_val, f[1]);
        if constexpr (U == 4) {
            tile_load<2, VALS>(t, b_col, b_val, f[2]);
            tile_load<3, VALS>(t, b_col, b_val, f[3]);
        }
        for (; left > U * TILE_STEP; left -= U * TILE_STEP) {
            tile_load<U, VALS>(t, b_col, b_val, g[0]);
            tile_load<U + 1, VALS>(t, b_col, b_val, g[1]);
            if constexpr (U == 4) {
                tile_load<U + 2, VALS>(t, b_col, b_val, g[2]);
                tile_load<U + 3, VALS>(t, b_col, b_val, g[3]);
            }
            use(f, t);
            t.template advance<U>();
#pragma unroll
            for (int u = 0; u < U; ++u) f[u] = g[u];
        }
        use(f, t);
    }
}

}  // namespace ocean
