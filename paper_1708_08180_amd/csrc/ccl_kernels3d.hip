// 3D volume labeling (the paper's method on a 3D grid): the same three
// phases over 3D tiles of 64 (x) x 16 (y) x 8 (z) voxels (4 slices under
// 6-connectivity).
//
//   local merge   the tile is taken in bundles of rows whose components are
//                 column intervals: two rows of two slices (2 x 2 rows) under
//                 18- and 26-connectivity, two rows of one slice under 6.
//                 The intervals are the union-find nodes.  Every touching
//                 pair of intervals of neighbouring bundles is found once
//                 from the row masks and joined in LDS.  The labels of a
//                 bundle's first row take, per column, 1 + the local root of
//                 that column's voxels (its "column labels"), whichever of
//                 the bundle's rows they lie in; the tile's local roots take
//                 labels[root] = root + 1.  Roots are foreground voxels, so
//                 a column label never stands where another value is due,
//                 and the forest is only ever entered at a root.
//   boundary      every voxel on a shared face is joined with its
//                 raster-earlier neighbours in other tiles; a tile's distinct
//                 pairs of local roots are collected in LDS and merged with
//                 the global union-find of the 2D path.
//   link          resolves the column labels and stores every voxel's final
//                 label.
#include <hip/hip_runtime.h>

#include "ccl.h"
#include "ccl_device.h"
#include "ccl_internal.h"
#include "ccl_merge.h"

namespace ccl {

namespace {

constexpr int kTY = 16;  // tile rows per slice

template <int CONN>
struct Geo {
    static constexpr int TZ = CONN == 6 ? 4 : 8;          // slices per tile
    static constexpr int ROWS = kTY * TZ;                 // tile rows; row z * 16 + y
    static constexpr int BR = CONN == 6 ? 2 : 4;          // rows per bundle
    static constexpr int NB = ROWS / BR;                  // bundles per tile; bundle bz * 8 + by
    static constexpr int NODES = NB * (CONN == 26 ? 32 : 64);
    static constexpr int NJ = CONN == 6 ? 2 : 4;          // earlier neighbours of a bundle
    static_assert(NB == 32, "eight threads per bundle of a 256-thread workgroup");
};

struct Vol {
    const uint8_t *vol;
    uint32_t *labels;
    int64_t pitch_y, pitch_z;
    int32_t D, H, W;
    int32_t tilesX, tilesY, tilesZ;
    uint32_t n;
};

__device__ __forceinline__ uint4 load_chunk3d(const Vol &v, int x0, int y, int z, int q) {
    if (y >= v.H || z >= v.D) return make_uint4(0u, 0u, 0u, 0u);
    return load_row16(v.vol + (int64_t)z * v.pitch_z + (int64_t)y * v.pitch_y, x0 + q * 16, v.W);
}

__device__ __forceinline__ void tile_of(const Vol &v, uint32_t t, int &tx, int &ty, int &tz) {
    const uint32_t TX = (uint32_t)v.tilesX, TY = (uint32_t)v.tilesY;
    tx = (int)(t % TX);
    ty = (int)((t / TX) % TY);
    tz = (int)(t / (TX * TY));
}

// Row masks of the tile whose first voxel is (x0, y0, z0), all threads.
template <int CONN>
__device__ __forceinline__ void load_masks(const Vol &v, int x0, int y0, int z0, uint64_t *msk) {
#pragma unroll
    for (int i = 0; i < Geo<CONN>::ROWS * 4 / 256; ++i) {
        const int c = (int)threadIdx.x + i * 256, r = c >> 2;
        ((uint16_t *)msk)[c] =
            (uint16_t)nonzero_bytes16(load_chunk3d(v, x0, y0 + (r % kTY), z0 + r / kTY, c & 3));
    }
}

// First row of bundle k; its rows are r, r + 1 and, where a bundle spans two
// slices, r + 16, r + 17 (raster order).
template <int CONN>
__device__ __forceinline__ int bundle_row(int k) {
    return (k >> 3) * (Geo<CONN>::BR / 2) * kTY + (k & 7) * 2;
}
__device__ __forceinline__ int bundle_row_offset(int i) { return (i & 1) + (i >> 1) * kTY; }

// First column of every interval of a bundle with rows w (its components:
// all voxels of one column are connected, and two adjacent columns are when
// some voxel of one neighbours some voxel of the other; under
// 18-connectivity voxels at opposite corners of the 2 x 2 rows do not).
template <int CONN>
__device__ __forceinline__ uint64_t bundle_starts(const uint64_t (&w)[4]) {
    const uint64_t m = w[0] | w[1] | w[2] | w[3];
    if (CONN == 26) return m & ~(m << 1);
    uint64_t p[4], c;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = w[i] << 1;
    if (CONN == 18)
        c = (w[0] & (p[0] | p[1] | p[2])) | (w[1] & (p[0] | p[1] | p[3])) | (w[2] & (p[0] | p[2] | p[3])) |
            (w[3] & (p[1] | p[2] | p[3]));
    else
        c = (w[0] & p[0]) | (w[1] & p[1]);
    return m & ~c;
}

template <int CONN>
struct K1Lds3d {
    using G = Geo<CONN>;
    uint32_t par[G::NODES];           // parents; a root's entry: kPixel | its smallest voxel
    uint32_t mp[G::NODES];            // joins still to make; at the end 1 + the node's root voxel
    uint16_t info[G::NODES];          // bundle << 6 | first column
    uint64_t msk[G::ROWS];            // row masks
    uint64_t M[G::NB], S[G::NB], E[G::NB];  // a bundle's columns, interval starts and ends
    uint64_t rf[G::NJ * G::NB];       // touching pairs (pair_requests) with each earlier neighbour
    uint64_t rl[CONN == 6 ? 1 : G::NJ * G::NB], rr[CONN == 6 ? 1 : G::NJ * G::NB];
    uint16_t base[G::NB];             // first node of every bundle
    uint16_t pre[G::NB * 8];          // first node at or after every eighth column
    uint32_t nodes, joins;
};

// Local merge of one tile.  Bound by instruction issue and by the chain of
// LDS round trips; nothing in it waits for another bundle: the touching
// pairs of all bundles are found at once, a lane per bundle and neighbour,
// from 64-bit masks, and each of the 256 threads then joins the pairs of
// eight columns of one bundle.  A pair's join is one LDS atomicMin that
// hooks the later interval under the earlier one; where the interval was
// hooked before, the two upper intervals are listed, and joined after all
// hooks have been compressed to trees of depth one, so that the walks are
// short.  256^3 voxels at p = 0.3, 26-connectivity: 23 us; the wavefront per
// slice that swept its rows one after the other and then joined each row with
// six neighbour rows took 172.
template <int CONN>
__global__ void __launch_bounds__(256) k1_local_merge3d(Vol v) {
    using G = Geo<CONN>;
    __shared__ K1Lds3d<CONN> sh;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tx, ty, tz;
    tile_of(v, xcd_remap(blockIdx.x, gridDim.x), tx, ty, tz);
    const int x0 = tx * kTileW, y0 = ty * kTY, z0 = tz * G::TZ;
    uint32_t *par = sh.par;
    load_masks<CONN>(v, x0, y0, z0, sh.msk);
    __syncthreads();
    auto rows_of = [&](int k, uint64_t (&w)[4]) {
        const uint64_t *m = &sh.msk[bundle_row<CONN>(k)];
        w[0] = m[0];
        w[1] = m[1];
        w[2] = CONN == 6 ? 0ull : m[kTY];
        w[3] = CONN == 6 ? 0ull : m[kTY + 1];
    };
    // every bundle's intervals (lane = bundle), numbered densely
    if (wave == 0) {
        uint64_t w[4];
        rows_of(lane & 31, w);
        const uint64_t m = w[0] | w[1] | w[2] | w[3];
        const uint64_t s = bundle_starts<CONN>(w);
        uint32_t nodes;
        const uint32_t b = wave_exclusive_scan(lane < G::NB ? (uint32_t)__popcll(s) : 0u, &nodes);
        if (lane < G::NB) {
            sh.M[lane] = m;
            sh.S[lane] = s;
            sh.E[lane] = band_ends(m, s);
            sh.base[lane] = (uint16_t)b;
        }
        if (lane == 0) {
            sh.nodes = nodes;
            sh.joins = 0u;
        }
    }
    __syncthreads();
    // touching pairs of bundle k with its earlier neighbours j: the bundles
    // before it in y (0) and z (1), and (18 / 26) the one before it in both
    // (2) and the one before it in z and after it in y (3)
    if (tid < G::NJ * G::NB) {
        const int k = tid & 31, j = tid >> 5, by = k & 7, bz = k >> 3;
        const bool ok = (j == 0 ? by > 0 : bz > 0) && (j != 2 || by > 0) && (j != 3 || by < 7);
        PairRequests q = {0ull, 0ull, 0ull};
        if (ok) {
            const int ku = k - (j == 0 ? 1 : j == 1 ? 8 : j == 2 ? 9 : 7);
            uint64_t w[4], u[4];
            rows_of(k, w);
            rows_of(ku, u);
            uint64_t st, l = 0ull, r = 0ull;
            if (CONN == 6) {
                st = j == 0 ? w[0] & u[1] : (w[0] & u[0]) | (w[1] & u[1]);
            } else {
                // the two lower rows facing the neighbour and the two upper
                // rows facing back (one each across a corner)
                const uint64_t t0 = j == 3 ? w[1] : w[0], t1 = j == 0 ? w[2] : j == 1 ? w[1] : 0ull;
                const uint64_t a0 = j == 0 ? u[1] : j == 1 ? u[2] : j == 2 ? u[3] : u[2];
                const uint64_t a1 = j == 0 || j == 1 ? u[3] : 0ull;
                const uint64_t T = t0 | t1, U = a0 | a1;
                st = T & U;
                if (CONN == 26) {
                    l = T & (U << 1);
                    r = T & (U >> 1);
                } else if (j < 2) {
                    l = (t0 & (a0 << 1)) | (t1 & (a1 << 1));
                    r = (t0 & (a0 >> 1)) | (t1 & (a1 >> 1));
                }
            }
            q = pair_requests(st, l, r, sh.M[k], sh.S[k], sh.E[k], sh.M[ku], sh.S[ku], sh.E[ku]);
        }
        sh.rf[tid] = q.f;
        if (CONN != 6) {
            sh.rl[tid] = q.l;
            sh.rr[tid] = q.r;
        }
    }
    // nodes: thread (bundle k, columns [8 q, 8 q + 8))
    const int k = tid >> 3, q = tid & 7;
    const uint64_t Ek = sh.E[k];
    const uint32_t e8 = (uint32_t)(Ek >> (8 * q)) & 0xFFu;
    const uint32_t first = (uint32_t)sh.base[k] + (uint32_t)__popcll(Ek & ((1ull << (8 * q)) - 1ull));
    sh.pre[tid] = (uint16_t)first;
    for (uint32_t s8 = (uint32_t)(sh.S[k] >> (8 * q)) & 0xFFu; s8; s8 &= s8 - 1u) {
        const uint32_t b = (uint32_t)__builtin_ctz(s8);
        const uint32_t n = first + (uint32_t)__builtin_popcount(e8 & ((1u << b) - 1u));
        sh.info[n] = (uint16_t)(((uint32_t)k << 6) | ((uint32_t)q << 3) | b);
        lds_st(&par[n], n);
    }
    __syncthreads();
    // hooks, neighbour by neighbour (the four neighbours' pairs in one loop,
    // so that their atomics are in flight together, measured 2.3 us slower)
#pragma unroll
    for (int j = 0; j < G::NJ; ++j) {
        // columns of the pairs: shared ones, then the two kinds of corners
        uint32_t m = ((const uint8_t *)sh.rf)[(j * G::NB + k) * 8 + q];
        if (CONN == 26 || (CONN == 18 && j < 2))
            m |= ((uint32_t)((const uint8_t *)sh.rl)[(j * G::NB + k) * 8 + q] << 8) |
                 ((uint32_t)((const uint8_t *)sh.rr)[(j * G::NB + k) * 8 + q] << 16);
        const int ku = max(0, k - (j == 0 ? 1 : j == 1 ? 8 : j == 2 ? 9 : 7));  // m is 0 without that neighbour
        const uint32_t ufirst = sh.pre[ku * 8 + q], ue8 = ((const uint8_t *)sh.E)[ku * 8 + q];
        for (; m; m &= m - 1u) {
            const uint32_t p = (uint32_t)__builtin_ctz(m), b = p & 7u;
            const uint32_t below = (1u << b) - 1u;
            const uint32_t lo = first + (uint32_t)__builtin_popcount(e8 & below);
            uint32_t up = ufirst + (uint32_t)__builtin_popcount(ue8 & below);
            if (CONN != 6) {
                if (p >= 16u) up += (ue8 >> b) & 1u;  // the interval that starts right of b
                else if (p >= 8u) up -= 1u;           // the one that ends left of b
            }
            const uint32_t old = atomicMin(&par[lo], up);
            if (old != lo && old != up) {
                // hooked before: its two upper intervals are to be joined
                const uint32_t i = atomicAdd(&sh.joins, 1u);
                if (i < (uint32_t)G::NODES) sh.mp[i] = old | (up << 16);
                else lds_link(par, old, up);
            }
        }
    }
    __syncthreads();
    const uint32_t nodes = sh.nodes, joins = min(sh.joins, (uint32_t)G::NODES);
    // an interval's smallest voxel: the first one of its first row that has any
    auto smallest = [&](uint32_t n) {
        const uint32_t in = sh.info[n];
        const int kn = (int)(in >> 6), s = (int)(in & 63u);
        const int e = s + __builtin_ctzll(sh.E[kn] >> s);
        const uint64_t I = (~0ull >> (63 - e)) & (~0ull << s);
        uint64_t w[4];
        rows_of(kn, w);
        uint64_t hit = 0ull;
        int i = G::BR;
#pragma unroll
        for (int c = G::BR - 1; c >= 0; --c) {
            if (w[c] & I) {
                hit = w[c] & I;
                i = c;
            }
        }
        return ((uint32_t)(bundle_row<CONN>(kn) + bundle_row_offset(i)) << 6) | (uint32_t)__builtin_ctzll(hit);
    };
    // every node finds the root of its tree of hooks; such a root's entry
    // becomes kPixel | its smallest voxel, which walks and joins still take
    // for a root's
    compress_nodes<256>(par, nodes, [&](uint32_t n) { lds_st(&par[n], kPixel | smallest(n)); });
    __syncthreads();
    for (uint32_t i = (uint32_t)tid; i < joins; i += 256u) {
        const uint32_t e = sh.mp[i];
        lds_link(par, parent_of(par, e & 0xFFFFu), parent_of(par, e >> 16));
    }
    __syncthreads();
    // every node finds its root.  The component's smallest voxel lies in an
    // interval of the root's slices (nodes are numbered slice by slice), as
    // does the one entered so far; intervals whose rows begin after that one
    // hold no better.  (In passes of their own over an array of their own,
    // 256^3 voxels: 23.0 us, so 22.5; 97 x 251 x 203, 6-connectivity: 10.5 and
    // 10.1.)
    constexpr uint32_t kSliceRows = kTY * G::BR / 2;
    compress_nodes<256>(par, nodes, [](uint32_t) {}, [&](uint32_t n, uint32_t r, uint32_t e) {
        const uint32_t in = sh.info[n], row = (e & (kPixel - 1u)) >> 6;
        if (in >> 9 == row / kSliceRows && (uint32_t)bundle_row<CONN>((int)(in >> 6)) <= row) {
            const uint32_t p = kPixel | smallest(n);
            if (p < e) atomicMin(&par[r], p);
        }
    });
    __syncthreads();
    auto index_of = [&](uint32_t row, uint32_t col) {
        return ((uint32_t)(z0 + (int)(row / kTY)) * (uint32_t)v.H + (uint32_t)(y0 + (int)(row % kTY))) *
                   (uint32_t)v.W + (uint32_t)x0 + col;
    };
    // the local roots' forest entries; mp[] takes every node's label
    for (uint32_t n = (uint32_t)tid; n < nodes; n += 256u) {
        uint32_t e = lds_ld(&par[n]);
        const bool root = e >= kPixel;
        if (!root) e = lds_ld(&par[e]);
        const uint32_t pos = e & (kPixel - 1u);
        const uint32_t g = index_of(pos >> 6, pos & 63u);
        if (root) v.labels[g] = g + 1u;
        sh.mp[n] = g + 1u;
    }
    __syncthreads();
    // column labels
#pragma unroll
    for (int i = 0; i < G::NB / 4; ++i) {
        const int kn = wave * (G::NB / 4) + i, row = bundle_row<CONN>(kn);
        if (y0 + row % kTY >= v.H || z0 + row / kTY >= v.D) continue;  // wave-uniform
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.base[kn]) + bits_below(uniform64(sh.E[kn]));
        const uint32_t val = lane_in(uniform64(sh.M[kn])) ? lds_ld(&sh.mp[n]) : 0u;
        if (x0 + lane < v.W) v.labels[index_of((uint32_t)row, (uint32_t)lane)] = val;
    }
}

// Boundary analysis of one tile: its low z, y and x faces against the faces
// they look at.  A pair of touching voxels is examined once: pairs whose
// step aside leaves the tile's own rows belong to the z face, then to the y
// face.
//
// The z and y faces are taken as joins of lines along x (one lane per join,
// 64-bit masks): under 18 and 26 a bundle's two own rows against the two they
// look at, and single rows across the corners between bundles; under 6 the
// straight pairs only.  A pair across a corner is left out where a foreground
// voxel lies between its two (one that touches both by a shorter step): both
// of that voxel's pairs are joined, here or by the local merge.  Touching
// columns are reduced to one per pair of runs (pair_requests), their column
// labels to the tile's distinct pairs (a hash table in LDS), and these are
// joined all at once.  Bound by the latency of its loads and of the global
// union-find.  256^3 voxels at p = 0.3, 26-connectivity: 28 us; testing every
// face voxel against its thirteen earlier neighbours took 101.
template <int CONN>
struct K2Lds3d {
    static constexpr int TZ = Geo<CONN>::TZ;
    static constexpr int LS = kTileW + 2;  // a line of column labels: columns -1 .. 64
    static constexpr int SLOTS = 256, LIST = 256;
    // rows of masks: z face (own 16, facing -1 .. 16), y face (own, facing)
    static constexpr int MZT = 0, MZU = kTY + 1, MYT = 2 * kTY + 2, MYU = MYT + 8, MROWS = MYU + 8;
    // lines of column labels of the bundles there: z face (own 8, facing
    // -1 .. 8), y face (own 4, facing 4)
    static constexpr int LZT = 0, LZU = 9, LYT = 18, LYU = 22, LINES = 26;
    static constexpr int NJ = CONN == 6 ? 12 : 34;
    unsigned long long tab[SLOTS], list[LIST];
    uint64_t m[MROWS];
    uint64_t x[2][2];         // x face: facing / own voxels (z, y), 64 per word
    uint64_t f[NJ], l[NJ], r[NJ];
    uint32_t lab[LINES * LS];
    uint32_t xl[2][32];       // x face: column labels of the facing / own bundles
    uint8_t el[MROWS], er[MROWS];  // a facing row's voxels in columns -1 and 64
    uint32_t count;
};

// Rows and lines of join j: the own rows t0 (and t1), the rows they look at
// u0 (and u1), for a join across a corner the row u0's side neighbour that t0
// looks at (us) and t0's own side neighbour (tp); -1: none.
struct Join3d { int t0, t1, u0, u1, us, tp, lt, lu; };

template <int CONN>
__device__ __forceinline__ Join3d join_of(int j) {
    using L = K2Lds3d<CONN>;
    if (CONN == 6) {
        if (j < 8) return {L::MZT + 2 * j, L::MZT + 2 * j + 1, L::MZU + 2 * j, L::MZU + 2 * j + 1, -1, -1, L::LZT + j, L::LZU + j};
        return {L::MYT + j - 8, -1, L::MYU + j - 8, -1, -1, -1, L::LYT + j - 8, L::LYU + j - 8};
    }
    const bool z = j < 24;
    // which of the face's bundles, and straight (0) or across the corner
    // before (1) or after (2) it
    const int b = z ? j & 7 : j < 28 ? j - 24 : j < 31 ? j - 27 : j - 31;
    const int kind = z ? j >> 3 : j < 28 ? 0 : j < 31 ? 1 : 2;
    const int t = (z ? L::MZT : L::MYT) + 2 * b, u = (z ? L::MZU : L::MYU) + 2 * b;
    const int lt = (z ? L::LZT : L::LYT) + b, lu = (z ? L::LZU : L::LYU) + b;
    if (kind == 0) return {t, t + 1, u, u + 1, -1, -1, lt, lu};
    if (kind == 1) return {t, -1, u - 1, -1, u, b > 0 ? t - 1 : -1, lt, lu - 1};
    return {t + 1, -1, u + 2, -1, u + 1, b < (z ? 7 : 3) ? t + 2 : -1, lt, lu + 1};
}

template <int CONN>
__global__ void __launch_bounds__(256) k2_boundary3d(Vol v) {
    using G = Geo<CONN>;
    using Lds = K2Lds3d<CONN>;
    constexpr bool DIAG = CONN != 6;
    constexpr int LS = Lds::LS;
    __shared__ Lds sh;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tx, ty, tz;
    tile_of(v, xcd_remap(blockIdx.x, gridDim.x), tx, ty, tz);
    const int x0 = tx * kTileW, y0 = ty * kTY, z0 = tz * G::TZ;
    const uint32_t W = (uint32_t)v.W, HW = (uint32_t)v.H * W;
    auto inside = [&](int z, int y, int x) {
        return (uint32_t)z < (uint32_t)v.D && (uint32_t)y < (uint32_t)v.H && (uint32_t)x < W;
    };
    auto voxel = [&](int z, int y, int x) { return v.vol + (int64_t)z * v.pitch_z + (int64_t)y * v.pitch_y + x; };
    // column label of the bundle of row (z, y), 0 outside the volume
    auto column = [&](int z, int y, int x) {
        if (!inside(z, y, x)) return 0u;
        return v.labels[(uint32_t)(CONN == 6 ? z : z & ~1) * HW + (uint32_t)(y & ~1) * W + (uint32_t)x];
    };
    // volume row of a row of masks (facing rows look out of the tile), and
    // whether it is needed
    auto row_of = [&](int r, int &z, int &y) {
        if (r < Lds::MYT) {
            z = r < Lds::MZU - 1 ? z0 : z0 - 1;
            y = y0 + (r < Lds::MZU - 1 ? r : r - Lds::MZU);
            return tz > 0;
        }
        const int i = r < Lds::MYU ? r - Lds::MYT : r - Lds::MYU;
        z = z0 + i;
        y = r < Lds::MYU ? y0 : y0 - 1;
        return ty > 0 && i < G::TZ;
    };
    sh.tab[tid] = 0ull;
    static_assert(Lds::SLOTS == 256 && Lds::MROWS * 4 <= 200, "one table slot and at most one load per thread");
    if (tid == 0) sh.count = 0u;
    if (tid < Lds::MROWS * 4) {
        int z, y;
        const bool need = row_of(tid >> 2, z, y);
        uint32_t m = 0u;
        if (need && inside(z, y, x0)) m = nonzero_bytes16(load_row16(voxel(z, y, 0), x0 + (tid & 3) * 16, v.W));
        ((uint16_t *)sh.m)[tid] = (uint16_t)m;
    } else if (DIAG && tid >= 200 && tid < 252) {
        const int i = (tid - 200) >> 1, r = i < kTY + 2 ? Lds::MZU - 1 + i : Lds::MYU + i - (kTY + 2);
        const int x = (tid & 1) ? x0 + kTileW : x0 - 1;
        int z, y;
        const bool need = row_of(r, z, y);
        const uint8_t b = need && inside(z, y, x) && *voxel(z, y, x) ? 1 : 0;
        if (tid & 1) sh.er[r] = b;
        else sh.el[r] = b;
    }
#pragma unroll
    for (int i = 0; i < (Lds::LINES + 3) / 4; ++i) {
        const int l = wave + 4 * i;
        // line -> (z, y) of its bundle; the facing ones of the z face start
        // one bundle before the tile
        const bool zf = l < Lds::LYT;
        const int b = l < Lds::LZU - 1 ? l : zf ? l - Lds::LZU : l < Lds::LYU ? l - Lds::LYT : l - Lds::LYU;
        const int z = zf ? (l < Lds::LZU - 1 ? z0 : z0 - 1) : z0 + (CONN == 6 ? b : 2 * b);
        const int y = zf ? y0 + 2 * b : l < Lds::LYU ? y0 : y0 - 1;
        if (l < Lds::LINES && (zf ? tz > 0 : ty > 0)) {  // wave-uniform
            sh.lab[l * LS + 1 + lane] = column(z, y, x0 + lane);
            if (DIAG && (lane == 0 || lane == 63)) {
                const int c = lane == 0 ? -1 : kTileW;
                sh.lab[l * LS + 1 + c] = column(z, y, x0 + c);
            }
        }
    }
    if (tx > 0) {
        const int z = z0 + tid / kTY, y = y0 + tid % kTY;
        const bool in = tid < G::ROWS && inside(z, y, x0);
        uint8_t b[2] = {0, 0};
        if (in) __builtin_memcpy(b, voxel(z, y, x0 - 1), 2);
        const uint64_t xu = __ballot(b[0] != 0), xt = __ballot(b[1] != 0);
        if (wave < G::ROWS / 64 && lane == 0) {
            sh.x[0][wave] = xu;
            sh.x[1][wave] = xt;
        }
        if (tid >= 192) {
            const int k = tid & 31, r = bundle_row<CONN>(k), s = (tid >> 5) & 1;
            sh.xl[s][k] = column(z0 + r / kTY, y0 + r % kTY, x0 - 1 + s);
        }
    }
    __syncthreads();
    // touching pairs of runs, a lane per join
    if (tid < Lds::NJ) {
        const Join3d j = join_of<CONN>(tid);
        const uint64_t t0 = sh.m[j.t0], t1 = j.t1 >= 0 ? sh.m[j.t1] : 0ull;
        const uint64_t u0 = sh.m[j.u0], u1 = j.u1 >= 0 ? sh.m[j.u1] : 0ull;
        const uint64_t T = t0 | t1, U = u0 | u1;
        uint64_t st = T & U, l = 0ull, r = 0ull;
        uint64_t S = T & ~(T << 1), Su = U & ~(U << 1);
        if (CONN == 6) {
            st = (t0 & u0) | (t1 & u1);
            S = band_starts<false>(t0, t1);
            Su = band_starts<false>(u0, u1);
        } else {
            auto left = [&](uint64_t w, int row) { return (w << 1) | (uint64_t)sh.el[row]; };
            auto right = [&](uint64_t w, int row) { return (w >> 1) | ((uint64_t)sh.er[row] << 63); };
            if (j.us < 0) {
                // diagonal steps stay in one row under 18-connectivity
                const uint64_t l0 = left(u0, j.u0), l1 = left(u1, j.u1), r0 = right(u0, j.u0), r1 = right(u1, j.u1);
                l = CONN == 26 ? T & (l0 | l1) : (t0 & l0) | (t1 & l1);
                r = CONN == 26 ? T & (r0 | r1) : (t0 & r0) | (t1 & r1);
            } else {
                const uint64_t b = sh.m[j.us] | (j.tp >= 0 ? sh.m[j.tp] : 0ull);  // voxels between
                st &= ~b;
                if (CONN == 26) {
                    l = T & left(u0, j.u0) & ~(b | (b << 1));
                    r = T & right(u0, j.u0) & ~(b | (b >> 1));
                }
            }
        }
        const PairRequests q = pair_requests(st, l, r, T, S, band_ends(T, S), U, Su, band_ends(U, Su));
        sh.f[tid] = q.f;
        sh.l[tid] = q.l;
        sh.r[tid] = q.r;
    }
    __syncthreads();
    auto ask = [&](uint32_t a, uint32_t b) {
        const unsigned long long key = ((unsigned long long)a << 32) | b;
        uint32_t h = ((a * 2654435761u) ^ (b * 2246822519u)) >> 24;  // 8 bits
        for (int probe = 0; probe < 4; ++probe) {
            const unsigned long long old = atomicCAS(&sh.tab[h], 0ull, key);
            if (old == key) return;
            if (old == 0ull) break;
            h = (h + 1u) & (uint32_t)(Lds::SLOTS - 1);
        }
        const uint32_t i = atomicAdd(&sh.count, 1u);
        if (i < (uint32_t)Lds::LIST) sh.list[i] = key;
        else g_union(v.labels, v.n, a - 1u, b - 1u);
    };
    // eight columns of one join per thread
    for (int i = tid; i < Lds::NJ * 8; i += 256) {
        const int c = i >> 3, q = i & 7;
        const Join3d j = join_of<CONN>(c);
        if (!(j.lt < Lds::LYT ? tz > 0 : ty > 0)) continue;
        uint32_t m = ((const uint8_t *)sh.f)[i];
        if (DIAG) m |= ((uint32_t)((const uint8_t *)sh.l)[i] << 8) | ((uint32_t)((const uint8_t *)sh.r)[i] << 16);
        const uint32_t *lt = &sh.lab[j.lt * LS + 1 + 8 * q], *lu = &sh.lab[j.lu * LS + 1 + 8 * q];
        for (; m; m &= m - 1u) {
            const int p = __builtin_ctz(m), b = p & 7;
            ask(lt[b], lu[b + (p >= 16 ? 1 : p >= 8 ? -1 : 0)]);
        }
    }
    // the x face by bundles, on the wavefront that has no second join
    if (tx > 0 && tid >= 192 && tid < 224) {
        const int k = tid & 31, by = k & 7, bz = k >> 3;
        // a bundle's voxels in the column: bit i as its row i
        auto rows = [&](int side, int kk) {
            const int r = bundle_row<CONN>(kk);
            const uint32_t w = (uint32_t)(sh.x[side][r >> 6] >> (r & 63));
            return CONN == 6 ? w & 3u : (w & 3u) | ((w >> 14) & 12u);
        };
        const uint32_t t = rows(1, k), a = sh.xl[1][k];
        if (CONN == 6) {
            if (t & rows(0, k)) ask(a, sh.xl[0][k]);
        } else if (t) {
            uint32_t touching = 0u;  // bit 3 (dz + 1) + dy + 1
#pragma unroll
            for (int dz = -1; dz <= 1; ++dz) {
#pragma unroll
                for (int dy = -1; dy <= 1; ++dy) {
                    const int ny = by + dy, nz = bz + dz, kk = k + 8 * dz + dy;
                    if (ny < 0 || ny > 7 || nz < 0 || nz > 3) continue;
                    const uint32_t u = rows(0, kk);
                    bool touch = false;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
#pragma unroll
                        for (int o = 0; o < 4; ++o) {
                            // steps from own row i to the neighbour's row o
                            const int sy = 2 * dy + (o & 1) - (i & 1), sz = 2 * dz + (o >> 1) - (i >> 1);
                            if (sy < -1 || sy > 1 || sz < -1 || sz > 1) continue;
                            if (CONN == 18 && sy != 0 && sz != 0) continue;
                            touch = touch || ((t >> i) & (u >> o) & 1u);
                        }
                    }
                    if (touch) touching |= 1u << (3 * dz + dy + 4);
                }
            }
            for (; touching; touching &= touching - 1u) {
                const int d = __builtin_ctz(touching);
                ask(a, sh.xl[0][k + 8 * (d / 3 - 1) + d % 3 - 1]);
            }
        }
    }
    __syncthreads();
    const uint32_t n = min(sh.count, (uint32_t)Lds::LIST);
    for (uint32_t i = (uint32_t)tid; i < n; i += 256u)
        g_union(v.labels, v.n, (uint32_t)(sh.list[i] >> 32) - 1u, (uint32_t)sh.list[i] - 1u);
}

// Link of one tile: wavefront w resolves the column labels of bundles
// 8 w .. 8 w + 7 and stores the labels of their rows.  Its time is the volume
// (1 byte a voxel) and the column labels (1) read and the labels (4) written:
// 22 us for 256^3 voxels; with a label stored and reread for every voxel 43.
template <int CONN>
__global__ void __launch_bounds__(256, 8) k3_link3d(Vol v) {
    using G = Geo<CONN>;
    constexpr int BPW = G::NB / 4;
    __shared__ uint64_t msk[G::ROWS];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tx, ty, tz;
    tile_of(v, xcd_remap(blockIdx.x, gridDim.x), tx, ty, tz);
    const int x0 = tx * kTileW, y0 = ty * kTY, z0 = tz * G::TZ;
    load_masks<CONN>(v, x0, y0, z0, msk);
    __syncthreads();
    // the tile's row r starts at org[line(r)]
    uint32_t *org = v.labels + (((uint64_t)z0 * v.H + y0) * v.W + x0);
    auto line = [&](int r) { return ((uint64_t)(r / kTY) * v.H + r % kTY) * v.W; };
    auto rows_of = [&](int k, uint64_t (&w)[4]) {
        const uint64_t *m = &msk[bundle_row<CONN>(k)];
        w[0] = uniform64(m[0]);
        w[1] = uniform64(m[1]);
        w[2] = CONN == 6 ? 0ull : uniform64(m[kTY]);
        w[3] = CONN == 6 ? 0ull : uniform64(m[kTY + 1]);
    };
    const bool full = x0 + kTileW <= v.W && y0 + kTY <= v.H && z0 + G::TZ <= v.D;
    const bool xin = x0 + lane < v.W;
    constexpr int BP = 4;  // bundles whose walks overlap
#pragma unroll 1
    for (int k0 = wave * BPW; k0 < (wave + 1) * BPW; k0 += BP) {
        uint32_t g[BP], p[BP];
#pragma unroll
        for (int i = 0; i < BP; ++i) {
            uint64_t w[4];
            rows_of(k0 + i, w);
            g[i] = lane_in(w[0] | w[1] | w[2] | w[3]) ? org[line(bundle_row<CONN>(k0 + i)) + lane] : 0u;
        }
        // first step of every walk; most local roots are roots or next to one
#pragma unroll
        for (int i = 0; i < BP; ++i) p[i] = g[i] ? v.labels[g[i] - 1u] : 0u;
#pragma unroll
        for (int i = 0; i < BP; ++i) {
            uint64_t w[4];
            rows_of(k0 + i, w);
            uint32_t f = p[i];
            if (p[i] < g[i]) f = g_root(v.labels, p[i] - 1u) + 1u;
#pragma unroll
            for (int c = 0; c < G::BR; ++c) {
                const int r = bundle_row<CONN>(k0 + i) + bundle_row_offset(c);
                if (full || (y0 + r % kTY < v.H && z0 + r / kTY < v.D && xin))
                    __builtin_nontemporal_store(lane_in(w[c]) ? f : 0u, org + line(r) + lane);
            }
        }
    }
}

}  // namespace

}  // namespace ccl

using namespace ccl;

extern "C" int ccl_label_3d(const uint8_t *vol, int32_t D, int32_t H, int32_t W, int64_t pitch_y,
                            int64_t pitch_z, int32_t connectivity, uint32_t *labels, void *stream) {
    if (!vol || !labels || D <= 0 || H <= 0 || W <= 0) return CCL_ERR_INVALID_ARG;
    if (pitch_y < (int64_t)W || pitch_z < (int64_t)H * pitch_y) return CCL_ERR_INVALID_ARG;
    if (connectivity != 6 && connectivity != 18 && connectivity != 26) return CCL_ERR_UNSUPPORTED;
    const uint64_t n = (uint64_t)D * (uint64_t)H * (uint64_t)W;
    if (n > 0xFFFFFFFFull) return CCL_ERR_TOO_LARGE;
    const unsigned __int128 vol_bytes = (unsigned __int128)(D - 1) * (uint64_t)pitch_z +
                                        (unsigned __int128)(H - 1) * (uint64_t)pitch_y + (uint64_t)W;
    if (byte_ranges_overlap(vol, vol_bytes, labels, (unsigned __int128)n * 4u)) return CCL_ERR_INVALID_ARG;
    Vol v;
    v.vol = vol;
    v.labels = labels;
    v.pitch_y = pitch_y;
    v.pitch_z = pitch_z;
    v.D = D;
    v.H = H;
    v.W = W;
    v.tilesX = (W + kTileW - 1) / kTileW;
    v.tilesY = (H + kTY - 1) / kTY;
    const int tz = connectivity == 6 ? Geo<6>::TZ : Geo<26>::TZ;
    v.tilesZ = (D + tz - 1) / tz;
    v.n = (uint32_t)n;
    const uint64_t tiles = (uint64_t)v.tilesX * v.tilesY * v.tilesZ;
    // the volumes accepted are those of at most 2^31 - 1 tile rows, counted
    // in tiles of 16 rows and 4 slices
    if ((uint64_t)v.tilesX * v.tilesY * (uint64_t)((D + 3) / 4) * 64u > 0x7FFFFFFFull) return CCL_ERR_TOO_LARGE;
    hipStream_t s = (hipStream_t)stream;
    auto launch = [&](auto k1, auto k2, auto k3) {
        hipLaunchKernelGGL(k1, dim3((uint32_t)tiles), dim3(256), 0, s, v);
        if (tiles > 1) hipLaunchKernelGGL(k2, dim3((uint32_t)tiles), dim3(256), 0, s, v);
        hipLaunchKernelGGL(k3, dim3((uint32_t)tiles), dim3(256), 0, s, v);
    };
    switch (connectivity) {
        case 6: launch(k1_local_merge3d<6>, k2_boundary3d<6>, k3_link3d<6>); break;
        case 18: launch(k1_local_merge3d<18>, k2_boundary3d<18>, k3_link3d<18>); break;
        default: launch(k1_local_merge3d<26>, k2_boundary3d<26>, k3_link3d<26>); break;
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e);
    return CCL_OK;
}
