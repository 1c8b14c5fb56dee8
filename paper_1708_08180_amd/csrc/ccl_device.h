// Device-side building blocks of the three labeling phases (gfx950, wave64).
//
// Tile model.  A tile is 64 pixels wide -- one lane of a 64-wide wavefront
// per column -- and TH rows tall (TH in {16, 32, 64, 128}).  A workgroup of NW
// wavefronts owns one tile at a time.  The local merge spreads a tile's bands,
// parts of eight columns and nodes over all its threads; in the link wavefront
// w owns rows [w*RPW, (w+1)*RPW) with RPW = TH / NW.  A tile row is a 64-bit
// foreground mask, so the paper's row scan plus row-column unification (Sec. II-A-2) collapses
// to mask arithmetic: binary labeling takes two rows at a time, and the
// components of such a band are column intervals found from its two masks;
// those intervals are the union-find nodes, joined with the intervals of the
// band above that they touch (LineForest).  Equal-value labeling keeps one
// node per run of equal values in a row.
//
// Forest encoding in global memory.  labels[p] holds 1 + parent(p); a root r
// holds r + 1 and background holds 0.  The final output is therefore itself a
// fully compressed forest, so the link phase can overwrite entries in place
// while other tiles still walk the forest.
//
// Workspace per tile, written by the local merge:
//   masks[...]      top-row, bottom-row, left-column, right-column foreground
//                   masks (boundary analysis; mask_words)
//   roots[...]      global raster index of the tile-local root of every cell
//                   on those four edges (boundary analysis)
//   rowmask[...]    the 64-bit foreground mask of every tile row, then per
//                   row the mask of the local root pixels whose component
//                   touches a shared tile edge, then (binary labeling) every
//                   two-row band's interval ends and first node (link)
//   slots[...]      one 16-bit record per union-find node (binary: per band
//                   interval; equal-value: per run, 64 slots per row): the
//                   tile-local pixel of the node's local root (link)
// Every root of an edge-touching component is also seeded in the forest,
// labels[root] = root + 1, before the boundary analysis runs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ccl {

constexpr int kTileW = 64;               // tile width == wavefront width
constexpr uint32_t kNone = 0xFFFFFFFFu;  // "no node"

// Edge masks of a tile: the top and bottom rows (one word each), then the
// left and the right column, one bit per row (one word per 64 rows each).
enum { kMaskTop = 0, kMaskBottom = 1, kMaskLeft = 2 };
__host__ __device__ constexpr int col_words(int th) { return (th + 63) / 64; }
__host__ __device__ constexpr int mask_words(int th) { return 2 + 2 * col_words(th); }
__host__ __device__ constexpr int mask_right(int th) { return kMaskLeft + col_words(th); }

// Run records per tile row: a 64-pixel row has at most 32 foreground runs,
// and at most 64 equal-value runs.
template <bool EQ>
__host__ __device__ constexpr int slots_per_row() { return EQ ? 64 : 32; }
constexpr int kSlotsPerRow = slots_per_row<false>();

__host__ __device__ constexpr int roots_per_tile(int th) { return 2 * kTileW + 2 * th; }
// 64-bit words per tile of the row data: TH row masks, TH edge-root masks,
// TH / 2 band interval-end masks, then TH / 2 16-bit band bases (first
// record of every band)
__host__ __device__ constexpr int rowmask_words(int th) { return 2 * th + th / 2 + th / 8; }
__host__ __device__ constexpr int rowmask_ends(int th) { return 2 * th; }
__host__ __device__ constexpr int rowmask_bases(int th) { return 2 * th + th / 2; }
__host__ __device__ constexpr int roots_top(int) { return 0; }
__host__ __device__ constexpr int roots_bottom(int) { return kTileW; }
__host__ __device__ constexpr int roots_left(int) { return 2 * kTileW; }
__host__ __device__ constexpr int roots_right(int th) { return 2 * kTileW + th; }

// One image as the kernels see it.
struct ImgView {
    const uint8_t *img;
    uint32_t *labels;
    uint64_t *masks;    // [tiles][mask_words(TH)]
    uint32_t *roots;    // [tiles][roots_per_tile(TH)]
    uint64_t *rowmask;  // [tiles][rowmask_words(TH)]: row masks, edge-root masks, row bases
    uint16_t *slots;    // [tiles][TH][slots_per_row]
    int64_t pitch;
    int32_t H, W;
    int32_t tilesX, tilesY;
    uint32_t n;         // H * W (<= 2^32 - 1)
};

// One image of a batch as the batch kernels see it (device descriptor).
// Tiles of all images are numbered consecutively: image i owns global tiles
// [tile_base, tile_base + tilesX*tilesY), and its workspace lives at those
// tile offsets.
struct BatchImage {
    const uint8_t *img;
    uint32_t *labels;
    int64_t pitch;
    int32_t H, W;
    int32_t tilesX, tilesY;
    uint32_t n;
    uint32_t tile_base;
};

// Workspace of a batch context, indexed by global tile.  tile_img[g] is the
// image that owns global tile g (written by the local merge, read by the
// two later phases).
struct BatchWs {
    uint64_t *masks;
    uint32_t *roots;
    uint64_t *rowmask;
    uint16_t *slots;
    uint32_t *tile_img;
};

// Kernel argument of the three batch kernels (one call).  tile_base holds
// the n images' first global tiles (ascending) and coarse every 64th of
// them, so the local merge finds a tile's image with two coalesced reads.
struct BatchArgs {
    const BatchImage *descs;
    const uint32_t *tile_base;
    const uint32_t *coarse;
    BatchWs w;
    uint32_t n, tiles;
};

// ---------------------------------------------------------- launch helpers

// Consecutive workgroup ids are spread round-robin over the 8 XCDs; remap
// them so that each XCD works on one contiguous run of tiles and
// horizontally adjacent tiles (which share image cache lines) meet in the
// same L2.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t bid, uint32_t nb) {
    constexpr uint32_t X = 8;
    const uint32_t q = nb / X, r = nb % X;
    const uint32_t xcd = bid % X, i = bid / X;
    return xcd * q + (xcd < r ? xcd : r) + i;
}

// ------------------------------------------------------------------ helpers

// Image that owns global tile g: the last image whose tile_base is <= g,
// i.e. the number of bases <= g minus one.  First among the coarse bases
// (every 64th image), then among the 64 images of that group; each lane
// compares one base.
__device__ __forceinline__ uint32_t batch_image_of(const BatchArgs &a, uint32_t g) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t nc = (a.n + 63u) >> 6;
    uint32_t cnt = 0;
    for (uint32_t j = 0; j < nc; j += 64) {
        const uint32_t k = j + lane;
        cnt += (uint32_t)__popcll(__ballot(k < nc && a.coarse[k] <= g));
    }
    const uint32_t k = ((cnt - 1u) << 6) + lane;
    return ((cnt - 1u) << 6) + (uint32_t)__popcll(__ballot(k < a.n && a.tile_base[k] <= g)) - 1u;
}


__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

__device__ __forceinline__ int bit(uint64_t m, int j) { return (int)((m >> j) & 1ull); }

template <typename T>
__device__ __forceinline__ T lds_ld(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <typename T>
__device__ __forceinline__ void lds_st(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Global forest accessors for the concurrent boundary phase.  Links are
// made with agent-scope atomicMin, which acts on the one coherent copy.
// Finds read through the caches (g_ld): a read may return an older parent
// than the current one, but the forest only ever gets coarser -- a parent
// is only replaced by one of its own ancestors, always a smaller index --
// so an old parent is still an ancestor, every walk still ends, and a node
// taken for a root by mistake is caught by the value the linking atomicMin
// returns (the link is then retried from there).  Reading the hot roots of
// large components from the caches instead of memory is what keeps the
// phase from serializing on them.
__device__ __forceinline__ uint32_t g_ld(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t g_min(uint32_t *p, uint32_t v) {
    return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------- LDS union-find

// Every parent is strictly smaller than its child, so `p >= x` both detects
// a root (p == x) and stops on anything that is not a valid parent; every
// loop below therefore strictly decreases its index and always terminates.

// Join the trees of a and b (Sec. II-A-3), the larger index under the
// smaller, without finding the roots first: the atomicMin lowers the larger
// node's parent to the smaller node and returns the parent it had.  If that
// was the node itself, a root was linked and the join is done; otherwise the
// node is now the smaller one's child, its old parent still has to be joined
// to it, and the step repeats on that pair.  The larger index of the pair
// drops every step, so the walk ends; every parent only ever moves to a
// smaller node connected to it, so no concurrent link is lost.  Callers
// mostly pass roots, which makes this a single atomic.
__device__ __forceinline__ void lds_link(uint32_t *par, uint32_t a, uint32_t b) {
    while (a != b) {
        if (a > b) { const uint32_t t = a; a = b; b = t; }
        const uint32_t old = atomicMin(&par[b], a);
        if (old >= b) return;
        b = old;
    }
}

// ------------------------------------------------------ global union-find

// Find steps after which a join also points its starting nodes at the root.
constexpr uint32_t kLongWalk = 256u;

// Roots of a and b in the global forest, found together so that the loads
// of both walks are in flight at once.  Path halving: a node whose parent
// is not a root is pointed at its grandparent with an atomicMin, which can
// only lower a parent to an ancestor.  steps counts the loop's passes.
__device__ __forceinline__ void g_find2(uint32_t *L, uint32_t &a, uint32_t &b, uint32_t &steps) {
    // every step issues both walks' loads unconditionally (a root re-reads
    // its own entry), so the two loads are in flight together and the
    // wavefront waits once per step
    while (true) {
        ++steps;
        uint32_t pa = g_ld(&L[a]) - 1u, pb = g_ld(&L[b]) - 1u;
        bool ra = pa >= a, rb = pb >= b;
        if (ra && rb) return;
        pa = ra ? a : pa;
        pb = rb ? b : pb;
        const uint32_t ga = g_ld(&L[pa]) - 1u, gb = g_ld(&L[pb]) - 1u;
        if (!ra) {
            if (ga >= pa) {
                a = pa;
                ra = true;
            } else {
                g_min(&L[a], ga + 1u);
                a = ga;
            }
        }
        if (!rb) {
            if (gb >= pb) {
                b = pb;
                rb = true;
            } else {
                g_min(&L[b], gb + 1u);
                b = gb;
            }
        }
        if (ra && rb) return;
    }
}

// Link the trees of a and b, the larger root under the smaller (Sec. II-B).
// When the atomicMin shows that b stopped being a root meanwhile, the value
// it returns is b's new parent and the link is retried from there, so no
// concurrent link is lost.
//
// A join whose walks took many steps (a long chain, as a spiral or a
// serpentine builds across tiles) points both of its starting nodes straight
// at the final root, so the next join along the same chain starts next to
// the root instead of walking it again.  Path halving alone only halves such
// a chain per walk.  Joins that found their roots quickly skip this.
__device__ __forceinline__ void g_union(uint32_t *L, uint32_t n, uint32_t a, uint32_t b) {
    if (a >= n || b >= n) return;
    const uint32_t a0 = a, b0 = b;
    uint32_t steps = 0;
    while (true) {
        g_find2(L, a, b, steps);
        if (a == b) break;
        if (a > b) { const uint32_t t = a; a = b; b = t; }
        const uint32_t old = g_min(&L[b], a + 1u) - 1u;
        if (old >= b) break;
        b = old;
    }
    if (steps > kLongWalk) {
        g_min(&L[a0], a + 1u);
        g_min(&L[b0], a + 1u);
    }
}

// Merge requests of one wavefront: every lane holds NS (a, b) slots (b ==
// kNone: empty).  Along a tile edge most requests repeat the same pair of
// tile-local roots, so the distinct pairs are collected first (one per
// lane, at most 64 at a time) and then merged by all lanes concurrently
// with join(a, b) (a lane without a pair gets kNone for both).
template <int NS, class Union>
__device__ __forceinline__ void union_requests(const uint32_t (&A)[NS], const uint32_t (&B)[NS],
                                               Union &&join) {
    const int lane = (int)(threadIdx.x & 63);
    uint64_t pend[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) pend[s] = __ballot(B[s] != kNone);
    bool more = true;
    while (more) {  // rounds of up to 64 distinct pairs, one per lane
        more = false;
        uint32_t ma = kNone, mb = kNone;
        int cnt = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            while (pend[s] && cnt < 64) {
                const int lead = __builtin_ctzll(pend[s]);
                const uint32_t PA = (uint32_t)__builtin_amdgcn_readlane((int)A[s], lead);
                const uint32_t PB = (uint32_t)__builtin_amdgcn_readlane((int)B[s], lead);
                if (lane == cnt) {
                    ma = PA;
                    mb = PB;
                }
#pragma unroll
                for (int q = s; q < NS; ++q) pend[q] &= ~__ballot(A[q] == PA && B[q] == PB);
                ++cnt;
            }
            more = more || pend[s] != 0ull;
        }
        join(ma, mb);  // one call site: lanes without a pair return at once
    }
}

// Root of x once no link is made any more (link phase).  A long walk (a
// component threaded through many tiles, such as a one-pixel-wide spiral)
// then points every node it passed at the root, so the tiles that walk
// there later stop short; a short one writes nothing.  The stores are the
// final root, the value every other writer of those entries stores too.
__device__ __forceinline__ uint32_t g_root(uint32_t *L, uint32_t x0) {
    uint32_t x = x0, v = L[x] - 1u, steps = 0;
    while (v < x) {
        x = v;
        v = L[x] - 1u;
        ++steps;
    }
    if (steps > 8u) {
        uint32_t y = x0;
        while (y > x) {
            const uint32_t ny = L[y] - 1u;
            if (ny >= y) break;
            L[y] = x + 1u;
            y = ny;
        }
    }
    return x;
}

// ------------------------------------------------------ tile-local labeling

__device__ __forceinline__ uint32_t global_index(const ImgView &v, int tx, int ty, int th,
                                                 uint32_t l) {
    const uint64_t y = (uint64_t)ty * th + (l >> 6);
    const uint64_t x = (uint64_t)tx * kTileW + (l & 63u);
    return (uint32_t)(y * (uint64_t)v.W + x);
}

// Top bit of every nonzero byte of w.
__device__ __forceinline__ uint32_t nonzero_tops(uint32_t w) {
    return (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
}

// Bit i (i < 16) set iff byte i of the 16 is nonzero: the top bits, 128
// each, are weighted by 1, 2, 4 .. 128 in a byte dot product over two words.
__device__ __forceinline__ uint32_t nonzero_bytes16(uint4 b) {
    const uint32_t lo = __builtin_amdgcn_udot4(
        nonzero_tops(b.y), 0x80402010u, __builtin_amdgcn_udot4(nonzero_tops(b.x), 0x08040201u, 0u, false), false);
    const uint32_t hi = __builtin_amdgcn_udot4(
        nonzero_tops(b.w), 0x80402010u, __builtin_amdgcn_udot4(nonzero_tops(b.z), 0x08040201u, 0u, false), false);
    return (lo >> 7) | (hi << 1);
}

// Pixels [x, x + 16) of an image row of W bytes, zero past its end.  One
// 16-byte load wherever the row holds 16 bytes: of the chunk itself, or, for
// the chunk that the row's end cuts, of the row's last 16 bytes, shifted
// down.  Rows need no alignment: gfx950 serves a 16-byte global load at any
// byte address.  Byte loads for rows that are not 16-byte aligned bound the
// local merge of such an image: 3001 x 4099 with a pitch of 4137 bytes took
// 67.6 us a call with them and takes 52.5 with these.
__device__ __forceinline__ uint4 load_row16(const uint8_t *row, int x, int W) {
    uint4 b = make_uint4(0u, 0u, 0u, 0u);
    if (x >= W) return b;
    if (x + 16 <= W) {
        __builtin_memcpy(&b, row + x, 16);
        return b;
    }
    if (W >= 16) {
        uint64_t h[2];
        __builtin_memcpy(h, row + (W - 16), 16);
        const int sh = 8 * (x + 16 - W);  // 8 .. 120 bits
        const uint64_t lo = sh < 64 ? (h[0] >> sh) | (h[1] << (64 - sh)) : h[1] >> (sh & 63);
        const uint64_t hi = sh < 64 ? h[1] >> sh : 0ull;
        return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
    }
    uint64_t lo = 0ull, hi = 0ull;  // W < 16: the row's only chunk (x == 0)
#pragma unroll 1
    for (int i = W - 1; i >= 0; --i) {
        hi = (hi << 8) | (lo >> 56);
        lo = (lo << 8) | row[i];
    }
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// 16 pixels of one tile row: row `row` of tile (tx, ty), columns
// [16q, 16q + 16), zero outside the image.
template <class V>
__device__ __forceinline__ uint4 load_chunk(const V &v, int tx, int ty, int th, int row, int q) {
    const int y = ty * th + row;
    if (y >= v.H) return make_uint4(0u, 0u, 0u, 0u);
    return load_row16(v.img + (int64_t)y * v.pitch, tx * kTileW + q * 16, v.W);
}

// ------------------------------------------------------ masks and lanes

// Lane predicate from a wave-uniform 64-bit mask (no VALU work).
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Number of set bits of m strictly below this lane.
__device__ __forceinline__ uint32_t bits_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Value of lane-1 / lane+1 (whole-wave DPP shifts; lane 0 / 63 get `edge`).
__device__ __forceinline__ uint32_t from_left(uint32_t v, uint32_t edge) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t from_right(uint32_t v, uint32_t edge) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x130, 0xF, 0xF, false);
}

__device__ __forceinline__ uint64_t run_starts(uint64_t d) { return d & ~(d << 1); }

// Exclusive prefix sum over the 64 lanes of a wavefront; *total gets the
// sum of all lanes.  DPP row shifts scan each 16-lane row, then the last
// lane of row 0 / row 1 is broadcast into rows 1 and 3 / 2 and 3.
__device__ __forceinline__ uint32_t wave_exclusive_scan(uint32_t x, uint32_t *total) {
    uint32_t v = x;
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31
    *total = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    return v - x;
}

// A value every lane holds identically, moved to scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Lane k's value of x (k wave-uniform), in scalar registers.
__device__ __forceinline__ uint64_t lane_value64(uint64_t x, int k) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), k);
    return ((uint64_t)hi << 32) | lo;
}

// Which (lower run, upper run) pairs of two adjacent lines are merged, as
// lane masks over the lower line d with the upper line u: every pair of runs
// that touch is taken exactly once, by the leftmost lower cell adjacent to
// the upper run.  8-connectivity: PL = the upper run containing column j-1
// (only at a lower run start), PM = the upper run starting at j (only at a
// lower run start whose above-left is empty), PR = the upper run starting at
// j+1.  4-connectivity: PM = the upper run containing j, at the lower run
// start or where the upper run starts.  On a tile's top edge the upper line
// continues into the neighbouring tiles: xl (bit 0 only) is set when the
// cell above-left of column 0 is foreground, xr (bit 63 only) when the cell
// above-right of column 63 is; inside a tile both are 0.
struct PairMasks { uint64_t pl, pm, pr; };

template <bool CONN8>
__device__ __forceinline__ PairMasks pair_masks(uint64_t d, uint64_t u, uint64_t xl = 0,
                                                uint64_t xr = 0) {
    const uint64_t S = run_starts(d);
    PairMasks p;
    if (CONN8) {
        p.pl = S & ((u << 1) | xl);
        p.pm = S & u & ~(u << 1);
        p.pr = d & (((u >> 1) & ~u) | xr);
    } else {
        p.pl = 0;
        p.pm = d & u & (S | ~(u << 1));
        p.pr = 0;
    }
    return p;
}

// Which intervals of a lower line touch which intervals of an upper line,
// as one request per touching pair.  Inputs, bit j = column j:
//   st / l / r   the lower line's column j touches the upper line's column
//                j / j - 1 / j + 1;
//   M, S, E      the lower line's columns, and the first and last columns of
//                its intervals (maximal segments; two of them may be adjacent);
//   Mu, Su, Eu   the same of the upper line.
// Result: f has one column per pair of intervals that share a column and
// touch (anywhere): the pair is the two intervals of that column.  l / r have
// the columns j where the lower interval that starts / ends at j touches the
// upper interval that ends at j - 1 / starts at j + 1 and shares no column
// with it.
struct PairRequests { uint64_t f, l, r; };

__host__ __device__ __forceinline__ PairRequests pair_requests(uint64_t st, uint64_t l, uint64_t r, uint64_t M,
                                                               uint64_t S, uint64_t E, uint64_t Mu, uint64_t Su,
                                                               uint64_t Eu) {
    // a diagonal touch of two intervals that share a column is a touch at
    // such a column: at j when the upper interval goes on to j, at the
    // neighbouring column when the lower interval goes on to it
    const uint64_t upl = Mu & ~Su;         // the upper intervals of j - 1 and j are one
    const uint64_t upr = Mu & ~(Su >> 1);  // those of j and j + 1 are one (where j + 1 is in one)
    const uint64_t c = st | (l & upl) | ((l & ~S) >> 1) | (r & upr) | ((r & ~E) << 1);
    // first touching column of every segment of columns shared by one pair:
    // adding the segments' first columns to their untouched columns carries
    // through those up to the first touching one (a carry never leaves its
    // segment, whose last column is left clear)
    const uint64_t D = M & Mu;
    const uint64_t Sb = D & (~(D << 1) | S | Su);
    const uint64_t Eb = D & (~(D >> 1) | E | Eu);
    PairRequests q;
    q.f = ((D & ~c & ~Eb) + Sb) & c;
    q.l = l & S & ~upl;
    q.r = r & E & ~upr;
    return q;
}

// ------------------------------------------------- two-row band nodes
//
// The binary local merge takes the tile two rows at a time.  Inside such a
// band every connected component is one contiguous interval of columns:
// under 8-connectivity the intervals are the runs of t | b (t the band's top
// row, b its bottom row); under 4-connectivity they are those runs split
// wherever neither row continues across the column boundary.  So the row
// scan and the row-column unification of Sec. II-A-2 reduce to a few 64-bit
// operations per band, and the union-find of Sec. II-A-3 runs over intervals
// and over half as many steps as rows.
//
// Node n of a tile is its n-th interval in band order, left to right inside
// a band, so a component's root, its smallest node, lies in the component's
// first band.

// First column of every interval of the band (t above b).
template <bool CONN8>
__device__ __forceinline__ uint64_t band_starts(uint64_t t, uint64_t b) {
    const uint64_t m = t | b;
    uint64_t s = m & ~(m << 1);
    if (!CONN8) s |= m & (m << 1) & ~(t & (t << 1)) & ~(b & (b << 1));
    return s;
}

// Last column of every interval, from the band's columns m = t | b and the
// interval starts s.
__device__ __forceinline__ uint64_t band_ends(uint64_t m, uint64_t s) { return m & (~(m >> 1) | (s >> 1)); }

// Local union-find over the intervals of a tile's lines (two-row bands, or
// rows in equal-value labeling), whose nodes are numbered densely line by
// line.  Nothing in it follows the lines one after the other: every touching
// pair of intervals of neighbouring lines is known beforehand
// (pair_requests), and each thread takes the pairs of eight columns of a
// line.  A root's entry is anything no smaller than its node.
//   hooks      a pair is one LDS atomicMin that hooks the lower interval
//              under the upper one; where it was hooked before, the two upper
//              intervals are listed as a join
//   compress   every node is pointed at the root of its tree of hooks
//   joins      the listed pairs, between roots or next to them
//   compress   every node is pointed at its root
// (Sec. II-A-3 with the larger node under the smaller.)  Hooks alone build
// trees as deep as the tile has lines; joining along them without the
// compression in between would walk them again and again.
// The local merge is bound by instruction issue and by the chain of LDS round
// trips between its barriers.  A wavefront that swept its bands one after the
// other, carrying each column's root in a register, issued more instructions
// in one long chain; local merge, both on one card: 4096 x 4096 p = 0.5,
// 8-connectivity 27.0 us with the sweep, 20.0 so, 4-connectivity 23.2 and 21.3;
// 8192 x 8192 smoothed 64 and 41; serpentine 56 and 30.
template <int LINES, int NODES, int JOINS, int INFO, int COLS = 8>
struct LineForest {
    static constexpr int kCols = COLS, kParts = 64 / COLS;  // columns per thread, threads per line
    uint32_t par[NODES];
    uint32_t join[JOINS];      // upper nodes of a join, 16 bits each
    uint16_t info[INFO ? INFO : 1];  // line << 6 | first column of a node's interval (where kept)
    uint64_t E[LINES];         // interval ends
    uint64_t f[LINES], l[LINES], r[LINES];  // touching pairs with the line above
    uint16_t base[LINES];      // first node of the line
    // first node at or after every part's first column (forest_nodes)
    uint16_t pre[INFO ? 1 : LINES * 64 / COLS];
    uint32_t joins;
    // columns [COLS q, COLS q + COLS) of line k's mask in m
    __device__ static uint32_t part(const uint64_t *m, int k, int q) {
        const uint32_t b = ((const uint8_t *)m)[k * 8 + q * COLS / 8];
        return COLS == 8 ? b : (b >> (COLS * q & 7)) & ((1u << COLS) - 1u);
    }
};

// First node at or after the first column of part q of line k, and the nodes
// of the intervals that start in the part (S: the line's interval starts):
// every node a root, with the entry root_entry(node, its first column).
template <class F, class Entry>
__device__ __forceinline__ void forest_nodes(F &sh, int k, int q, uint64_t S, Entry &&root_entry) {
    constexpr uint32_t C = F::kCols, kMask = (1u << C) - 1u;
    const uint64_t E = sh.E[k];
    const uint32_t e = (uint32_t)(E >> (C * q)) & kMask;
    const uint32_t first = (uint32_t)sh.base[k] + (uint32_t)__popcll(E & ((1ull << (C * q)) - 1ull));
    sh.pre[k * F::kParts + q] = (uint16_t)first;
    for (uint32_t s = (uint32_t)(S >> (C * q)) & kMask; s; s &= s - 1u) {
        const uint32_t b = (uint32_t)__builtin_ctz(s);
        const uint32_t n = first + (uint32_t)__builtin_popcount(e & ((1u << b) - 1u));
        lds_st(&sh.par[n], root_entry(n, C * (uint32_t)q + b));
    }
}

// Hook of node lo under node up, or a join of the node it was hooked under.
template <int LINES, int NODES, int JOINS, int INFO, int COLS>
__device__ __forceinline__ void forest_hook(LineForest<LINES, NODES, JOINS, INFO, COLS> &sh, uint32_t lo, uint32_t up) {
    const uint32_t old = atomicMin(&sh.par[lo], up);
    if (old < lo && old != up) {
        const uint32_t j = atomicAdd(&sh.joins, 1u);
        if (j < (uint32_t)JOINS) sh.join[j] = old | (up << 16);
        else lds_link(sh.par, old, up);
    }
}

// The pairs m (columns of the part: shared ones, then the two kinds of
// corners) of a line whose part has the interval ends e and the first node
// `first`, with a line that has u and ufirst.
template <bool DIAG, class F>
__device__ __forceinline__ void forest_hooks(F &sh, uint32_t m, uint32_t e, uint32_t first, uint32_t u, uint32_t ufirst) {
    for (; m; m &= m - 1u) {
        const uint32_t p = (uint32_t)__builtin_ctz(m), b = p & 7u, below = (1u << b) - 1u;
        const uint32_t lo = first + (uint32_t)__builtin_popcount(e & below);
        uint32_t up = ufirst + (uint32_t)__builtin_popcount(u & below);
        if (DIAG) {
            if (p >= 16u) up += (u >> b) & 1u;  // the interval that starts right of b
            else if (p >= 8u) up -= 1u;         // the one that ends left of b
        }
        forest_hook(sh, lo, up);
    }
}

template <bool DIAG, class F>
__device__ __forceinline__ uint32_t forest_pairs(const F &sh, int k, int q) {
    uint32_t m = F::part(sh.f, k, q);
    if (DIAG) m |= (F::part(sh.l, k, q) << 8) | (F::part(sh.r, k, q) << 16);
    return m;
}

// Hooks of part q of line k with the line above it, after forest_nodes.
template <bool DIAG, class F>
__device__ __forceinline__ void forest_hooks(F &sh, int k, int q) {
    const int i = k * F::kParts + q;
    forest_hooks<DIAG>(sh, forest_pairs<DIAG>(sh, k, q), F::part(sh.E, k, q), sh.pre[i], F::part(sh.E, k - 1, q),
                       sh.pre[i - F::kParts]);
}

// Every node a root with its own number as its entry, NT threads: before the
// nodes are known (16-byte stores, 4 nodes each).
template <int NT>
__device__ __forceinline__ void forest_roots(uint32_t *par, int nodes) {
    for (int i = (int)threadIdx.x; i < nodes / 4; i += NT) {
        const uint32_t n = 4u * (uint32_t)i;
        ((uint4 *)par)[i] = make_uint4(n, n + 1u, n + 2u, n + 3u);
    }
}

// Info of the nodes that start in part q of line k (S: the line's interval
// starts) and the part's hooks with the line `above` lines before it (0:
// none), after forest_roots.  (With the nodes' entries set in a phase of their
// own before the hooks, and the pairs found after the numbering instead of
// beside it: local merge of 4096 x 4096 smoothed 13.9 us, so 13.0; 64 mixed
// images 438 us a call, so 432; noise 55.5 and 55.0.)
template <bool DIAG, class F>
__device__ __forceinline__ void forest_line(F &sh, int k, int q, uint64_t S, int above) {
    constexpr uint32_t C = F::kCols, kMask = (1u << C) - 1u;
    const uint64_t before = (1ull << (C * q)) - 1ull;
    const uint64_t E = sh.E[k];
    const uint32_t e = (uint32_t)(E >> (C * q)) & kMask;
    const uint32_t first = (uint32_t)sh.base[k] + (uint32_t)__popcll(E & before);
    for (uint32_t s = (uint32_t)(S >> (C * q)) & kMask; s; s &= s - 1u) {
        const uint32_t b = (uint32_t)__builtin_ctz(s);
        sh.info[first + (uint32_t)__builtin_popcount(e & ((1u << b) - 1u))] =
            (uint16_t)(((uint32_t)k << 6) | (C * (uint32_t)q + b));
    }
    if (above == 0) return;
    const uint64_t Eu = sh.E[k - above];
    forest_hooks<DIAG>(sh, forest_pairs<DIAG>(sh, k, q), e, first, (uint32_t)(Eu >> (C * q)) & kMask,
                       (uint32_t)sh.base[k - above] + (uint32_t)__popcll(Eu & before));
}

// Parent of node n, n itself for a root.
__device__ __forceinline__ uint32_t parent_of(const uint32_t *par, uint32_t n) {
    const uint32_t p = lds_ld(&par[n]);
    return p < n ? p : n;
}

// Points every node at its root and calls done(n) for the roots and then(n,
// root, the root's entry as it was read) for the others.  A node's
// owner alone stores to it, always an ancestor, and a walk stops on any entry
// that is no smaller than its node.  (Two walks at a time per thread, to
// overlap their loads, measured slower: the kernel is short of issue slots.)
template <int NT, class Done, class Then>
__device__ __forceinline__ void compress_nodes(uint32_t *par, uint32_t nodes, Done &&done, Then &&then) {
    for (uint32_t n = threadIdx.x; n < nodes; n += NT) {
        uint32_t p = lds_ld(&par[n]);
        if (p >= n) {
            done(n);
            continue;
        }
        uint32_t g;
        while (true) {
            g = lds_ld(&par[p]);
            if (g >= p) break;
            p = g;
            lds_st(&par[n], p);
        }
        then(n, p, g);
    }
}
template <int NT, class Done>
__device__ __forceinline__ void compress_nodes(uint32_t *par, uint32_t nodes, Done &&done) {
    compress_nodes<NT>(par, nodes, done, [](uint32_t, uint32_t, uint32_t) {});
}

}  // namespace ccl
