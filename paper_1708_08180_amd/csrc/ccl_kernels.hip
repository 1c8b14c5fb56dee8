// The three labeling kernels (gfx950) for one image and for a batch, and
// their launchers.
//
//   local merge        Sec. II-A (Kernel 1): tile-local merge with coarse
//                      labeling over two-row bands (equal-value: runs);
//                      writes the tile's edge masks and edge-cell roots, its
//                      row masks, band data and per-interval records to the
//                      workspace, and seeds labels[root] = root + 1 for roots
//                      whose component touches a shared tile edge.
//   boundary analysis  Sec. II-B (Kernel 2): union-find on tile-edge cells
//                      only, one wavefront per tile (its top and left
//                      edges); the only phase with global atomics.
//   link               Sec. II-C: reads each tile's row masks and records,
//                      resolves each edge-touching local root once in the
//                      global forest and writes the dense output labels
//                      (1 + root, 0 for background); its per-tile body is in
//                      ccl_link.h, shared with the statistics link.
//
// The per-tile bodies are device functions shared by the single-image
// kernels (one workgroup per tile; four tiles per workgroup for the
// boundary analysis) and the batch kernels (the same bodies over one global
// numbering of the tiles of all images).

#include <type_traits>

#include "ccl_device.h"
#include "ccl_internal.h"
#include "ccl_link.h"
#include "ccl_merge.h"

namespace ccl {

// ------------------------------------------------------------- local merge

// Equal-value local merge (every value class labeled, Sec. II-A's
// "same property" test): nodes are the runs of equal values of every row,
// lines are rows, and touching pairs are those of equal value.  2160 x 3840
// in six levels, 8-connectivity: 20 us; sweeping the rows of each wavefront
// one after the other took 39.5.  The sweep was faster where nearly every run is
// hooked or joined: 4096 x 4096 columns, 4-connectivity, 41 us against 56, a
// checkerboard under 8-connectivity 56 against 94.
template <int TH>
struct K1EqLds {
    // Room for every join: a run of m pixels touches at most (m + 3) / 2 runs of
    // its value in the row above, the first of which is its hook, so a row of 64
    // lists at most 64.  (Joins that did not fit 32 per row were made at once,
    // among the uncompressed hooks: local merge of a 4096 x 4096 checkerboard,
    // 8-connectivity, 343 us; so 94.)
    static constexpr int JOINS = 64 * TH;
    alignas(16) LineForest<TH, TH * 64, JOINS, 0> f;
    uint64_t S[TH];         // per row: run starts
    uint64_t flg[TH];       // per row: local roots of edge-touching components
    uint32_t nodes;
    // the tile's bytes, in the joins' place until the masks are made
    __device__ uint8_t *pix() { return (uint8_t *)f.join; }
};

// Kernel 1 body for tile t of image v, equal-value labeling.  Ends after a
// workgroup barrier, so the caller may reuse the LDS for another tile.
template <int TH, int NW, bool CONN8>
__device__ __forceinline__ void k1_tile_eq(const ImgView &v, uint32_t t, K1EqLds<TH> &sh) {
    static_assert(TH <= 64, "one lane per row");
    constexpr int SPR = slots_per_row<true>();
    constexpr int NT = NW * 64;
    constexpr int CH = TH * 4;                  // 16-byte chunks per tile
    constexpr int LPT = (CH + NT - 1) / NT;     // chunks per thread
    auto &F = sh.f;
    uint32_t *par = F.par;
    uint64_t *flg = sh.flg;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
    const uint32_t TX = (uint32_t)v.tilesX;
    const int tx = (int)(t % TX), ty = (int)(t / TX);
    const bool hasUp = ty > 0, hasDown = ty + 1 < v.tilesY;
    const bool hasLeft = tx > 0, hasRight = tx + 1 < v.tilesX;
    // columns / rows of the tile inside the image
    const int wlim = min(kTileW, v.W - tx * kTileW), hlim = min(TH, v.H - ty * TH);
    const uint64_t cols = wlim == 64 ? ~0ull : ((1ull << wlim) - 1ull);

#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int c = tid + i * NT;
        if (c < CH) ((uint4 *)sh.pix())[c] = load_chunk(v, tx, ty, TH, c >> 2, c & 3);
    }
    if (tid < TH) flg[tid] = 0ull;
    if (tid == 0) F.joins = 0u;
    __syncthreads();
    // run starts of every row, and which columns equal the row above
    // straight, to its left and to its right (held in the forest's pair
    // masks until the pairs are known); 16 columns per thread, compared by
    // bytes
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int c = tid + i * NT;
        if (c >= CH) break;
        const int r = c >> 2, q = c & 3;
        const uint8_t *pr = sh.pix() + r * kTileW + q * 16, *pu = pr - (r > 0 ? kTileW : 0);
        const uint4 w = *(const uint4 *)pr, u = *(const uint4 *)pu;
        // the 16 bytes one column to the left / right (what lies beyond the
        // tile's columns is masked)
        auto left = [](uint4 x, uint32_t before) {
            return make_uint4((x.x << 8) | before, __builtin_amdgcn_alignbyte(x.y, x.x, 3),
                              __builtin_amdgcn_alignbyte(x.z, x.y, 3), __builtin_amdgcn_alignbyte(x.w, x.z, 3));
        };
        auto right = [](uint4 x, uint32_t after) {
            return make_uint4(__builtin_amdgcn_alignbyte(x.y, x.x, 1), __builtin_amdgcn_alignbyte(x.z, x.y, 1),
                              __builtin_amdgcn_alignbyte(x.w, x.z, 1), (x.w >> 8) | (after << 24));
        };
        auto differ = [](uint4 x, uint4 y) {
            return nonzero_bytes16(make_uint4(x.x ^ y.x, x.y ^ y.y, x.z ^ y.z, x.w ^ y.w));
        };
        const uint32_t in = r < hlim ? (uint32_t)(cols >> (16 * q)) & 0xFFFFu : 0u;
        const uint32_t inu = r > 0 ? in : 0u;
        const uint32_t first = q == 0 ? 1u : 0u;  // column 0 is in this chunk
        ((uint16_t *)sh.S)[c] = (uint16_t)((differ(w, left(w, q > 0 ? pr[-1] : 0u)) | first) & in);
        ((uint16_t *)F.f)[c] = (uint16_t)(~differ(w, u) & inu);
        if (CONN8) {
            const uint32_t last = (uint32_t)((cols >> 1) >> (16 * q)) & 0xFFFFu;  // columns with a right neighbour
            ((uint16_t *)F.l)[c] = (uint16_t)(~differ(w, left(u, q > 0 ? pu[-1] : 0u)) & inu & ~first);
            ((uint16_t *)F.r)[c] = (uint16_t)(~differ(w, right(u, q < 3 ? pu[16] : 0u)) & inu & last);
        } else {
            ((uint16_t *)F.l)[c] = 0;
            ((uint16_t *)F.r)[c] = 0;
        }
    }
    __syncthreads();
    // runs numbered densely, row by row; the touching pairs of every row
    // with the row above (lane = row)
    if (wave == 0) {
        const uint64_t S = lane < TH ? sh.S[lane] : 0ull, Su = lane > 0 && lane < TH ? sh.S[lane - 1] : 0ull;
        const uint64_t M = lane < hlim ? cols : 0ull;
        const uint64_t E = band_ends(M, S), Eu = band_ends(cols, Su);
        uint32_t nodes;
        const uint32_t b = wave_exclusive_scan((uint32_t)__popcll(S), &nodes);
        if (lane < TH) {
            F.E[lane] = E;
            F.base[lane] = (uint16_t)b;
            const PairRequests q = pair_requests(F.f[lane], F.l[lane], F.r[lane], M, S, E, cols, Su, Eu);
            F.f[lane] = q.f;
            F.l[lane] = q.l;
            F.r[lane] = q.r;
        }
        if (lane == 0) sh.nodes = nodes;
    }
    __syncthreads();
    // a root's entry is kPixel | its first pixel, the smallest of its
    // component (runs are numbered in raster order)
    for (int i = tid; i < TH * 8; i += NT)
        forest_nodes(F, i >> 3, i & 7, sh.S[i >> 3],
                     [&](uint32_t, uint32_t c) { return kPixel | (uint32_t)((i >> 3) * kTileW) | c; });
    __syncthreads();
    for (int i = tid; i < TH * 8; i += NT)
        if (i >= 8) forest_hooks<CONN8>(F, i >> 3, i & 7);
    __syncthreads();
    const uint32_t nodes = sh.nodes, joins = min(F.joins, (uint32_t)K1EqLds<TH>::JOINS);
    // (Also without joins: chains are as deep as the tile where runs go straight
    // down, and the walks of the record phase, eight columns apart, meet on
    // eight of the LDS banks.  Local merge of 4096 x 4096 columns, 4-connectivity: 96 us
    // without it, 56 so; a checkerboard, which hooks nothing, 30 and 33.)
    compress_nodes<NT>(par, nodes, [](uint32_t) {});
    __syncthreads();
    if (joins) {  // workgroup-uniform
        for (uint32_t i = (uint32_t)tid; i < joins; i += NT) {
            const uint32_t e = F.join[i];
            lds_link(par, parent_of(par, e & 0xFFFFu), parent_of(par, e >> 16));
        }
        __syncthreads();
    }
    // records: the first pixel of the node's component, which is also left as
    // the node's entry (a walk that meets it there has found what it looks for)
    uint16_t *sl = v.slots + (size_t)t * TH * SPR;
    for (int i = tid; i < TH * 8; i += NT) {
        const int r = i >> 3, q = i & 7;
        const uint32_t first = F.pre[i], base = F.base[r], e8 = ((const uint8_t *)F.E)[i];
        for (uint32_t s8 = (uint32_t)(sh.S[r] >> (8 * q)) & 0xFFu; s8; s8 &= s8 - 1u) {
            const uint32_t n = first + (uint32_t)__builtin_popcount(e8 & ((1u << __builtin_ctz(s8)) - 1u));
            uint32_t p = lds_ld(&par[n]);
            if (p < kPixel) {
                do p = lds_ld(&par[p]);
                while (p < kPixel);
                lds_st(&par[n], p);
            }
            sl[r * SPR + (int)(n - base)] = (uint16_t)p;
        }
    }
    __syncthreads();
    uint64_t *rw = v.rowmask + (size_t)t * rowmask_words(TH);
    if (tid < TH) rw[tid] = sh.S[tid];
    // edge masks and edge-cell roots for the boundary analysis; every such
    // root is seeded in the forest (lanes of one component store the same
    // word) and marked in the edge-root masks.  Edge k goes to wavefront
    // k mod NW.
    {
        uint64_t *mk = v.masks + (size_t)t * mask_words(TH);
        uint32_t *rt = v.roots + (size_t)t * roots_per_tile(TH);
        // cells taking part in the top / bottom row
        const uint64_t mTop = cols, mBot = TH - 1 < hlim ? cols : 0ull;
        auto root_g = [&](uint32_t n) {
            const uint32_t pos = lds_ld(&par[n]) & (kPixel - 1u);
            atomicOr((unsigned long long *)&flg[pos >> 6], 1ull << (pos & 63u));
            return global_index(v, tx, ty, TH, pos);
        };
        auto put = [&](uint32_t *dst, uint32_t g) {
            *dst = g;
            v.labels[g] = g + 1u;
        };
        if (wave == 0) {
            if (hasUp && lane_in(mTop)) put(&rt[roots_top(TH) + lane], root_g(bits_below(uniform64(F.E[0]))));
            if (lane == 0) {
                mk[kMaskTop] = mTop;
                mk[kMaskBottom] = mBot;
            }
        }
        if (wave == 1 % NW && hasDown && lane_in(mBot))
            put(&rt[roots_bottom(TH) + lane], root_g((uint32_t)F.base[TH - 1] + bits_below(uniform64(F.E[TH - 1]))));
        // per row (lane = row): cells in the left / right column
        const bool lb = lane < hlim, rb = lb && wlim == 64;
        if (wave == 2 % NW) {
            if (hasLeft && lb) put(&rt[roots_left(TH) + lane], root_g((uint32_t)F.base[lane]));
            const uint64_t m = __ballot(lb);
            if (lane == 0) mk[kMaskLeft] = m;
        }
        if (wave == 3 % NW) {
            if (hasRight && rb)
                put(&rt[roots_right(TH) + lane], root_g((uint32_t)F.base[lane] + (uint32_t)__popcll(sh.S[lane]) - 1u));
            const uint64_t m = __ballot(rb);
            if (lane == 0) mk[mask_right(TH)] = m;
        }
    }
    __syncthreads();  // every wavefront's marks are in
    if (tid < TH) rw[TH + tid] = flg[tid];
    __syncthreads();  // LDS may be reused for another tile
}

// ------------------------------------------------------ boundary analysis

// One wavefront per tile: the tile's top edge against the tile above (64
// lanes, one per column; it also takes the diagonal pairs that cross the
// tile's upper corners) and its left edge against the tile on its left (TH
// lanes, one per row; pairs inside one tile row only), so every adjacent
// foreground pair that crosses tiles is examined by exactly one edge.  All
// masks and edge-cell roots are loaded up front; the neighbours' roots come
// from lane shifts.  Each lane holds up to four merge requests (two per
// edge), which are deduplicated and merged together.
template <int TH, bool CONN8>
__device__ __forceinline__ void k2_tile(const ImgView &v, uint32_t t) {
    constexpr int RT = roots_per_tile(TH);
    constexpr int MW = mask_words(TH);
    constexpr int LH = col_words(TH);  // left-edge cells per lane
    const int lane = lane_id();
    const uint32_t TX = (uint32_t)v.tilesX;
    const uint32_t tx = t % TX, ty = t / TX;
    const bool hasT = ty > 0, hasL = tx > 0, hasR = tx + 1u < TX;
    const uint64_t *mk = v.masks;
    const uint32_t *rts = v.roots;
    uint64_t dT = 0, uT = 0, xl = 0, xr = 0, dL[LH], uL[LH];
    uint32_t aT = kNone, rT = kNone, eTL = kNone, eTR = kNone, aL[LH], rL[LH];
    if (hasT) {
        const uint32_t tu = t - TX;
        dT = mk[(size_t)t * MW + kMaskTop];
        uT = mk[(size_t)tu * MW + kMaskBottom];
        if (hasL) {
            xl = mk[(size_t)(tu - 1u) * MW + kMaskBottom] >> 63;
            eTL = rts[(size_t)(tu - 1u) * RT + roots_bottom(TH) + 63];
        }
        if (hasR) {
            xr = (mk[(size_t)(tu + 1u) * MW + kMaskBottom] & 1ull) << 63;
            eTR = rts[(size_t)(tu + 1u) * RT + roots_bottom(TH)];
        }
        aT = rts[(size_t)t * RT + roots_top(TH) + lane];
        rT = rts[(size_t)tu * RT + roots_bottom(TH) + lane];
    }
#pragma unroll
    for (int h = 0; h < LH; ++h) {
        const int r = 64 * h + lane;
        dL[h] = uL[h] = 0ull;
        aL[h] = rL[h] = kNone;
        if (hasL) {
            dL[h] = mk[(size_t)t * MW + kMaskLeft + h];
            uL[h] = mk[(size_t)(t - 1u) * MW + mask_right(TH) + h];
            if (r < TH) {
                aL[h] = rts[(size_t)t * RT + roots_left(TH) + r];
                rL[h] = rts[(size_t)(t - 1u) * RT + roots_right(TH) + r];
            }
        }
    }
    // roots of the cells above-left / above-right (left edge: above / below)
    const uint32_t bTl = from_left(rT, eTL), bTr = from_right(rT, eTR);
    uint32_t A[2 + 2 * LH], B[2 + 2 * LH];
    {
        const PairMasks p = pair_masks<CONN8>(dT, uT, xl, xr);
        // at lane 0 the above-left cell lies in the tile to the left, so
        // PL and PM can both hold there; elsewhere they exclude each other
        B[0] = lane_in(p.pl) ? bTl : (lane_in(p.pm) ? rT : kNone);
        B[1] = lane_in(p.pr) ? bTr : (lane_in(p.pl & p.pm) ? rT : kNone);
        A[0] = A[1] = aT;
    }
    // the left edge as lines of 64 rows; the rows next to a chunk boundary
    // come from the neighbouring chunk, the tile's own first and last rows
    // have none (their corner pairs belong to the top edges)
#pragma unroll
    for (int h = 0; h < LH; ++h) {
        const uint64_t cl = h > 0 ? uL[h - 1] >> 63 : 0ull;
        const uint64_t cr = h + 1 < LH ? (uL[h + 1] & 1ull) << 63 : 0ull;
        const uint32_t el = h > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)rL[h - 1], 63) : kNone;
        const uint32_t er = h + 1 < LH ? (uint32_t)__builtin_amdgcn_readlane((int)rL[h + 1], 0) : kNone;
        const uint32_t bLl = from_left(rL[h], el), bLr = from_right(rL[h], er);
        const PairMasks p = pair_masks<CONN8>(dL[h], uL[h], cl, cr);
        B[2 + 2 * h] = lane_in(p.pl) ? bLl : (lane_in(p.pm) ? rL[h] : kNone);
        B[3 + 2 * h] = lane_in(p.pr) ? bLr : (lane_in(p.pl & p.pm) ? rL[h] : kNone);
        A[2 + 2 * h] = A[3 + 2 * h] = aL[h];
    }
    union_requests<2 + 2 * LH>(A, B, [&](uint32_t a, uint32_t b) { g_union(v.labels, v.n, a, b); });
}

// Equal-value boundary analysis for tile t: like k2_tile, but a pair of
// cells across the edge is merged when their image values are equal (read
// straight from the image), and every such pair is proposed -- the
// deduplication keeps one union per distinct pair of roots.
template <int TH, bool CONN8>
__device__ __forceinline__ void k2_tile_eq(const ImgView &v, uint32_t t) {
    constexpr int RT = roots_per_tile(TH);
    constexpr uint32_t kOut = 0x100u, kOutUp = 0x200u;  // no byte equals these
    const int lane = lane_id();
    const uint32_t TX = (uint32_t)v.tilesX;
    const uint32_t tx = t % TX, ty = t / TX;
    const bool hasT = ty > 0, hasL = tx > 0, hasR = tx + 1u < TX;
    const int x0 = (int)tx * kTileW, y0 = (int)ty * TH;
    const int wlim = min(kTileW, v.W - x0), hlim = min(TH, v.H - y0);
    const uint32_t *rts = v.roots;
    uint32_t vT = kOut, vU = kOutUp, vUL = kOutUp, vUR = kOutUp, vC = kOut, vN = kOutUp;
    uint32_t aT = kNone, rT = kNone, eTL = kNone, eTR = kNone, aL = kNone, rL = kNone;
    if (hasT) {
        const uint32_t tu = t - TX;
        const uint8_t *row = v.img + (int64_t)y0 * v.pitch + x0;  // this tile's top row
        const uint8_t *up = row - v.pitch;                         // the row above it
        if (lane < wlim) {
            vT = row[lane];
            vU = up[lane];
            aT = rts[(size_t)t * RT + roots_top(TH) + lane];
            rT = rts[(size_t)tu * RT + roots_bottom(TH) + lane];
        }
        if (hasL) {
            vUL = up[-1];
            eTL = rts[(size_t)(tu - 1u) * RT + roots_bottom(TH) + 63];
        }
        if (hasR) {
            vUR = up[kTileW];
            eTR = rts[(size_t)(tu + 1u) * RT + roots_bottom(TH)];
        }
    }
    if (hasL && lane < hlim) {
        const uint8_t *p = v.img + (int64_t)(y0 + lane) * v.pitch + x0;
        vC = p[0];
        vN = p[-1];
        aL = rts[(size_t)t * RT + roots_left(TH) + lane];
        rL = rts[(size_t)(t - 1u) * RT + roots_right(TH) + lane];
    }
    // neighbours across the edge: above-left / above-right (top edge), the
    // left cells of the rows above / below (left edge, inside the tile rows)
    const uint32_t vUl = from_left(vU, vUL), vUr = from_right(vU, vUR);
    const uint32_t bTl = from_left(rT, eTL), bTr = from_right(rT, eTR);
    const uint32_t vNu = from_left(vN, kOutUp), vNd = from_right(vN, kOutUp);
    const uint32_t bLu = from_left(rL, kNone), bLd = from_right(rL, kNone);
    uint32_t A[6], B[6];
    A[0] = A[1] = A[2] = aT;
    A[3] = A[4] = A[5] = aL;
    B[0] = vT == vU ? rT : kNone;
    B[1] = CONN8 && vT == vUl ? bTl : kNone;
    B[2] = CONN8 && vT == vUr ? bTr : kNone;
    B[3] = vC == vN ? rL : kNone;
    B[4] = CONN8 && vC == vNu ? bLu : kNone;
    B[5] = CONN8 && vC == vNd ? bLd : kNone;
    union_requests<6>(A, B, [&](uint32_t a, uint32_t b) { g_union(v.labels, v.n, a, b); });
}

// ------------------------------------------------------ single-image kernels

template <int TH, int NW, bool CONN8, bool EQ>
__global__ void __launch_bounds__(NW * 64) k1_local_merge(ImgView v) {
    const uint32_t t = xcd_remap(blockIdx.x, gridDim.x);
    if constexpr (EQ) {
        __shared__ K1EqLds<TH> sh;
        k1_tile_eq<TH, NW, CONN8>(v, t, sh);
    } else {
        __shared__ K1BandLds<TH, NW, CONN8> sh;
        k1_tile_bands<TH, NW, CONN8>(v, t, sh, [] {});
    }
}

template <int TH, bool CONN8, bool EQ>
__global__ void __launch_bounds__(256) k2_boundary(ImgView v, uint32_t tiles) {
    // the same XCD-contiguous tile ranges as the local merge and the link:
    // the forest chains of a region's components stay in one XCD's L2
    const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(xcd_remap(blockIdx.x, gridDim.x) * 4u + (threadIdx.x >> 6)));
    if (t >= tiles) return;  // wave-uniform
    if (EQ) k2_tile_eq<TH, CONN8>(v, t);
    else k2_tile<TH, CONN8>(v, t);
}

template <int TH, int NW, bool EQ>
__global__ void __launch_bounds__(NW * 64) k3_link(ImgView v) {
    __shared__ uint32_t fin[TH * kTileW];
    constexpr int SPR = slots_per_row<EQ>();
    const uint32_t t = xcd_remap(blockIdx.x, gridDim.x);
    k3_tile<TH, NW, EQ>(v, t, v.rowmask + (size_t)t * rowmask_words(TH), v.slots + (size_t)t * TH * SPR, fin);
}

// ------------------------------------------------------------- small images

// A small image in one workgroup and one launch: the local merge's forest over
// the whole image, whose lines are the 64-column words of its bands in raster
// order, with joins between neighbouring words of a band; the labels are
// written from LDS.  Such a call is bound by launches and by the latency of a
// phase, not by work: 64 x 64 of noise, p = 0.5, takes 11.6 us in three launches
// and 6.1 so, 120 x 160, 8-connectivity, 15.6 and 12.4.
// small_image() holds where the line lies.
template <bool CONN8>
constexpr int kSmallLines = CONN8 ? 256 : 192;  // room for, a multiple of 64

template <bool CONN8>
struct SmallLds {
    static constexpr int LINES = kSmallLines<CONN8>;
    static constexpr int NODES = LINES * (CONN8 ? 32 : 64);
    // Room for every join: a line's intervals touch at most 33 of the line
    // above (its 64 columns and, under 8-connectivity, one beside each end),
    // and along a line the touching pairs are one fewer than the intervals on
    // both sides; each lower interval's first pair is a hook, so a line lists
    // at most 32 joins, and one more with the word before.  (With 4096 entries the
    // joins that did not fit were made at once, among the uncompressed hooks:
    // columns staggered every other row, 8-connectivity, 128 x 192, 58.5 us a
    // call; so 16.1.)
    static constexpr int JOINS = 33 * LINES;
    alignas(16) LineForest<LINES, NODES, JOINS, NODES> f;
    uint64_t m[2][LINES];  // top / bottom row masks of every line
    uint32_t part[LINES / 64], nodes;
};

template <bool CONN8>
__global__ void __launch_bounds__(1024) label_small(ImgView v) {
    constexpr int NT = 1024;
    __shared__ SmallLds<CONN8> sh;
    auto &F = sh.f;
    uint32_t *par = F.par;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int WX = (v.W + kTileW - 1) / kTileW, NB = (v.H + 1) / 2, lines = NB * WX;
    // line / WX for line < 256
    const uint32_t inv = 65536u / (uint32_t)WX + 1u;
    auto band_of = [&](uint32_t line) { return (line * inv) >> 16; };
    forest_roots<NT>(par, lines * (CONN8 ? 32 : 64));
    for (int c = tid; c < lines * 8; c += NT) {
        const int row = (c >> 2) & 1, q = c & 3;  // eight chunks per line
        const uint32_t line = (uint32_t)c >> 3, k = band_of(line);
        const int y = 2 * (int)k + row, x = (int)(line - k * (uint32_t)WX) * kTileW + q * 16;
        uint32_t bits = 0u;
        if (y < v.H) bits = nonzero_bytes16(load_row16(v.img + (int64_t)y * v.pitch, x, v.W));
        ((uint16_t *)&sh.m[row][line])[q] = (uint16_t)bits;
    }
    if (tid == 0) F.joins = 0u;
    __syncthreads();
    // every line's intervals, and their numbering (a line per thread)
    uint32_t ex = 0u;
    if (wave < SmallLds<CONN8>::LINES / 64) {
        const bool in = tid < lines;
        const uint64_t t0 = in ? sh.m[0][tid] : 0ull, b0 = in ? sh.m[1][tid] : 0ull;
        const uint64_t S = band_starts<CONN8>(t0, b0);
        uint32_t total;
        ex = wave_exclusive_scan((uint32_t)__popcll(S), &total);
        F.E[tid] = band_ends(t0 | b0, S);
        if (lane == 0) sh.part[wave] = total;
    }
    __syncthreads();
    if (wave < SmallLds<CONN8>::LINES / 64) {
        uint32_t before = 0u, all = 0u;
#pragma unroll
        for (int j = 0; j < SmallLds<CONN8>::LINES / 64; ++j) {
            before += j < wave ? sh.part[j] : 0u;
            all += sh.part[j];
        }
        F.base[tid] = (uint16_t)(before + ex);
        if (tid == 0) sh.nodes = all;
        // touching pairs with the line above (the same word of the band
        // above); its corner columns look into the words beside it
        PairRequests p = {0ull, 0ull, 0ull};
        if (tid >= WX && tid < lines) {
            const int up = tid - WX;
            const uint32_t w = (uint32_t)tid - band_of((uint32_t)tid) * (uint32_t)WX;
            const uint64_t t0 = sh.m[0][tid], b0 = sh.m[1][tid], tu = sh.m[0][up], u = sh.m[1][up];
            uint64_t l = 0ull, r = 0ull;
            if (CONN8) {
                l = t0 & ((u << 1) | (w > 0u ? sh.m[1][up - 1] >> 63 : 0ull));
                r = t0 & ((u >> 1) | (w + 1u < (uint32_t)WX ? sh.m[1][up + 1] << 63 : 0ull));
            }
            p = pair_requests(t0 & u, l, r, t0 | b0, band_starts<CONN8>(t0, b0), F.E[tid], tu | u,
                              band_starts<CONN8>(tu, u), F.E[up]);
        }
        F.f[tid] = p.f;
        F.l[tid] = p.l;
        F.r[tid] = p.r;
    }
    __syncthreads();
    for (int i = tid; i < lines * 8; i += NT) {
        const int k = i >> 3;
        forest_line<CONN8>(F, k, i & 7, band_starts<CONN8>(sh.m[0][k], sh.m[1][k]), k >= WX ? WX : 0);
        if ((i & 7) == 0 && k > 0 && (uint32_t)k != band_of((uint32_t)k) * (uint32_t)WX) {
            // the band goes on from the word before
            const uint64_t t0 = sh.m[0][k], b0 = sh.m[1][k], tl = sh.m[0][k - 1] >> 63, bl = sh.m[1][k - 1] >> 63;
            const bool on = CONN8 ? ((tl | bl) & (t0 | b0) & 1ull) != 0 : (((tl & t0) | (bl & b0)) & 1ull) != 0;
            if (on) forest_hook(F, (uint32_t)F.base[k], (uint32_t)F.base[k] - 1u);
        }
    }
    __syncthreads();
    const uint32_t nodes = sh.nodes, joins = min(F.joins, (uint32_t)SmallLds<CONN8>::JOINS);
    // roots' entries become kPixel | smallest pixel, row << 14 | column (see
    // k1_tile_bands)
    constexpr uint32_t kRow = 1u << 14;
    auto smallest = [&](uint32_t n) {
        const uint32_t in = F.info[n], line = in >> 6, s = in & 63u, k = band_of(line);
        const uint64_t tr = sh.m[0][line] >> s, er = F.E[line] >> s;
        const uint32_t dt = tr ? (uint32_t)__builtin_ctzll(tr) : 64u;
        const bool top = dt <= (uint32_t)__builtin_ctzll(er);
        const uint32_t x = (line - k * (uint32_t)WX) * (uint32_t)kTileW + s + (top ? dt : 0u);
        return (2u * k + (top ? 0u : 1u)) * kRow | x;
    };
    compress_nodes<NT>(par, nodes, [&](uint32_t n) { lds_st(&par[n], kPixel | smallest(n)); });
    __syncthreads();
    if (joins) {  // workgroup-uniform
        for (uint32_t i = (uint32_t)tid; i < joins; i += NT) {
            const uint32_t e = F.join[i];
            lds_link(par, parent_of(par, e & 0xFFFFu), parent_of(par, e >> 16));
        }
        __syncthreads();
    }
    compress_nodes<NT>(par, nodes, [](uint32_t) {}, [&](uint32_t n, uint32_t r, uint32_t e) {
        // a root without a top-row pixel, and a node of the same band
        const uint32_t first = band_of((uint32_t)F.info[n] >> 6) * (uint32_t)WX;
        if (r >= (uint32_t)F.base[first]) {
            const uint32_t p = kPixel | smallest(n);
            if (p < e) atomicMin(&par[r], p);
        }
    });
    __syncthreads();
    // labels, a line's two rows at a time
    for (int k = wave; k < lines; k += NT / 64) {
        const uint32_t band = band_of((uint32_t)k);
        const uint32_t x = ((uint32_t)k - band * (uint32_t)WX) * (uint32_t)kTileW + (uint32_t)lane;
        const uint64_t t0 = uniform64(sh.m[0][k]), b0 = uniform64(sh.m[1][k]);
        uint32_t val = 0u;
        if (lane_in(t0 | b0)) {
            uint32_t e = lds_ld(&par[(uint32_t)F.base[k] + bits_below(uniform64(F.E[k]))]);
            if (e < kPixel) e = lds_ld(&par[e]);
            e -= kPixel;
            val = (e / kRow) * (uint32_t)v.W + (e & (kRow - 1u)) + 1u;
        }
        if (x >= (uint32_t)v.W) continue;
        uint32_t *out = v.labels + (size_t)(2u * band) * (uint32_t)v.W + x;
        *out = lane_in(t0) ? val : 0u;
        if (2 * (int)band + 1 < v.H) out[v.W] = lane_in(b0) ? val : 0u;
    }
}

// ------------------------------------------------------------ batch kernels

template <int TH>
__device__ __forceinline__ ImgView batch_view(const BatchImage &b, const BatchWs &w) {
    ImgView v;
    v.img = b.img;
    v.labels = b.labels;
    v.masks = w.masks + (size_t)b.tile_base * mask_words(TH);
    v.roots = w.roots + (size_t)b.tile_base * roots_per_tile(TH);
    v.rowmask = w.rowmask + (size_t)b.tile_base * rowmask_words(TH);
    v.slots = w.slots + (size_t)b.tile_base * TH * kSlotsPerRow;
    v.pitch = b.pitch;
    v.H = b.H;
    v.W = b.W;
    v.tilesX = b.tilesX;
    v.tilesY = b.tilesY;
    v.n = b.n;
    return v;
}

// The batch kernels are the single-image ones over one global numbering of
// the tiles of all images: one workgroup per tile for the local merge and
// the link, four tiles per workgroup for the boundary analysis.  The host
// sizes the grids for every call.
template <int TH, int NW, bool CONN8>
__global__ void __launch_bounds__(NW * 64) k1_batch(BatchArgs a) {
    __shared__ K1BandLds<TH, NW, CONN8> sh;
    const uint32_t g = xcd_remap(blockIdx.x, gridDim.x);
    if (g >= a.tiles) return;  // workgroup-uniform
    const uint32_t i = batch_image_of(a, g);
    if (threadIdx.x == 0) a.w.tile_img[g] = i;
    const BatchImage &d = a.descs[i];
    k1_tile_bands<TH, NW, CONN8>(batch_view<TH>(d, a.w), g - d.tile_base, sh, [] {});
}

template <int TH, bool CONN8>
__global__ void __launch_bounds__(256) k2_batch(BatchArgs a) {
    const uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(xcd_remap(blockIdx.x, gridDim.x) * 4u + (threadIdx.x >> 6)));
    if (g >= a.tiles) return;  // wave-uniform
    const BatchImage &d = a.descs[a.w.tile_img[g]];
    k2_tile<TH, CONN8>(batch_view<TH>(d, a.w), g - d.tile_base);
}

template <int TH, int NW>
__global__ void __launch_bounds__(NW * 64) k3_batch(BatchArgs a) {
    __shared__ uint32_t fin[TH * kTileW];
    const uint32_t g = xcd_remap(blockIdx.x, gridDim.x);
    if (g >= a.tiles) return;  // workgroup-uniform
    const BatchImage &d = a.descs[a.w.tile_img[g]];
    k3_tile<TH, NW, false>(batch_view<TH>(d, a.w), g - d.tile_base, a.w.rowmask + (size_t)g * rowmask_words(TH),
                           a.w.slots + (size_t)g * TH * kSlotsPerRow, fin);
}

// ---------------------------------------------------------------- launchers

template <int TH, int NW, bool CONN8, bool EQ>
static hipError_t launch_plain_t(const ImgView &v, hipStream_t stream, hipEvent_t *ev) {
    const uint32_t tiles = (uint32_t)v.tilesX * (uint32_t)v.tilesY;
    // a grid that HIP would refuse: the later phases must not run on a
    // workspace that the local merge has not written
    if (!grid_fits(tiles, (NW > TH / 16 ? NW : TH / 16) * 64u)) return hipErrorInvalidConfiguration;
    if (ev) (void)hipEventRecord(ev[0], stream);
    hipLaunchKernelGGL((k1_local_merge<TH, NW, CONN8, EQ>), dim3(tiles), dim3(NW * 64), 0, stream, v);
    if (ev) (void)hipEventRecord(ev[1], stream);
    if (tiles > 1)
        hipLaunchKernelGGL((k2_boundary<TH, CONN8, EQ>), dim3((tiles + 3) / 4), dim3(256), 0, stream,
                           v, tiles);
    if (ev) (void)hipEventRecord(ev[2], stream);
    with_link_waves<TH>(tiles, [&](auto nw3) {
        constexpr int NW3 = decltype(nw3)::value;
        hipLaunchKernelGGL((k3_link<TH, NW3, EQ>), dim3(tiles), dim3(NW3 * 64), 0, stream, v);
    });
    if (ev) (void)hipEventRecord(ev[3], stream);
    return hipGetLastError();
}

// Boundary analysis only (binary labeling), for callers with a local merge
// and a link of their own.
template <int TH, bool CONN8>
static hipError_t launch_boundary_t(const ImgView &v, hipStream_t stream) {
    const uint32_t tiles = (uint32_t)v.tilesX * (uint32_t)v.tilesY;
    if (tiles > 1)
        hipLaunchKernelGGL((k2_boundary<TH, CONN8, false>), dim3((tiles + 3) / 4), dim3(256), 0, stream,
                           v, tiles);
    return hipGetLastError();
}

template <int TH, int NW, bool CONN8>
static void batch_kernels_t(BatchKernels *k) {
    k->k1 = (const void *)k1_batch<TH, NW, CONN8>;
    k->k2 = (const void *)k2_batch<TH, CONN8>;
    k->k3 = (const void *)k3_batch<TH, link_waves<TH>()>;
    k->block1 = NW * 64;
    k->block3 = link_waves<TH>() * 64;
    k->block2 = 256;
    k->tiles_per_group2 = 4;
}

bool config_supported(int th, int nw) {
    switch (th) {
        case 16: return nw == 1 || nw == 2 || nw == 4 || nw == 8;
        case 32: return nw == 1 || nw == 2 || nw == 4 || nw == 8 || nw == 16;
        case 64: return nw == 1 || nw == 2 || nw == 4 || nw == 8 || nw == 16;
        case 128: return nw == 2 || nw == 4 || nw == 8 || nw == 16;
        default: return false;
    }
}

#define CCL_FOR_EACH_CONFIG(X) CCL_FOR_EACH_LOW_CONFIG(X) X(128, 2) X(128, 4) X(128, 8) X(128, 16)

// Tile configurations compiled for equal-value labeling.
#define CCL_FOR_EACH_EQ_CONFIG(X) X(16, 4) X(32, 2) X(32, 8) X(64, 4) X(64, 8)

bool config_supported_equal(int th, int nw) {
#define CCL_CASE(T, N) \
    if (th == T && nw == N) return true;
    CCL_FOR_EACH_EQ_CONFIG(CCL_CASE)
#undef CCL_CASE
    return false;
}

hipError_t launch_plain(const ImgView &v, int th, int nw, int conn, hipStream_t s, hipEvent_t *ev,
                        bool equal) {
    if (equal) {
#define CCL_CASE(T, N)                                                        \
    if (th == T && nw == N)                                                   \
        return conn == 8 ? launch_plain_t<T, N, true, true>(v, s, ev)         \
                         : launch_plain_t<T, N, false, true>(v, s, ev);
        CCL_FOR_EACH_EQ_CONFIG(CCL_CASE)
#undef CCL_CASE
        return hipErrorInvalidValue;
    }
#define CCL_CASE(T, N)                                                        \
    if (th == T && nw == N)                                                   \
        return conn == 8 ? launch_plain_t<T, N, true, false>(v, s, ev)        \
                         : launch_plain_t<T, N, false, false>(v, s, ev);
    CCL_FOR_EACH_CONFIG(CCL_CASE)
#undef CCL_CASE
    return hipErrorInvalidValue;
}

// One launch up to the lines where noise takes no longer in it than in three
// and the worst pattern (a checkerboard under 4-connectivity, columns or staggered
// columns under 8) at most 2 % longer than in the three launches that ran every
// size before.  us a call, three launches and one:
//   4-connectivity: 4 x 4096 (128 lines) checkerboard 9.3 and 9.2; 64 x 320 (160)
//     checkerboard 10.7 and 10.8, noise 1.2 times as fast; 4 x 5120 (160)
//     checkerboard 9.3 and 10.9; 128 x 256 (256) 10.5 and 16.2;
//   8-connectivity, at most one row of 32-row tiles: 32 x 640 (160) columns 10.0
//     and 10.2, noise 1.2 times as fast; 8 x 4096 (256) columns 9.2 and 14.1;
//   8-connectivity, more rows, where three launches join tiles below each other:
//     56 x 512 (224) staggered columns 17.4 and 17.7, noise 1.1 times as fast;
//     512 x 64 (256) staggered columns 18.6 and 19.9.
bool small_image(int H, int W, int conn) {
    const int64_t lines = ((int64_t)H + 1) / 2 * (((int64_t)W + kTileW - 1) / kTileW);
    if (conn == 4) return lines <= (H >= 48 ? 160 : 128);
    return lines <= (H >= 48 ? 224 : 160);
}

hipError_t launch_small(const ImgView &v, int conn, hipStream_t s) {
    if (conn == 8) hipLaunchKernelGGL(label_small<true>, dim3(1), dim3(1024), 0, s, v);
    else hipLaunchKernelGGL(label_small<false>, dim3(1), dim3(1024), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_boundary(const ImgView &v, int th, int conn, hipStream_t s) {
    const bool c8 = conn == 8;
    switch (th) {
        case 16: return c8 ? launch_boundary_t<16, true>(v, s) : launch_boundary_t<16, false>(v, s);
        case 32: return c8 ? launch_boundary_t<32, true>(v, s) : launch_boundary_t<32, false>(v, s);
        case 64: return c8 ? launch_boundary_t<64, true>(v, s) : launch_boundary_t<64, false>(v, s);
        default: return hipErrorInvalidValue;
    }
}

bool batch_kernels(int th, int nw, int conn, BatchKernels *out) {
#define CCL_CASE(T, N)                                                                   \
    if (th == T && nw == N) {                                                            \
        if (conn == 8) batch_kernels_t<T, N, true>(out);                                 \
        else batch_kernels_t<T, N, false>(out);                                          \
        return true;                                                                     \
    }
    CCL_FOR_EACH_CONFIG(CCL_CASE)
#undef CCL_CASE
    return false;
}

}  // namespace ccl
