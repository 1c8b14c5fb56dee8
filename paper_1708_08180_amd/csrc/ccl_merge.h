// Local merge (Sec. II-A) of one tile, binary labeling, shared by the labeling
// kernels and the kernel that also gathers component statistics.
#pragma once

#include "ccl_device.h"

namespace ccl {

// Entry of a settled node: kPixel | its root's tile-local pixel (3D: voxel).
constexpr uint32_t kPixel = 0x80000000u;

// Binary local merge over two-row bands.
template <int TH, int NW, bool CONN8>
struct K1BandLds {
    static constexpr int NB = TH / 2;
    static constexpr int NODES = NB * (CONN8 ? 32 : 64);  // a band's most intervals
    // eight columns of a band per thread, four where that leaves threads idle
    alignas(16) LineForest<NB, NODES, 16 * TH, NODES, (NB * 8 >= NW * 64 ? 8 : 4)> f;
    uint64_t msk[TH];  // per row: foreground mask
    uint64_t flg[TH];  // per row: local roots of edge-touching components
    uint32_t nodes;
};

// Kernel 1 body for tile t of image v, binary labeling.  Writes the tile's
// row masks, edge-root masks, band interval ends and band bases, one record
// per node (the tile-local pixel of its root), the edge masks and the roots
// of the edge cells, and seeds those roots in the forest.  then() runs at the
// end, when every node's entry is kPixel | its root's pixel and the flag masks
// are whole.  Ends after a workgroup barrier.
template <int TH, int NW, bool CONN8, class Then>
__device__ __forceinline__ void k1_tile_bands(const ImgView &v, uint32_t t, K1BandLds<TH, NW, CONN8> &sh, Then &&then) {
    constexpr int NB = TH / 2;
    constexpr int NT = NW * 64;
    constexpr int CH = TH * 4;               // 16-byte chunks per tile
    constexpr int LPT = (CH + NT - 1) / NT;  // chunks per thread
    auto &F = sh.f;
    uint32_t *par = F.par;
    uint64_t *msk = sh.msk;
    uint64_t *flg = sh.flg;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
    const uint32_t TX = (uint32_t)v.tilesX;
    const int tx = (int)(t % TX), ty = (int)(t / TX);
    const bool hasUp = ty > 0, hasDown = ty + 1 < v.tilesY;
    const bool hasLeft = tx > 0, hasRight = tx + 1 < v.tilesX;

    uint4 px[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int c = tid + i * NT;
        px[i] = c < CH ? load_chunk(v, tx, ty, TH, c >> 2, c & 3) : make_uint4(0u, 0u, 0u, 0u);
    }
    forest_roots<NT>(par, K1BandLds<TH, NW, CONN8>::NODES);  // while the pixels are on their way
    for (int r = tid; r < TH; r += NT) flg[r] = 0ull;
    if (tid == 0) F.joins = 0u;
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int c = tid + i * NT;
        if (c < CH) ((uint16_t *)msk)[c] = (uint16_t)nonzero_bytes16(px[i]);
    }
    __syncthreads();
    // every band's intervals, one band per lane: nodes are numbered densely
    // (an exclusive scan of the bands' interval counts)
    if (wave == 0) {
        const uint64_t bt = lane < NB ? msk[2 * lane] : 0ull, bb = lane < NB ? msk[2 * lane + 1] : 0ull;
        const uint64_t s = band_starts<CONN8>(bt, bb);
        uint32_t nodes;
        const uint32_t b = wave_exclusive_scan((uint32_t)__popcll(s), &nodes);
        if (lane < NB) {
            F.E[lane] = band_ends(bt | bb, s);
            F.base[lane] = (uint16_t)b;
        }
        if (lane == 0) sh.nodes = nodes;
    }
    // the touching pairs of every band with the band above, one band per
    // lane (on a wavefront that does not scan)
    if (wave == (NW > 1 ? 1 : 0) && lane < NB && lane > 0) {
        const uint64_t t0 = msk[2 * lane], u = msk[2 * lane - 1];
        const uint64_t M = t0 | msk[2 * lane + 1], Mu = u | msk[2 * lane - 2];
        const uint64_t S = band_starts<CONN8>(t0, msk[2 * lane + 1]);
        const uint64_t Su = band_starts<CONN8>(msk[2 * lane - 2], u);
        const PairRequests q = pair_requests(t0 & u, CONN8 ? t0 & (u << 1) : 0ull, CONN8 ? t0 & (u >> 1) : 0ull, M, S,
                                             band_ends(M, S), Mu, Su, band_ends(Mu, Su));
        F.f[lane] = q.f;
        F.l[lane] = q.l;
        F.r[lane] = q.r;
    }
    __syncthreads();
    using Forest = decltype(sh.f);
    for (int i = tid; i < NB * Forest::kParts; i += NT) {
        const int k = i / Forest::kParts;
        forest_line<CONN8>(F, k, i % Forest::kParts, band_starts<CONN8>(msk[2 * k], msk[2 * k + 1]), k > 0 ? 1 : 0);
    }
    __syncthreads();
    const uint32_t nodes = sh.nodes, joins = min(F.joins, (uint32_t)(16 * TH));
    // an interval's smallest pixel: its first top-row pixel, else its first
    // pixel (a bottom-row one, at the start column)
    auto smallest = [&](uint32_t n) {
        const uint32_t in = F.info[n], k = in >> 6, s = in & 63u;
        const uint64_t tr = msk[2 * k] >> s, er = F.E[k] >> s;
        const uint32_t dt = tr ? (uint32_t)__builtin_ctzll(tr) : 64u;
        const bool top = dt <= (uint32_t)__builtin_ctzll(er);
        return ((2u * k + (top ? 0u : 1u)) << 6) | (s + (top ? dt : 0u));
    };
    // every node finds the root of its tree of hooks; such a root's entry
    // becomes kPixel | its smallest pixel, which walks and joins still take
    // for a root's (it is no smaller than any node)
    compress_nodes<NT>(par, nodes, [&](uint32_t n) { lds_st(&par[n], kPixel | smallest(n)); });
    __syncthreads();
    if (joins) {  // workgroup-uniform
        for (uint32_t i = (uint32_t)tid; i < joins; i += NT) {
            const uint32_t e = F.join[i];
            lds_link(par, parent_of(par, e & 0xFFFFu), parent_of(par, e >> 16));
        }
        __syncthreads();
    }
    // every node finds its root.  Where the root has no top-row pixel, the
    // component's smallest pixel may be the top-row pixel of another of its
    // intervals in the band (once one has been entered, only of one that
    // starts before it); e's pixel lies in the root's band.  (In a pass of
    // its own after the roots were settled, local merge of 4096 x 4096 p = 0.5,
    // 8-connectivity: 21.5 us, so 20.0.)
    compress_nodes<NT>(par, nodes, [](uint32_t) {}, [&](uint32_t n, uint32_t r, uint32_t e) {
        const uint32_t in = F.info[n];
        if ((e & (kPixel - 1u)) >> 7 == in >> 6 && ((e & 64u) || (in & 63u) < (e & 63u))) {
            const uint32_t p = kPixel | smallest(n);
            if (p < e) atomicMin(&par[r], p);
        }
    });
    __syncthreads();
    // records: the smallest pixel of the node's component
    uint16_t *sl = v.slots + (size_t)t * TH * kSlotsPerRow;
    for (uint32_t n = (uint32_t)tid; n < nodes; n += NT) {
        uint32_t e = lds_ld(&par[n]);
        if (e < kPixel) {
            e = lds_ld(&par[e]);
            lds_st(&par[n], e);
        }
        sl[n] = (uint16_t)e;
    }
    uint64_t *rw = v.rowmask + (size_t)t * rowmask_words(TH);
    for (int r = tid; r < TH; r += NT) rw[r] = msk[r];
    if (tid < NB) {
        rw[rowmask_ends(TH) + tid] = F.E[tid];
        ((uint16_t *)(rw + rowmask_bases(TH)))[tid] = F.base[tid];
    }
    // edge masks and edge-cell roots for the boundary analysis; every such
    // root is seeded in the forest (lanes of one component store the same
    // word) and marked in the edge-root masks.  The four edges go to four
    // wavefronts (edge k to wavefront k mod NW), so their root loads and
    // stores overlap.
    {
        uint64_t *mk = v.masks + (size_t)t * mask_words(TH);
        uint32_t *rt = v.roots + (size_t)t * roots_per_tile(TH);
        const uint64_t mTop = uniform64(msk[0]), mBot = uniform64(msk[TH - 1]);
        auto root_g = [&](uint32_t n) {
            uint32_t e = lds_ld(&par[n]);  // n's root, or already the root's entry
            if (e < kPixel) e = lds_ld(&par[e]);
            const uint32_t pos = e & (kPixel - 1u);
            atomicOr((unsigned long long *)&flg[pos >> 6], 1ull << (pos & 63u));
            return global_index(v, tx, ty, TH, pos);
        };
        auto put = [&](uint32_t *dst, uint32_t g) {
            *dst = g;
            v.labels[g] = g + 1u;
        };
        const uint32_t bbLast = (uint32_t)F.base[NB - 1];
        if (wave == 0) {
            if (hasUp && lane_in(mTop)) put(&rt[roots_top(TH) + lane], root_g(bits_below(uniform64(F.E[0]))));
            if (lane == 0) {
                mk[kMaskTop] = mTop;
                mk[kMaskBottom] = mBot;
            }
        }
        if (wave == 1 % NW && hasDown && lane_in(mBot))
            put(&rt[roots_bottom(TH) + lane], root_g(bbLast + bits_below(uniform64(F.E[NB - 1]))));
        // per row (lane = row, 64 rows at a time): the band's first / last
        // interval holds the row's cell in the left / right column
        if (wave == 2 % NW || wave == 3 % NW) {
#pragma unroll
            for (int h = 0; h < col_words(TH); ++h) {
                const int r = 64 * h + lane;
                const uint64_t mr = r < TH ? msk[r] : 0ull;
                const bool lb = (mr & 1ull) != 0, rb = (mr >> 63) != 0;
                const uint32_t bFirst = r < TH ? (uint32_t)F.base[r >> 1] : 0u;
                const uint32_t nInt = r < TH ? (uint32_t)__popcll(F.E[r >> 1]) : 0u;
                const uint64_t mLeft = __ballot(lb), mRight = __ballot(rb);
                if (wave == 2 % NW) {
                    if (hasLeft && lb) put(&rt[roots_left(TH) + r], root_g(bFirst));
                    if (lane == 0) mk[kMaskLeft + h] = mLeft;
                }
                if (wave == 3 % NW) {
                    if (hasRight && rb) put(&rt[roots_right(TH) + r], root_g(bFirst + nInt - 1u));
                    if (lane == 0) mk[mask_right(TH) + h] = mRight;
                }
            }
        }
    }
    __syncthreads();  // every wavefront's marks are in
    for (int r = tid; r < TH; r += NT) rw[TH + r] = flg[r];
    then();
    __syncthreads();  // LDS may be reused for another tile
}

}  // namespace ccl
