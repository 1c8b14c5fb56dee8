// Per-component statistics of a canonical labeling: area, inclusive
// bounding box and the sums of the pixels' column and row indices (the
// size and location of every component, which is what the applications in
// the paper's introduction use the labels for).
//
// A component's root is the pixel whose label is its own raster index + 1.
// Roots are numbered in raster order, so records come out in increasing
// label order:
//   st_roots     one 64-bit root mask per 64-pixel row word (lane = pixel)
//                and the number of roots per block of 256 words;
//   st_scan      exclusive scan of the block counts (one workgroup); only for
//                images of many blocks, in others every block of st_bases
//                adds up the counts before its own;
//   st_bases     exclusive scan inside each block: the first record index
//                of every word, and the records of its roots initialised;
//                the total;
//   st_accum     a wavefront takes 16 rows of a 64-pixel column and gathers
//                the labels that fill much of it one at a time, from lane
//                masks; what is left goes run by run (runs of equal labels in
//                a row).  Both add to a hash table in LDS keyed by label per
//                128 x 128 block, which is added to the records once per slot
//                with global atomics.
#include <hip/hip_runtime.h>

#include "ccl.h"
#include "ccl_device.h"
#include "ccl_internal.h"

namespace ccl {

namespace {

constexpr int kWordsPerBlock = 256;
constexpr uint32_t kEmpty = 0u;  // no component has label 0

__global__ void __launch_bounds__(256) st_roots(const uint32_t *L, uint32_t W, uint32_t WW,
                                                 uint32_t words, uint64_t *mask, uint32_t *bsum) {
    __shared__ uint32_t part[4];
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr int kWords = kWordsPerBlock / 4, kBatch = 16;
    uint32_t cnt = 0;
#pragma unroll 1
    for (int i0 = 0; i0 < kWords; i0 += kBatch) {
        const uint32_t w0 = blockIdx.x * kWordsPerBlock + (uint32_t)(wave * kWords + i0);
        if (w0 >= words) break;  // wave-uniform
        uint32_t y = w0 / WW, wx = w0 - y * WW;
        // the batch's loads are in flight together
        uint32_t l[kBatch], p[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const uint32_t x = wx * (uint32_t)kTileW + (uint32_t)lane;
            const bool in = w0 + (uint32_t)i < words && x < W;
            p[i] = y * W + x;
            // outside the image its own index, never a root's label (0 is one's
            // where p + 1 wraps around, H * W being close to 2^32)
            l[i] = in ? L[p[i]] : p[i];
            if (++wx == WW) {
                wx = 0u;
                ++y;
            }
        }
        uint64_t mine = 0ull;  // lane i: word i's mask
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const uint64_t m = __ballot(l[i] == p[i] + 1u);
            if (lane == i) mine = m;
            cnt += (uint32_t)__popcll(m);
        }
        if (lane < kBatch && w0 + (uint32_t)lane < words) mask[w0 + (uint32_t)lane] = mine;
    }
    if (lane == 0) part[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) bsum[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Blocks whose counts every block of st_bases adds up by itself.  The sums
// read nb * nb / 2 counts from the L2, 8 MB at 2048 blocks (32 Mi pixels where
// W is a multiple of 64); a scan is a launch of its own.  Counting background
// only, with the sums and with the scan: 1080 x 1920 12.7 and 15.6 us, 4096 x
// 4096 (1024 blocks) 30.4 and 32.7, 4096 x 8192 (2048) 53.9 and 55.9, 8192 x 8192
// (4096) 97.8 and 100.0, 12288 x 12288 (9216) 249.9 and 246.5; between 2048 and
// 8192 blocks there is 2 % in it.
constexpr uint32_t kSelfScanBlocks = 2048u;

__global__ void __launch_bounds__(1024) st_scan(uint32_t *bsum, uint32_t nb) {
    __shared__ uint32_t s[1024];
    const uint32_t tid = threadIdx.x;
    const uint32_t per = (nb + 1023u) / 1024u;
    const uint32_t b0 = tid * per, b1 = min(nb, b0 + per);
    uint32_t acc = 0;
    for (uint32_t b = b0; b < b1; ++b) acc += bsum[b];
    s[tid] = acc;
    __syncthreads();
    for (uint32_t off = 1; off < 1024u; off <<= 1) {
        const uint32_t v = tid >= off ? s[tid - off] : 0u;
        __syncthreads();
        s[tid] += v;
        __syncthreads();
    }
    uint32_t run = s[tid] - acc;
    for (uint32_t b = b0; b < b1; ++b) {
        const uint32_t t = bsum[b];
        bsum[b] = run;
        run += t;
    }
}

// SELF: bsum holds the blocks' counts, else their exclusive prefix.
template <bool SELF>
__global__ void __launch_bounds__(kWordsPerBlock) st_bases(const uint64_t *mask, const uint32_t *bsum,
                                                uint32_t words, uint32_t W, uint32_t WW,
                                                uint32_t *base, ccl_component *out, uint32_t cap,
                                                uint32_t *n_out) {
    __shared__ uint32_t part[2][4];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t w = blockIdx.x * kWordsPerBlock + tid;
    const uint64_t m = w < words ? mask[w] : 0ull;
    uint32_t before = 0u;
    if (SELF) {
        for (uint32_t j = tid; j < blockIdx.x; j += kWordsPerBlock) before += bsum[j];
        wave_exclusive_scan(before, &before);
    }
    uint32_t wtot;
    const uint32_t ex = wave_exclusive_scan((uint32_t)__popcll(m), &wtot);
    if (lane == 0) {
        part[0][wave] = before;
        part[1][wave] = wtot;
    }
    __syncthreads();
    uint32_t b = SELF ? 0u : bsum[blockIdx.x], total = 0u;
#pragma unroll
    for (uint32_t j = 0; j < 4u; ++j) {
        if (SELF) b += part[0][j];
        total += part[1][j];
    }
    if (blockIdx.x + 1u == gridDim.x && tid == 0) *n_out = b + total;
    b += ex;
#pragma unroll
    for (uint32_t j = 0; j < 4u; ++j) b += j < wave ? part[1][j] : 0u;
    if (w >= words) return;
    base[w] = b;
    const uint32_t y = w / WW, p0 = y * W + (w - y * WW) * (uint32_t)kTileW;
    uint64_t mm = m;
    uint32_t id = b;
    while (mm) {
        const uint32_t j = (uint32_t)__builtin_ctzll(mm);
        mm &= mm - 1ull;
        if (id < cap) {
            ccl_component &r = out[id];
            r.label = p0 + j + 1u;
            r.area = 0u;
            r.x_min = 0xFFFFFFFFu;
            r.y_min = 0xFFFFFFFFu;
            r.x_max = 0u;
            r.y_max = 0u;
            r.sum_x = 0ull;
            r.sum_y = 0ull;
        }
        ++id;
    }
}

__device__ __forceinline__ void add_global(ccl_component &r, uint32_t len, uint32_t xmn, uint32_t xmx,
                                           uint32_t ymn, uint32_t ymx, uint64_t sxv, uint64_t syv) {
    atomicAdd(&r.area, len);
    atomicMin(&r.x_min, xmn);
    atomicMax(&r.x_max, xmx);
    atomicMin(&r.y_min, ymn);
    atomicMax(&r.y_max, ymx);
    atomicAdd((unsigned long long *)&r.sum_x, (unsigned long long)sxv);
    atomicAdd((unsigned long long *)&r.sum_y, (unsigned long long)syv);
}

// Record index of the component whose root pixel is r (its label - 1).
__device__ __forceinline__ uint32_t record_of(uint32_t r, uint32_t W, uint32_t WW,
                                              const uint64_t *mask, const uint32_t *base) {
    const uint32_t rx = r % W;
    const uint32_t w = (r / W) * WW + rx / (uint32_t)kTileW;
    return base[w] + (uint32_t)__popcll(mask[w] & ((1ull << (rx & 63u)) - 1ull));
}

// Block of 128 x 128 pixels, a wavefront per 64 columns and 16 rows.  The hash
// table is keyed by label, so an addition needs no global read; the record
// index is looked up once per table slot when the block flushes.  Bound by the
// chain of LDS round trips in a wavefront and by the flushes of components
// that reach many blocks (atomics on one record follow each other).  At most
// 80 scalar registers (eight wavefronts per SIMD), so that two workgroups
// share a compute unit; with 112 one ran at a time.  Gathering a label over a
// wavefront's strip makes its eight LDS additions once per strip instead of
// once per row.  2160 x 3840 smoothed labels: 40 to 52 us by the field drawn with
// blocks of 64 x 256 that added run by run, 26 to 43 so.  Blocks of 128 x 256
// took 15 to 30 % less on large images of large components, but up to 7 % more
// where components are many and small (4-connectivity, p = 0.3), with half as
// many workgroups to share them.
constexpr int kAccWaves = 16, kAccStripRows = 16;
constexpr int kAccCols = 2 * kTileW;
constexpr int acc_rows(int waves) { return waves / 2 * kAccStripRows; }
constexpr int kAccRows = acc_rows(kAccWaves);
constexpr int kAccSlots = 1024;
// A workgroup takes up to this many blocks below each other, as many as leave
// two workgroups per compute unit (kAccGroups), and flushes when its table is
// half full, or at the end: where components are few and large, as many
// blocks share one flush.  4096 x 4096 p = 0.5, 8-connectivity: 115 us a call
// with a flush per block, 82 so; 6000 x 7000 smoothed 108 us, against 227 with
// the blocks of 64 columns.  With half the workgroups 2160 x 3840 smoothed
// takes 42 us instead of 50, but dense small components lose 4 %.
constexpr uint32_t kAccMaxBlocks = 8u, kAccGroups = 512u;
// the table's 32-bit coordinate sums hold a workgroup whose pixels all have one
// label
static_assert((uint64_t)kAccCols * kAccRows * kAccMaxBlocks * (kAccRows * kAccMaxBlocks - 1u) <= 0xFFFFFFFFull &&
                  (uint64_t)kAccCols * kAccRows * kAccMaxBlocks * (kAccCols - 1) <= 0xFFFFFFFFull,
              "coordinate sums relative to the workgroup's first pixel fit 32 bits");
// Wavefronts per block: 16, but 4 (blocks of 32 rows) or 8 (64 rows) on images
// of few blocks.  There a block of 128 x 128 leaves the chip idle while one
// workgroup adds the runs of 16384 pixels, whose components may also be more
// than its table has slots for; on larger images the small blocks' flushes of
// one large component follow each other.  Worst over noise of p = 0.1 .. 0.9,
// smoothed fields and blobs, as a share of the speed of 64 x 256 blocks:
//   128 x 128    16 waves 0.60, 8 0.97, 4 1.08
//   480 x 640    (75 blocks of 32 rows) 0.83, 1.15, 1.00
//   640 x 800    (140; 70 of 64 rows) 0.94, 1.06, 0.84
//   720 x 1280   (240; 120) 1.00, 1.00, 0.74
//   1080 x 1920  (510; 255) 1.02, 0.85, 0.54
//   60 x 8192    (128; 64) 0.78, 0.76, 1.00
inline int acc_waves(uint32_t H, uint32_t W) {
    const uint64_t cols = ((uint64_t)W + kAccCols - 1u) / kAccCols;
    auto blocks = [&](int waves) { return cols * (((uint64_t)H + acc_rows(waves) - 1u) / acc_rows(waves)); };
    if (blocks(4) <= (H <= 64u ? 128u : 96u)) return 4;
    return blocks(8) <= 128u ? 8 : kAccWaves;
}
// Labels gathered over the strip at most (with 256-row blocks 1, 2, 4 and 8
// measured 28.1, 27.6, 29.0 and 30.3 us), and the pixels a gathered label must have had for another
// one to be tried: a strip of small components is cheaper run by run.
constexpr int kAccGather = 2;
constexpr uint32_t kAccGatherPixels = 24u;

// SEVERAL: more than one block per workgroup.
template <int WAVES, bool SEVERAL>
__global__ void __launch_bounds__(WAVES * 64, 8) st_accum(const uint32_t *L, uint32_t H, uint32_t W,
                                                          uint32_t WW, const uint64_t *mask,
                                                          const uint32_t *base, ccl_component *out,
                                                          uint32_t cap, uint32_t blocks) {
    const uint32_t per = SEVERAL ? blocks : 1u;
    // extents and sums relative to the first block's first pixel (a sum is at
    // most 2^17 * 1023)
    __shared__ uint32_t key[kAccSlots], area[kAccSlots], xmn[kAccSlots], ymn[kAccSlots],
        xmx[kAccSlots], ymx[kAccSlots], sx[kAccSlots], sy[kAccSlots];
    __shared__ uint32_t used;
    constexpr int NT = WAVES * 64;
    constexpr uint32_t kRows = acc_rows(WAVES);
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto clear = [&] {
        for (int i = tid; i < kAccSlots; i += NT) {
            key[i] = kEmpty;
            area[i] = 0u;
            xmn[i] = ymn[i] = 0xFFFFFFFFu;
            xmx[i] = ymx[i] = 0u;
            sx[i] = sy[i] = 0u;
        }
        if (tid == 0) used = 0u;
    };
    clear();
    __syncthreads();
    const uint32_t bx = blockIdx.x * (uint32_t)kAccCols, by = blockIdx.y * kRows * per;
    const uint32_t xr = (uint32_t)(wave & 1) * kTileW;  // the wavefront's first column and row in the block
    const uint32_t n = H * W;
    const uint32_t x = bx + xr + (uint32_t)lane;
    const bool xin = x < W;
    auto to_record = [&](uint32_t l, uint32_t len, uint32_t xa, uint32_t xb, uint32_t ya, uint32_t yb,
                         uint32_t sxv, uint32_t syv) {
        const uint32_t id = record_of(l - 1u, W, WW, mask, base);
        if (id < cap)
            add_global(out[id], len, bx + xa, bx + xb, by + ya, by + yb, (uint64_t)len * bx + sxv,
                       (uint64_t)len * by + syv);
    };
    // Adds one run (or a strip's pixels of one label) to the LDS table.
    auto add_lds = [&](uint32_t l, uint32_t len, uint32_t xa, uint32_t xb, uint32_t ya, uint32_t yb,
                       uint32_t sxv, uint32_t syv) {
        uint32_t h = (l * 2654435761u) >> 22;  // 10 bits
        for (int probe = 0; probe < 16; ++probe) {
            const uint32_t kk = atomicCAS(&key[h], kEmpty, l);
            if (kk == kEmpty || kk == l) {
                if (SEVERAL && kk == kEmpty) atomicAdd(&used, 1u);
                atomicAdd(&area[h], len);
                atomicMin(&xmn[h], xa);
                atomicMax(&xmx[h], xb);
                atomicMin(&ymn[h], ya);
                atomicMax(&ymx[h], yb);
                atomicAdd(&sx[h], sxv);
                atomicAdd(&sy[h], syv);
                return;
            }
            h = (h + 1u) & (uint32_t)(kAccSlots - 1);
        }
        // table full around h: straight to the record
        to_record(l, len, xa, xb, ya, yb, sxv, syv);
    };
#pragma unroll 1
    for (uint32_t j = 0; j < per && by + j * kRows < H; ++j) {  // workgroup-uniform
        const uint32_t yw = j * kRows + (uint32_t)(wave >> 1) * kAccStripRows;
        // all the strip's rows are loaded first, so the loads overlap
        uint32_t lv[kAccStripRows];
#pragma unroll
        for (int k = 0; k < kAccStripRows; ++k) {
            const uint32_t y = by + yw + (uint32_t)k;
            const uint32_t l = xin && y < H ? L[y * W + x] : 0u;
            lv[k] = l <= n ? l : 0u;  // (labels above H*W: not canonical)
        }
#pragma unroll 1
        for (int g = 0; g < kAccGather; ++g) {
            // a label still in the strip: the topmost one of the first column
            // that has any
            uint32_t c = 0u;
#pragma unroll
            for (int k = kAccStripRows - 1; k >= 0; --k) c = lv[k] ? lv[k] : c;
            const uint64_t any = __ballot(c != 0u);
            if (!any) break;
            const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)c, __builtin_ctzll(any));
            // its pixels per column (lanes) and per row; they leave the strip
            uint32_t cnt = 0u, area = 0u, sr = 0u, ymask = 0u;
            uint64_t xmask = 0ull;
#pragma unroll
            for (int k = kAccStripRows - 1; k >= 0; --k) {
                const bool is = lv[k] == l;
                const uint64_t m = __ballot(is);
                cnt += is ? 1u : 0u;
                lv[k] = is ? 0u : lv[k];
                xmask |= m;
                ymask |= m ? 1u << k : 0u;
                area += (uint32_t)__popcll(m);
                if (k > 0) sr += area;  // the pixels of rows >= k, summed over k >= 1: every pixel's row
            }
            uint32_t sc;  // column sum, at most 16 * 2016
            wave_exclusive_scan(cnt * (uint32_t)lane, &sc);
            if (lane == 0)
                add_lds(l, area, xr + (uint32_t)__builtin_ctzll(xmask), xr + 63u - (uint32_t)__builtin_clzll(xmask),
                        yw + (uint32_t)__builtin_ctz(ymask), yw + 31u - (uint32_t)__builtin_clz(ymask),
                        area * xr + sc, area * yw + sr);
            if (area < kAccGatherPixels) break;
        }
#pragma unroll
        for (int k = 0; k < kAccStripRows; ++k) {
            const uint32_t y = yw + (uint32_t)k;
            const uint32_t l = lv[k];
            const uint32_t ll = from_left(l, 0u), lr = from_right(l, 0u);
            const uint64_t E = __ballot(l != 0u && l != lr);
            if (!E) continue;  // wave-uniform
            if (l == 0u || l == ll) continue;
            // this lane starts a run of equal labels; it ends at the first run
            // end at or after it
            const uint32_t e = (uint32_t)lane + (uint32_t)__builtin_ctzll(E >> lane);
            const uint32_t len = e - (uint32_t)lane + 1u, xa = xr + (uint32_t)lane, xb = xr + e;
            add_lds(l, len, xa, xb, y, y, len * (xa + xb) / 2u, len * y);
        }
        __syncthreads();
        const bool last = j + 1u == per || by + (j + 1u) * kRows >= H;
        if (SEVERAL) {
            const bool full = used > (uint32_t)kAccSlots / 2u;
            __syncthreads();  // every wavefront has read it before the next block counts on
            if (!last && !full) continue;
        }
        for (int i = tid; i < kAccSlots; i += NT) {
            const uint32_t l = key[i];
            if (l == kEmpty) continue;
            to_record(l, area[i], xmn[i], xmx[i], ymn[i], ymx[i], sx[i], sy[i]);
        }
        if (!SEVERAL || last) break;
        __syncthreads();
        clear();
        __syncthreads();
    }
}

}  // namespace

size_t stats_workspace_bytes(int32_t H, int32_t W) {
    const size_t WW = ((size_t)W + kTileW - 1) / kTileW;
    const size_t words = (size_t)H * WW;
    const size_t nb = (words + kWordsPerBlock - 1) / kWordsPerBlock;
    return align_up(words * sizeof(uint64_t), 256) + align_up(words * sizeof(uint32_t), 256) +
           align_up(nb * sizeof(uint32_t), 256);
}

}  // namespace ccl

using namespace ccl;

extern "C" int ccl_component_stats(const uint32_t *labels, int32_t H, int32_t W,
                                   ccl_component *out, int64_t capacity, uint32_t *n_out,
                                   void *stream) {
    if (!labels || !n_out || H <= 0 || W <= 0 || capacity < 0 || (capacity > 0 && !out))
        return CCL_ERR_INVALID_ARG;
    if ((uint64_t)H * (uint64_t)W > 0xFFFFFFFFull) return CCL_ERR_TOO_LARGE;
    hipStream_t s = (hipStream_t)stream;
    void *ws = nullptr;
    std::unique_lock<std::mutex> held;
    int rc = stream_workspace(s, stats_workspace_bytes(H, W), &ws, &held);
    if (rc != CCL_OK) return rc;
    const uint32_t WW = (uint32_t)((W + kTileW - 1) / kTileW);
    const uint32_t words = (uint32_t)H * WW;
    const uint32_t nb = (words + kWordsPerBlock - 1) / kWordsPerBlock;
    char *p = (char *)ws;
    uint64_t *mask = (uint64_t *)p;
    uint32_t *base = (uint32_t *)(p + align_up((size_t)words * sizeof(uint64_t), 256));
    uint32_t *bsum = (uint32_t *)((char *)base + align_up((size_t)words * sizeof(uint32_t), 256));
    const uint32_t cap = capacity > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)capacity;
    hipLaunchKernelGGL(st_roots, dim3(nb), dim3(256), 0, s, labels, (uint32_t)W, WW, words, mask, bsum);
    if (nb <= kSelfScanBlocks) {
        hipLaunchKernelGGL(st_bases<true>, dim3(nb), dim3(kWordsPerBlock), 0, s, mask, bsum, words, (uint32_t)W, WW,
                           base, out, cap, n_out);
    } else {
        hipLaunchKernelGGL(st_scan, dim3(1), dim3(1024), 0, s, bsum, nb);
        hipLaunchKernelGGL(st_bases<false>, dim3(nb), dim3(kWordsPerBlock), 0, s, mask, bsum, words, (uint32_t)W, WW,
                           base, out, cap, n_out);
    }
    const uint32_t cols = ((uint32_t)W + kAccCols - 1u) / kAccCols, rows = ((uint32_t)H + kAccRows - 1u) / kAccRows;
    const uint64_t per = min((uint64_t)kAccMaxBlocks, max((uint64_t)1, (uint64_t)cols * rows / kAccGroups));
    const dim3 grid(cols, (rows + (uint32_t)per - 1u) / (uint32_t)per);
    auto accumulate = [&](auto kernel, dim3 g, int waves) {
        hipLaunchKernelGGL(kernel, g, dim3(waves * 64), 0, s, labels, (uint32_t)H, (uint32_t)W, WW, mask, base, out, cap,
                           (uint32_t)per);
    };
    const int waves = acc_waves((uint32_t)H, (uint32_t)W);
    const dim3 small(cols, ((uint32_t)H + acc_rows(waves) - 1u) / acc_rows(waves));
    if (waves == 4) accumulate(st_accum<4, false>, small, 4);
    else if (waves == 8) accumulate(st_accum<8, false>, small, 8);
    else if (per > 1u) accumulate(st_accum<kAccWaves, true>, grid, kAccWaves);
    else accumulate(st_accum<kAccWaves, false>, grid, kAccWaves);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e);
    return CCL_OK;
}
