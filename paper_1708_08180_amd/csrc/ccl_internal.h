// Host-side interface between the C ABI layer and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>

#include "ccl.h"
#include "ccl_device.h"

namespace ccl {

// True when (tile_h, waves) names a compiled kernel configuration.
bool config_supported(int th, int nw);

// The three batch kernels of one configuration.  Each takes one BatchArgs
// by value.  Grids: local merge and link one workgroup (block1 / block3
// threads) per tile; boundary analysis one workgroup (block2 threads) per
// tiles_per_group2 tiles.
struct BatchKernels {
    const void *k1, *k2, *k3;
    unsigned block1, block2, block3;
    unsigned tiles_per_group2;
};
bool batch_kernels(int th, int nw, int conn, BatchKernels *out);

// True when (tile_h, waves) is compiled for equal-value labeling.
bool config_supported_equal(int th, int nw);

// Enqueue the three phases for one image on `s`.  With ev != nullptr,
// ev[0..3] are recorded before phase 1, between the phases and after phase 3.
// equal: label every equal-value class instead of the nonzero foreground.
hipError_t launch_plain(const ImgView &v, int th, int nw, int conn, hipStream_t s,
                        hipEvent_t *ev = nullptr, bool equal = false);

// Images that label_small takes whole (binary labeling; one launch, no
// workspace), and that launch.
bool small_image(int H, int W, int conn);
hipError_t launch_small(const ImgView &v, int conn, hipStream_t s);

// The boundary analysis of binary labeling for one image on `s`, without the
// other phases (tiles of at most 64 rows).
hipError_t launch_boundary(const ImgView &v, int th, int conn, hipStream_t s);
// The supported tile configurations of at most 64 rows (X(tile_h, waves)).
#define CCL_FOR_EACH_LOW_CONFIG(X)                                                          \
    X(16, 1) X(16, 2) X(16, 4) X(16, 8) X(32, 1) X(32, 2) X(32, 4) X(32, 8) X(32, 16) \
        X(64, 1) X(64, 2) X(64, 4) X(64, 8) X(64, 16)

// Workspace layout for one image: edge masks, edge-cell roots, row masks
// (row foreground and edge-root masks), run slots.
struct WsLayout {
    size_t tiles;
    size_t mask_bytes;
    size_t root_bytes;
    size_t rowmask_bytes;
    size_t slot_bytes;
    size_t total;
};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline WsLayout ws_layout(int H, int W, int th, bool equal = false) {
    WsLayout l;
    const size_t tx = ((size_t)W + kTileW - 1) / kTileW;
    const size_t ty = ((size_t)H + th - 1) / th;
    l.tiles = tx * ty;
    l.mask_bytes = align_up(l.tiles * (size_t)mask_words(th) * sizeof(uint64_t), 256);
    l.root_bytes = align_up(l.tiles * (size_t)roots_per_tile(th) * sizeof(uint32_t), 256);
    l.rowmask_bytes = align_up(l.tiles * (size_t)rowmask_words(th) * sizeof(uint64_t), 256);
    const size_t spr = equal ? (size_t)slots_per_row<true>() : (size_t)slots_per_row<false>();
    l.slot_bytes = align_up(l.tiles * (size_t)th * spr * sizeof(uint16_t), 256);
    l.total = l.mask_bytes + l.root_bytes + l.rowmask_bytes + l.slot_bytes;
    return l;
}

// Whether a launch of `groups` workgroups of `threads` threads is one that HIP
// accepts: fewer than 2^32 threads in all.
inline bool grid_fits(uint64_t groups, unsigned threads) { return groups * threads <= 0xFFFFFFFFull; }

// Shared by the entry points.
int fail_hip(hipError_t e);
// The library's workspace for (current device, stream), at least `need`
// bytes (grown on demand, in stream order).  *held receives the cache lock,
// to be kept until the kernels that use the buffer are enqueued.
int stream_workspace(hipStream_t s, size_t need, void **out, std::unique_lock<std::mutex> *held);
// Frees the cached workspace of (current device, s), in stream order on s.
void release_stream_workspace(hipStream_t s);
// Image arguments: a non-null image of H x W >= 1 bytes per row pitch >= W
// and H * W <= 2^32 - 1.
int validate_image_only(const void *img, int32_t H, int32_t W, int64_t pitch);
// The same, and a non-null label buffer of H * W u32 whose bytes do not
// overlap the image's.
int validate_image(const void *img, int32_t H, int32_t W, int64_t pitch, const void *labels);
// True when [a, a + na) and [b, b + nb) share a byte.
bool byte_ranges_overlap(const void *a, unsigned __int128 na, const void *b, unsigned __int128 nb);
// Tile configuration of a call: the caller's, else the tuning table's, else the
// built-in one.  *builtin (may be null): neither chose one.
int resolve_config(int H, int W, int conn, const ccl_config *cfg, int *th, int *nw, bool *builtin = nullptr);
void default_config(int H, int W, int conn, int *th, int *nw, bool *builtin = nullptr);
// Wavefronts the local merge of one image runs with where nobody chose a
// configuration (the other phases and the workspace depend on the tile height
// alone): 8 for up to 512 32-row tiles under 4-connectivity, whose bands hold
// twice the intervals, so that the loops over a tile's nodes take one pass while
// wavefront slots are idle.  us a call with 4 and with 8, noise p = 0.5: 480 x
// 640 16.2 and 15.6, 720 x 1280 (460 tiles) 17.5 and 17.1, 1080 x 1920 (1020)
// 19.8 and 19.7, where smoothed fields take 21.9 and 22.3; 1200 x 2000 (1216
// tiles, more than the chip's slots hold at once with 8) 21.1 and 22.7.  Under
// 8-connectivity 8 is never faster: 480 x 640 18.9 both, 1200 x 2000 25.5 and 28.1.
inline int merge_waves(const ImgView &v, int th, int nw, int conn) {
    return th == 32 && nw == 4 && conn == 4 && (int64_t)v.tilesX * v.tilesY <= 512 ? 8 : nw;
}
// The kernels' view of one image whose workspace (ws_layout(H, W, th,
// equal).total bytes, 256-byte aligned) starts at ws.
ImgView make_view(const uint8_t *img, int32_t H, int32_t W, int64_t pitch, uint32_t *labels,
                  void *ws, int th, bool equal = false);

}  // namespace ccl
