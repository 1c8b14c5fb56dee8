"""The kernels and grids that calls launch, over the sizes the entry points
accept: HIP refuses a launch of 2^32 threads or more, so images of very few
rows or columns, which have many tiles for their pixels, decide what still
fits.  Runs without a GPU (launches are recorded, not made)."""
import pytest

from tests.launches import COUNT, IMG, LABELS, OUT, record


def _plain(H, W, conn=8, cfg=None):
    return ("ccl_label_2d_ex", [IMG, H, W, W, conn, LABELS, None, 0, cfg, None])


def _equal(H, W, conn=8, cfg=None):
    return ("ccl_label_2d_equal", [IMG, H, W, W, conn, LABELS, cfg, None])


def _accepted(results):
    for rc, launches in results:
        assert rc == 0 and launches and not any(l[4] for l in launches), (rc, launches)


def test_equal_value_thin_images(tmp_path):
    # the most tiles of 64 rows that four wavefronts each can take
    most = (2 ** 32 - 1) // 256
    res = record([_equal(1, 64 * most), _equal(64 * most, 1, 4), _equal(1, 64 * (most // 2)), _equal(2160, 3840)], tmp_path)
    _accepted(res)
    assert [ls[0][3] for _, ls in res] == [256, 256, 512, 512]


@pytest.mark.parametrize("conn", [4, 8])
def test_link_of_thin_images(tmp_path, conn):
    # 32-row tiles of one and two wavefronts: the local merge needs 64 and 128
    # threads a tile, and the link no more than 128
    most = (2 ** 32 - 1) // 128
    calls = [_plain(1, 64 * most - 5, conn, ("cfg", 32, nw)) for nw in (1, 2)]
    calls += [_plain(32 * most // 2, 1, conn, ("cfg", 32, 2)), _equal(1, 64 * most - 5, conn, ("cfg", 32, 2))]
    calls += [("ccl_label_2d_stats", [IMG, 1, 64 * most - 5, 64 * most - 5, conn, LABELS, OUT, 1, COUNT, ("cfg", 32, nw), None])
              for nw in (1, 2)]
    _accepted(record(calls, tmp_path))
    # elsewhere four wavefronts
    for _, ls in record([_plain(480, 640, conn), _plain(480, 640, conn, ("cfg", 32, 1))], tmp_path):
        assert ls[-1][3] == 256


def test_nothing_runs_when_a_launch_is_refused(tmp_path):
    # sixteen wavefronts a tile do not fit; the boundary analysis and the link
    # would read a workspace that no local merge has written
    n = 600000000
    calls = [_plain(1, n, 8, ("cfg", 64, 16)), _plain(1, n, 4, ("cfg", 32, 16)), _plain(n, 1, 8, ("cfg", 128, 16)),
             _equal(1, 1200000000), ("ccl_label_2d_timed", [IMG, 1, n, n, 8, LABELS, ("cfg", 64, 16), None, 0]),
             ("ccl_label_2d_stats", [IMG, 1, n, n, 8, LABELS, OUT, 1, COUNT, ("cfg", 64, 16), None]),
             ("ccl_label_2d_stats", [IMG, n, 1, 1, 4, LABELS, OUT, 1, COUNT, ("cfg", 16, 1), None])]
    for rc, launches in record(calls, tmp_path):
        assert rc == 4 and not launches


@pytest.mark.parametrize("fn", ["ex", "noalloc"])
def test_sizes_of_one_launch(tmp_path, fn):
    # (size, connectivity): one launch up to the line, three beyond it
    one = [(1, 1, 4), (320, 64, 4), (2, 8192, 4), (48, 384, 4), (319, 1, 4), (32, 512, 4), (320, 64, 8), (32, 640, 8),
           (2, 10240, 8), (46, 384, 8), (48, 576, 8), (120, 160, 8), (448, 64, 8), (447, 1, 8)]
    three = [(321, 64, 4), (2, 8193, 4), (120, 160, 4), (511, 1, 4), (32, 513, 4), (32, 641, 8), (46, 449, 8), (2, 10241, 8),
             (449, 64, 8), (48, 577, 8), (160, 160, 8), (512, 64, 8)]
    calls = [_plain(*s) if fn == "ex" else ("ccl_label_2d_noalloc", [IMG, s[0], s[1], s[1], s[2], LABELS, None])
             for s in one + three]
    for size, (rc, ls) in zip(one + three, record(calls, tmp_path)):
        assert rc == 0 and len(ls) == (1 if size in one else 3 if size[0] > 32 or size[1] > 64 else 2), (size, ls)


def test_tuning_leaves_small_images_in_one_launch(tmp_path):
    table = tmp_path / "tuning.jsonl"
    table.write_text('{"class": 14, "conn": 8, "tile_h": 64, "waves": 2, "ms": 0.01}\n')
    small, noalloc = _plain(120, 160), ("ccl_label_2d_noalloc", [IMG, 120, 160, 160, 8, LABELS, None])
    thin = _plain(20000, 1)  # of the same class, with too many lines
    calls = [small, ("ccl_tuning_load", [str(table)]), small, noalloc, thin, _plain(120, 160, 8, ("cfg", 64, 2)),
             ("ccl_autotune", [IMG, 120, 160, 160, 8, LABELS, 1, None, None, None]), small, thin]
    res = record(calls, tmp_path)
    assert all(rc == 0 for rc, _ in res)
    assert [len(res[i][1]) for i in (0, 2, 3, 7)] == [1, 1, 1, 1]
    assert res[4][1][0][0] == "k1_local_merge<64, 2, true, false>"
    assert len(res[5][1]) == 3
    assert len(res[8][1]) == 3 and res[8][1][0][0] != "k1_local_merge<32, 4, true, false>"


def test_timed_call_launches_what_the_plain_call_does(tmp_path):
    calls = []
    for H, W, conn in ((480, 640, 8), (480, 640, 4), (1080, 1920, 8), (2160, 3840, 4)):
        for cfg in (None, ("cfg", 32, 4), ("cfg", 64, 8)):
            calls += [_plain(H, W, conn, cfg), ("ccl_label_2d_timed", [IMG, H, W, W, conn, LABELS, cfg, None, 0])]
    res = record(calls, tmp_path)
    _accepted(res)
    for k in range(0, len(res), 2):
        assert res[k] == res[k + 1], calls[k]


@pytest.mark.parametrize("fn", ["ex", "noalloc", "timed"])
def test_wavefronts_of_the_merge(tmp_path, fn):
    # 8 on up to 512 tiles of 32 rows under 4-connectivity, else 4
    sizes = [(480, 640, 4, 512), (512, 2048, 4, 512), (513, 2048, 4, 256), (852, 3840, 4, 256), (480, 640, 8, 256),
             (852, 3840, 8, 256), (2160, 3840, 4, 256)]
    call = {"ex": lambda h, w, c: _plain(h, w, c),
            "noalloc": lambda h, w, c: ("ccl_label_2d_noalloc", [IMG, h, w, w, c, LABELS, None]),
            "timed": lambda h, w, c: ("ccl_label_2d_timed", [IMG, h, w, w, c, LABELS, None, None, 0])}[fn]
    res = record([call(h, w, c) for h, w, c, _ in sizes], tmp_path)
    _accepted(res)
    assert [ls[0][3] for _, ls in res] == [s[3] for s in sizes]
