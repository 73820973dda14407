"""What a call launches, through the library's own planner on the host
(quick_launch_plan, quick_grouped_launch_plan): which sizes run in the
wave-split form and which in a kernel that a configuration names."""
import ctypes
import os
import re

import pytest

import paper_2402_10076_amd as Q


@pytest.fixture(autouse=True)
def no_tune_table():
    Q.tune_table_clear()
    yield
    Q.tune_table_clear()


def wave(M, N, K, **kw):
    return Q.launch_plan(M, N, K, **kw)["variant"] == 0


def test_automatic_launch_is_reported(tmp_path):
    p = Q.launch_plan(1024, 4096, 8192)
    assert p["variant"] == 0 and p["tile_m"] % 16 == 0 and p["tile_n"] % 16 == 0
    assert p["k_ranges"] in (1, 2, 4, 8) and p["launches"] == 1 + (p["split_k"] >= 4)
    # where the rules stay with a nameable kernel it is the one select_config reports
    for M, N, K in ((1, 4096, 4096), (16, 12288, 4096)):
        p = Q.launch_plan(M, N, K)
        assert {f: p[f] for f in ("variant", "split_k", "tile_m", "tile_n")} == Q.select_config(M, N, K)
        assert p["k_ranges"] == 0 and p["launches"] == 1
    # a recorded configuration, and the automatic choice recorded as such
    t = tmp_path / "t.txt"
    t.write_text("quick-tune 1\n1024 4096 8192 2 2 128 32\n512 4096 8192 0 0 0 0\n")
    Q.tune_table_load(str(t))
    assert Q.launch_plan(1024, 4096, 8192) == dict(variant=2, split_k=2, tile_m=128, tile_n=32, k_ranges=0,
                                                   launches=2)
    assert wave(512, 4096, 8192) and wave(1024, 4096, 8192, cfg=Q.make_config())


def test_explicit_launch_is_the_configuration():
    c = Q.make_config(variant=6, split_k=2, tile_m=64, tile_n=32)
    assert Q.launch_plan(100, 4096, 4096, cfg=c) == dict(c.as_dict(), k_ranges=0, launches=2)
    assert Q.launch_plan(100, 4096, 4096, cfg=Q.make_config(variant=2, split_k=1))["launches"] == 1
    # the gated form pairs n-tiles: its stream kernel has two per wave
    assert Q.launch_plan(1, 4096, 4096)["tile_n"] == 1 and Q.launch_plan(1, 4096, 4096, gated=True)["tile_n"] == 2


def test_launch_plan_errors():
    assert Q.launch_plan(0, 4096, 4096) == dict.fromkeys(
        ("variant", "split_k", "tile_m", "tile_n", "k_ranges", "launches"), 0)
    assert Q.grouped_launch_plan(0, 8, 4096, 4096)["launches"] == 0
    L = Q.lib()
    p = ctypes.byref(Q.QuickLaunch())
    assert L.quick_launch_plan(1, 4096, 4096, None, 0, None) == Q.QUICK_ERR_INVALID_ARG
    assert L.quick_launch_plan(1, 4096, 4000, None, 0, p) == Q.QUICK_ERR_SHAPE
    assert L.quick_launch_plan(1 << 16, 32768, 128, None, 0, p) == Q.QUICK_ERR_SHAPE
    assert L.quick_launch_plan(1, 4112, 4096, None, 1, p) == Q.QUICK_ERR_SHAPE            # gated: N % 32
    bad = Q.make_config(variant=4)
    assert L.quick_launch_plan(1, 4096, 4096, ctypes.byref(bad), 0, p) == Q.QUICK_ERR_INVALID_ARG
    assert L.quick_grouped_launch_plan(8, 0, 4096, 4096, None, p) == Q.QUICK_ERR_SHAPE
    assert L.quick_grouped_launch_plan(8, 4, 4096, 4096, None, None) == Q.QUICK_ERR_INVALID_ARG


def test_grouped_launch_is_reported():
    p = Q.grouped_launch_plan(1024, 8, 28672, 4096)
    assert p["variant"] == 0 and p["split_k"] == 1 and p["launches"] == 1
    p = Q.grouped_launch_plan(1024, 8, 28672, 4096, cfg=Q.make_config(variant=2, split_k=2, tile_m=64, tile_n=32))
    assert p == dict(variant=2, split_k=2, tile_m=64, tile_n=32, k_ranges=0, launches=2)
    # 512 experts x 2^25 columns: more tiles than a grid of the wave-split form
    # holds, whatever their size, so the tiled kernel's resident workgroups run
    assert Q.grouped_launch_plan(32, 512, 1 << 25, 128)["variant"] == Q.VARIANT_STREAMK


# Which form the automatic choice takes where the lines of its rules lie: (M,
# N, K), sizes at which the other form was timed and is slower.
STREAM = [(3, 640, 27520), (4, 3408, 21632), (13, 816, 15488), (16, 1056, 8192), (4, 6432, 12672), (2, 5392, 25728),
          (2, 8192, 28672), (2, 7248, 12032), (2, 31232, 14592)]
STREAM_LEFT = [(16, 384, 11136), (16, 5120, 5120), (3, 9744, 11008), (4, 4560, 19584), (8, 5536, 6272),
               (2, 21504, 21760)]


@pytest.mark.parametrize("M,N,K", STREAM)
def test_few_rows_stay_with_the_stream_kernel(M, N, K):
    assert Q.launch_plan(M, N, K)["variant"] == Q.VARIANT_STREAM


@pytest.mark.parametrize("M,N,K", STREAM_LEFT)
def test_few_rows_leave_the_stream_kernel(M, N, K):
    assert Q.select_config(M, N, K)["variant"] == Q.VARIANT_STREAM and wave(M, N, K)


SLICED = [(16, 53168, 256), (16, 42448, 640), (12, 37232, 896), (10, 17504, 5376), (10, 12288, 4096),
          (16, 27648, 5120)]
SLICED_LEFT = [(16, 15360, 5120), (16, 22016, 4096), (13, 12400, 4736)]


@pytest.mark.parametrize("M,N,K", SLICED)
def test_nine_rows_on_stay_with_the_sliced_kernel(M, N, K):
    assert Q.launch_plan(M, N, K)["variant"] == Q.VARIANT_KSTREAM


@pytest.mark.parametrize("M,N,K", SLICED_LEFT)
def test_nine_rows_on_leave_the_sliced_kernel(M, N, K):
    assert Q.select_config(M, N, K)["variant"] == Q.VARIANT_KSTREAM and wave(M, N, K)


@pytest.mark.parametrize("M,N,K,form", [(10, 14240, 256, 2), (14, 8528, 256, 2), (9, 14240, 128, 2),
                                        (10, 14240, 384, 0)])
def test_nine_rows_on_short_k(M, N, K, form):
    assert Q.select_config(M, N, K)["variant"] == Q.VARIANT_TILED
    assert Q.launch_plan(M, N, K)["variant"] == form


@pytest.mark.parametrize("M,N,K,waves,tiles", [
    (2, 64048, 1024, 2, 2), (1, 30688, 1280, 4, 2), (2, 31568, 1664, 4, 2), (2, 23216, 1152, 4, 2),
    (7, 40496, 1152, 2, 2), (6, 57968, 1280, 2, 2),                          # short K
    (1, 57344, 8192, 4, 1), (1, 22016, 4096, 4, 1), (4, 22016, 4096, 4, 2), (3, 34320, 2304, 4, 2),
    (1, 8880, 11008, 8, 1), (1, 4096, 4096, 8, 1)])
def test_stream_kernel_shape(M, N, K, waves, tiles):
    assert Q.select_config(M, N, K) == dict(variant=Q.VARIANT_STREAM, split_k=waves, tile_m=0, tile_n=tiles)


TILED = [(26, 40192, 11776), (28, 24352, 23936), (32, 57344, 8192), (18, 35168, 4864), (23, 57712, 1920),
         (19, 3904, 23040), (44, 33408, 9472), (61, 33088, 8960),
         (220, 3504, 128), (24, 5536, 128), (98, 5120, 640), (54, 32288, 896), (43, 24656, 128),
         (1784, 1936, 1408), (580, 5840, 1408), (612, 5744, 512),
         (2026, 704, 2176), (1806, 720, 6784), (1731, 576, 12544),
         (512, 8192, 28672), (1024, 8192, 28672), (744, 4848, 22272), (1070, 7120, 18432)]
TILED_LEFT = [(27, 8816, 3840), (32, 12288, 4096), (33, 40192, 11776), (32, 27648, 5120), (41, 38800, 12544),
              (1448, 5760, 15872), (1029, 7808, 7808), (316, 23424, 7808), (500, 512, 640), (1000, 8192, 640), (200, 4096, 1024), (53, 24000, 768), (53, 24000, 1024), (141, 3264, 640), (177, 2704, 768),
              (1177, 2496, 896), (1000, 704, 2176), (2026, 1104, 2176), (878, 8272, 2560),
              (1505, 1248, 24960), (512, 10240, 8192), (256, 22016, 4096), (64, 4096, 4096)]


@pytest.mark.parametrize("M,N,K", TILED)
def test_more_rows_stay_with_the_tiled_kernel(M, N, K):
    assert Q.launch_plan(M, N, K)["variant"] in (Q.VARIANT_TILED, Q.VARIANT_STREAMK)


@pytest.mark.parametrize("M,N,K", TILED_LEFT)
def test_more_rows_leave_the_tiled_kernel(M, N, K):
    assert wave(M, N, K)


@pytest.mark.parametrize("M,N,K,waves", [(1, 26688, 10112, 4), (2, 26624, 12416, 4), (1, 10912, 9088, 4),
                                         (3, 16384, 8448, 4), (2, 9056, 9088, 8), (6, 22784, 2176, 4)])
def test_stream_kernel_shape_gated(M, N, K, waves):
    """The waves are chosen for the pairs of n-tiles that the gated form has."""
    p = Q.launch_plan(M, N, K, gated=True)
    assert (p["variant"], p["split_k"], p["tile_n"]) == (Q.VARIANT_STREAM, waves, 2)
    # set by the caller: kept
    p = Q.launch_plan(M, N, K, gated=True, cfg=Q.make_config(variant=1, split_k=8))
    assert (p["split_k"], p["tile_n"]) == (8, 2)


@pytest.mark.parametrize("M,N,K,form", [(16, 16544, 19968, 2), (12, 19136, 22912, 2), (13, 38528, 8448, 0)])
def test_largest_matrices_gated(M, N, K, form):
    assert wave(M, N, K) and Q.launch_plan(M, N, K, gated=True)["variant"] == form


@pytest.mark.parametrize("M,N,K,form", [(32, 55296, 1152, 2), (32, 41696, 768, 2), (24, 55904, 3968, 2),
                                        (41, 12384, 640, 0), (32, 22016, 4096, 0), (24, 35584, 6144, 0),
                                        (30, 42496, 6528, 0), (24, 12992, 22016, 2)])
def test_more_rows_gated(M, N, K, form):
    assert Q.launch_plan(M, N, K, gated=True)["variant"] == form


GATED = [(48, 28672, 4096), (64, 22016, 4096), (128, 12288, 4096), (256, 16384, 6144), (44, 33408, 9472),
         (128, 10240, 8192)]


@pytest.mark.parametrize("table", [False, True])
@pytest.mark.parametrize("M,N,K", GATED)
def test_automatic_gated_call_is_never_refused(M, N, K, table):
    """The tiled plan of these sizes has 16-column waves on 64 or 128 rows,
    which cannot pair a gate tile with its up tile: the automatic choice takes
    another form, with the committed tune table and without, and only a
    configuration that the caller names is refused."""
    if table:
        Q.tune_table_load(os.path.join(os.path.dirname(Q.LIB_PATH), "tune_mi355x.txt"))
    else:
        sel = Q.select_config(M, N, K)
        assert sel["tile_m"] > 32 and sel["tile_n"] == 16
    p = Q.launch_plan(M, N, K, gated=True)
    assert p["variant"] == 0 or p["tile_n"] == 32
    assert Q.launch_plan(M, N, K, gated=True, cfg=Q.make_config()) is not None
    with pytest.raises(Q.QuickError):
        Q.launch_plan(M, N, K, gated=True, cfg=Q.make_config(variant=2, split_k=1, tile_m=64, tile_n=16))


def _source_shapes(name, lower):
    """(rows, columns, K ranges[, rows of the lower tiles]) of the wave-split shapes in the library's source."""
    src = open(os.path.join(os.path.dirname(Q.LIB_PATH), "csrc", "quick_gemm.hip")).read()
    body = re.search(r"#define %s\(X\)(.*?[^\\])\n" % name, src, re.S).group(1)
    rows = [[float(v.rstrip("f")) for v in m.split(",")] for m in re.findall(r"X\((.*?)\)", body)]
    return {(int(16 * r[0]), int(16 * r[1] * r[2]), int(8 // r[2])) + ((int(16 * r[8]),) if lower else ())
            for r in rows}


def test_gpu_tests_run_every_wave_split_shape():
    """The sizes of test_wave_split_gpu.py run every shape of the form; gated
    ones and two K slices with each epilogue are among them; of the grouped
    form the full-height and, where it has one, the lower tiles."""
    import test_wave_split_gpu as t
    plans = [Q.launch_plan(*s) for s in t.SIZES]
    run = {(p["tile_m"], p["tile_n"], p["k_ranges"]) for p in plans if p["variant"] == 0}
    assert run == _source_shapes("QUICK_WSPLIT_SHAPES", False)
    assert {p["split_k"] for p in plans if p["variant"] == 0} >= {1, 2, 4, 8}
    long_one_range = {(p["tile_m"], p["tile_n"]) for s, p in zip(t.SIZES, plans)
                      if p["variant"] == 0 and p["k_ranges"] == 1 and s[2] // 128 >= 9}
    assert long_one_range >= {(m, n) for m, n, k in run if k == 1 and (m, n) != (96, 512)}
    for gated in (False, True):
        assert any(p["variant"] == 0 and p["split_k"] == 2
                   for p in (Q.launch_plan(*s, gated=gated) for s in t.EPILOGUES))
    bodies = set()
    for counts, N, K in t.GROUPS:
        p = Q.grouped_launch_plan(sum(counts), len(counts), N, K)
        for r in counts:
            tile = p["tile_m"], p["tile_n"], p["k_ranges"]
            bodies |= {tile + (-(-r // -(-r // tile[0])),)} if r else set()
    for tm, tn, kr, low in _source_shapes("QUICK_WSPLIT_GRP_SHAPES", True):
        rows = [b[3] for b in bodies if b[:3] == (tm, tn, kr)]
        assert any(r > low for r in rows) or low == tm, (tm, tn, kr)
        assert any(r <= low for r in rows), (tm, tn, kr)
