"""The host side of the tiled GEMM (gemm_tile_plan.h), compiled with g++: where its kernels'
loads read, and which products qx_gemm and qx_gemm_a8 give to it. CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="session")
def tile_model(tmp_path_factory):
    """Runs tests/host/tile_model.cpp with one argument and a standard input: its lines."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("tile") / "tile_model")
    subprocess.run([gxx, "-O2", "-std=c++17", "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "tile_model.cpp"),
                    os.path.join(ROOT, "paper_2505_07531_amd", "csrc", "qx_api.cpp"), "-o", exe, "-pthread"], check=True)

    def run(what, text=""):
        return subprocess.run([exe, what], input=text, capture_output=True, text=True, check=True,
                              timeout=300).stdout.splitlines()
    return run


def test_tile_loads_stay_in_their_buffers(tile_model):
    """Every load of activations, codes and tables that the range check lets through reads
    inside its buffer, whether the check leaves the scalar offset out or takes it from the
    size: partial tiles of every number of rows, last super-rounds of one chunk."""
    lines = tile_model("reads")
    assert len(lines) > 100
    bad = [line for line in lines if line.split()[5:] != ["0", "0", "0"]]
    assert not bad, (len(bad), bad[:8])


def test_tile_order(tile_model):
    """Every tile is numbered once, and no XCD's run of tiles takes in many more weight tiles
    than an equal share of them needs (nx / 8 of them times the groups of activation tiles)."""
    cases = [(nx, my) for nx in (1, 2, 7, 8, 31, 64, 86) for my in (1, 2, 7, 8, 9, 10, 15, 16, 17, 25, 33, 57, 65)]
    for (nx, my), line in zip(cases, tile_model("order", "".join(f"{nx} {my}\n" for nx, my in cases))):
        once, most = (int(v) for v in line.split())
        assert once, (nx, my)
        assert most <= nx * ((my + 7) // 8) // 8 * 1.3 + 2, (nx, my, most)


FORMATS = {f"{'uc'[kind]}{b}g{g}": (b, kind, g) for b in (3, 4) for kind in (0, 1) for g in (32, 64, 128)}
FORMATS["q4x"] = (4, 2, 64)


def routes(tile_model, cases):
    """The kernel of each (format, int8 rows, n, k, m)."""
    return tile_model("route", "".join("%d %d %d %d %d %d %d\n" % (*FORMATS[f], a8, n, k, m) for f, a8, n, k, m in cases))


# (format, int8 rows, n, k, m): us in gemm.hip, us in the tiled shape that had taken the product
SMALL_TILES = {
    ("c4g32", 0, 11008, 4096, 24): (26.4, 31.2), ("c4g32", 0, 22016, 5120, 24): (54.6, 71.7),
    ("c4g32", 0, 11008, 4096, 48): (36.9, 43.5), ("c4g32", 1, 11008, 4096, 48): (41.7, 45.5),
    ("c4g64", 0, 22016, 8192, 24): (61.5, 76.2), ("c4g64", 1, 22016, 1024, 24): (13.9, 18.0),
    ("c4g128", 0, 22016, 2048, 24): (16.5, 18.6), ("q4x", 0, 12288, 4096, 24): (21.9, 23.7),
    ("c3g32", 0, 18944, 8192, 24): (53.0, 54.4), ("u4g128", 0, 12288, 5120, 24): (21.6, 23.5),
    ("u4g32", 0, 22016, 2048, 24): (15.5, 17.5), ("u3g128", 0, 22016, 1024, 24): (9.5, 11.5),
    ("q4x", 0, 14336, 1024, 48): (12.7, 16.7), ("u4g128", 0, 18944, 2048, 48): (19.8, 22.3),
    ("u4g128", 0, 18016, 3072, 50): (27.4, 31.5), ("c4g64", 0, 20432, 3072, 36): (36.0, 44.0), ("c4g64", 1, 20432, 3072, 62): (40.8, 46.9),
    ("c3g32", 0, 20432, 3072, 36): (34.7, 37.1), ("c4g64", 1, 13824, 5120, 30): (32.6, 37.5), ("c4g128", 1, 18016, 512, 24): (8.8, 10.7),
    ("u4g64", 0, 3346, 512, 50): (5.1, 5.7), ("c4g128", 0, 960, 512, 56): (5.2, 5.8), ("u4g128", 0, 1536, 1024, 44): (6.0, 6.6),
    ("u4g128", 0, 5781, 768, 39): (6.8, 7.9), ("c4g64", 0, 3305, 512, 24): (5.2, 5.8), ("c4g32", 0, 4121, 12288, 24): (40.3, 46.3),
    ("u3g128", 0, 4672, 512, 41): (5.9, 6.5), ("c4g64", 1, 15840, 1280, 54): (20.5, 22.9),
}


def test_short_and_tall_products_of_few_rows(tile_model):
    """17 to 64 rows, several rounds of blocks: the formats and chunk counts at which the
    32 x 32 tiles of gemm.hip measured faster than the tiled shapes go there."""
    got = dict(zip(SMALL_TILES, routes(tile_model, SMALL_TILES)))
    assert all(r == "gemm" for r in got.values()), got
    # and those that measured slower there stay: (33.7, 28.3), (16.6, 11.1), (29.2, 27.5), (5.1, 5.0) us
    keep = [("c4g32", 0, 8192, 8192, 24), ("c3g128", 0, 4096, 5120, 24), ("c4g32", 0, 4368, 9216, 24), ("u4g128", 0, 1241, 640, 50)]
    assert all(r in "EFGH" for r in routes(tile_model, keep))
    # the sizes by which test_gpu_tile.py runs that kernel in every format
    edges = [(f, 0, n, k, m) for f in FORMATS for n, k, m in ((12305, 640, 21), (12309, 1024, 50))]
    assert set(routes(tile_model, edges)) == {"gemm"}


def test_third_activation_tile_of_the_small_batch_kernel(tile_model):
    """33 to 48 rows on small matrices of 29 to 32 chunks stay with gemm_skinny.hip where it
    measured faster (us there / in the tiled shape that had taken them)."""
    small = {("c4g128", 0, 4096, 4096, 33): (10.2, 12.0), ("c4g128", 0, 4096, 4096, 48): (10.9, 11.7),
             ("u3g64", 0, 4096, 4096, 33): (9.2, 10.4), ("c3g128", 0, 2048, 4096, 40): (8.4, 9.2),
             ("u4g32", 0, 3072, 4096, 40): (9.3, 10.0), ("u3g64", 0, 1376, 3840, 33): (8.2, 9.3), ("u4g128", 0, 4096, 4096, 40): (9.8, 10.3)}
    got = dict(zip(small, routes(tile_model, small)))
    assert all(r == "skinny" for r in got.values()), got
    # slower there (12.0 / 10.9, 10.3 / 10.2, 9.1 / 8.9, 9.4 / 8.9, 19.1 / 14.4), and 49 rows and more
    keep = [("c3g32", 0, 4096, 4096, 33), ("u4g128", 0, 4096, 4096, 48), ("u4g128", 0, 1376, 4096, 40),
            ("c3g128", 0, 3072, 3712, 48), ("c3g128", 0, 8192, 4096, 40), ("c4g128", 0, 4096, 4096, 49)]
    assert all(r in "EFGH" for r in routes(tile_model, keep))


def test_int8_rows_of_uniform_weights(tile_model):
    """More than 64 int8 rows: sizes at which gemm_a8.hip measured faster than the tiled shape
    that had taken them (us there / in that shape)."""
    there = {("u3g128", 1, 8192, 4096, 600): (69.9, 88.4), ("u4g128", 1, 8192, 4096, 600): (70.7, 77.6),
             ("u3g64", 1, 8192, 1024, 600): (24.2, 29.9), ("u4g128", 1, 22016, 1024, 600): (52.1, 62.5),
             ("u3g128", 1, 2000, 4096, 2048): (54.0, 60.2), ("u4g64", 1, 4096, 1024, 1000): (19.4, 22.2)}
    got = dict(zip(there, routes(tile_model, there)))
    assert all(r == "gemm_a8" for r in got.values()), got
    # faster in a tiled shape (us in gemm_a8.hip / there)
    here = {("u3g64", 1, 11008, 4096, 512): (96, 86), ("u4g128", 1, 11008, 4096, 1000): (207, 119),
            ("u3g32", 1, 22016, 1024, 2048): (212, 178), ("u4g32", 1, 4096, 4096, 1000): (83, 66)}
    got = dict(zip(here, routes(tile_model, here)))
    assert all(r in "ABCDE" for r in got.values()), got


def test_table_formats_with_one_round_of_64x64_tiles(tile_model):
    """257 to 512 tiles of 64 x 64 in rows of up to 64 chunks: us in gemm.hip / in shape E."""
    there = {("c4g128", 0, 8192, 4096, 200): (43.5, 48.7), ("c4g128", 0, 2000, 4096, 1000): (43.6, 48.4),
             ("c3g32", 0, 8192, 4096, 200): (43.8, 46.5), ("c4g64", 1, 2000, 4096, 1000): (51.8, 57.9),
             ("q4x", 1, 8192, 1024, 200): (18.0, 20.4), ("c4g128", 1, 8192, 4096, 200): (49.1, 52.0)}
    got = dict(zip(there, routes(tile_model, there)))
    assert all(r == "gemm" for r in got.values()), got
    here = {("c3g128", 0, 8192, 4096, 200): (40.6, 38.1), ("c4g32", 0, 11008, 4096, 96): (68.6, 67.3)}
    got = dict(zip(here, routes(tile_model, here)))
    assert all(r == "E" for r in got.values()), got


def test_uniform_3_bit_g32_against_blocks_it_has(tile_model):
    """gemm.hip has no 128 x 256 blocks for 3-bit codes in groups of 32: its products are compared
    with the 128 x 64 tiles that run (us there / in the tiled shape)."""
    sizes = {("u3g32", 0, 11008, 4096, 600): (106, 79), ("u3g32", 0, 4096, 4096, 2048): (119, 88),
             ("u3g32", 0, 16384, 4096, 512): (110, 85), ("u3g32", 0, 8192, 11008, 1000): (292, 218),
             ("u3g32", 0, 11008, 4096, 300): (55.8, 54.8), ("u3g32", 0, 4096, 4096, 600): (55.5, 53.6)}
    got = dict(zip(sizes, routes(tile_model, sizes)))
    assert all(r in "ABCDE" for r in got.values()), got
    assert routes(tile_model, [("u3g32", 0, 4096, 4096, 400)]) == ["gemm"]  # 39.1 there, 41.0 in E


def test_gpu_sizes_reach_every_built_shape(tile_model):
    """The sizes that test_gpu_tile.py runs select every shape that is built, in every format
    and with both kinds of activations: a change of the cost model that takes a kernel out of
    that test's reach, or out of reach altogether, fails here."""
    from test_gpu_tile import sizes
    name = {v: f for f, v in FORMATS.items()}
    built = {}
    for line in tile_model("reads"):
        b, kind, g, a8, shape = line.split()[:5]
        built.setdefault((name[int(b), int(kind), int(g)], int(a8)), set()).add(shape)
    assert len(built) == 2 * len(FORMATS)
    for (f, a8), shapes in built.items():
        b, kind, g = FORMATS[f]
        got = set(routes(tile_model, [(f, a8, *s) for s in sizes((b, kind, g), a8)]))
        assert got >= shapes, (f, a8, shapes - got)


def test_uniform_fp16_rows_against_the_tiles_that_run(tile_model):
    """More than 64 fp16 rows of uniform weights: gemm.hip is priced by the tiles that it launches,
    with its weight tiles padded to the 8 XCDs (us there / in the tiled shape)."""
    there = {("u4g128", 0, 2496, 11008, 267): (55.2, 62.4), ("u4g64", 0, 3040, 5120, 489): (42.4, 46.6),
             ("u4g128", 0, 4277, 4096, 707): (50.3, 53.8), ("u4g128", 0, 3968, 4096, 816): (50.3, 53.6),
             ("u4g64", 0, 4128, 5120, 500): (60.5, 64.1), ("u4g128", 0, 4656, 13824, 200): (83.7, 98.2)}
    got = dict(zip(there, routes(tile_model, there)))
    assert all(r == "gemm" for r in got.values()), got
    here = {("u3g128", 0, 17024, 14336, 285): (272, 230), ("u3g64", 0, 1168, 1280, 2162): (36, 22),
            ("u3g64", 0, 4448, 8192, 1447): (280, 147), ("u4g64", 0, 4237, 3072, 778): (59, 44),
            ("u3g64", 0, 320, 2048, 2332): (34, 17)}
    got = dict(zip(here, routes(tile_model, here)))
    assert all(r in "ABCDEFGH" for r in got.values()), got


def test_int8_rows_of_codebook_3_avoid_the_spilling_shape(tile_model):
    """The 128 x 64 wave tile spills 16 registers for g64 (us in B / in D), 6 for g128, where it is the faster."""
    d = {("c3g64", 1, 18352, 3072, 1279): (260, 188), ("c3g64", 1, 21632, 3072, 784): (211, 164)}
    assert set(routes(tile_model, d)) == {"D"}
    assert routes(tile_model, [("c3g128", 1, 8192, 5120, 2048)]) == ["B"]  # 192 us, 215 in D


def test_int8_rows_of_codebook_3_never_ask_for_small_tiles(tile_model):
    """gemm.hip has no 32 x 32 tiles for int8 rows of codebook-3 g64 and g128: 17 to 64 of them
    always find a tiled shape."""
    cases = [(f, 1, n, 128 * c, m) for f in ("c3g64", "c3g128") for n in (1, 40, 4096, 8200, 12300, 16390, 18000, 20480, 28672, 300000)
             for c in (1, 2, 4, 5, 8, 12, 16, 24, 32, 64, 86, 112, 1024) for m in (17, 32, 33, 48, 64)]
    assert set(routes(tile_model, cases)) <= set("EFGH")
