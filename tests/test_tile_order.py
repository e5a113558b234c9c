"""csrc/tile_order.h on the CPU: every tile of a grid belongs to exactly one workgroup, and no XCD
(workgroup id mod 8) is given much more than its share of the tiles."""
import os
import subprocess

import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2405_01943_amd", "csrc",
                      "tile_order.h")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#define __device__
#define __forceinline__ inline
#include HEADER
using namespace dass;
int main(int argc, char **argv)
{
    if (argc == 4) {   // tokens, columns, kernel: which tile
        const int64_t T = atoll(argv[1]), n = atoll(argv[2]);
        const char k = argv[3][0];
        printf("%d", (k == 's' ? sparse_tile_shape(T, n) : dense_tile_shape(T, n, k == 'g')).which);
        return 0;
    }
    const uint32_t tt = atoi(argv[1]), tn = atoi(argv[2]);
    const TileOrder o = argc > 5 ? make_tile_order(tt, tn, atoi(argv[3]) != 0, atoi(argv[4]), atoi(argv[5]))
                                 : make_tile_order(tt, tn, atoi(argv[3]) != 0, atoi(argv[4]));
    std::vector<int> seen((size_t)tt * tn, 0);
    uint32_t per_xcd[8] = {0}, worst = 0;
    for (uint32_t b = 0; b < o.blocks; ++b) {
        uint32_t t, n;
        if (!tile_of_block(o, b, t, n))
            continue;
        if (t >= tt || n >= tn)
            return printf("tile %u,%u outside\n", t, n), 1;
        ++seen[(size_t)t * tn + n];
        ++per_xcd[b % 8];
    }
    for (size_t i = 0; i < seen.size(); ++i)
        if (seen[i] != 1)
            return printf("tile %zu taken %d times\n", i, seen[i]), 1;
    for (uint32_t x : per_xcd)
        worst = x > worst ? x : worst;
    printf("%u %u\n", worst, o.band);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_order")
    src, exe = d / "driver.cpp", d / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", f'-DHEADER="{HEADER}"', "-o", str(exe), str(src)], check=True)
    return str(exe)


@pytest.mark.parametrize("max_band", [4, 8])
@pytest.mark.parametrize("cached", [0, 1])
@pytest.mark.parametrize("tiles_t,tiles_n", [
    (1, 1), (1, 86), (3, 7), (5, 9), (6, 192), (8, 16), (13, 43),   # small grids, ragged bands
    (64, 64), (128, 16), (64, 65), (47, 88),                                   # either side of the change of order (4096 tiles)
    (37, 192), (36, 192), (100, 97), (1024, 86), (1024, 12)])       # patches; super-rows that do not divide; short columns
def test_every_tile_once_and_evenly(driver, tiles_t, tiles_n, cached, max_band):
    out = subprocess.run([driver, str(tiles_t), str(tiles_n), str(cached), str(max_band)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    worst, band = (int(v) for v in out.stdout.split())
    n = tiles_t * tiles_n
    if band:
        assert band <= max_band
        assert worst == (n + 7) // 8
    else:   # whole patches of 32 dealt to the XCDs
        assert worst <= n / 8 * 1.1 + 64


@pytest.mark.parametrize("tiles_t,tiles_n,cached,run_tiles,runs", [
    (128, 16, 1, 4096, False), (16, 224, 0, 4096, False),      # whole patches that go round evenly
    (64, 16, 1, 4096, True), (12, 224, 0, 4096, True),         # up to 1024 tiles; patches that do not
    (64, 16, 1, 1023, False), (63, 16, 1, 1023, True), (96, 20, 1, 1023, False), (96, 12, 1, 1023, True),
    (16384, 1, 1, 4096, True), (5000, 7, 1, 4096, True)])      # grids narrower than a patch
def test_which_order(driver, tiles_t, tiles_n, cached, run_tiles, runs):
    out = subprocess.run([driver, str(tiles_t), str(tiles_n), str(cached), "4", str(run_tiles)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    worst, band = (int(v) for v in out.stdout.split())
    assert (band > 0) == runs
    if runs:
        assert worst == (tiles_t * tiles_n + 7) // 8


def _which(driver, tokens, columns, kernel):
    return int(subprocess.run([driver, str(tokens), str(columns), kernel], capture_output=True, text=True, check=True).stdout)


def test_gpu_tests_take_every_tile(driver):
    """The shapes of the GPU tests that are meant for the tiles of the matrix-core kernels take them."""
    import test_gpu_calib
    import test_gpu_forward
    import test_gpu_sparse_down
    for T, d, d_int, gated, down in test_gpu_forward.TILE_SHAPES:
        assert (_which(driver, T, d_int, "gated"), _which(driver, T, d, "down")) == (gated, down), (T, d, d_int)
        assert _which(driver, 700, d_int, "gated") == 2     # its chunks
    for shapes, kernel in ((test_gpu_calib.TILE_SHAPES, "gated"), (test_gpu_sparse_down.TILE_SHAPES, "sparse")):
        for T, columns, which in shapes:
            assert _which(driver, T, columns, kernel) == which, (kernel, T, columns)
    for taken in ([s[3] for s in test_gpu_forward.TILE_SHAPES], [s[4] for s in test_gpu_forward.TILE_SHAPES],
                  [s[2] for s in test_gpu_calib.TILE_SHAPES], [s[2] for s in test_gpu_sparse_down.TILE_SHAPES]):
        assert set(taken) == {0, 1, 2}
