"""The rule by which fp64 products get their tiles (csrc/gemm64_tiles.h), compiled on the host: the batches of test_gpu_split.TILE_WIDTHS run on the
tiles they are named after, and both sides of a line are where its comment says."""
import subprocess

import pytest

from paper_2605_02218_amd import build as B
from test_gpu_split import TILE_WIDTHS

PROGRAM = r"""
#include <stdio.h>
#include "gemm64_tiles.h"
int main() {
  const char* names[] = {"16x16", "32x32", "64x32", "64x48", "64x64", "64x80", "64x96"};
  long m, n, k, batch;
  int triangle, f64;
  while (scanf("%ld %ld %ld %ld %d %d", &m, &n, &k, &batch, &triangle, &f64) == 6) puts(names[covspec::plain_tile(m, n, k, batch, triangle, f64)]);
}
"""


@pytest.fixture(scope="module")
def tile(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "tiles.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", B.CSRC, str(d / "tiles.cpp"), "-o", str(d / "tiles")], check=True, capture_output=True)

    def ask(m, n, k, batch, triangle=0, f64=1):
        text = "%d %d %d %d %d %d\n" % (m, n, k, batch, triangle, f64)
        return subprocess.run([str(d / "tiles")], input=text, capture_output=True, text=True, check=True, timeout=20).stdout.strip()
    return ask


@pytest.mark.parametrize("name", list(TILE_WIDTHS))
def test_batches_run_on_the_tiles_they_are_named_after(tile, name):
    images, tokens, rank = TILE_WIDTHS[name]
    block, order = (rank + 64 + 63) // 64 * 64, (tokens + 63) // 64 * 64
    got = tile(block, order, order, images)
    if name == "16x16-over":
        assert got != "16x16"
        return
    assert got == name.split("-")[0]
    width = int(got.split("x")[1])
    if got in ("64x96", "64x48") or name.endswith("partial"):
        assert order % width != 0
    if name == "16x16-most":
        assert block // 16 * (order // 16) * images == 256


def test_every_tile_has_a_batch(tile):
    assert {n.split("-")[0] for n in TILE_WIDTHS} == {"16x16", "32x32", "64x32", "64x48", "64x64", "64x80", "64x96"}


@pytest.mark.parametrize("shape,want", [
    ((192, 1664, 1664, 4), "64x80"), ((384, 1280, 1280, 12), "64x96"), ((256, 640, 640, 64), "64x64"), ((192, 192, 1664, 1, 1), "16x16"),
    ((192, 192, 1664, 3, 1), "16x16"), ((192, 192, 1664, 4, 1), "32x32"), ((256, 256, 640, 64, 1), "32x32"), ((1024, 1024, 512, 1, 1, 0), "32x32"),
    ((4096, 4096, 512, 8, 0, 0), "64x64")])
def test_lines(tile, shape, want):
    assert tile(*shape) == want
