"""CPU check of the set-up launch's grid: every vertex of every view and every tile has its thread, and no grid dimension
passes 2^32 threads, also where views times vertices do (launches past it are refused)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_02482_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
DRIVER = r'''
#include "vs_api.hip"
int main(int, char** a) {
  uint32_t proj = 0, tiles = 0;
  const dim3 g = setup_blocks(atoll(a[1]), atoll(a[2]), atoll(a[3]), atoi(a[4]), proj, tiles);
  printf("%u %u %u %u\n", g.x, g.y, proj, tiles);
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    src, exe = d / "driver.hip", d / "driver"
    src.write_text(DRIVER)
    subprocess.check_call([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-w", "-I", os.path.join(ROOT, "include"), "-I",
                           CSRC, "-Wl,--unresolved-symbols=ignore-all", str(src), "-o", str(exe)])
    return lambda *x: [int(v) for v in subprocess.check_output([str(exe), *map(str, x)], text=True).split()]


@pytest.mark.parametrize("verts,tiles16,tiles_bin,views", [
    (3, 1, 1, 1), (257, 1000, 0, 1), (357_000, 64 * 4096, 64 * 304, 64), (2 ** 28, 100 * 64, 100 * 4, 100),
    (2 ** 31, 16, 16, 16), (16 * 2 ** 26, 3, 7, 4), (5, 65_535, 65_535, 65_535)])
def test_set_up_grid(driver, verts, tiles16, tiles_bin, views):
    x, y, proj, tiles = driver(verts, tiles16, tiles_bin, views)
    assert y == views and x * 256 < 2 ** 32
    assert proj * 256 >= verts and tiles * 256 >= tiles16
    assert (x - proj) * views >= tiles + -(-tiles_bin // 256)   # blocks (x - proj) * views + view: all of them, each once
