"""The launches of the library as the host decides on them: a host program (tests/launch_geometry_driver.cpp) stands in for
the runtime's launch call and looks at each one."""
import os
import subprocess

import pytest

from paper_2407_08296_amd import build as qg_build
from paper_2407_08296_amd import qgalore as qg
from test_gpu_linear import TWO_GROUPS, TWO_GROUPS_GRAD_INPUT

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    qg.lib()
    exe = str(tmp_path_factory.mktemp("launch") / "launch_geometry_driver")
    lib_dir = os.path.dirname(os.path.abspath(qg.LIB_PATH))
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "c++", "-std=c++17", "-O1",
                    "-I", os.path.join(qg_build.ROOT, "include"), os.path.join(HERE, "launch_geometry_driver.cpp"), "-rdynamic",
                    "-L", lib_dir, "-l:" + os.path.basename(qg.LIB_PATH), "-Wl,-rpath," + lib_dir, "-o", exe], check=True)

    def run(what, *sizes):
        p = subprocess.run([exe, what, *map(str, sizes)], capture_output=True, text=True, timeout=300)
        assert p.returncode == 0, p.stdout + p.stderr
        return [tuple(int(v) for v in line.split()) for line in p.stdout.splitlines()[:-1]]   # (workgroups, threads)
    return run


@pytest.mark.parametrize("count,m,n,r", [
    (1, 8, 8, 8), (3, 768, 768, 256), (16, 4096, 4096, 1024),
    (32767, 32768, 8, 8), (32768, 32768, 8, 8),       # 512 row tiles of 64 per matrix: 2^24 tiles in all, and 512 fewer
    (40000, 65536, 8, 8), (700, 1 << 21, 8, 8),       # more; fewer and longer matrices
    (20000, 72, 72, 72), (1, 1 << 27, 8, 8),          # two block columns; the longest single matrix
])
def test_grids_of_a_refresh(driver, count, m, n, r):
    """They stay within what a launch can hold, for every batch that the entry point accepts."""
    driver("refresh", count, m, n, r)


@pytest.mark.parametrize("n,k,want", [
    (2048, 2000, (256, 512)), (2047, 2040, (512, 256)), (2047, 2048, (256, 512)),   # whole rows of the weight; odd ones
    (2042, 1016, (512, 256)), (2042, 2040, (256, 512)),                             # even rows
    (2048, 2049, (512, 256)), (2047, 5461, (256, 512)),                             # a contraction of unaligned rows
])
def test_two_groups_on_a_weight_with_k_slow(driver, n, k, want):
    """1000 tokens.  128 x 64 tiles in two groups of waves (512 threads) where the weight's rows start 16-byte aligned or the
    contraction is long, else 64 x 64 tiles (256 threads): grad_input of the layer k <- n, and the forward pass of the same weight stored transposed."""
    assert driver("grad_input", 1000, k, n)[0] == want
    assert driver("t_forward", 1000, n, k)[0] == want


@pytest.mark.parametrize("what,tokens,n,k,threads", [
    ("forward", 2048, 2048, 520, 256), ("forward", 2000, 2000, 767, 256), ("forward", 2048, 2048, 768, 512),
    ("grad_input", 1024, 4096, 512, 256), ("grad_input", 1024, 4096, 1535, 256), ("grad_input", 1024, 4096, 1536, 512),   # whole
    ("grad_input", 1000, 3000, 512, 512), ("grad_input", 1000, 3000, 543, 256), ("grad_input", 1000, 3000, 545, 512),    # ragged
])
def test_shortest_contraction_of_two_groups_on_large_tiles(driver, what, tokens, n, k, threads):
    """128 x 128 tiles, at most a workgroup per CU: n columns, contraction k."""
    tiles = -(-tokens // 128) * -(-n // 128)
    sizes = (tokens, n, k) if what == "forward" else (tokens, k, n)
    assert driver(what, *sizes) == [(-(-tiles // 8) * 8, threads)]


@pytest.mark.parametrize("tokens,n,k,want", [
    (32, 17408, 2048, (544, 256)), (20, 24576, 768, (768, 256)),       # 272 and 384 tiles of 64 x 64: contraction over four waves
    (32, 16384, 2048, (512, 256)), (64, 12288, 2048, (192, 512)),      # up to 512 tiles of 32 x 32; 192 of 64 x 64, two groups
    (32, 24576, 511, (768, 256)), (64, 12288, 511, (768, 256)),        # a short contraction
])
def test_few_rows_in_the_forward_pass(driver, tokens, n, k, want):
    assert driver("forward", tokens, n, k) == [want]


@pytest.mark.parametrize("tokens,m,n,split", [
    (1000, 2048, 768, True), (500, 2048, 1280, True), (2000, 4096, 320, True),      # at least twice the tokens
    (1000, 1999, 768, False), (2000, 2048, 320, False), (1000, 768, 768, False),    # less, or a short contraction
    (500, 4096, 1280, False),                                                       # grad_W in a launch of its own: two groups
    (602, 2416, 1207, False), (536, 3315, 1144, False),                             # unaligned rows of x, of dy
    (1000, 2048, 512, True), (1000, 500, 768, True),                                # up to 512 tiles; up to a contraction of 511
])
def test_grad_input_of_a_transposed_weight(driver, tokens, m, n, split):
    """513 to 768 tiles of 32 x 32: split over waves, or 64 x 64 tiles; alone and beside grad_W it is the same kernel."""
    tiles32, tiles64 = -(-tokens // 32) * -(-n // 32), -(-tokens // 64) * -(-n // 64)
    up8 = lambda v: -(-v // 8) * 8
    assert driver("t_grad_input", tokens, m, n) == [(up8(tiles32 if split else tiles64), 512 if m == 4096 and not split else 256)]
    both = driver("t_backward", tokens, m, n)
    if len(both) == 2:
        assert both[0] == driver("t_grad_input", tokens, m, n)[0]
    else:
        grad_w = [up8(-(-m // t) * -(-n // t)) for t in (32, 64)]
        assert both[0][0] - up8(tiles32 if split else tiles64) in grad_w


@pytest.mark.parametrize("tm,tn,layout,tokens,cols,k", TWO_GROUPS)
def test_tiles_of_two_groups(driver, tm, tn, layout, tokens, cols, k):
    tiles = -(-tokens // tm) * -(-cols // tn)
    assert driver("forward" if layout == "fast" else "t_forward", tokens, cols, k) == [(-(-tiles // 8) * 8, 512)]


@pytest.mark.parametrize("tm,tn,tokens,m,n", TWO_GROUPS_GRAD_INPUT)
def test_tiles_of_two_groups_in_grad_input(driver, tm, tn, tokens, m, n):
    tiles = -(-tokens // tm) * -(-n // tn)
    assert driver("backward", tokens, m, n)[0] == driver("grad_input", tokens, m, n)[0] == (-(-tiles // 8) * 8, 512)


@pytest.mark.parametrize("what", ["forward", "t_forward"])
@pytest.mark.parametrize("k,two", [(576, False), (608, False), (640, True), (656, False), (944, False), (960, True), (976, True)])
def test_shortest_contraction_of_two_groups_on_128x64_tiles(driver, what, k, two):
    """With a partial last step, which one group takes alone, longer than without."""
    assert driver(what, 1800, 624, k) == [(152, 512) if two else (296, 256)]     # 15 x 10 and 29 x 10 tiles
