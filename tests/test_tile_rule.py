"""The rules that pick a tile (csrc/tile_rule.hpp), compiled for the host.  A GEMM's block tile: on shapes timed with every tile in whole steps, in a
sustained loop, it does not take one that is clearly slower than another: 0.4 % of a step and more, where the step's times differ by 0.2-0.3 %
(the dense row-wise up-projections apart, whose two largest tiles spill: those taken are 0.7 and 2 % from the best)."""
import shutil
import subprocess
from pathlib import Path

import pytest

from test_gpu_big_tiles import SIZES as BIG_SIZES
from test_gpu_k_major import SIZES as K_MAJOR_SIZES
from test_gpu_pick import SHAPES as PICK_SHAPES

RULE = Path(__file__).resolve().parents[1] / "paper_2503_16672_amd" / "csrc" / "tile_rule.hpp"
MAIN = """
#include "%s"
#include <cstdio>
int main() {
  char epi; int sparse, f8, M, N, K, gemms;
  while (std::scanf(" %%d %%d %%c %%d %%d %%d %%d", &sparse, &f8, &epi, &M, &N, &K, &gemms) == 7) {
    const ffn24::EpiCost e = epi == 'p' ? ffn24::EPI_PLAIN : epi == 'f' ? ffn24::EPI_FP8 : ffn24::EPI_FP8_SPILLS;
    std::printf("%%d\\n", ffn24::pick_tile(sparse, f8, e, M, N, K, gemms));
  }
}
"""

# sparse, fp8, epilogue (p: plain or bf16, f: fp8, s: fp8 dense row-wise up-projection), M, N, K, GEMMs in the launch -> tiles that do
# (0: 256 x 256, 1: 256 x 128, 2: 128 x 128, 3: 128 x 64, 4: 64 x 64); in the comment the step's time against 256 x 256, us
MEASURED = [
    ((0, 0, "p", 15616, 2304, 4864, 1), {0}),      # 2.1 rounds: 256 x 128 +31 of 1704
    ((0, 0, "p", 14336, 4096, 4096, 1), {0}),      # 3.5 rounds: +18 of 1793
    ((0, 0, "p", 10240, 10240, 2560, 1), {0}),     # 6.3 rounds: +31 of 2055
    ((0, 0, "p", 11776, 1024, 3584, 1), {0}),      # 0.7 rounds: 256 x 128 +24, 128 x 128 +29 of 576
    ((0, 0, "p", 12544, 768, 3328, 1), {0}),       # 0.6 rounds: 128 x 128 +31 of 530
    ((0, 0, "p", 8704, 3840, 3328, 1), {0}),       # 2.0 rounds: +47 of 941
    ((0, 0, "p", 5376, 4352, 1280, 1), {1}),       # 1.4 rounds: 256 x 128 -25, 128 x 128 +12 of 369
    ((0, 0, "p", 4608, 4352, 1280, 1), {2}),       # 1.2 rounds: 128 x 128 -34, 256 x 128 -23 of 344
    ((0, 0, "p", 6144, 5888, 2816, 1), {1}),       # 2.2 rounds: 256 x 128 -30 of 884
    ((0, 0, "p", 9984, 2304, 4608, 1), {1}),       # 1.4 rounds: 256 x 128 -29 of 1109
    ((0, 0, "p", 2048, 1024, 4096, 1), {3}),       # dense down-projection of 32 large tiles: 128 x 64 -84, 128 x 128 -73, 64 x 64 -72 of 250
    ((0, 0, "p", 2816, 3840, 9216, 1), {0}),       # dense down-projection, 0.6 rounds: 256 x 128 -4, 128 x 128 +120 of 1154
    ((0, 0, "p", 10496, 1024, 3328, 1), {0, 2}),   # dense down-projection, 0.6 rounds: 256 x 128 +15, 128 x 128 +9 of 504
    ((0, 1, "p", 4096, 2560, 7936, 1), {0}),       # dense down-projection, 0.6 rounds: 256 x 128 +22, 128 x 128 +23 of 510
    ((0, 1, "f", 8704, 5888, 3072, 1), {1}),       # 3.1 rounds: 256 x 128 -42, 128 x 128 -12 of 881
    ((0, 1, "f", 8192, 8192, 2048, 1), {1}),       # 4.0 rounds: -34 of 751
    ((0, 1, "f", 4608, 14080, 2048, 1), {1}),      # 3.9 rounds: -38 of 781
    ((0, 1, "s", 6144, 7168, 2048, 1), {0, 2}),    # 2.6 rounds: 256 x 128 +1, 128 x 128 +5 of 690
    ((0, 1, "s", 5120, 5888, 2304, 1), {0, 2}),    # 1.8 rounds: 128 x 128 -11, 256 x 128 0 of 544
    ((1, 0, "p", 8192, 2048, 8192, 1), {0}),       # one full round: 256 x 128 +63 of 1075
    ((1, 0, "p", 1024, 1024, 4096, 1), {4}),       # 16 large tiles: 64 x 64 -78, 128 x 64 -69 of 170
    ((1, 0, "p", 3584, 1792, 5888, 1), {1}),       # 0.4 rounds: 256 x 128 -38, 128 x 128 -39 of 471
    ((1, 0, "p", 5376, 1280, 4352, 2), {0}),       # both weight gradients, 0.8 rounds together: 256 x 128 +21 of 346
    ((1, 0, "p", 4096, 1024, 16384, 2), {1}),      # 0.5 rounds together: 256 x 128 -60, 128 x 128 -14 of 688
    ((0, 0, "p", 9984, 4608, 2304, 2), {0}),       # 5.5 rounds together, dense: 256 x 128 -2 of 1273
]


@pytest.fixture(scope="module")
def picks(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("tile_rule")
    (d / "main.cpp").write_text(MAIN % RULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", str(d / "main"), str(d / "main.cpp")], check=True)

    def run(queries):
        text = "\n".join(" ".join(str(x) for x in q) for q in queries)
        return [int(x) for x in subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return run


@pytest.mark.parametrize("i", range(len(MEASURED)), ids=["-".join(str(x) for x in q) for q, _ in MEASURED])
def test_tile_of_measured_shapes(picks, i):
    assert picks([MEASURED[i][0]])[0] in MEASURED[i][1]


def test_shapes_of_the_pick_tests_take_every_tile(picks):
    """The GPU test of the pick runs each block tile, of the bf16 and of the row-wise fp8 up-projection."""
    for f8, epilogue in ((0, "p"), (1, "f")):
        assert picks([(0, f8, epilogue, Fh, T, D, 1) for T, D, Fh, _ in PICK_SHAPES]) == [tile for *_, tile in PICK_SHAPES]
    assert {tile for *_, tile in PICK_SHAPES} == set(range(5))


def test_shape_of_the_big_tile_tests_takes_them_everywhere(picks):
    """The first size of the GPU test of the 256 x 256 tile runs every GEMM of every kind of step with it, and its slices of 512 tokens (Y, dX) and
    256 features (dW1, dW2) run with smaller tiles."""
    T, D, F = BIG_SIZES[0]
    products = lambda t, f: [(0, 0, "p", f, t, D, 1), (0, 1, "p", f, t, D, 1), (0, 1, "f", f, t, D, 1), (0, 1, "s", f, t, D, 1),
                             *((sp, f8, "p", t, D, f, 1) for sp in (0, 1) for f8 in (0, 1))]
    gradients = lambda t, f: [(sp, f8, "p", f, D, t, 2) for sp in (0, 1) for f8 in (0, 1)]
    assert set(picks(products(T, F) + gradients(T, F))) == {0}
    assert 0 not in picks(products(512, F)) and 0 not in picks(gradients(T, 256))


def test_sizes_of_the_k_major_tests_take_every_tile(picks, tmp_path):
    """... in each of the GEMMs that they name; and those beside which the re-compression rides take the three tiles that it may."""
    every = set(range(5))
    assert set(picks([(0, 0, "p", F, T, D, 1) for T, D, F in K_MAJOR_SIZES])) == every                     # up-projection
    for sparse in (0, 1):
        assert set(picks([(sparse, 0, "p", T, D, F, 1) for T, D, F in K_MAJOR_SIZES])) == every            # down-projection, dX
        assert set(picks([(sparse, 0, "p", F, D, T, 2) for T, D, F in K_MAJOR_SIZES])) == every            # weight gradients together
        assert set(picks([(sparse, 0, "p", F, D, T, 1) for T, D, F in K_MAJOR_SIZES])) == every            # ... alone
    split = [s for s in K_MAJOR_SIZES if s[2] >= 1024 and not (s[0] > 2048 and s[2] > 1280)]
    (tmp_path / "main.cpp").write_text("""
#include "%s"
#include <cstdio>
using namespace ffn24;
int main() {
  int T, D, F;
  while (std::scanf("%%d %%d %%d", &T, &D, &F) == 3) {
    const int dx = pick_tile(true, false, EPI_PLAIN, T, D, F);
    std::printf("%%d %%d\\n", pick_pair_tile(false, 256, F - 256, D, T, 2), side_rides(true, dx, T, D, F) ? dx : -1);
  }
}
""" % RULE)
    subprocess.run(["g++", "-std=c++17", "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    run = lambda sizes: [tuple(map(int, line.split())) for line in
                         subprocess.run([str(tmp_path / "main")], input="\n".join(" ".join(map(str, s)) for s in sizes), capture_output=True, text=True, check=True).stdout.splitlines()]
    assert {pair for pair, _ in run(split)} == every
    assert {rides for _, rides in run(K_MAJOR_SIZES)} == {-1, 2, 3, 4}


def test_two_full_gemms_take_the_large_tile_alone_too(tmp_path):
    """Where two GEMMs together take the 256 x 256 tile and each fills whole rounds with it, they are launched apart with that tile: one of
    them by itself has to pick it as well."""
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    (tmp_path / "main.cpp").write_text("""
#include "%s"
using namespace ffn24;
int main() {
  int seen = 0;
  for (int sparse = 0; sparse < 2; sparse++) for (int f8 = 0; f8 < 2; f8++)
    for (int M = 256; M <= 32768; M += 256) for (int N = 256; N <= 8192; N += 256) for (int K = 256; K <= 16384; K += 768) {
      if (tile_count(TILES_SPARSE[0], M, N) %% CHIP_CUS || pick_tile(sparse, f8, EPI_PLAIN, M, N, K, 2) != 0) continue;
      seen++;
      if (pick_tile(sparse, f8, EPI_PLAIN, M, N, K, 1) != 0) return 1;
    }
  return seen ? 0 : 2;
}
""" % RULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    assert subprocess.run([str(tmp_path / "main")]).returncode == 0


# fp8, 256 x 256 tiles of one launch, K, least rounds of one -> apart
TOGETHER = [
    ((0, 966, 6912, 1), 1), ((0, 966, 6912, 2), 1), ((0, 658, 3584, 1), 1), ((0, 720, 3584, 2), 1), ((1, 406, 7680, 1), 1),
    ((0, 512, 4096, 2), 0), ((0, 256, 8192, 2), 0), ((0, 1024, 16384, 2), 0),      # whole rounds
    ((0, 928, 1280, 2), 0), ((0, 980, 2048, 1), 0), ((1, 398, 5120, 1), 0),        # short reductions
    ((0, 532, 5888, 2), 0), ((0, 1029, 8704, 1), 0),                               # a round saved together
    ((0, 189, 8192, 1), 0),                                                        # less than a round each
]


def test_launches_apart(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    (tmp_path / "main.cpp").write_text('#include "%s"\n#include <cstdio>\nint main() { int f, n, K, r; while (std::scanf("%%d %%d %%d %%d", &f, &n, &K, &r) == 4) '
                                       'std::printf("%%d\\n", ffn24::apart_is_better(f, n, K, r)); }\n' % RULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    text = "\n".join(" ".join(str(x) for x in q) for q, _ in TOGETHER)
    got = subprocess.run([str(tmp_path / "main")], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert [int(x) for x in got] == [a for _, a in TOGETHER]


def test_rides_beside_dx_at_measured_shapes(tmp_path):
    """The feature-wise re-compression beside the dX GEMM: where whole steps were faster so, with each of the three tiles, and not where they were
    slower by 1 % and more."""
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    rides = [((256, 512, 2048), 4), ((1536, 512, 2048), 4), ((768, 768, 3072), 4), ((1280, 768, 3072), 4), ((512, 1024, 4096), 4), ((4096, 512, 1024), 3), ((8192, 256, 512), 3),
             ((8192, 512, 512), 2), ((2304, 1024, 1280), 2), ((4096, 1024, 1024), 2), ((3072, 1024, 1280), 2)]
    apart = [(1024, 1024, 4096), (2048, 1024, 2048), (1536, 1024, 2560), (2048, 768, 3072), (2048, 512, 4096), (1024, 1536, 2048), (1280, 1280, 5120)]
    (tmp_path / "main.cpp").write_text("""
#include "%s"
#include <cstdio>
using namespace ffn24;
int main() {
  int T, D, F;
  while (std::scanf("%%d %%d %%d", &T, &D, &F) == 3) {
    const int tile = pick_tile(true, false, EPI_PLAIN, T, D, F);
    std::printf("%%d\\n", side_rides(true, tile, T, D, F) ? tile : -1);
  }
}
""" % RULE)
    subprocess.run(["g++", "-std=c++17", "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    text = "\n".join(" ".join(map(str, x)) for x in [s for s, _ in rides] + apart)
    got = [int(x) for x in subprocess.run([str(tmp_path / "main")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    assert got == [tile for _, tile in rides] + [-1] * len(apart)


def test_in_place_or_copied_at_measured_shapes(tmp_path):
    """Operands read k-major or brought into panel form first: whichever was the faster by 1 % and more (copies: up to 17 %, in place: up to 21 %)."""
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    acts_in = [(256, 512, 2048), (512, 2048, 8192), (512, 2048, 12288), (1024, 1024, 1024), (512, 8192, 4096), (8192, 4096, 8192), (16384, 4096, 16384), (16384, 4096, 8192), (32768, 512, 512),
               (65536, 256, 256), (65536, 1024, 2048), (131072, 1024, 1024), (131072, 768, 768), (131072, 512, 2048)]
    acts_copied = [(256, 4096, 16384), (1024, 4096, 16384), (2048, 4096, 16384), (256, 8192, 28672), (2048, 8192, 28672), (256, 4096, 8192), (512, 4096, 12288), (1024, 8192, 16384)]
    long = [(65536, 512, 512), (65536, 512, 1024), (65536, 256, 1024), (131072, 256, 512), (131072, 512, 512), (262144, 512, 512)]      # 2:4 only
    weights_in = [(1024, 1024, 4096, 0), (256, 4096, 16384, 0), (8192, 2048, 8192, 1), (16384, 4096, 16384, 1), (8192, 8192, 2048, 0), (16384, 4096, 1024, 0)]
    weights_copied = [(65536, 2048, 512, 0), (65536, 2048, 512, 1), (131072, 1024, 512, 1), (16384, 8192, 1024, 0), (65536, 4096, 1024, 1)]
    call = lambda f, a: f"{f}({', '.join(map(str, a))})"
    checks = ([call("acts_in_place", (*a, d)) for a in acts_in for d in (0, 1)] + ["!" + call("acts_in_place", (*a, d)) for a in acts_copied for d in (0, 1)]
              + ["!" + call("acts_in_place", (*a, 0)) for a in long] + [call("acts_in_place", (*a, 1)) for a in long]
              + [call("weights_in_place", a) for a in weights_in] + ["!" + call("weights_in_place", a) for a in weights_copied])
    (tmp_path / "main.cpp").write_text('#include "%s"\n#include <cstdio>\nusing namespace ffn24;\nint main() { const bool ok[] = {%s}; for (bool b : ok) std::printf("%%d\\n", b); }\n'
                                       % (RULE, ", ".join(checks)))
    subprocess.run(["g++", "-std=c++17", "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    got = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True, check=True).stdout.split()
    assert [c for c, ok in zip(checks, got, strict=True) if ok != "1"] == []


def test_featurewise_tile_of_measured_shapes(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    small = [(128, 64), (128, 16384), (16384, 64), (2560, 768), (1280, 1216), (2048, 2048)]            # 64 x 64 tiles 1.2-2.5 x faster
    large = [(5248, 896), (1792, 3712), (512, 12288), (10112, 768), (16384, 512), (8064, 8256), (1 << 20, 1 << 20)]   # 128 x 256 tiles 1.1-2.8 x
    checks = " && ".join([f"featurewise_small({a}, {b})" for a, b in small] + [f"!featurewise_small({a}, {b})" for a, b in large])
    (tmp_path / "main.cpp").write_text('#include "%s"\nusing namespace ffn24;\nint main() { return %s ? 0 : 1; }\n' % (RULE, checks))
    subprocess.run(["g++", "-std=c++17", "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    assert subprocess.run([str(tmp_path / "main")]).returncode == 0


def test_held_columns_of_measured_shapes(tmp_path):
    """quantise_e4m3 per column: one launch where it was the faster one, three launches where they were (by 4 % and more)."""
    held = [(1, 8), (1, 16384), (64, 16384), (512, 8192), (512, 16384), (640, 16384), (1024, 8192), (1024, 24576), (1024, 65536), (1280, 16384), (1536, 512), (1536, 8192), (1536, 16384), (1536, 32768)]
    not_held = [(1, 32768), (1, 1 << 24), (8, 1 << 20), (64, 1 << 20), (256, 32768), (256, 1 << 18), (512, 20480), (512, 1 << 17), (640, 32768), (768, 20480), (896, 16384), (1024, 9216),
                (1024, 98304), (1152, 12288), (1536, 10240), (1536, 98304), (1536, 1 << 17), (1537, 512), (2048, 4096), (4096, 1024), (8192, 12896), (1 << 24, 8), (1 << 24, 1 << 24)]
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    checks = " && ".join([f"held_columns({r}, {c})" for r, c in held] + [f"!held_columns({r}, {c})" for r, c in not_held])
    (tmp_path / "main.cpp").write_text('#include "%s"\nusing namespace ffn24;\nint main() { return %s ? 0 : 1; }\n' % (RULE, checks))
    subprocess.run(["g++", "-std=c++17", "-o", str(tmp_path / "main"), str(tmp_path / "main.cpp")], check=True)
    assert subprocess.run([str(tmp_path / "main")]).returncode == 0
