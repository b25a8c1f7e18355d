"""Host-side checks of the streaming GEMM's choice of a tile (csrc/gemm_tiles.h, compiled by itself): that every tile
is reached, by the shapes of the GPU test among others, and that recorded shapes get a tile that was fast there."""
import os
import random
import subprocess

import pytest

from test_gpu_parity import STREAMING_SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_00422_amd", "csrc")
DRIVER = """
#include <cstdio>
#include "gemm_tiles.h"
int main() {
    printf("%d", GD_NTILES);
    for (const GdTile& t : GD_TILES) printf(" %d %d %d %d %d", t.ntl, t.wk, t.nb, t.wn, t.resident);
    printf("\\n");
    long long M, K, N;
    int r, a4;
    while (scanf("%lld %lld %lld %d %d", &M, &K, &N, &r, &a4) == 5) printf("%d\\n", gd_pick(M, K, N, r, 256, a4 != 0));
}
"""


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("tiles")
    (d / "pick.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(d / "pick"), str(d / "pick.cpp")], check=True)

    def run(shapes, a4=0):
        out = subprocess.run([str(d / "pick")], input="".join("%d %d %d %d %d\n" % (*s, a4) for s in shapes), text=True,
                             capture_output=True, check=True).stdout.split("\n")
        run.tiles = [tuple(t) for t in zip(*[iter(map(int, out[0].split()[1:]))] * 5)]
        return [int(x) for x in out[1:1 + len(shapes)]]

    return run


def test_every_tile_is_reached(pick):
    """By one in three hundred of random shapes at least (a tile that never is is a kernel that nothing runs), with either
    kind of codes, and by the shapes of the GPU test."""
    rng = random.Random(0)
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random())                 # noqa: E731
    shapes = [(log(17, 4097), 128 * log(1, 225), log(32, 28673), rng.choice([0, 8, 32, 64, 96])) for _ in range(6000)]
    for a4 in (0, 1):
        got = pick(shapes, a4)
        for i in range(len(pick.tiles)):
            assert got.count(i) >= 20, (i, pick.tiles[i], got.count(i))
    assert set(pick(STREAMING_SHAPES)) == set(range(len(pick.tiles)))
    assert set(pick(STREAMING_SHAPES, 1)) == set(range(len(pick.tiles)))


# (tokens, K, N, rank), nibble codes: tiles within 4 % of the best of fifteen, measured with three layers in turn, as
# (32-channel tiles, wavefronts that share K, wavefronts side by side).  The first lines are those where constants
# fitted to plain codes alone, with no share of the ranks, had lost time (in microseconds: best, and what was taken).
RECORDED = [
    ((18, 1280, 126, 0), 1, [(1, 4, 1)]),                            # 5.7, 7.1
    ((25, 1280, 492, 64), 1, [(1, 4, 1)]),                           # 7.9, 9.7
    ((25, 1280, 492, 64), 0, [(1, 4, 1)]),                           # 8.3, 9.0
    ((484, 1152, 528, 0), 1, [(1, 4, 1)]),                           # 7.7, 9.4
    ((17, 5120, 25600, 32), 1, [(2, 2, 1)]),                         # 16.6, 20.5
    ((1024, 28672, 8192, 64), 0, [(2, 1, 4)]),                       # 179, 210
    ((3696, 13312, 378, 96), 0, [(3, 2, 1), (1, 1, 4)]),             # 46, 66: 348 tiles of 64 x 64, every XCD fetches all codes
    ((3418, 25600, 304, 0), 0, [(3, 2, 1)]),                         # 57, 89: likewise
    ((4096, 4096, 12288, 96), 0, [(4, 1, 4)]),                       # 243, 268
    ((2048, 11008, 4096, 32), 0, [(4, 1, 4), (2, 1, 4)]),            # 77.4, 78.4
    ((4096, 8192, 28672, 64), 0, [(3, 1, 4)]),                       # 788; 830 by thresholds
    ((4096, 28672, 8192, 64), 0, [(4, 1, 4)]),                       # 673; 711
    ((2048, 4096, 22016, 64), 0, [(3, 1, 4), (2, 1, 4)]),            # 210, 213; 260
    ((2048, 25600, 5120, 64), 0, [(5, 1, 4)]),
    ((64, 8192, 28672, 64), 0, [(2, 2, 1)]),
    ((64, 8192, 8192, 64), 0, [(1, 4, 1)]),
]


@pytest.mark.parametrize("shape,a4,tiles", RECORDED)
def test_recorded_shapes_take_a_fast_tile(pick, shape, a4, tiles):
    i = pick([shape], a4)[0]
    ntl, wk, _, wn, _ = pick.tiles[i]
    assert (ntl, wk, wn) in tiles


# ---- the sparse GEMM's tiles (same header)
# Short rows of K and low ranks, where constants fitted to a slower epilogue had lost time against the kernel of before that
# epilogue (microseconds: that one, what was taken, now).
@pytest.mark.parametrize("shape,tiles", [
    ((24, 512, 270, 0), [(1, 1, 2), (1, 1, 4)]),                     # 4.8, 5.9, 4.6
    ((23, 384, 868, 0), [(1, 1, 2), (1, 1, 4)]),                     # 4.8, 5.9, 4.6
    ((25, 384, 666, 0), [(1, 1, 2), (1, 1, 4)]),                     # 5.0, 6.0, 4.8
    ((806, 512, 11140, 16), [(1, 1, 4), (3, 1, 4)]),                 # 22.6, 25.7, below 18.8
    ((806, 1408, 11140, 16), [(1, 1, 4), (3, 1, 4)]),                # 30.0, 33.0, 25.3
    ((385, 1408, 21018, 16), [(1, 1, 4), (3, 1, 4)]),                # (5, 1, 4): 34.3
])
def test_short_rows_take_a_fast_tile(pick, shape, tiles):
    i = pick([shape])[0]
    ntl, wk, _, wn, _ = pick.tiles[i]
    assert (ntl, wk, wn) in tiles


SPARSE_DRIVER = """
#include <cstdio>
#include "gemm_tiles.h"
int main() {
    printf("%d\\n", GS_NTILES);
    long long M, K, N;
    int r;
    while (scanf("%lld %lld %lld %d", &M, &K, &N, &r) == 4) {
        int dense = -1;
        const int sparse = gs_pick(M, K, N, r, 256, &dense);
        // the dense kernel's tile that comes with the answer is the one it would be launched with (not looked at: -1)
        if (dense != (M > GS_MIN_TOKENS ? gd_pick(M, K, N, r, 256, false) : -1)) return 1;
        printf("%d\\n", sparse);
    }
}
"""


@pytest.fixture(scope="module")
def sparse_pick(tmp_path_factory):
    d = tmp_path_factory.mktemp("sparse_tiles")
    (d / "pick.cpp").write_text(SPARSE_DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(d / "pick"), str(d / "pick.cpp")], check=True)

    def run(shapes):
        out = subprocess.run([str(d / "pick")], input="".join("%d %d %d %d\n" % s for s in shapes), text=True,
                             capture_output=True, check=True).stdout.split()
        run.tiles = int(out[0])
        return [int(x) for x in out[1:]]

    return run


def test_every_sparse_tile_is_reached(sparse_pick):
    from test_gpu_sparse import SHAPES
    rng = random.Random(1)
    log = lambda lo, hi: int(lo * (hi / lo) ** rng.random())                 # noqa: E731
    got = sparse_pick([(log(17, 4097), 128 * log(1, 225), log(32, 28673), rng.choice([0, 8, 32, 64, 96])) for _ in range(6000)])
    for i in range(sparse_pick.tiles):
        assert got.count(i) >= 20, (i, got.count(i))
    assert sorted(set(sparse_pick(SHAPES))) == list(range(sparse_pick.tiles))   # each of them by one: none is left to the dense kernel


# (tokens, K, N, rank), tile (-1: dense kernel), both sides in microseconds: pass over the codes and sparse kernel, dense kernel
@pytest.mark.parametrize("shape,tiles", [
    ((4096, 28672, 8192, 64), [2]),              # 36 + 475, 647
    ((2048, 25600, 5120, 64), [1]),              # 17 + 158, 192
    ((2048, 4096, 22016, 64), [0]),              # 5 + 176, 183
    ((4096, 8192, 8192, 64), [2]),               # 12 + 183, 237
    ((64, 28672, 8192, 64), [-1]),
    ((1031, 5120, 1024, 64), [-1]),              # 2 + 26, 22
])
def test_recorded_shapes_take_the_faster_kernel(sparse_pick, shape, tiles):
    assert sparse_pick([shape])[0] in tiles


RESIDENT_DRIVER = """
#include <cstdio>
#include "gemm_tiles.h"
int main() {
    for (int r = 0; r <= 128; ++r)
        for (int i = 0; i < GD_NTILES; ++i) {
            const GdTile& v = GD_TILES[i];
            // a cost of two rounds and nothing else: how many workgroups does it put side by side?
            GdTile probe = v;
            probe.start = probe.idle = probe.low = 0.0f;
            for (int s = 0; s < 4; ++s) { probe.base[s] = 0.0f; probe.slice[s] = 1.0f; }
            const long long bn = 32LL * v.ntl * v.wn, K = 128LL * v.wk * 1000;
            int side = 0;
            for (int s = 1; s <= 8; ++s)                // s x 256 tiles: one round of 1000 slices up to what is resident
                if (gd_cost(probe, 64, K, s * 256 * bn, r, 256, false) < 1500.0f) side = s;
            printf("%d %d %d %zu %d\\n", r, i, v.resident, gd_lds_bytes(v, r), side);
        }
}
"""


def test_workgroups_side_by_side_fit_the_lds(tmp_path):
    """At every rank up to 128: the epilogue's rows of T grow with it.  Up to 112, which the costs were fitted to, all of
    what the table says."""
    (tmp_path / "res.cpp").write_text(RESIDENT_DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp_path / "res"), str(tmp_path / "res.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "res")], text=True, capture_output=True, check=True).stdout.split("\n")
    for line in out[:-1]:
        r, i, resident, lds, side = map(int, line.split())
        assert side * lds <= 160 * 1024, (r, i, side, lds)
        assert side == min(resident, 160 * 1024 // lds), (r, i)
        if r <= 112:
            assert side == resident, (r, i)
