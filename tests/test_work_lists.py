"""The work lists of the fused product, on the CPU: the library's layout code
built with the host compiler into a small program that is asked for the
default segment length of layouts too large to build here (their streams'
lengths are all that it needs) and for the tile shape of a box."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2308_07487_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "sdc_internal.h"
// box L0 L1 L2 precision -> tiles in box order, tiles
// kind(periodic|radial) n_streams pairs_per_stream lag_groups sched(index) -> length, streams cut, most tasks
int main(int argc, char** argv) {
    sdc::Layout lay;
    if (!std::strcmp(argv[1], "box")) {
        sdc_bin_spec b{};
        b.kind = SDC_BINS_PERIODIC_SC;
        for (int a = 0; a < 3; ++a) b.cells[a] = atoi(argv[2 + a]);
        std::vector<float> pos;
        for (int x = 0; x < b.cells[0]; ++x)
            for (int y = 0; y < b.cells[1]; ++y)
                for (int z = 0; z < b.cells[2]; ++z) pos.insert(pos.end(), {(float)x, (float)y, (float)z});
        std::string err;
        if (sdc::build_layout(pos.data(), (int64_t)pos.size() / 3, &b, atoi(argv[5]), 96, &lay, &err) != SDC_OK) return 1;
        std::printf("%d %d\n", (int)lay.linear, (int)lay.n_tiles);
        return 0;
    }
    lay.kind = std::strcmp(argv[1], "radial") ? SDC_BINS_PERIODIC_SC : SDC_BINS_RADIAL;
    const long n = atol(argv[2]), len = atol(argv[3]);
    const int groups = atoi(argv[4]), sched = atoi(argv[5]);
    for (long k = 0; k < n; ++k) {
        sdc::KStream s{};
        s.p1 = (int)len;
        lay.streams.push_back(s);
    }
    const long most = (long)sdc::max_fused_tasks(sched);
    const int seg = sdc::fitted_segment(lay, lay.streams, groups, 256 * sdc::wg_per_cu(sched), sched, true);
    std::printf("%d %ld %ld\n", seg, n * ((len + seg - 1) / seg), most);
}
"""


@pytest.fixture(scope="module")
def prog(tmp_path_factory):
    d = tmp_path_factory.mktemp("work_lists")
    (d / "main.cpp").write_text(MAIN)
    out = d / "work_lists"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                           str(d / "main.cpp"), os.path.join(CSRC, "sdc_layout.cpp"), "-o", str(out)])
    return lambda *a: [int(x) for x in subprocess.check_output([str(out), *map(str, a)], text=True).split()]


ONE, TWO, SPLIT = 0, 1, 2  # schedules: one-pass, two-pass, lag-split


@pytest.mark.parametrize("tiles,groups,sched", [
    (5360, 32, TWO),     # sc 70^3, 256 lags: 9.6e6 tasks with 96 pairs, 2.9e7 with 32
    (7000, 32, TWO),     # the largest at 256 lags
    (3800, 32, SPLIT),   # eight waves per workgroup: half as many tasks
    (32768, 1, TWO),     # sc 128^3, 8 lags
    (20797, 2, ONE),     # sc 110^3 FP32, 32 lags
])
def test_large_periodic_samples_fit_one_launch(prog, tiles, groups, sched):
    seg, streams, most = prog("periodic", tiles, tiles, groups, sched)
    assert streams * groups <= most < 2 ** 32 / 256
    assert streams * 256 < 2 ** 32  # the pair counts: one workgroup per stream
    assert tiles * -(-tiles // 96) * groups <= most  # as it did in segments of 96 pairs


@pytest.mark.parametrize("points,groups", [(600_000, 16), (1_600_000, 128), (4_000_000, 128)])
def test_large_radial_samples_fit_one_launch(prog, points, groups):
    tiles = -(-points // 64)
    seg, streams, most = prog("radial", tiles, tiles, groups, TWO)
    assert streams * groups <= most


def test_sample_beyond_one_launch_keeps_its_subsets(prog):
    """sc 110^3 x 1024 lags: at most the tasks of 96-pair segments."""
    seg, streams, most = prog("periodic", 20797, 20797, 128, TWO)
    assert streams <= 20797 * -(-20797 // 96) and streams * 128 < 2 ** 30


@pytest.mark.parametrize("tiles,groups,sched,kind,seg", [(729, 32, TWO, "periodic", 32), (8, 8, TWO, "periodic", 1),
                                                         (1024, 16, TWO, "radial", 64)])
def test_ordinary_samples(prog, tiles, groups, sched, kind, seg):
    """sc 36^3 x 256 lags, sc 8^3 x 64 lags, 65 536 points x 128 lags."""
    assert prog(kind, tiles, tiles, groups, sched)[0] == seg


@pytest.mark.parametrize("kind,tiles,groups,sched", [
    ("periodic", 125, 1, ONE), ("periodic", 125, 2, ONE), ("periodic", 64, 4, ONE), ("periodic", 64, 8, ONE),
    ("periodic", 27, 9, TWO), ("radial", 125, 1, ONE), ("radial", 313, 8, ONE), ("periodic", 128, 8, SPLIT)])
def test_rounds_are_counted(prog, kind, tiles, groups, sched):
    """The length has the least rounds x (pairs + 1) of all up to the cap; sc 20^3 x
    8 lags in BF16x3 (125 tiles, one group) took segments of 8, 10% over 32."""
    slots = 256 * (2 if sched == TWO else 1)

    def cost(seg):
        k = -(-tiles // seg)
        return -(-tiles * k * groups // slots) * (-(-tiles // k) + 1)

    seg, _, _ = prog(kind, tiles, tiles, groups, sched)
    cap = min(tiles, 64 if kind == "radial" else 32)
    assert tiles * tiles * groups < cap * cap * slots  # few enough pairs per slot
    assert seg <= cap and cost(seg) == min(cost(s) for s in range(1, cap + 1))


FP32, BF16, FP16, X3 = 0, 1, 2, 3


@pytest.mark.parametrize("L,bricks,order,taken", [
    ((36, 36, 36), 729, 729, ()),
    ((94, 191, 1), 282, 281, ()),                  # 0.4% of the tiles: slower in every precision
    ((63, 109, 1), 109, 108, (BF16, FP16)),        # 0.9%
    ((112, 142, 1), 252, 249, (BF16, FP16, FP32)),  # 1.2%
    ((34, 94, 1), 51, 50, (BF16, FP16, FP32)),     # 2.0%: BF16x3 lost 9%
    ((90, 90, 1), 130, 127, (BF16, FP16, FP32, X3)),
    ((27, 27, 27), 324, 308, (BF16, FP16, FP32, X3)),
])
def test_tile_shape_by_precision(prog, L, bricks, order, taken):
    assert prog("box", *L, -1) == [int(order < bricks), order]
    for p in (FP32, BF16, FP16, X3):
        linear, tiles = prog("box", *L, p)
        assert linear == (p in taken), p
        assert tiles == order if linear else tiles == bricks
