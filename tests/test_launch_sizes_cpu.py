"""The quantizers' cut of a job into workgroups (large pattern tables), compiled for the host: what a chip of 256 CUs that hands
workgroups out as places become free would take for it, against the work spread evenly.  No GPU is needed."""
import heapq
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = """
#include "pk_cut.h"
#include <stdio.h>
int main()
{
    int n_tiles, n_streams, ragged, by_lds, waves, waves_per_cu, multiple;   // waves 0: two_blocks_per_pass(blocks, streams, patterns, bits, given)
                                                                             // waves -1: eight_waves, by_lds and multiple workgroups per CU of either
    long long tiles;
    while (scanf("%d %d %lld %d %d %d %d %d", &n_tiles, &n_streams, &tiles, &ragged, &by_lds, &waves, &waves_per_cu, &multiple) == 8) {
        if (waves == 0) {
            printf("%d 0\\n", pk::two_blocks_per_pass(n_tiles, n_streams, ragged, by_lds, multiple != 0));
            continue;
        }
        if (waves == -1) {
            const pk::Job j = {n_tiles, n_streams, tiles, ragged != 0, 4.f};
            printf("%d 0\\n", pk::eight_waves(pk::cut_pairs(j, by_lds, 8, 16, 4), pk::cut_streams(j, multiple, 4, 16, 1), n_tiles));
            continue;
        }
        const pk::Cut c = pk::cut_streams({n_tiles, n_streams, tiles, ragged != 0, 4.f}, by_lds, waves, waves_per_cu, multiple);
        printf("%d %g\\n", c.tiles, c.cost);
    }
    return 0;
}
"""
# (workgroups that the LDS holds, waves, waves that registers allow, tiles side by side)
SHAPES = [(1, 12, 12, 12), (2, 4, 12, 4), (1, 4, 8, 4), (1, 8, 8, 8), (2, 8, 16, 4), (1, 8, 12, 2), (1, 12, 12, 3), (3, 4, 16, 1)]
STAGING = 4


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("cut")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2510_05176_amd", "csrc"), str(d / "driver.cpp"),
                    "-o", str(d / "driver")], check=True)

    def run(jobs):
        text = "\n".join(" ".join(str(int(v)) for v in j) for j in jobs)
        lines = subprocess.run([str(d / "driver")], input=text, check=True, capture_output=True, text=True).stdout.splitlines()
        return [(int(t), float(cost)) for t, cost in (line.split() for line in lines)]
    return run


def _makespan(jobs, places):
    """Jobs started in order, each as soon as a place is free."""
    free = [0.0] * places
    for j in jobs:
        heapq.heapreplace(free, free[0] + j)
    return max(free)


def _loss(lengths, t, shape):
    """Time of the cut over that of the same work in equal shares with one workgroup per stream (and one round of a workgroup's waves,
    which nothing avoids)."""
    by_lds, waves, waves_per_cu, multiple = shape
    beside = max(1, min(by_lds, waves_per_cu // waves))
    chunks = [min(t, n - s) for s in range(0, max(lengths), t) for n in lengths if n > s]
    took = _makespan([c * beside + STAGING for c in chunks], 256 * beside)
    return took / (sum(lengths) / 256 + STAGING * -(-len(lengths) // (256 * beside)) + multiple * beside)


def test_cut_leaves_no_round_nearly_empty(cut):
    """Any number of streams and any length: at most 1.5 times the evenly spread work where a CU takes one workgroup, 1.9 times where it takes
    several (one alone is counted here as slow as among others, which it is not).  One workgroup per CU, computed from the tiles of
    all streams, takes a second round as long as the first from 257 streams on."""
    rng = random.Random(3)
    jobs = [(n, s) for s in (8, 64, 200, 256, 257, 260, 288, 320, 384, 400, 511, 513, 640, 1024, 3000) for n in (1, 2, 5, 16, 33, 64, 128, 500)]
    jobs += [(rng.randint(1, 600), rng.randint(1, 2000)) for _ in range(60)]
    for shape in SHAPES:
        for (n, s), (t, _) in zip(jobs, cut([(n, s, n * s, 0, *shape) for n, s in jobs])):
            assert t > 0 and t % shape[3] == 0
            loss = _loss([n] * s, t, shape)
            assert loss < (1.5 if shape[0] == 1 else 1.9), (shape, n, s, t, loss)


def test_cut_of_a_ragged_job_follows_the_tiles_that_exist(cut):
    """Sequences of very different lengths, one long one among short ones among them: at most 1.7 times the evenly spread work."""
    rng = random.Random(4)
    jobs = [[512] + [8] * 15, [512] * 2 + [30] * 30, [128] * 3, [64, 1]]
    jobs += [[rng.randint(1, hi) for _ in range(rng.randint(2, 40))] for hi in (8, 64, 512, 2000) for _ in range(6)]
    jobs = [[n for n in j for _ in range(8)] for j in jobs]   # eight heads of a sequence
    for shape in SHAPES:
        for j, (t, _) in zip(jobs, cut([(max(j), len(j), sum(j), 1, *shape) for j in jobs])):
            assert t > 0 and t % shape[3] == 0
            loss = _loss(j, t, shape)
            assert loss < 1.7, (shape, max(j), len(j), sum(j), t, loss)


def test_cut_of_extreme_jobs(cut):
    """A single tile, a single stream of millions of vectors, hundreds of thousands of streams."""
    jobs = [(1, 1, 1, 0), (1, 1, 0, 1), (1 << 17, 1, 1 << 17, 0), (1, 1 << 19, 1 << 19, 0), (1 << 17, 1 << 12, 1 << 29, 0), (1 << 15, 4096, 1 << 15, 1)]
    for shape in SHAPES:
        for t, _ in cut([(*j, *shape) for j in jobs]):
            assert 0 < t < 1 << 20 and t % shape[3] == 0


def test_many_waves_need_many_groups(cut):
    """A flush of one or two blocks over thousands of streams, beside a table that leaves room for two workgroups of four waves: those, and
    not one of twelve of which ten idle.  Beside a table that leaves room for one workgroup, and in long jobs of a stream per CU, twelve."""
    four, twelve, alone = (2, 4, 12, 4), (1, 12, 12, 12), (1, 4, 12, 4)
    for n, s in ((1, 4096), (2, 4096), (4, 2048), (1, 288), (2, 1024)):
        few, many, single = cut([(n, s, n * s, 0, *shape) for shape in (four, twelve, alone)])
        assert few[1] < many[1] < single[1], (n, s)
    few, many = cut([(128, 256, 128 * 256, 0, *shape) for shape in (four, twelve)])
    assert many[1] < few[1]


def test_two_blocks_per_pass_need_blocks(cut):
    """One or a few blocks per stream, however many streams, never take two per pass (the second would repeat the first); jobs of many
    blocks do, with no difference between table sizes that are padded to the same number of rows."""
    def two(blocks, streams, P, bits, given=0):
        return cut([(blocks, streams, 0, P, bits, 0, 0, given)])[0][0]
    for P in (1, 64, 112, 113, 120, 127, 128):
        assert not two(1, 4096, P, 2) and not two(2, 1 << 16, P, 2) and not two(64, 8, P, 2) and not two(128, 256, P, 2, given=1)
        assert two(128, 256, P, 2) and two(16, 1024, P, 2)
        assert two(128, 256, P, 4) == two(128, 256, -(-P // 16) * 16, 4)


@pytest.mark.parametrize("by_lds", [(2, 2), (3, 3)])   # workgroups per CU beside 256 and beside 136 patterns of 128 channels
def test_eight_waves_need_many_blocks(cut, by_lds):
    """V beside a large table: jobs whose blocks give every CU at most a workgroup or two of four waves take those (an eight-wave
    workgroup takes four blocks at least), jobs of many blocks the eight-wave ones; also ragged, by the blocks that exist."""
    def eight(blocks, streams, tiles=None, ragged=0):
        return cut([(blocks, streams, tiles or blocks * streams, ragged, by_lds[0], -1, 0, by_lds[1])])[0][0]
    for blocks, streams in ((4, 8), (16, 8), (32, 8), (64, 8), (4, 32), (16, 32), (4, 128), (1, 4096), (3, 2048)):
        assert not eight(blocks, streams), (blocks, streams)
    for blocks, streams in ((64, 128), (256, 8), (4, 512), (128, 256), (2048, 4)):
        assert eight(blocks, streams), (blocks, streams)
    assert eight(512, 128, 20000, 1) and not eight(32, 16, 200, 1)


def test_two_blocks_per_pass_share_evenly(cut):
    """What counts is how many blocks a workgroup has: an odd few leave the last one to be searched twice, few are not worth it, fewer are
    enough beside larger tables."""
    def two(blocks, streams, P):
        return cut([(blocks, streams, 0, P, 2, 0, 0, 0)])[0][0]
    for P in (40, 64, 100, 128):
        assert two(8, 2048, P) and two(14, 1024, P) and two(20, 1024, P) and two(16, 512, P) and two(32, 512, P) and two(16, 320, P)
        assert not any(two(b, n, P) for b, n in ((3, 4096), (5, 4096), (9, 1024), (10, 512), (20, 256), (4, 4096), (16, 256)))
    assert two(6, 1024, 128) and not two(6, 1024, 64) and not two(10, 1024, 16) and two(12, 1024, 16)
