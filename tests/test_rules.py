"""The size rules of the launches, from a host build of their header.  (CPU only.)"""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2206_00470_amd", "csrc")
LLC = 256 << 20   # bytes of the last-level cache


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, "-o", exe, os.path.join(HERE, "rules_check.cpp")])
    return lambda *a: int(subprocess.check_output([exe, *map(str, a)], text=True))


@pytest.mark.parametrize("dim,per_store", [(4, 4), (50, 1), (64, 4), (100, 4), (512, 4), (1000, 4)])
def test_a_pulled_output_is_streamed_only_past_the_last_level_cache(rule, dim, per_store):
    """A reader finds a smaller output in the cache."""
    line = LLC // (4 * dim)
    assert rule("pull_streams", line, dim, per_store) == 0
    assert rule("pull_streams", line + 1, dim, per_store) == 1
    assert rule("pull_streams", (32 << 20) // (4 * dim) + 1, dim, per_store) == 0
    assert rule("pull_streams", 2**31 - 2**20, dim, per_store) == 1


def test_rows_that_write_lines_in_parts_are_not_streamed(rule):
    """Rows of one float per lane wider than a wavefront never, rows of 257 to
    512 floats that share 64-byte pieces not into a large output."""
    for dim in (65, 130, 301, 511):
        for gb in (0.3, 1, 5, 20):
            assert rule("pull_streams", int(gb * 1e9) // (4 * dim), dim, 1) == 0
    assert rule("pull_streams", 10**9 // 1024, 256, 1) == 0     # an unaligned output
    for dim, large in ((260, 0), (300, 0), (500, 0), (272, 1), (400, 1), (512, 1), (100, 1), (252, 1), (516, 1), (1000, 1)):
        assert rule("pull_streams", 5 * 10**8 // (4 * dim), dim, 4) == 1
        for gb in (2, 5, 20):
            assert rule("pull_streams", gb * 10**9 // (4 * dim), dim, 4) == large


@pytest.mark.parametrize("groups_per_block", [64, 16, 4])
def test_small_pulls_keep_one_row_per_group(rule, groups_per_block):
    """Four rows per group where the groups would not all run at once anyway."""
    line = 2048 * groups_per_block
    for n in (1, 1000, line):
        assert rule("pull_rows", n, groups_per_block, 4) == 1
    for n in (line + 1, 2**31 - 2**20):
        assert rule("pull_rows", n, groups_per_block, 4) == 4
        assert rule("pull_rows", n, groups_per_block, 1) == 4
        assert rule("pull_rows", n, groups_per_block, 8) == 1   # eight floats per lane are enough in flight


@pytest.mark.parametrize("dim,lanes,tiled,separate", [(64, 16, 120_000, 200_000), (128, 32, 64_000, 200_000),
                                                      (200, 64, 24_000, 64_000), (140, 64, 20_000, 47_000),
                                                      (50, 64, 28_000, 125_000)])
def test_a_prepare_beside_a_long_merge_takes_no_tiles(rule, dim, lanes, tiled, separate):
    assert tiled <= rule("push_prepare_tiled_keys", dim, lanes) < separate


def test_a_prepare_beside_the_merge_of_wide_rows_takes_tiles(rule):
    assert rule("push_prepare_tiled_keys", 300, 64) > 96 * 4096


@pytest.mark.parametrize("layout", ["dense", "interleaved", "rowwise", "bf16"])
def test_merges_stream_rows_that_leave_few_lines_in_parts(rule, layout):
    """Rows that can exceed the last-level cache are streamed at the widths that
    gain from it, in each layout; narrow or one-float-per-lane rows are not."""
    args = dict(dense=(0, 0, 0), interleaved=(0, 0, 1), rowwise=(1, 0, 0), bf16=(0, 1, 0))[layout]
    row = {"rowwise": lambda d: 4 * d + 4, "bf16": lambda d: 6 * d}.get(layout, lambda d: 8 * d)
    yes = dict(dense=[16, 32, 48, 64, 80, 96, 100, 140, 200, 256, 300, 500, 512, 1000],
               interleaved=[16, 28, 32, 36, 48, 60, 64, 68, 96, 100, 140, 200, 300, 512, 1000],
               rowwise=[64, 68, 80, 96, 100, 128, 200, 300, 130, 250, 301, 511], bf16=[32, 64, 96, 100, 140, 200, 300, 512])
    no = dict(dense=[4, 20, 28, 36, 60, 68, 13, 50, 63, 65, 101, 127, 130, 250, 511],
              interleaved=[4, 20, 24, 13, 50, 63, 65, 101, 130, 250, 511],
              rowwise=[4, 16, 20, 28, 32, 48, 60, 13, 50, 65, 101, 127],
              bf16=[4, 16, 20, 28, 36, 48, 60, 68, 50, 65, 101, 130, 301])
    for d in yes[layout]:
        line = LLC // row(d)
        assert rule("merge_streams", line, d, *args) == 0, d
        assert rule("merge_streams", line + 1, d, *args) == 1, d
    for d in no[layout]:
        assert rule("merge_streams", 2**31 - 2**20, d, *args) == 0, d


@pytest.mark.parametrize("dim,triples,tiled,separate", [(64, 1300, 198_900, 276_000), (256, 1000, 153_000, 367_200),
                                                        (512, 1000, 45_900, 153_000), (64, 28_000, 92_000, 196_000)])
def test_key_work_beside_the_complex_gradient_takes_few_tiles(rule, dim, triples, tiled, separate):
    assert tiled <= rule("kge_tiled_keys", dim, triples) < separate
