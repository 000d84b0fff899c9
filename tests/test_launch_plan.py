"""The rule that picks kernel and tile of a GEMM (csrc/jet_plan.h), on the host: all kernels give the same bits, so a
changed rule would drop one from the GPU tests without any of them failing."""
import pytest

import launch_plan as lp
from test_gpu_gemm import (CACHE_CASES, CHUNK_CASES, FEW_ROW_CASES, RAGGED_CASES, SAMPLED_CHUNK_CASES, SAMPLED_WGRAD_CHUNK_CASES,
                           STRIP_CASES, TILE_CASES, WGRAD_CHUNK_CASES)
from test_gpu_mfma import KERNEL_CASES

CASES = ([(M, N, K, label) for M, N, K, label in RAGGED_CASES] +
         [(M, N, 128 * g, label) for M, N, g, label in TILE_CASES + FEW_ROW_CASES])


@pytest.mark.parametrize("M,N,K,label", CASES)
def test_the_gpu_cases_run_what_their_labels_say(M, N, K, label):
    assert lp.name(M, N, K) == label.split(":")[0]


@pytest.mark.parametrize("T,groups,kernel", KERNEL_CASES)
def test_the_group_sum_cases_run_on_the_kernels_they_name(T, groups, kernel):
    assert lp.name(T, 1024, 128 * groups) == kernel


@pytest.mark.parametrize("M,N,groups,depth", STRIP_CASES)
def test_the_strip_cases_run_strips_of_their_depth(M, N, groups, depth):
    assert lp.name(M, N, 128 * groups) == "strips" and lp.strip_depth(M, N, 128 * groups) == depth


def test_every_strip_kernel_has_a_case_of_one_pass_and_one_of_more():
    seen = {(depth, -(-M // 8), groups > 32) for M, _, groups, depth in STRIP_CASES}
    assert seen >= {(depth, blocks, more) for depth in (1, 3) for blocks in (1, 2) for more in (False, True)} | {(2, 1, False), (2, 1, True)}


@pytest.mark.parametrize("M,N,groups,kernel,past", CACHE_CASES)
def test_the_cache_policy_cases_run_the_policy_they_name(M, N, groups, kernel, past):
    assert lp.name(M, N, 128 * groups) == kernel and lp.past_the_caches(M, N, 128 * groups) == past


CHUNKS = ([(lp.launches(M, N, 128 * g), g, label) for M, N, g, label in CHUNK_CASES + SAMPLED_CHUNK_CASES],
          [(lp.launches(N, K, M, row_scales=True), M // 128, label) for M, N, K, label in WGRAD_CHUNK_CASES + SAMPLED_WGRAD_CHUNK_CASES])


@pytest.mark.parametrize("launches,groups,label", CHUNKS[0] + CHUNKS[1])
def test_the_chunk_cases_run_what_their_labels_say(launches, groups, label):
    kernel, tiles = launches[0]
    assert f"{kernel}: {tiles} tiles" == label


SEVERAL_TILES = ({"big 256x256", "wide 256x128", "small 128x128", "small deep 128x128"}, {"big 256x256", "small 128x128"})


@pytest.mark.parametrize("cases,kernels", zip(CHUNKS, SEVERAL_TILES), ids=("fprop", "wgrad"))
def test_the_chunk_cases_cross_tiles(cases, kernels):
    """Every kernel that gets several tiles per workgroup: a chunk behind the first one that starts in a later tile and ends in
    another, three chunks and more; and (256x128 and 128x128 with four stages are not chosen for so few groups) one or two
    groups, where four steps are two tiles or more."""
    for kernel in kernels:
        of = [(launches[0][1], g) for launches, g, _ in cases if launches[0][0] == kernel]
        assert any(g % 4 and tiles >= 3 and tiles * g > 8 for tiles, g in of), kernel
        assert kernel in ("wide 256x128", "small deep 128x128") or any(g <= 2 and tiles >= 4 for tiles, g in of), kernel


@pytest.mark.parametrize("row_scales", (False, True))
def test_which_kernels_get_several_tiles_per_workgroup(row_scales):
    several = set()
    for I in (17, 100, 129, 257, 300, 385, 520, 641, 771, 897, 1000, 1024, 1025, 1300, 2048, 4096, 16384):
        for J in (*range(128, 8448, 384), *range(8448, 60000, 1408), 16384, 28672, 55296):
            for G in (1, 2, 3, 7, 9, 17, 32, 40, 111, 216):
                if lp.name(I, J, 128 * G, row_scales=row_scales).split()[0] not in ("panel", "strips"):
                    several |= {k for k, tiles in lp.launches(I, J, 128 * G, row_scales) if tiles > 1}
    assert several == SEVERAL_TILES[row_scales]


def test_every_tile_has_a_gpu_case():
    named = {label.split(":")[0] for *_, label in CASES}
    assert set(lp.tiles()) | {"strips", "split columns 256x256"} <= named
    # each panel with more than one chunk of 16 scales (48x112 is taken for shorter reductions only)
    for tile in lp.tiles():
        groups = [K // 128 for _, _, K, label in CASES if label.split(":")[0] == tile]
        if tile.startswith("panel") and tile != "panel 48x112":
            assert max(groups) > 15, (tile, groups)


def test_every_tile_is_chosen_somewhere_and_fits_its_kernel():
    seen = set()
    for I in (1, 7, 16, 17, 32, 33, 48, 64, 65, 80, 96, 97, 128, 129, 200, 256, 257, 400, 512, 700, 1000, 1024, 1025, 4096, 16384, 17408):
        for J in (128, 256, 384, 1024, 4096, 5120, 6144, 8320, 9600, 12416, 14336, 14464, 16512, 19072, 27648, 28672, 55296):
            for R in (128, 1024, 4096, 14336, 27648):
                for row_scales in (False, True):
                    k, bm, bn, split = lp.plan(I, J, R, row_scales)
                    seen.add(lp.name(I, J, R, row_scales=row_scales))
                    assert k == "panel" or J % bn == 0                        # only panels have ragged columns
                    assert k != "strips" or I <= 16
                    assert not row_scales or k in ("big", "small", "small deep", "split rows", "split columns")
                    if k.startswith("split"):
                        assert split % 256 == 0 and 0 < split < (I if k == "split rows" else J)
                        rest = (I - split, J) if k == "split rows" else (I, J - split)
                        for part in ((split, J) if k == "split rows" else (I, split), rest):
                            sub = lp.plan(*part, R, row_scales, whole=False)[0]
                            assert sub != "strips" and not sub.startswith("split")
    assert set(lp.tiles()) | {"strips", "split rows 256x256", "split columns 256x256"} <= seen


@pytest.mark.parametrize("M,N,K,within", [
    # the tiles within 5 % of the fastest, weights from HBM or from the caches
    (160, 16384, 1024, ("small deep 128x128", "small 128x128", "half 128x64")), (112, 16384, 1024, ("half 128x64",)),
    (257, 16384, 1024, ("small 128x128", "wide 256x128")), (400, 4096, 4096, ("half 128x64", "panel 128x64")),
    (400, 4096, 1024, ("half 128x64", "panel 128x64")), (1024, 2048, 2048, ("half 128x64", "panel 128x64")),
    (600, 3072, 1024, ("half 128x64",)), (700, 7168, 5120, ("wide 256x128",)), (1024, 5120, 27648, ("wide 256x128",)),
    (257, 28672, 4096, ("big 256x256", "small deep 128x128", "wide 256x128")), (350, 11008, 2048, ("wide 256x128", "small 128x128")),
    (1, 1024, 5120, ("strips",)), (8, 8192, 2048, ("strips",)), (1, 5120, 2560, ("strips",)), (16, 2048, 2048, ("strips",)),
])
def test_shapes_that_a_rule_without_a_time_per_round_got_wrong(M, N, K, within):
    """A cost of rounds x lines alone took a tile that was 5 to 37 % slower than another one (and than the kernels before
    that rule); the strips' share of full passes and rounds alone, panels that were 5 to 20 % slower."""
    assert lp.name(M, N, K) in within


def test_part_of_a_split_problem_never_runs_strips():
    """The skinny kernel writes rows of J elements; the rows of a part are further apart."""
    for I in range(1, 17):
        assert lp.plan(I, 4096, 4096)[0] == "strips"
        assert lp.plan(I, 4096, 4096, whole=False)[0] != "strips"


@pytest.mark.parametrize("d", [1, 2, 3, 5, 7, 8, 24, 127, 1736, 65535, 65536, 8388607, 1 << 27, (1 << 31) - 1])
def test_quotients_without_a_division(d):
    """Tile origins of the tile kernel: multiples of the divisor and their neighbours, and both ends of the range."""
    top = (1 << 31) - 1
    multiples = {k * d for k in (1, 2, 3, 5, 1000, top // d // 2, top // d - 1, top // d)}
    for n in {0, 1, top - 1, top} | {m + e for m in multiples for e in (-1, 0, 1)}:
        if 0 <= n <= top:
            assert lp.lib().jet_quotient(n, d) == n // d, (n, d)


def test_scales_are_read_where_a_copy_has_put_them():
    placed = {lp.chunk(lane=lane)[0]: 4 * lane for lane in range(64)}
    assert len(placed) == 64
    for row in range(16):
        for step in range(4):
            assert lp.chunk(row=row, step=step)[1] == placed[row, step]
            # four neighbouring columns are one 16-byte read
            assert lp.chunk(row=row, step=step)[1] == lp.chunk(row=row & ~3, step=step)[1] + 4 * (row & 3)


def test_scales_of_a_step_lie_in_different_banks():
    """A 4-byte read takes 32 banks at a time; lanes of equal rows read the same word."""
    for step in range(4):
        assert len({lp.chunk(row=row, step=step)[1] // 4 % 32 for row in range(16)}) == 16
