"""Which gradient GEMMs share a launch, asked on the host."""
from paper_2506_19645_amd import binding as B
from tests import test_gpu_gemm_pairs as pairs


TILES = {0: (256, 256), 1: (192, 256), 3: (128, 128), 4: (64, 128), 5: (64, 64)}
SLOTS = 256   # workgroups of persistent tiles that run at once


def tiles(M, N, G, tile):
    bm, bn = TILES[tile]
    return -(-M // bm) * -(-N // bn) * G


def test_gpu_tests_reach_every_pair_kernel_and_every_order():
    seen = set()
    for swi, T, n, h, fr, hs in pairs.PAIRS:
        for first, (N, K) in ((True, (fr, h)), (False, (h, 2 * fr if swi else fr))):
            r = B.gemm_pair_route(T, n, N, K)
            if r < 0:
                continue
            tile, wgrad_first, one_each, epi = r % 16, bool(r & 16), bool(r & 32), ("gelu", "swiglu")[swi] if first else "plain"
            seen |= {(tile, epi), r}
            if tile > 1 or n % TILES[tile][0] == 0 or N % TILES[tile][1] == 0:
                continue
            dgrad, wgrad = tiles(n, N, T, tile), tiles(K, N, T, tile)
            if (wgrad if wgrad_first else dgrad) > SLOTS:
                seen.add(("first walks", tile, wgrad_first))
            if (dgrad if wgrad_first else wgrad) > SLOTS and not one_each:
                seen.add(("second walks a share", tile, wgrad_first))
            if dgrad > SLOTS and not (wgrad_first and one_each):
                seen.add(("data gradient walks", epi))
    missing = {(tile, e) for tile in TILES for e in ("gelu", "swiglu", "plain")} - seen
    # persistent tiles: either GEMM first, the second by the tile and in shares; others: either first, always by the tile
    missing |= ({0, 16, 32, 48, 17, 33, 35, 51, 36, 52, 37, 53} | {1, 49}) - seen
    missing |= {(walk, tile, wf) for walk in ("first walks", "second walks a share") for tile in (0, 1) for wf in (False, True)} - seen
    missing |= {("data gradient walks", e) for e in ("gelu", "swiglu")} - seen
    assert not missing, sorted(map(str, missing))


def test_most_blocks_that_run_one_by_one_would_pair():
    runs = [pairs.paired(*b[:5]) for b in pairs.BLOCKS]
    assert sum(runs) >= 40, (sum(runs), len(runs))


def test_training_steps_pair_their_gradient_gemms_unless_one_is_a_long_chain():
    for T, n, h, fr in ((2, 256, 768, 1536), (4, 1111, 2048, 1408), (4, 8192, 2048, 2048), (8, 147, 1536, 768)):
        assert B.gemm_pair_route(T, n, fr, h) >= 0
    assert B.gemm_pair_route(2, 7476, 512, 1024) == -1        # 8 x 512 columns from 7476 rows: tiles that share a contraction
    assert B.gemm_pair_route(0, 1, 8, 8) == B.gemm_pair_route(1, 1 << 31, 8, 8) == -2


def test_a_pair_is_as_long_as_its_last_tile():
    """A data gradient that is a long chain on half of the compute units, and a weight gradient of many short tiles that the
    other half would have to take: backward passes with the two in one launch took 404 us for 314, 92 for 82, 97 for 88."""
    for T, n, N, K in ((1, 198, 4096, 28672), (2, 211, 2048, 5632), (2, 141, 2048, 7168), (1, 690, 2048, 14336)):
        assert B.gemm_pair_route(T, n, N, K) == -1


def test_the_stores_to_all_ranks_count_in_a_pair():
    """Few large tiles that store to 16 or 8 ranks each: forward passes took 194 us for 154, 206 for 165, 119 for 102 in a pair of
    128 x 128 tiles."""
    for T, n, h, hs, K in ((16, 4979, 512, 328, 112), (16, 6745, 512, 128, 128), (8, 7723, 512, 128, 256)):
        r = B.gemm_shared_pair_route(T, n, h, hs, K)
        assert r == -1 or r % 16 > 3 or r // 256 > 1


def test_a_pair_sums_the_ranks_in_the_groups_of_two_launches():
    """The bits depend neither on whether the private columns share the launch nor on how the residual stream is stored."""
    paired = 0
    for T in (2, 4, 8, 16):
        for n in (65, 136, 200, 390, 777, 1300, 2056, 3500):
            for h, hs, K in ((1024, 512, 512), (2048, 512, 1376), (4096, 2048, 512), (4096, 1024, 1376), (4096, 8, 72), (1032, 520, 2752)):
                r = B.gemm_shared_pair_route(T, n, h, hs, K)
                alone = B.gemm_route(B.GEMM_NT, 6, 1, n, hs, K, T)
                if r >= 0:
                    paired += 1
                    assert r // 256 == max(1, alone // 256), (T, n, h, hs, K)
    assert paired > 100


def test_gpu_tests_reach_every_pair_of_private_and_shared_columns():
    """Every tile with the shared sums in groups and directly (1 group); persistent tiles of which a workgroup walks several, by the
    private columns first and by either part second, in shares (shared columns first take products too large for a test)."""
    seen, walks = set(), set()
    for T, n, h, fr, hs in pairs.SHARED:
        r = B.gemm_shared_pair_route(T, n, h, hs, fr)
        if r < 0:
            continue
        tile, groups, shared_first, one_each = r % 16, r // 256, bool(r & 16), bool(r & 32)
        seen.add((tile, groups > 1))
        if tile < 2:
            private, shared = tiles(n, h - hs, T, tile), tiles(n, hs, groups, tile)
            if not shared_first and private > SLOTS:
                walks.add("private first")
            if (private if shared_first else shared) > SLOTS and not one_each:
                walks.add("private shares" if shared_first else "shared shares")
    assert seen == {(tile, groups) for tile in TILES for groups in (False, True)}
    assert walks == {"private first", "private shares", "shared shares"}
    assert B.gemm_shared_pair_route(8, 128, 1536, 768, 2048) == -1   # the private columns stream their weights
    assert B.gemm_shared_pair_route(8, 96, 4096, 4096, 512) == -2
