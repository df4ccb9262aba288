"""Calls that a line of the dispatch once sent to the slower of two kernels (the measured times stand at launch_forward), and
the claims that tests on the GPU make about the kernels their calls are sent to."""
import pytest

from tests import dispatch
from tests import test_gpu_dispatch as on_gpu
from tests import test_gpu_small_tiles as on_small_tiles


@pytest.mark.parametrize("b, n, hq, hkv, d, seqlens, shares", [
    (2, 1900, 14, 2, 128, True, 2), (2, 1900, 14, 2, 64, True, 2), (2, 1600, 16, 8, 64, True, 2), (4, 1700, 8, 8, 128, True, 2),
    (4, 1700, 8, 2, 128, True, 1), (2, 1400, 20, 4, 128, True, 1),                                  # one KV head to an XCD
    (1, 1900, 28, 4, 64, False, 2), (1, 1900, 28, 4, 128, False, 1), (1, 1700, 32, 8, 64, False, 1),
])
def test_split_where_nearly_every_place_is_taken(b, n, hq, hkv, d, seqlens, shares):
    assert dispatch.forward(b, n, hq, hkv, d, 128, seqlens=seqlens).shares == shares


@pytest.mark.parametrize("b, n, hq, hkv, seqlens, tiles, shares", [
    (64, 100, 3, 3, False, 1, 1), (8, 250, 12, 4, False, 1, 1), (24, 190, 6, 2, False, 1, 1), (300, 60, 3, 1, False, 1, 1), (2000, 10, 3, 3, False, 1, 1),
    (4, 900, 16, 16, True, 1, 1), (3, 3000, 8, 8, True, 1, 1), (8, 500, 12, 4, True, 1, 1), (8, 500, 16, 16, True, 1, 1), (32, 200, 3, 1, True, 1, 1),
    (64, 130, 3, 3, False, 2, 1), (64, 127, 6, 2, True, 2, 1), (4, 600, 28, 4, True, 2, 1), (16, 300, 12, 4, True, 2, 1), (2, 5000, 16, 16, True, 2, 1), (4, 450, 12, 4, False, 2, 2),
])
def test_64_row_tiles_of_width_128(b, n, hq, hkv, seqlens, tiles, shares):
    """Tiles of an odd group: alone or with the next one in a workgroup."""
    x = dispatch.forward(b, n, hq, hkv, 128, 64, seqlens=seqlens)
    assert (x.tiles, x.shares) == (tiles, shares)


def test_short_chains_of_shared_heads_are_not_split():
    assert dispatch.forward(64, 100, 4, 2, 128, 64)[3:6] == (2, 1, 1) and dispatch.forward(40, 200, 3, 1, 128, 32).shares == 1


@pytest.mark.parametrize("b, n, hq, hkv, seqlens, tiles, shares", [
    (64, 130, 3, 3, False, 1, 1), (1, 1000, 40, 8, False, 1, 1), (200, 180, 3, 1, False, 1, 1), (150, 250, 3, 1, False, 1, 1),
    (16, 300, 28, 4, True, 1, 1), (4, 900, 12, 4, True, 1, 1), (32, 200, 28, 4, True, 1, 1), (600, 128, 9, 3, True, 1, 1), (300, 60, 3, 3, False, 1, 1), (4, 2000, 16, 16, True, 1, 1),
    (100, 250, 3, 1, False, 2, 1), (2, 5000, 12, 4, True, 2, 1), (2, 4096, 12, 4, False, 2, 1), (4, 500, 12, 4, False, 1, 2),
])
def test_64_row_tiles_of_width_64(b, n, hq, hkv, seqlens, tiles, shares):
    """Tiles of an odd group: alone or with the next one in a workgroup."""
    x = dispatch.forward(b, n, hq, hkv, 64, 64, seqlens=seqlens)
    assert (x.tiles, x.shares) == (tiles, shares)


@pytest.mark.parametrize("b, n, hq, hkv, d, seqlens, heads, tiles", [
    (2000, 10, 4, 2, 128, False, 2, 1), (2000, 10, 4, 2, 64, False, 2, 1), (300, 30, 4, 2, 64, False, 2, 1), (2000, 10, 3, 1, 64, False, 1, 1), (300, 30, 3, 3, 64, True, 1, 1),
    (64, 20, 8, 2, 64, False, 2, 1), (300, 30, 8, 2, 64, False, 4, 1),
    (64, 130, 3, 3, 64, False, 1, 2), (4, 900, 12, 4, 64, True, 1, 2), (3, 3000, 8, 8, 64, True, 1, 2), (16, 300, 28, 4, 64, True, 1, 2), (200, 180, 3, 1, 64, False, 1, 2),
    (100, 250, 3, 1, 64, False, 1, 4), (8, 500, 28, 4, 64, True, 1, 4), (1, 8192, 28, 4, 64, False, 1, 4), (300, 60, 4, 2, 64, False, 2, 2), (2000, 10, 3, 1, 128, False, 1, 4),
])
def test_32_row_tiles(b, n, hq, hkv, d, seqlens, heads, tiles):
    """Heads and adjacent tiles of a workgroup, where key blocks are not dealt to several sets of waves."""
    x = dispatch.forward(b, n, hq, hkv, d, 32, seqlens=seqlens)
    assert (x.heads, x.tiles, x.shares) == (heads, tiles, 1)


@pytest.mark.parametrize("b, n, hq, hkv, d, tiles", [
    (1, 589, 12, 4, 128, 1), (1, 589, 12, 4, 64, 1), (16, 100, 3, 1, 128, 1), (8, 200, 12, 4, 64, 1), (8, 200, 12, 4, 128, 1), (1, 800, 28, 4, 128, 2), (1, 3000, 28, 4, 64, 2),
])
def test_score_half_of_64_row_tiles(b, n, hq, hkv, d, tiles):
    x = dispatch.scores(b, n, hq, hkv, d, 64)
    assert x.score and (x.heads, x.tiles) == (1, tiles)


@pytest.mark.parametrize("hq, hkv, n, d, bm, causal, fp8, dtype", on_gpu.SHARED_HEADS)
def test_shared_heads_are_compared_with_single_ones(hq, hkv, n, d, bm, causal, fp8, dtype):
    kw = dict(causal=causal, qk_fp8=fp8, workspace=True)
    shared, single = dispatch.forward(1, n, hq, hkv, d, bm, **kw), dispatch.forward(1, n, hq, hkv, d, bm, single_head=True, **kw)
    assert shared.heads > 1 and single.heads == 1 and shared.shares == single.shares == 1


@pytest.mark.parametrize("b, n, hq, hkv, d, bm", on_gpu.TURNED)
def test_turned_places_are_compared_with_places_in_order(b, n, hq, hkv, d, bm):
    plain, counted = dispatch.forward(b, n, hq, hkv, d, bm), dispatch.forward(b, n, hq, hkv, d, bm, seqlens=True)
    assert plain.turn[1] > plain.turn[0] > 0 and counted.turn == (0, 0, 0) and plain.shares == counted.shares == 1


def test_every_kernel_is_run_by_the_comparisons_of_forms():
    """Every instantiated form, by the calls that are compared with each other on the GPU."""
    ran = set()
    for b, n, hq, hkv, d, bm, causal, _ in on_gpu.CASES + on_gpu.SMALL_TILES + on_gpu.FEW_TILES:
        many = b * (1 + 150000 // (b * hq * n * (1 if causal else 2)))
        ran |= {dispatch.forward(b, n, hq, hkv, d, bm, causal), dispatch.forward(b, n, hq, hkv, d, bm, causal, single_head=True),
                dispatch.forward(many, n, hq, hkv, d, bm, causal)}
    for hq, hkv, n, d, bm, causal, fp8, _ in on_gpu.SHARED_HEADS:
        ran |= {dispatch.forward(1, n, hq, hkv, d, bm, causal, single_head=x, qk_fp8=fp8, workspace=True) for x in (False, True)}
    ran |= {dispatch.scores(*x) for x in on_gpu.SCORES}
    forms = dispatch.instantiated()
    assert len(forms) >= 40 and not forms - {x[:7] for x in ran}


@pytest.mark.parametrize("hq, hkv, d, bm", on_small_tiles.PREDICATE)
def test_the_predicate_meets_adjacent_tiles(hq, hkv, d, bm):
    x = dispatch.forward(on_small_tiles.PREDICATE_BATCH, on_small_tiles.PREDICATE_TOKENS, hq, hkv, d, bm, gate_mode=1)
    assert x.tiles == 128 // bm and x.shares == 1 and (on_small_tiles.PREDICATE_TOKENS // bm) % x.tiles


@pytest.mark.parametrize("hq, hkv, d, bm", on_small_tiles.WITH_LENGTHS)
def test_lengths_meet_adjacent_tiles(hq, hkv, d, bm):
    x = dispatch.forward(len(on_small_tiles.LENGTHS), max(on_small_tiles.LENGTHS), hq, hkv, d, bm, seqlens=True)
    assert x.tiles == 128 // bm and x.shares == 1


@pytest.mark.parametrize("hq, hkv, d, bm, n, lengths", on_gpu.IN_PLACE_ORDER + on_gpu.COUNTED_OFF)
def test_work_items_of_elements_with_lengths(hq, hkv, d, bm, n, lengths):
    """Counted off where more than one workgroup comes to a CU and the pairs of an XCD fit a row of lanes."""
    x = dispatch.forward(len(lengths), n, hq, hkv, d, bm, seqlens=True)
    assert x.counted == ((hq, hkv, d, bm, n, lengths) in on_gpu.COUNTED_OFF)
