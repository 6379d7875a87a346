"""CPU test of the rules that choose the kernel and the key ranges of an attention call
(launch_rules.hpp), compiled for the host: the calls the rules were measured at."""
import os
import shutil
import subprocess
from collections import namedtuple

import pytest

Rule = namedtuple("Rule", "fwd_few fwd_splits bwd_few ways k by_xcd rotated_entries together_entries terms_first "
                          "dkv_chunk dkv_ring joined", defaults=[1, 0, 0, 0, 0, 0, 0])


@pytest.fixture(scope="module")
def rules(repo_root, tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("rules") / "rules")
    src = os.path.join(repo_root, "tests", "host_rules", "rules_main.cpp")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", src, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def ask(D, pairs, Nq, hist, block_rows=0, in_order=False):
        """hist = resident rows, of all streams or of each"""
        hist = hist if isinstance(hist, list) else [hist]
        line = f"{D} {pairs} {Nq} {block_rows} {int(in_order)} {len(hist)} {' '.join(map(str, hist))}\n"
        out = subprocess.run([exe], input=line, capture_output=True, text=True, check=True).stdout
        return Rule(*map(int, out.split()))
    return ask


@pytest.mark.parametrize("D,pairs,Nq,hist,want", [
    (128, 12, 4680, 28080, Rule(0, 4, 0, 2, 7)),   # one production stream: 444 workgroups
    (128, 48, 4680, 28080, Rule(0, 1, 0, 1, 1)),   # four
    (128, 2, 252, 189, Rule(4, 1, 4, 1, 1)),       # a few rows
    (64, 16, 4680, 20280, Rule(0, 3, 0, 2, 4)),
])
def test_named_sizes(rules, D, pairs, Nq, hist, want):
    got = rules(D, pairs, Nq, hist)
    # what a call's other route would be cut into does not matter
    assert got.fwd_few == want.fwd_few and got.bwd_few == want.bwd_few
    assert want.fwd_few or got.fwd_splits == want.fwd_splits
    assert want.bwd_few or (got.ways, got.k) == (want.ways, want.k)


def test_outputs_over_inputs_take_the_routes_that_read_first(rules):
    for D, pairs, Nq, hist in [(128, 2, 252, 189), (128, 12, 4680, 28080), (64, 6, 2080, 1560), (128, 31, 2080, 1040)]:
        got = rules(D, pairs, Nq, hist, in_order=True)
        assert got.fwd_few == 0 and got.bwd_few == 0 and got.ways == 1
    assert rules(128, 480, 128, 5728, in_order=True).fwd_splits == 4 and rules(128, 480, 128, 5728).fwd_splits == 1


def test_ranges_of_streams_of_different_lengths(rules):
    """One short stream does not keep the launch from being cut (four streams of 0, 7, 9 and 10 frames of 768
    tokens, 72 workgroups: 236 us uncut, 62 in seven ranges), nor do causal blocks."""
    assert rules(128, 4, 2304, [0, 5376, 6912, 7680], block_rows=768).fwd_splits >= 5
    assert rules(64, 9, 4218, [1406, 2812, 16872], block_rows=1406).fwd_splits >= 4


def test_order_of_streams_of_different_lengths(rules):
    """A contiguous eighth of the workgroups per XCD while the heaviest eighth has little more than its share."""
    for heads in (3, 8):  # pairs that do not divide evenly over the XCDs, and that do
        for hist in ([28080] * 8, [28080] * 7 + [0], [15600, 14040], [9000] * 5 + [9900]):
            assert rules(128, heads * len(hist), 4680, hist).by_xcd == 1
        for hist in ([0, 15600], [500] * 5 + [9900], [0, 28080, 28080, 0]):
            assert rules(128, heads * len(hist), 9360, hist).by_xcd == 0
            # every workgroup on a CU of its own
            assert rules(128, heads * len(hist), 128, hist).by_xcd == 1


def test_ranges_of_launches_with_64_wide_heads(rules):
    """Four workgroups fit a CU at D = 64: sizes that an estimate with three left uncut (240 workgroups x 165 tiles
    110 us uncut, 65 in three or four ranges; 480 x 341 239 uncut, 194 - 200 in three to five; 256 x 165 106, 66)."""
    assert rules(64, 40, 720, 4560, block_rows=240).fwd_splits in (3, 4)
    assert rules(64, 96, 520, 10400).fwd_splits > 2
    assert rules(64, 32, 960, 4320, block_rows=480).fwd_splits in (3, 4)


def test_forward_with_few_rows_gives_way_where_the_general_kernel_is_faster(rules):
    """Sizes measured with both: a second or third workgroup on a few CUs only, short walks, and streams of
    different lengths, whose longest walk the general kernel cuts."""
    for call in [(64, 6, 1560, 17160), (64, 3, 2970, 12870, 990), (128, 192, 96, 96), (128, 160, 126, 126, 63), (64, 12, 792, 11880),
                 (128, 6, 1440, 3900), (128, 576, 96, 160, 32), (64, 640, 390, 390), (128, 384, 54, 72),
                 (64, 32, 1040, [2600, 1560, 4680, 2600, 0, 1040, 2080, 0]), (128, 480, 126, [63, 630, 630, 63])]:
        assert rules(*call).fwd_few == 0, call
    for call in [(128, 4, 32, 288), (64, 8, 570, 2570), (128, 12, 390, 3120), (128, 16, 240, 4240), (64, 32, 960, 2624), (128, 64, 320, 608), (64, 200, 130, 650), (128, 32, 768, 960)]:
        assert rules(*call).fwd_few != 0, call


def test_backward_with_few_rows_gives_way_where_the_general_kernels_are_faster(rules):
    """Blocks of 128 rows just above and below the lines, at both head sizes, short walks and long ones."""
    for call in [(128, 24, 696, 696), (128, 32, 640, 640), (128, 48, 330, 660, 126), (64, 24, 1040, 1040), (64, 32, 960, 1280), (64, 48, 640, 1600),
                 (64, 256, 128, 448), (128, 30, 390, 7800)]:
        assert rules(*call).bwd_few == 0, call
    for call in [(128, 16, 480, 2400), (128, 32, 390, 520), (64, 48, 390, 520), (64, 32, 390, 7800), (128, 2, 128, 448), (128, 48, 330, 330), (64, 120, 200, 260), (64, 128, 130, 30)]:
        assert rules(*call).bwd_few != 0, call


def test_split_of_the_dq_walk_only_where_it_gains(rules):
    """Sizes measured both ways; and a helper per item where the walks of the items differ."""
    for call in [(128, 120, 480, 2400), (128, 96, 640, 4480), (128, 96, 480, 2080), (64, 60, 1024, 1536), (64, 128, 640, 2240), (64, 144, 640, 2240),
                 (64, 36, 1500, 4000), (128, 192, 480, 2400)]:
        assert rules(*call).ways == 1, call
    for call, ways in [((128, 3, 4680, 28080), (3,)), ((128, 5, 4680, 15600), (2, 3)), ((128, 12, 4680, 28080), (2,)), ((128, 14, 4680, 18720), (3,)),
                       ((128, 20, 4680, 18720), (2, 3)), ((64, 16, 4680, 18720), (2,)), ((64, 4, 4680, 25000), (3,))]:
        assert rules(*call).ways in ways, call
    for D in (64, 128):
        for pairs in range(4, 130, 6):
            uneven = rules(D, pairs, 1560, [1560, 17160])
            assert uneven.k == 1 or uneven.ways == 1


def test_forward_rotates_its_chunk_only_with_few_chunk_tiles_per_wave(rules):
    for D, pairs, most, entries in [(64, 24, 12, 384), (128, 4, 8, 896)]:  # four waves: tiles of 32 chunk rows
        assert rules(D, pairs, 32 * most, 64).fwd_few == 4 and rules(D, pairs, 32 * most, 64).rotated_entries == entries
        assert rules(D, pairs, 32 * most + 1, 64).rotated_entries == 0
    for D, most, entries in [(64, 20, 384), (128, 16, 896)]:  # eight
        assert rules(D, 1, 32 * most, 2048).fwd_few == 8 and rules(D, 1, 32 * most, 2048).rotated_entries == entries
        assert rules(D, 1, 32 * most + 1, 2048).rotated_entries == 0
    for D in (64, 128):
        assert rules(D, 12, 4680, 28080).rotated_entries == 0  # the general kernel
        assert rules(D, 4, 64, 64, in_order=True).rotated_entries == 0


def test_waves_turn_short_chunks_together(rules):
    """Launches of eight waves only, on both sides of the most tiles and (cos, sin); a forward rotates for itself where they do."""
    for D, pairs, Nq, hist, together in [(64, 2, 31, 248, 384), (64, 6, 32, 288, 384), (64, 4, 33, 264, 384), (64, 2, 255, 510, 384), (64, 2, 256, 0, 384),
                                         (64, 3, 256, 256, 384), (64, 1, 257, 257, 0), (128, 2, 63, 567, 512), (128, 12, 64, 512, 512), (128, 1, 65, 585, 0),
                                         (64, 2, 64, 64, 0), (128, 2, 64, 256, 0)]:
        got = rules(D, pairs, Nq, hist)
        assert got.together_entries == together and (got.fwd_few == 8 or not together), (D, pairs, Nq, hist)
        assert got.rotated_entries >= got.together_entries


def test_waves_of_launches_with_few_rows(rules):
    """Eight only where every workgroup has a CU to itself and its waves have enough tiles."""
    for call, fwd, bwd in [((64, 2, 64, 256), 8, 4), ((64, 16, 260, 780), 8, 4), ((64, 30, 216, 1404), 8, 4), ((64, 24, 405, 4455), 4, 4),
                           ((128, 2, 64, 256), 4, 4), ((128, 16, 234, 468), 8, 4), ((128, 3, 672, 448), 8, 8),
                           ((128, 64, 90, 0), 4, 4), ((128, 16, 330, 1210), 8, 4), ((64, 12, 108, 810), 8, 8), ((128, 4, 192, 1900), 8, 8), ((64, 1, 32, 0), 4, 4)]:
        assert (rules(*call).fwd_few, rules(*call).bwd_few) == (fwd, bwd), call


def test_row_terms_of_a_backward_with_few_rows_come_first_for_long_chunks_over_short_rings(rules):
    for call, want in [((128, 3, 672, 448), 1), ((128, 3, 384, 1151), 1), ((128, 3, 384, 1152), 0), ((128, 3, 383, 0), 0),
                       ((64, 3, 512, 1023), 1), ((64, 3, 512, 1024), 0), ((64, 3, 511, 0), 0), ((64, 1, 2048, [0, 5000]), 0)]:
        assert rules(*call).bwd_few and rules(*call).terms_first == want, call


def test_key_blocks_of_shorter_streams_do_not_count(rules):
    """A ring launch's kernel goes by the blocks that have keys: one long stream among empty ones is a few workgroups, whatever
    the grid (16 pairs of 64, 2340 rows in one stream of eight, 19 blocks each)."""
    assert rules(64, 16, 260, [2340] + [0] * 7).dkv_ring == 0
    assert rules(64, 16, 260, [2340] * 8).dkv_ring == 1
    assert rules(64, 24, 2080, [4160] + [1] * 7).dkv_ring == rules(64, 3, 2080, [4160 + 7 * 128]).dkv_ring


def test_kernel_of_dk_and_dv_by_key_blocks_and_length_of_the_walk(rules):
    """D = 64, on both sides of each line: roles and two waves with a workgroup per CU, one wave with more, D = 128 roles only."""
    for Nq, pairs, want in [(832, 36, 0), (833, 36, 2), (896, 36, 2), (390, 64, 0), (390, 65, 1), (2176, 15, 2), (2176, 16, 1), (4680, 1, 2), (4680, 6, 2), (4680, 7, 1)]:
        assert rules(64, pairs, Nq, 3000).dkv_chunk == want, (Nq, pairs)
        assert rules(128, pairs, Nq, 3000).dkv_chunk == 0
    for Nq, pairs, hist, want in [(832, 2, 3840, 0), (833, 2, 3840, 2), (512, 7, 3840, 0), (512, 9, 3584, 0), (512, 9, 3585, 1), (2048, 8, 4096, 2),
                                  (2048, 8, 4097, 1)]:
        assert rules(64, pairs, Nq, hist).dkv_ring == want, (Nq, pairs, hist)
        assert rules(128, pairs, Nq, hist).dkv_ring == 0


def test_ring_and_chunk_in_one_launch_only_where_it_gains(rules):
    """Sizes measured both ways, and the calls whose routes or outputs keep them apart."""
    for call in [(128, 12, 4680, 28080), (128, 48, 4680, 28080), (128, 32, 1200, 5400), (64, 8, 4680, 6240), (64, 16, 4680, 18720), (64, 2, 4680, 18720), (64, 4, 4680, 18720),
                 (64, 16, 1200, 4200), (64, 1, 4680, 6240), (64, 16, 1200, 1800), (128, 48, 600, 1200)]:
        assert rules(*call).joined == 1, call
        assert rules(*call, block_rows=call[2] // 3).joined == 0 and rules(*call, in_order=True).joined == 0
        assert rules(*call[:3], 0).joined == 0
    for call in [(128, 5, 4680, 18720), (128, 8, 3120, 14040), (128, 5, 4680, 4680), (64, 4, 4680, 4680), (64, 5, 4680, 9360), (64, 4, 4680, 23400), (64, 6, 4680, 23400), (64, 50, 512, 2560), (64, 60, 260, 2340),
                 (64, 2, 128, 512), (128, 2, 252, 189)]:
        assert rules(*call).joined == 0, call
    # blocks with keys: three empty streams beside a full one do not make it eleven rounds
    assert rules(128, 12, 4680, [28080, 0, 0, 0]).joined == 0
