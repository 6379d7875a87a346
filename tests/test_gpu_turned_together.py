"""The forward of a few rows whose eight waves turn the chunk's keys together before the walk, against the same call behind
the rotation pre-pass: bit-identical outputs, gradients and staged operands, at the edges of its tiles and of its rule."""
import pytest

import test_gpu_rotating_forward as rotating

pytestmark = pytest.mark.gpu
P64, P128 = (12, 10, 10), (22, 21, 21)


@pytest.mark.parametrize("D,pairs,gh,gw,B,H,group,C,Fc,bf,resident", [
    (64, P64, 1, 31, 1, 2, 1, 8, 1, 0, 8),       # a row short of a tile, ragged ring
    (64, P64, 4, 8, 2, 3, 1, 9, 1, 0, 9),        # one tile
    (64, P64, 3, 11, 1, 2, 2, 8, 1, 0, 8),       # one row past it, candidates
    (64, P64, 15, 17, 1, 2, 1, 2, 1, 0, 2),      # 255 rows
    (64, P64, 16, 16, 1, 2, 1, 3, 1, 0, 0),      # eight tiles, empty ring: every wave starts with its chunk tile
    (64, P64, 16, 16, 1, 3, 1, 3, 1, 0, 1),      # behind one ring tile each
    (64, P64, 8, 16, 1, 2, 2, 4, 2, 1, 1),       # causal blocks: later blocks see more tiles
    (64, P64, 1, 257, 1, 1, 1, 3, 1, 0, 1),      # one row too many
    (128, P128, 7, 9, 1, 2, 1, 9, 1, 0, 9),      # 63 rows
    (128, P128, 8, 8, 2, 2, 3, 8, 1, 0, 8),      # the most at D = 128
    (128, P128, 5, 13, 1, 1, 1, 9, 1, 0, 9),     # one row too many
    (128, (64, 0, 0), 2, 4, 1, 2, 1, 70, 8, 3, 64),  # 512 (cos, sin), causal blocks of three frames
    (128, (64, 0, 0), 1, 7, 1, 2, 1, 80, 9, 0, 72),  # 576: each wave its own
])
def test_the_same_bits_as_behind_the_pre_pass(D, pairs, gh, gw, B, H, group, C, Fc, bf, resident):
    rotating.test_the_same_bits_as_behind_the_pre_pass(D, pairs, gh, gw, B, H, group, C, Fc, bf, resident)
