"""Host-only: both directions of an fp32 call compute logits the same way.

fp32 has two product methods, one per tile edge; the backward's recomputed logit is the forward's, bit for bit, only where both
directions run on the same edge.  (Both bf16 edges add up the same products in the same order.)"""
import random

import pytest

from conftest import tile_edges


@pytest.mark.parametrize("N,d,V", [
    (128 * 159, 64, 128), (128 * 160, 64, 128), (128 * 319, 64, 128), (128 * 320, 64, 128), (1024, 512, 4096), (600, 512, 6200),
    (1170, 96, 2500), (2000, 1024, 2400), (128 * 319 + 1, 8, 100), (1, 8, 128 * 319 + 1)])
def test_one_edge_for_both_directions(N, d, V):
    forward, backward = tile_edges(N, d, V, "f32")
    assert forward == backward


def test_one_edge_for_both_directions_everywhere():
    r = random.Random(3)
    for _ in range(400):
        forward, backward = tile_edges(int(2 ** r.uniform(0, 15)), 8 * r.randint(1, 256), int(2 ** r.uniform(0, 17)), "f32")
        assert forward == backward


def test_address_windows_leave_room_for_the_offsets_bias():
    """289 rows of 2 d bytes, 512 of the tile's columns and 3072 of bias in 2^32: the next hidden size runs on the generic loop."""
    from paper_2511_17599_amd import binding as B
    last = max(d for d in range(7430000, 7432000, 8) if 289 * 2 * d + 512 + 3072 < 2 ** 32)
    for d, loop in ((last, "tuned"), (last + 8, "generic")):
        assert f"loop={loop} " in B.flce_plan_describe(1, d, 1, B.FLCE_DTYPE_BF16)
