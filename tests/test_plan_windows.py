"""Host-only: the forward's vocabulary windows fill whole rounds of workgroups, the callers that cannot pass a workspace are
accepted at the same sizes as with ceil(256 / row blocks) windows, and the plan's tiles are those of the loop that runs."""
import random

import pytest

from paper_2511_17599_amd import binding as B
from conftest import set_plan


def _windows(N, d, V, dt=B.FLCE_DTYPE_BF16):
    f = dict(kv.split("=") for kv in B.flce_plan_describe(N, d, V, dt).split()[2:])
    return int(f["windows"]), int(f["tiles"].split("/")[0])


@pytest.mark.parametrize("seed", range(4))
def test_windows_leave_little_of_a_round_unused(seed):
    """The tiles a workgroup's place on the chip walks one after the other (launches of one round of row block x window items,
    each as long as its longest window), counted for every number of windows there could be: the plan's is within 6 % or two
    tiles of the least (20 % at hidden sizes under 512, where what an item costs beyond its tiles weighs as much as a
    tile).  Partials: at most 8 rounds of items, or as many windows as cover the CUs with 256-row blocks."""
    r = random.Random(seed)
    for _ in range(200):
        N, V, d = r.randint(1, 60000), r.randint(1, 200000), 32 * r.randint(1, 128)
        win, tile = _windows(N, d, V)
        rb, vt = -(-N // tile), -(-V // tile)
        places = 256 if tile == 256 else 512                 # one workgroup per CU, or two
        cover = min(max(4, -(-256 // -(-N // 256))), -(-V // 256))
        assert 1 <= win <= vt and rb * win <= max(8 * 256, rb * cover)

        def in_sequence(w):
            return -(-rb * w // places) * -(-vt // w)
        least = min(in_sequence(w) for w in range(min(4, vt), max(cover, min(vt, 8 * 256 // rb)) + 1))
        assert in_sequence(win) <= max((1.06 if d >= 512 else 1.2) * least, least + 2), (N, d, V)


def test_one_window_more_than_a_round_holds_is_avoided():
    for N, d, V, before in ((1030, 2048, 20011, 52), (3300, 2048, 65536, 20)):
        win, tile = _windows(N, d, V)
        rb = -(-N // 256)
        assert tile == 256 and before * rb > 256 >= win * rb


@pytest.mark.parametrize("d,V", [(4096, 128256), (768, 50257), (256, 600)])
def test_static_scratch_takes_the_same_shapes(d, V):
    """4 N + 12 * windows * Npad + 4 * ceil(V / 1024) * d bytes and the 256-byte aligned rest, windows = ceil(256 / row
    blocks), against the 16 MiB array: the last row count that fits is taken, the next one refused.  The address of H is
    misaligned, which is looked at after the size and before anything is launched, so a size that is taken shows as another
    error than a size that is not."""
    up = lambda x: -(-x // 256) * 256

    def need(N):
        rb, vt = -(-N // 256), -(-V // 256)
        win = min(max(4, -(-256 // rb)), vt)
        return (256 + up(12 * win * rb * 256) + 3 * up(4 * rb) + up(-(-V // 1024) * d * 4) + up(4 * d) + up(4 * N))

    def call(N):
        p = 4096
        return B.flce_forward_static(p + 8, p, p, N, d, V, -100, B.FLCE_REDUCE_MEAN, B.FLCE_DTYPE_BF16, p, p)
    lo, hi = 1, 1 << 22
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if need(mid) <= B.FLCE_STATIC_SCRATCH_BYTES else (lo, mid)
    assert call(hi) == B.FLCE_ERR_WORKSPACE
    for N in (1, lo // 3, lo - 1, lo):
        assert call(N) in (B.FLCE_ERR_BAD_ARG, B.FLCE_ERR_HIP)     # (the latter where there is no GPU to ask for the array)


@pytest.mark.parametrize("knobs,N,d,V", [({"FLCE_VC_TILES": 4096}, 100, 4096, 1050000), ({"FLCE_GENERIC": 1}, 300, 256, 5000),
                                         ({}, 300, 131072, 50000)])
def test_the_generic_loop_is_planned_with_its_own_tiles(monkeypatch, knobs, N, d, V):
    """bf16 out of the tuned loop's reach (a vocabulary chunk beyond 4 GiB, a long row, the knob): 256-row tiles, and no more
    windows than there are of those."""
    set_plan(monkeypatch, **knobs)
    assert "loop=generic" in B.flce_plan_describe(N, d, V, B.FLCE_DTYPE_BF16)
    win, tile = _windows(N, d, V)
    assert tile == 256 and win <= -(-V // 256)


@pytest.mark.parametrize("tile", [128, 256])
def test_the_tile_edge_can_be_asked_for(monkeypatch, tile):
    """Both directions of a tuned bf16 call, whatever the rule would take; the generic and the fp32 loop have their own."""
    set_plan(monkeypatch, FLCE_TILE=tile)
    for N, d, V in ((300, 200, 2100), (8192, 4096, 128256), (2048, 1024, 32000)):
        assert f" tiles={tile}/{tile} " in B.flce_plan_describe(N, d, V, B.FLCE_DTYPE_BF16)
        assert f" tiles={tile}/" not in B.flce_plan_describe(N, d, V, B.FLCE_DTYPE_F32) or tile == 128
    set_plan(monkeypatch, FLCE_GENERIC=1)
    assert " tiles=256/256 " in B.flce_plan_describe(300, 200, 2100, B.FLCE_DTYPE_BF16)
