"""Host-only: the forward's vocabulary windows fill whole rounds of 256 workgroups, and the callers that cannot pass a
workspace are accepted at the same sizes as with ceil(256 / row blocks) windows."""
import random

import pytest

from paper_2511_17599_amd import binding as B
from conftest import set_plan


def _windows(N, d, V, dt=B.FLCE_DTYPE_BF16):
    f = dict(kv.split("=") for kv in B.flce_plan_describe(N, d, V, dt).split()[2:])
    return int(f["windows"]), int(f["tiles"].split("/")[0])


@pytest.mark.parametrize("seed", range(4))
def test_no_more_work_in_sequence_than_before(seed):
    r = random.Random(seed)
    for _ in range(200):
        N, V, d = r.randint(1, 60000), r.randint(1, 200000), 32 * r.randint(1, 128)
        win, tile = _windows(N, d, V)
        rb, vt = -(-N // tile), -(-V // tile)
        old = min(max(4, -(-256 // -(-N // 256))), -(-V // 256))   # (of the 256-row plan)
        if tile == 256:                                      # one workgroup per CU
            seq = lambda w: -(-rb * w // 256) * (-(-vt // w) + 8.0 / (0.0242 * d))
        else:                                                # two
            end = 1.5 / (0.28 * -(-d // 32) + 0.9)
            seq = lambda w: (1.3 if rb * w <= 256 else 2 * -(-rb * w // 512)) * (-(-vt // w) + end)
        assert 1 <= win <= vt and seq(win) <= seq(old)
        assert rb * win <= max(8 * 256, rb * old)            # partials: bounded by 8 rounds of items
    # one more than a round is what it avoids: 5 row blocks
    win, tile = _windows(1030, 2048, 20011)
    assert tile == 256 and win * 5 <= 256


def test_static_scratch_takes_the_same_shapes():
    """4 N + 12 * windows * Npad + 4 * ceil(V / 1024) * d bytes and the 256-byte aligned rest, windows = ceil(256 / row
    blocks), against the 16 MiB array: one row on either side of the limit (fake addresses: a call that is accepted
    would launch, so only the refusal is called)."""
    up = lambda x: -(-x // 256) * 256

    def need(N, d, V):
        rb, vt = -(-N // 256), -(-V // 256)
        win = min(max(4, -(-256 // rb)), vt)
        return (256 + up(12 * win * rb * 256) + 3 * up(4 * rb) + up(-(-V // 1024) * d * 4) + up(4 * d) + up(4 * N))
    for d, V in ((4096, 128256), (768, 50257), (256, 600)):
        lo, hi = 1, 1 << 22
        while lo + 1 < hi:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if need(mid, d, V) <= B.FLCE_STATIC_SCRATCH_BYTES else (lo, mid)
        p = 4096
        call = lambda N: B.flce_forward_static(p, p, p, N, d, V, -100, B.FLCE_REDUCE_MEAN, B.FLCE_DTYPE_BF16, p, p)
        assert call(hi) == B.FLCE_ERR_WORKSPACE


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
