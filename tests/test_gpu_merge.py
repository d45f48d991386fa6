"""The window merge at the edges of its dispatch: up to 8 parts per row one thread merges them; beyond that 16 threads do up
to 4096 rows (64 blocks of 64 rows) and 4 from there on; with the loss of the call summed by the merge itself (forward) or by
a second launch (merge of slices handed over)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import flce_oracle as O                       # noqa: E402
from paper_2511_17599_amd import binding as B             # noqa: E402
from paper_2511_17599_amd import inputs as I              # noqa: E402
from paper_2511_17599_amd.runner import session_for       # noqa: E402
from conftest import set_plan                             # noqa: E402


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("N,windows", [(1, 8), (257, 9), (300, 64), (77, 70), (2305, 65), (4096, 20), (4097, 20)])
def test_forward_with_many_windows(monkeypatch, N, windows):
    """One and several blocks of rows; the windows of a thread full (64 = 16 x 4), partly filled (65 = 13 x 5, three threads
    without any) and one fewer than there are threads for (9)."""
    set_plan(monkeypatch, FLCE_WINDOWS=windows)
    wl = I.Workload(f"merge_{N}_{windows}", N, 32, 70 * 256 - 3, "bf16", "uniform", ignore_frac=0.2, seed=300 + N)
    x = I.make_inputs(wl)
    x["y"][N // 2] = wl.V + 5                                # one row out of range: dropped and flagged
    print(f"[case] {wl.name}", flush=True)
    s = session_for(wl, x)
    status = torch.full((1,), -1, dtype=torch.int32, device=s.device)
    n_valid = torch.full((1,), -1, dtype=torch.int64, device=s.device)
    f = O.forward(I.to_f64(x["H"]), I.to_f64(x["W"]), x["y"], wl.ignore_index, wl.reduction)

    def check():
        lse = s.lse.double().cpu().numpy()
        # fp32 logits (|z| < 1 here) and a sum of up to 18000 exponentials, pairwise in blocks of 16: about 1e-6 of lse ~ 10
        assert np.abs(lse - f["lse"]).max() <= 2e-6 * np.abs(f["lse"]).max()
        assert abs(float(s.loss.item()) - f["loss"]) <= 1e-5 * max(abs(f["loss"]), 1e-30)

    for _ in range(2):                                       # twice: the arrival count starts over
        s.loss.fill_(float("nan"))
        assert s.forward() == B.FLCE_OK
        st, nv = s.device_status()
        assert st == B.FLCE_ERR_TARGET_RANGE and nv == f["n_valid"]
        check()
    assert B.flce_forward_static(s.H, s.W, s.y, s.N, s.d, s.V, s.ignore_index, s.red, s.dt, s.loss, s.lse, status,
                                 n_valid, s.stream()) == B.FLCE_OK
    assert status.item() == B.FLCE_ERR_TARGET_RANGE and n_valid.item() == f["n_valid"]
    check()


@pytest.mark.parametrize("parts", [1, 8, 9, 33, 64])
@pytest.mark.parametrize("N", [5, 700, 4200])
def test_merge_of_given_partials(parts, N):
    """Triples made here, some of them the identity (nothing seen: m = -inf, a = 0), against a merge in 64 bits."""
    r = np.random.default_rng(parts * 1000 + N)
    m = r.normal(0, 30, (parts, N)).astype(np.float32)
    a = r.uniform(1, 500, (parts, N)).astype(np.float32)
    empty = r.random((parts, N)) < 0.3
    empty[r.integers(0, parts, N), np.arange(N)] = False     # every row has seen something
    m[empty], a[empty] = -np.inf, 0.0
    zt = np.zeros((parts, N), dtype=np.float32)
    zt[r.integers(0, parts, N), np.arange(N)] = r.normal(0, 5, N)
    y = r.integers(0, 1000, N)
    y[::3] = -100
    M = m.max(0).astype(np.float64)
    want = M + np.log((a * np.exp(m.astype(np.float64) - M)).sum(0))
    loss = (want - zt.sum(0))[y != -100].mean()
    d = lambda v: torch.from_numpy(v).cuda()
    out = torch.empty(1, device="cuda"), torch.empty(N, device="cuda")
    nb = B.flce_merge_workspace_bytes(N)
    ws = torch.full((nb,), 0x5A, dtype=torch.uint8, device="cuda")
    dm, da, dz, dy = d(m), d(a), d(zt), d(y)
    assert B.flce_merge_partials(dm, da, dz, parts, dy, N, 1000, -100, B.FLCE_REDUCE_MEAN, out[0], out[1], ws, nb,
                                 torch.cuda.current_stream()) == B.FLCE_OK
    assert B.flce_last_device_status(ws, torch.cuda.current_stream()) == (B.FLCE_OK, int((y != -100).sum()))
    # fp32: one rounding of |lse| <= 150, and 2^x at arguments to a few hundred (2^-24 of the argument, times ln 2)
    assert np.abs(out[1].double().cpu().numpy() - want).max() <= 4e-5
    assert abs(out[0].item() - loss) <= 4e-5
