"""Timing consensus of 17 to 64 ranks, whose two votes one launch makes with
sixteen lanes a unit, against the CPU oracle: every number of registers a lane
and both kinds of times, unit counts that leave a wave and a workgroup partly
filled, per-unit results of both kinds, one or none, and fingerprint rows that
leave a majority vote every kind of candidate."""
import ctypes

import numpy as np
import pytest
import torch

from test_gpu_timing import _case, _inputs, _oracle

pytestmark = pytest.mark.gpu

c3 = pytest.importorskip("paper_2608_11034_amd.c3")
DEV = "cuda"


def fingerprint_rows(U, R, rng):
    """[U, R]: one value; one rank apart; a strict majority in the upper ranks
    with all others distinct; the same in two values; halves, in a row and
    mixed; all distinct; three values; bare majorities and half of the ranks,
    scattered; a majority of one of many small classes."""
    rows = np.empty((U, R), np.int64)
    for u in range(U):
        k = u % 11
        row = np.full(R, 7, np.int64)
        if k == 1:
            row[rng.integers(0, R)] = 3
        elif k == 2:
            row[: (R - 1) // 2] = 100 + np.arange((R - 1) // 2)
        elif k == 3:
            row[: (R - 1) // 2] = 100
        elif k == 4:
            row[: R // 2] = 100
        elif k == 5:
            row[rng.permutation(R)[: R // 2]] = 100
        elif k == 6:
            row = 100 + rng.permutation(R)
        elif k == 7:
            row = rng.integers(0, 3, size=R)
        elif k == 8:
            row[rng.permutation(R)[: (R - 1) // 2]] = 100 + rng.integers(0, 2, size=(R - 1) // 2)
        elif k == 9:
            row[rng.permutation(R)[: R - R // 2]] = 100 + rng.integers(0, 9, size=R - R // 2)
        elif k == 10:
            row = rng.integers(0, 5, size=R)
            row[rng.permutation(R)[: R // 2 + 1]] = 9
        rows[u] = row
    # values that differ in one half of the word only
    return np.where(rng.random((U, 1)) < 0.5, rows, rows << 32) * 3 - 5


@pytest.mark.parametrize("kinds", ["both", "fp", "time", "none"])
@pytest.mark.parametrize("R", [17, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("G,T,W", [(1, 1, 16), (5, 21, 4), (13, 43, 70)])
def test_wide_timing(R, f64, G, T, W, kinds):
    _case("timing wide", R, f64, G, T, W, kinds)
    rng = np.random.default_rng(R * 100 + T)
    _, tau = _inputs(R, G, T, seed=R + T, f64=f64)
    fp = fingerprint_rows(T * G, R, rng).reshape(T, G, R)
    fo_ref, to_ref, ver_ref = _oracle(fp, tau, W)
    dfp, dtau = torch.from_numpy(fp).to(DEV), torch.from_numpy(tau).to(DEV)

    def outs():
        return (torch.full((T * G,), 0xEE, dtype=torch.uint8, device=DEV),
                torch.full((T * G,), -5, dtype=torch.int64, device=DEV),
                torch.full((T * G,), -7, dtype=torch.int32, device=DEV))
    fo, to = (outs() if kinds in ("both", k) else None for k in ("fp", "time"))
    ver = torch.empty((R * G, 24), dtype=torch.uint8, device=DEV)
    ws = torch.empty(c3.timing_consensus_workspace_size(R, G, T, W), dtype=torch.uint8, device=DEV)
    p = lambda x: ctypes.c_void_p(x.data_ptr())
    three = lambda o: tuple(p(x) for x in o) if o else (ctypes.c_void_p(0),) * 3
    rc = c3.lib().c3_timing_consensus(p(dfp), p(dtau), c3.EV_F64 if f64 else c3.EV_F32, R, G, T,
                                      c3.KAPPA_DEFAULT, W, *three(fo), *three(to), p(ver), p(ws),
                                      ws.numel(), ctypes.c_void_p(0))
    assert rc == 0
    torch.cuda.synchronize()
    for out, ref in ((fo, fo_ref), (to, to_ref)):
        if out is not None:
            assert np.array_equal(out[0].cpu().numpy(), ref[0])
            assert np.array_equal(out[1].cpu().numpy().view(np.uint64), ref[1])
            assert np.array_equal(out[2].cpu().numpy(), ref[2])
    v = c3.verdicts_numpy(ver)
    for k, rk in (("flags", "flags"), ("first_divergent_iter", "first_div"),
                  ("divergent_count", "div_count"), ("slow_count", "slow_count"),
                  ("max_window_slow", "max_window"), ("first_straggler_window", "first_window")):
        assert np.array_equal(v[k], ver_ref[rk]), k


# more units than sixteen lanes each can be launched for (2^28): a thread per
# unit.  One row read for every unit, and timing rows equal but for a few.
def test_units_past_the_group_launch():
    _case("units past the group launch")
    n, R = (1 << 28) + 3, 17
    row = torch.ones(R, dtype=torch.float64, device=DEV)
    row[5] = 9.0
    st, bm, mj = c3.consensus(row, c3.STATISTICAL, R=R, n_units=n, replica_stride=8, unit_stride=0)
    torch.cuda.synchronize()
    assert int(st.min()) == int(st.max()) == 1 and int(bm.min()) == int(bm.max()) == 1 << 5
    assert int(mj.min()) == int(mj.max()) == 9      # the ninth of the sixteen ones
    del st, bm, mj
    G, T = 16, (1 << 24) + 1
    fp = torch.full((T, G, R), 77, dtype=torch.int64, device=DEV)
    tau = torch.ones((T, G, R), dtype=torch.float32, device=DEV)
    fp[T - 1, 3, 4] = 1
    tau[5:25, 7, 16] = 2.0
    ver, _, _ = c3.timing_consensus(fp, tau, window=16, per_unit=False)
    v = c3.verdicts_numpy(ver).reshape(R, G)
    assert v["first_divergent_iter"][4, 3] == T - 1 and v["divergent_count"].sum() == 1
    assert v["slow_count"][16, 7] == v["slow_count"].sum() == 20
    assert v["first_straggler_window"][16, 7] == 0 and v["max_window_slow"][16, 7] == 16
    del fp, tau, ver
    torch.cuda.empty_cache()
