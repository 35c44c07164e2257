"""GPU parity of the optimizer-boundary check (Sec. 9): the AdamW replay
kernel bit for bit against the oracle, and the whole check (replay,
signatures, exact vote, localize) against the oracle's check.

All through the C ABI (c3_adamw_slice, c3_signature, c3_consensus,
c3_localize).  Inputs: seeded normal state plus special values (NaN payloads,
infinities, signed zeros, subnormals, negative second moments, overflow).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from oracle import adamw
from parity import compare_all_records

pytestmark = pytest.mark.gpu

c3 = pytest.importorskip("paper_2608_11034_amd.c3")
DEV = "cuda"


def _case(*a):
    print("CASE", *a, flush=True)


def _state(R, numel, seed, specials=True):
    rng = np.random.default_rng(seed)
    sig = (0.02, 1e-3, 1e-4, 1e-6)
    host = []
    for t in range(4):
        x = (rng.standard_normal(numel) * sig[t]).astype(np.float32)
        if t == 3:
            x = np.abs(x)
        if specials and numel >= 64:
            idx = rng.choice(numel, size=max(8, numel // 50), replace=False)
            pool = np.array([np.nan, np.inf, -np.inf, 0.0, -0.0, 1e-40, -1e-42, 3e38, -3e38,
                             1e-20, -1e-3], np.float32)
            x[idx] = rng.choice(pool, size=idx.size)
            nan_idx = idx[np.isnan(x[idx])]
            x.view(np.uint32)[nan_idx] |= rng.integers(0, 1 << 22, nan_idx.size, dtype=np.uint32)
        reps = []
        for r in range(R):
            y = x.copy()
            if r and numel:                        # replicas differ in a few places
                j = rng.integers(0, numel, 3)
                y.view(np.uint32)[j] ^= np.uint32(1) << rng.integers(0, 32, 3).astype(np.uint32)
            reps.append(y)
        host.append(reps)
    dev = [[torch.from_numpy(y).to(DEV) for y in reps] for reps in host]
    return host, dev


HPS = [dict(lr=1e-3, betas=(0.9, 0.999), eps=1e-8, weight_decay=0.1, step=1),
       dict(lr=3e-4, betas=(0.9, 0.95), eps=1e-8, weight_decay=0.1, step=1000),
       dict(lr=1e-2, betas=(0.3, 0.99), eps=1e-6, weight_decay=0.0, step=7),      # w >= 1/2
       dict(lr=5e-4, betas=(0.5, 0.999), eps=1e-8, weight_decay=0.01, step=2)]


def _hp(h):
    return c3.adamw_hparams(h["lr"], h["betas"], h["eps"], h["weight_decay"], h["step"])


def _oracle(host, off, n, h):
    out = []
    for r in range(len(host[0])):
        ins = [x[r][off:off + n] for x in host]
        out.append(adamw.adamw_step(*ins, lr=h["lr"], beta1=h["betas"][0], beta2=h["betas"][1],
                                    eps=h["eps"], weight_decay=h["weight_decay"], step=h["step"]))
    return np.stack([np.stack(o) for o in out])       # [R, 3, n]


@pytest.mark.parametrize("R,numel,off,n", [
    (1, 4096, 0, 4096),                 # 128-bit path, one replica
    (3, 70000, 65536, 4464),            # 128-bit path, tail slice
    (8, 200001, 65536, 65536),          # 128-bit path, full slice
    (8, 200001, 196608, 3393),          # ragged tail: 32-bit path
    (2, 1000, 3, 997),                  # unaligned offset: 32-bit path
    (5, 300, 0, 1),                     # one element
])
@pytest.mark.parametrize("hi", range(len(HPS)))
def test_adamw_slice_bit_exact(R, numel, off, n, hi):
    h = HPS[hi]
    _case("adamw", R, numel, off, n, h)
    host, dev = _state(R, numel, seed=R * 1000 + hi)
    out = c3.adamw_slice(*dev, off, n, _hp(h))
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    ref = _oracle(host, off, n, h)
    bad = got.view(np.uint32) != ref.view(np.uint32)
    assert not bad.any(), (f"{int(bad.sum())} mismatches, first at {np.argwhere(bad)[:3].tolist()}: "
                           f"{got[bad][:3]} vs {ref[bad][:3]}")
    # the replicas' own state is only read
    assert np.array_equal(dev[1][R - 1].cpu().numpy().view(np.uint32), host[1][R - 1].view(np.uint32))


def test_adamw_slice_leaves_state_untouched_and_n0_is_noop():
    _case("adamw untouched")
    host, dev = _state(3, 9000, seed=7)
    out = torch.full((3, 3, 16), 7.0, device=DEV)
    c3.adamw_slice(*dev, 100, 0, _hp(HPS[0]), out=out)
    c3.adamw_slice(*dev, 4, 16, _hp(HPS[0]), out=out)
    torch.cuda.synchronize()
    for t in range(4):
        for r in range(3):
            assert np.array_equal(dev[t][r].cpu().numpy().view(np.uint32), host[t][r].view(np.uint32))
    ref = _oracle(host, 4, 16, HPS[0])
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.view(np.uint32))


def test_adamw_slice_row_stride():
    _case("adamw stride")
    host, dev = _state(4, 5000, seed=9)
    for off, n, stride in ((1000, 1024, 1024), (4000, 1000, 1024), (3, 997, 1001), (4992, 8, 1024)):
        out = torch.full((4, 3, stride), -5.0, device=DEV)
        c3.adamw_slice(*dev, off, n, _hp(HPS[1]), out=out, out_stride=stride)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        ref = _oracle(host, off, n, HPS[1])
        assert np.array_equal(got[:, :, :n].view(np.uint32), ref.view(np.uint32)), (off, n, stride)
        assert (got[:, :, n:] == -5.0).all()                   # padding untouched


def test_adamw_slice_rejects_bad_arguments_on_device():
    _case("adamw errors")
    _, dev = _state(2, 1024, seed=8, specials=False)
    with pytest.raises(c3.C3Error):
        c3.adamw_slice(*dev, 1000, 100, _hp(HPS[0]))
    with pytest.raises(c3.C3Error):
        c3.adamw_slice(*dev, 0, 10, c3.adamw_hparams(step=0))
    with pytest.raises(c3.C3Error):
        c3.adamw_slice(dev[0], dev[1], dev[2], dev[3][:1], 0, 10, _hp(HPS[0]))


def _gpu_check(chk, k, hp):
    rec, st, bm, mj, outl, und, cnt = chk.run(k, hp)
    torch.cuda.synchronize()
    counts = cnt.cpu().numpy()
    o = c3.outliers_numpy(outl, cnt)
    return dict(records=c3.records_numpy(rec), status=st.cpu().numpy(),
                bitmap=bm.cpu().numpy().view(np.uint64), majority=mj.cpu().numpy(),
                unit=o["chunk"], replica=o["replica"], majority_replica=o["majority_replica"],
                undecided=und.cpu().numpy()[:min(int(counts[1]), und.numel())], counts=counts)


def _compare_check(g, ref):
    compare_all_records(g["records"], ref["records"])
    assert np.array_equal(g["status"], ref["status"])
    assert np.array_equal(g["bitmap"], ref["bitmap"])
    agree = ref["status"] != oracle.INCONCLUSIVE
    assert np.array_equal(g["majority"][agree], ref["majority"][agree])
    loc = ref["localize"]
    assert np.array_equal(g["counts"], loc["counts"])
    assert np.array_equal(g["unit"], loc["unit"])
    assert np.array_equal(g["replica"], loc["replica"])
    assert np.array_equal(g["majority_replica"], loc["majority"])
    assert np.array_equal(g["undecided"], loc["undecided"])


@pytest.mark.parametrize("tile", [0, 1024, 16384, 262144])
def test_boundary_check_small_workload_every_slice(tile):
    w = workloads.make(6, device=DEV, scale="small")
    host = [[t.cpu().numpy() for t in x] for x in w.state]
    chk = c3.OptimizerBoundaryCheck(*w.state, slice_elems=w.slice_elems, tile_bytes=tile)
    hp = _hp(w.hparams)
    n_slices = -(-w.numel // w.slice_elems)
    for k in range(n_slices + 1):                      # one wrap-around
        _case("boundary small", tile, k)
        g = _gpu_check(chk, k, hp)
        ref = adamw.boundary_check(host, k, w.hparams, w.slice_elems)
        _compare_check(g, ref)
        upd = chk.updated_slices(k).cpu().numpy()
        for r in range(w.R):
            for j in range(3):
                assert np.array_equal(upd[r, j].view(np.uint32), ref["outputs"][r][j].view(np.uint32))
        if k % n_slices in w.fault_slices:
            assert g["counts"][0] > 0
        else:
            assert g["counts"][0] == 0 and (g["status"] == oracle.AGREE).all()


@pytest.mark.parametrize("R,numel,S", [(2, 2 * 1024 + 13, 1024), (3, 767, 256), (16, 4096, 4096),
                                       (5, 10 * 768 + 1, 768)])
def test_boundary_check_ragged_slices_and_replica_counts(R, numel, S):
    host, dev = _state(R, numel, seed=numel + R)
    h = HPS[R % len(HPS)]
    chk = c3.OptimizerBoundaryCheck(*dev, slice_elems=S)
    n_slices = -(-numel // S)
    for k in list(range(n_slices)) + [n_slices, 7 * n_slices + 1]:
        _case("boundary ragged", R, numel, S, k)
        g = _gpu_check(chk, k, _hp(h))
        _compare_check(g, adamw.boundary_check(host, k, h, S))


def test_boundary_check_full_workload_fault_and_clean_slices():
    """The benchmark's workload (8 replicas x 134M-parameter AdamW state) at
    the slices holding the planted faults and at two clean ones, in the
    benchmark's launch configuration; the oracle sees only those slices."""
    w = workloads.make(6, device=DEV, scale="full")
    chk = c3.OptimizerBoundaryCheck(*w.state, slice_elems=w.slice_elems)
    hp = _hp(w.hparams)
    n_slices = -(-w.numel // w.slice_elems)
    clean = [k for k in (0, n_slices - 1, n_slices // 2) if k not in w.fault_slices][:2]
    for k in sorted(set(w.fault_slices)) + clean:
        _case("boundary full", k)
        g = _gpu_check(chk, k, hp)
        off, n = adamw.slice_bounds(k, w.numel, w.slice_elems)
        host = [[t[off:off + n].cpu().numpy() for t in x] for x in w.state]
        ref = adamw.boundary_check(host, 0, w.hparams, w.slice_elems)
        _compare_check(g, ref)
        planted = {(f.tensor, f.replica) for f, s in zip(w.faults, w.fault_slices) if s == k}
        found_inputs = {(int(u), int(r)) for u, r in zip(g["unit"], g["replica"]) if u < 4}
        assert found_inputs == planted
    del chk, w
    torch.cuda.empty_cache()


# slices of an odd number of blocks, in whole-KiB tiles that do not divide
# them; the last slice ends inside a tile and inside a block
@pytest.mark.parametrize("S", [256 * 33, 256 * 257, 256 * 500, 256 * 2047])
def test_boundary_check_odd_slices(S):
    R, h = 2, HPS[1]
    host, dev = _state(R, S + 3 * S // 4 + 101, seed=S)
    chk = c3.OptimizerBoundaryCheck(*dev, slice_elems=S)
    for k in (0, 1):
        _case("boundary odd", S, k)
        _compare_check(_gpu_check(chk, k, _hp(h)), adamw.boundary_check(host, k, h, S))
