"""Wide groups: the statistical vote of sixteen lanes per unit, the lists in
two launches and the confirmation of up to 64 replicas by a wave per group, at
the sizes where they can go wrong, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

c3 = pytest.importorskip("paper_2608_11034_amd.c3")
DEV = "cuda"


def _stat(t, kappa=oracle.KAPPA_DEFAULT):
    R = t.shape[1]
    st, bm, mj = c3.consensus(torch.from_numpy(t).to(DEV), c3.STATISTICAL, kappa=kappa)
    ost, obm, omj = oracle.vote_statistical(t, kappa, replica_axis=1)
    assert np.array_equal(st.cpu().numpy(), ost)
    words = (R + 63) // 64
    assert np.array_equal(bm.cpu().numpy().view(np.uint64).reshape(-1, words), obm.reshape(-1, words))
    assert np.array_equal(mj.cpu().numpy(), omj)


# R at the edges of each number of registers a lane; unit counts that leave a
# wave, a workgroup and nothing partly filled
@pytest.mark.parametrize("R", [17, 31, 32, 33, 63, 64, 65, 128, 129, 191, 192, 193, 255, 256])
@pytest.mark.parametrize("U", [1, 3, 16, 37])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_statistical_groups(R, U, dt):
    print("CASE groups", R, U, dt, flush=True)
    rng = np.random.default_rng(R * 100 + U)
    _stat(np.exp(0.02 * rng.standard_normal((U, R))).astype(dt))
    # ties, zeros of both signs, subnormals, missing values up to and past half
    t = rng.integers(-2, 3, size=(U, R)).astype(dt) * dt(np.finfo(dt).smallest_subnormal)
    t[rng.random((U, R)) < 0.1] = -0.0
    for i in range(U):
        bad = rng.permutation(R)[: [0, 1, R // 2 - 1, R // 2, (R + 1) // 2, R][i % 6]]
        t[i, bad] = rng.choice([np.nan, np.inf, -np.inf], size=len(bad))
    _stat(t)


# one value but for a few (MAD 0: quartiles, then range), and kappa that flags
# most; magnitudes whose middle sum is large but finite
@pytest.mark.parametrize("R", [33, 130, 256])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_statistical_fallbacks(R, dt):
    print("CASE fallbacks", R, dt, flush=True)
    rng = np.random.default_rng(R)
    U = 21
    t = np.ones((U, R), dt)
    for i in range(U):
        at = rng.permutation(R)
        t[i, at[: i * R // (2 * U)]] += rng.standard_normal(i * R // (2 * U)).astype(dt)
    _stat(t)
    _stat(t, 0.1)
    _stat((rng.standard_normal((U, R)) * (np.finfo(dt).max / 64)).astype(dt))


# one workgroup up to 4,096 units, two launches up to 1,048,576, three above;
# one and several bitmap words, lists cut short
@pytest.mark.parametrize("R", [3, 66, 130, 256])
@pytest.mark.parametrize("U", [4096, 4097, 5120, 5121, 1048576, 1048577])
def test_localize_sizes(U, R):
    print("CASE localize", U, R, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(U + R)
    W = (R + 63) // 64
    st = torch.zeros(U, dtype=torch.uint8, device=DEV)
    bm = torch.zeros((U, W), dtype=torch.int64, device=DEV)
    pick = torch.rand(U, generator=gen, device=DEV)
    out = pick < 0.02
    bm[out, 0] = 5 if R == 3 else -(1 << 63) | 1
    if W > 1:
        bm[out, W - 1] = 3
    st[out] = 1
    st[pick > 0.99] = 2
    st[0] = 2
    bm[U - 1, 0] = 2
    st[U - 1] = 1
    mj = torch.ones(U, dtype=torch.int32, device=DEV)
    s, b = st.cpu().numpy(), bm.cpu().numpy().view(np.uint64)
    bits = ((b[:, :, None] >> np.arange(64, dtype=np.uint64)) & np.uint64(1)).reshape(U, -1) if U < 10_000 else None
    if bits is None:
        want = [(int(u), 64 * w + k) for u in np.nonzero(b.any(1))[0] for w in range(W)
                for k in range(64) if (int(b[u, w]) >> k) & 1]
    else:
        want = [tuple(x) for x in np.argwhere(bits)]
    und_want = np.nonzero(s == 2)[0]
    counts = [len(want), len(und_want), int(b.any(1).sum())]
    for cap in (len(want), 7):
        outl, und, cnt = c3.localize(st, bm, mj, None, R=R, out_cap=cap, und_cap=cap)
        assert cnt.cpu().tolist() == counts
        o = c3.outliers_numpy(outl, cnt)
        assert [(int(a), int(r)) for a, r in zip(o["chunk"], o["replica"])] == want[:cap]
        n = min(cap, len(und_want))
        assert und.cpu().numpy()[:n].tolist() == und_want[:n].tolist()
    noalloc = c3.localize_noalloc(st, bm, mj, None, R=R, out_cap=7)
    assert noalloc[2].cpu().tolist() == counts


# segments of 64 iterations: one, part of one, several, shared by one, two and
# four waves; ragged groups; every window length class and dense bits
@pytest.mark.parametrize("R", [17, 33, 64])
@pytest.mark.parametrize("T,G", [(1, 3), (63, 8), (64, 9), (65, 16), (128, 5), (129, 64), (260, 17),
                                 (700, 33)])
@pytest.mark.parametrize("W", [1, 2, 16, 63, 64])
def test_confirm_groups(R, T, G, W):
    print("CASE confirm groups", R, T, G, W, flush=True)
    rng = np.random.default_rng(R * 1000 + T + W)
    slow = np.where(rng.random((G, R)) < 0.2, rng.choice([0.4, 0.55, 1.0], size=(G, R)), 0.03)
    pack = lambda b: (b.astype(np.uint64) << np.arange(R, dtype=np.uint64)).sum(-1).astype(np.uint64)
    fp, tm = pack(rng.random((T, G, R)) < 0.01), pack(rng.random((T, G, R)) < slow)
    v = c3.verdicts_numpy(c3.confirm(torch.from_numpy(fp.view(np.int64)).to(DEV),
                                     torch.from_numpy(tm.view(np.int64)).to(DEV), R, W))
    ref = oracle.confirm(fp, tm, R, W)
    for k, rk in (("flags", "flags"), ("first_divergent_iter", "first_div"),
                  ("divergent_count", "div_count"), ("slow_count", "slow_count"),
                  ("max_window_slow", "max_window"), ("first_straggler_window", "first_window")):
        assert np.array_equal(v[k], ref[rk]), k


# rows that are not dense: padded, replica-major, every other unit
@pytest.mark.parametrize("R", [17, 32, 33, 64, 130, 192, 256])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_statistical_strides(R, dt):
    print("CASE strides", R, dt, flush=True)
    rng = np.random.default_rng(R)
    U, es = 37, np.dtype(dt).itemsize
    t = np.exp(0.05 * rng.standard_normal((U, R))).astype(dt)
    t[rng.random((U, R)) < 0.02] = np.nan
    ost, obm, omj = oracle.vote_statistical(t, oracle.KAPPA_DEFAULT, replica_axis=1)

    def check(ev, replica_stride, unit_stride):
        st, bm, mj = c3.consensus(torch.from_numpy(ev).to(DEV), c3.STATISTICAL, R=R, n_units=U,
                                  replica_stride=replica_stride, unit_stride=unit_stride)
        assert np.array_equal(st.cpu().numpy(), ost) and np.array_equal(mj.cpu().numpy(), omj)
        words = (R + 63) // 64
        assert np.array_equal(bm.cpu().numpy().view(np.uint64).reshape(-1, words),
                              obm.reshape(-1, words))
    check(np.ascontiguousarray(t.T), U * es, es)                            # replica-major
    wide = np.full((2 * U, R + 3), np.nan, dt)
    wide[::2, :R] = t
    check(wide, es, 2 * (R + 3) * es)                                       # padded, every other row
    apart = np.full((U, 2 * R), np.inf, dt)
    apart[:, ::2] = t
    check(apart, 2 * es, 2 * R * es)                                        # every other value


# the sum of the middle two values and the differences overflow
@pytest.mark.parametrize("R", [18, 33, 34, 256])
def test_statistical_overflow(R):
    print("CASE overflow", R, flush=True)
    rng = np.random.default_rng(R)
    big = np.finfo(np.float64).max
    rows = [np.full(R, big), np.full(R, -big), np.where(np.arange(R) % 2, big, -big),
            np.where(np.arange(R) < R // 3, 1.0, big), np.where(np.arange(R) < R // 3, 1.0, -big),
            big * rng.random(R), -big * rng.random(R), big * (2 * rng.random(R) - 1),
            big * (0.9 + 0.1 * rng.random(R)), -big * (0.9 + 0.1 * rng.random(R))]
    t = np.stack(rows + [rng.permutation(r) for r in rows])
    for kappa in (oracle.KAPPA_DEFAULT, 0.01, 1e300):
        _stat(t, kappa)


# more groups than one launch has waves for
def test_confirm_past_the_wave_launch():
    print("CASE confirm past the wave launch", flush=True)
    R, G = 17, (1 << 26) + 5
    fp = torch.zeros((1, G), dtype=torch.int64, device=DEV)
    tm = torch.zeros((1, G), dtype=torch.int64, device=DEV)
    fp[0, G - 1], tm[0, 9] = 1 << 16, 1 << 3
    v = c3.confirm(fp, tm, R, 4).view(torch.int32).view(R, G, 6)
    torch.cuda.synchronize()
    assert int(v[16, G - 1, 1]) == 0 and int(v[16, G - 1, 2]) == 1 and int(v[3, 9, 3]) == 1
    assert int(v[:, :, 2].sum()) == 1 and int(v[:, :, 3].sum()) == 1
    del v, fp, tm
    torch.cuda.empty_cache()
