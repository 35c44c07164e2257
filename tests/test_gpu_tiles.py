"""The signature's tiles: chunk sizes that are no power of two, element types
side by side in one launch, and the two kernels that fold a tile (a workgroup,
or one wave for small tiles in large numbers), against the CPU oracle and
against each other bit for bit."""
import math
from fractions import Fraction

import numpy as np
import pytest
import torch

import oracle
import workloads
from parity import compare_all_records

pytestmark = pytest.mark.gpu

c3 = pytest.importorskip("paper_2608_11034_amd.c3")
DEV = "cuda"
KIB = 1024
CODE = {torch.float32: workloads.F32, torch.bfloat16: workloads.BF16, torch.float16: workloads.F16,
        torch.uint8: workloads.RAW}


def _tensor(dtype, n, gen, special=True):
    if dtype == torch.uint8:
        return torch.randint(0, 256, (n,), generator=gen, device=DEV, dtype=dtype)
    t = torch.randn(n, generator=gen, device=DEV).to(dtype)
    if special and n > 40:
        t[n // 3] = float("nan")
        t[n // 2] = float("inf")
        t[-1] = float("nan")             # in the partial last segment, where there is one
    return t


def _sign(reps, chunk, tile=0, grid_blocks=0):
    plan = c3.SignaturePlan(reps, chunk, tile)
    rec = plan.new_records()
    plan.run(rec, plan.new_workspace(), grid_blocks=grid_blocks)
    torch.cuda.synchronize()
    return rec


def _oracle(reps, chunk):
    metas = [(CODE[t.dtype], tuple(t.shape)) for t in reps[0]]
    return oracle.signature([[workloads.host_bytes(t) for t in rep] for rep in reps], metas, chunk)


# tile sizes by default: the chunk itself up to 256 KiB, then 2 x 160, 2 x 250
# and 4 x 250 KiB, and 3 x 257 KiB of which the last is 1 KiB shorter than the
# others (770 KiB); tensors end inside, at and just past tiles and chunks
@pytest.mark.parametrize("chunk_kib", [5, 33, 100, 160, 255, 257, 320, 500, 770, 1000])
def test_chunk_sizes_mixed_types(chunk_kib):
    chunk = chunk_kib * KIB
    print("CASE chunk", chunk_kib, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(chunk_kib)
    base = []
    for dtype in (torch.bfloat16, torch.float32, torch.uint8, torch.float16, torch.bfloat16):
        es = torch.empty(0, dtype=dtype).element_size()
        for nbytes in (0, es, chunk // 2, chunk - es, chunk, chunk + es, 2 * chunk + 161 * KIB + 7 * es):
            base.append(_tensor(dtype, nbytes // es, gen))
    reps = [[t.clone() for t in base] for _ in range(2)]
    reps[1][6].view(torch.uint8)[-1] ^= 1
    rec = c3.records_numpy(_sign(reps, chunk))
    compare_all_records(rec, _oracle(reps, chunk))
    assert (rec["sig"][0] != rec["sig"][1]).sum() == 1


# launches on both sides of the rule's tile counts; one replica alone (a
# workgroup per tile) against the same replica among others (a wave per tile):
# the records must be the same bits, sums included
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16, torch.uint8])
@pytest.mark.parametrize("chunk_kib,tiles,R", [(16, 257, 4), (33, 160, 13), (48, 130, 16), (64, 129, 64)])
def test_wave_tiles_same_bits(dtype, chunk_kib, tiles, R):
    chunk = chunk_kib * KIB
    print("CASE wave tiles", dtype, chunk_kib, tiles, R, flush=True)
    es = torch.empty(0, dtype=dtype).element_size()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(chunk_kib)
    # two tensors, the first ending 3 elements into a 16-byte segment
    half = (tiles // 2 - 1) * chunk // es
    base = [_tensor(dtype, half + 515 * 16 // es + 3, gen), _tensor(dtype, half, gen, special=False)]
    reps = [base] + [[t.clone() for t in base] for _ in range(R - 1)]
    together = _sign(reps, chunk)
    alone = _sign([reps[R - 1]], chunk)
    assert torch.equal(together, alone.expand(R, *alone.shape[1:]))
    compare_all_records(c3.records_numpy(alone), _oracle([base], chunk))


# runs of one to sixteen consecutive tiles per wave, crossing tensors, types
# and replicas, in as many workgroups as wanted and in three
@pytest.mark.parametrize("tiles", [1500, 20_000, 140_000])
def test_wave_runs(tiles):
    print("CASE wave runs", tiles, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(tiles)
    n = tiles // 2 // 3 * KIB
    base = [_tensor(torch.uint8, n + 1, gen), _tensor(torch.bfloat16, n // 2 + 1, gen),
            _tensor(torch.float32, n // 4 - 1, gen)]
    reps = [base, [t.clone() for t in base]]
    rec = _sign(reps, KIB)
    compare_all_records(c3.records_numpy(rec[:1]), _oracle([base], KIB))
    assert torch.equal(rec[0], rec[1])
    assert torch.equal(rec, _sign(reps, KIB, grid_blocks=3))
    # the same chunks in smaller tiles go through partials
    wide = _sign(reps, 4 * KIB, tile=KIB)
    compare_all_records(c3.records_numpy(wide[:1]), _oracle([base], 4 * KIB))


# partials of 2 to 33 tiles a chunk: combined by one thread (up to four tiles)
# or by sixteen lanes, in the finalize kernel, the one-workgroup tail (up to
# 256 records of them, beyond that finalized first) and the check's tail
@pytest.mark.parametrize("tiles", [2, 4, 5, 16, 17, 33])
@pytest.mark.parametrize("R,chunks", [(2, 3), (5, 60), (3, 90), (8, 300), (33, 8), (40, 30)])
def test_partials_combined_alike(tiles, R, chunks):
    print("CASE partials", tiles, R, chunks, flush=True)
    chunk = tiles * KIB
    gen = torch.Generator(device=DEV)
    gen.manual_seed(tiles * 100 + chunks)
    n = chunks // 2 * chunk // 4
    base = [_tensor(torch.float32, n + 77, gen), _tensor(torch.float32, n - 300, gen, special=False)]
    reps = [base] + [[t.clone() for t in base] for _ in range(R - 1)]
    reps[R - 1][0].view(torch.uint8)[chunk + 5] ^= 4
    plan = c3.SignaturePlan(reps, chunk, KIB)
    outs = plan.new_check_outputs()
    ws = torch.empty(plan.check_workspace_size(), dtype=torch.uint8, device=DEV)
    plan.run_check(outs, ws)
    rec, st, bm, mj, outl, und, cnt = outs
    apart = _sign(reps, chunk, tile=KIB)
    st2, bm2, mj2 = c3.consensus(apart, c3.EXACT)
    outl2, und2, cnt2 = c3.localize(st2, bm2, mj2, apart)
    torch.cuda.synchronize()
    assert torch.equal(rec, apart)
    assert torch.equal(st, st2) and torch.equal(bm, bm2) and torch.equal(mj, mj2)
    assert torch.equal(cnt, cnt2)
    assert np.array_equal(c3.outliers_numpy(outl, cnt), c3.outliers_numpy(outl2, cnt2))
    if R <= 8:
        compare_all_records(c3.records_numpy(rec), _oracle(reps, chunk))


# the plan as a kernel argument (up to 3.5 KB of it, and 8,192 tiles under 256
# KiB) and staged in the workspace; a second call that says its plan is still
# there reads the tensors as they are then
@pytest.mark.parametrize("R,T,n", [(2, 1, 5000), (2, 9, 900), (2, 10, 900), (2, 11, 900), (2, 12, 900),
                                   (32, 5, 300), (64, 3, 300), (64, 4, 300), (2, 2, 1024 * 1024 // 4 * 2),
                                   (2, 2, 1024 * 1024 // 4 * 2 + 1), (3, 70, 500), (2, 130, 3000)])
def test_plan_argument_and_staged(R, T, n):
    print("CASE plan", R, T, n, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(R * 100 + T)
    types = (torch.float32, torch.bfloat16, torch.uint8) if n < 10_000 else (torch.float32,)
    base = [_tensor(types[i % len(types)], n + i, gen) for i in range(T)]
    reps = [base] + [[t.clone() for t in base] for _ in range(R - 1)]
    for chunk, tile in ((KIB, 0), (3 * KIB, KIB), (KIB * 1024, 0)):
        plan = c3.SignaturePlan(reps, chunk, tile)
        outs = plan.new_check_outputs()
        ws = torch.empty(plan.check_workspace_size(), dtype=torch.uint8, device=DEV)
        plan.run_check(outs, ws)
        first = outs[0].clone()
        compare_all_records(c3.records_numpy(outs[0][:2]), _oracle(reps[:2], chunk))
        assert outs[6].cpu().tolist() == [0, 0, 0]
        reps[R - 1][T - 1].view(torch.uint8)[7] ^= 1
        plan.run_check(outs, ws, plan_staged=True)
        assert outs[6].cpu().tolist() == ([1, 0, 1] if R > 2 else [0, 1, 0])
        reps[R - 1][T - 1].view(torch.uint8)[7] ^= 1
        sig_ws = plan.new_workspace()
        rec = plan.new_records()
        plan.run(rec, sig_ws)
        plan.run(rec, sig_ws, plan_staged=True)
        torch.cuda.synchronize()
        assert torch.equal(rec, first)


# 256 KiB tiles up to and past the numbers that still take the plan as an
# argument, of one tensor and of two: on 64 replicas and alone
@pytest.mark.parametrize("T,tiles", [(1, 512), (1, 513), (2, 96), (2, 97)])
def test_plan_argument_large_tiles(T, tiles):
    print("CASE plan, large tiles", T, tiles, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(tiles)
    rep = [torch.randn(tiles * 65536 - 5 - t, generator=gen, device=DEV) for t in range(T)]
    alone = _sign([rep], 1024 * KIB)
    assert torch.equal(_sign([rep] * 64, 1024 * KIB), alone.expand(64, *alone.shape[1:]))
    compare_all_records(c3.records_numpy(alone), _oracle([rep], 1024 * KIB))


# sums of squares of fp32 chunks that are no power of two, whose tiles are
# folded on the way, against the exact sums: the exact result rounded once is
# off by 4e-17 to 6e-17 (2-norm, relative), and the chains between two folds may
# add as much again
@pytest.mark.parametrize("chunk_kib", [48, 96, 100, 160, 500, 1000])
def test_squares_of_fp32(chunk_kib):
    print("CASE squares", chunk_kib, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(chunk_kib)
    chunks = 48
    x = torch.randn(chunks * chunk_kib * KIB // 4, generator=gen, device=DEV)
    rec = c3.records_numpy(_sign([[x]], chunk_kib * KIB))[0]
    rows = x.cpu().numpy().astype(np.float64).reshape(chunks, -1)
    err = [float((Fraction(float(q)) - e) / e)
           for q, e in zip(rec["sumsq"], (Fraction(math.fsum((r * r).tolist())) for r in rows))]
    assert math.sqrt(np.mean(np.square(err))) < 1.2e-16


# the same for the optimizer check's slices of an odd number of KiB: seven
# records of four replicas
def test_squares_of_optimizer_slices():
    print("CASE squares of slices", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    S = 2047 * 256
    state = [[torch.randn(S, generator=gen, device=DEV) * s for _ in range(4)]
             for s in (0.02, 1e-3, 1e-4, 1e-6)]
    state[3] = [v.abs_() for v in state[3]]
    chk = c3.OptimizerBoundaryCheck(*state, slice_elems=S)
    rec = c3.records_numpy(chk.run(0, c3.adamw_hparams(3e-4, (0.9, 0.95), 1e-8, 0.1, 1000))[0])
    err = []
    for r in range(4):
        for u, t in enumerate([x[r] for x in state] + list(chk.updated[r])):
            d = t.double().cpu().numpy()
            e = Fraction(math.fsum((d * d).tolist()))
            err.append(float((Fraction(float(rec["sumsq"][r, u])) - e) / e))
    assert math.sqrt(np.mean(np.square(err))) < 1.2e-16


# the optimizer check's records are those of the signature over its seven
# slices with the same tile, sums included: a slice that ends inside a block, a
# NaN
@pytest.mark.parametrize("tile_kib", [1, 16, 32, 64, 256])
@pytest.mark.parametrize("n", [65536, 65536 - 4097])
def test_optimizer_records_are_signatures(tile_kib, n):
    print("CASE optimizer tile", tile_kib, n, flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    state = [[torch.randn(65536 + n, generator=gen, device=DEV) * s for _ in range(2)]
             for s in (0.02, 1e-3, 1e-4, 1e-6)]
    state[3] = [v.abs_() for v in state[3]]
    state[1][1][65536 + 5000] = float("nan")
    chk = c3.OptimizerBoundaryCheck(*state, slice_elems=65536, tile_bytes=tile_kib * KIB)
    rec = chk.run(1, c3.adamw_hparams(3e-4, (0.9, 0.95), 1e-8, 0.1, 1000))[0]
    slices = [[t[r][65536:] for t in state] + [chk.updated[r, j, :n].clone() for j in range(3)]
              for r in range(2)]
    torch.cuda.synchronize()
    assert torch.equal(rec.view(-1, 64), _sign(slices, 262144, tile_kib * KIB).view(-1, 64))


# the tile that a plan object names at the call is the one that is taken
def test_plan_tile_set_later():
    print("CASE tile set later", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    x = torch.randn(5000, generator=gen, device=DEV)
    plan = c3.SignaturePlan([[x], [x]], 4 * KIB, KIB)
    rec, ws = plan.new_records(), plan.new_workspace()
    plan.tile_bytes = 2 * KIB
    plan.run(rec, ws)
    assert torch.equal(rec, _sign([[x], [x]], 4 * KIB, 2 * KIB))
    outs = plan.new_check_outputs()
    check_ws = torch.empty(plan.check_workspace_size(), dtype=torch.uint8, device=DEV)
    plan.tile_bytes = 3000
    with pytest.raises(c3.C3Error):
        plan.run(rec, ws)
    with pytest.raises(c3.C3Error):
        plan.run_check(outs, check_ws)
