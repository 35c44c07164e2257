"""The C ABI library loads and exports every symbol include/c3.h declares.

Host-side checks only: symbol presence, the chunk plan and workspace sizes,
status strings and argument validation that returns before any GPU work.
"""
import ctypes
import os
import re

import numpy as np
import pytest

import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "c3.h")

c3 = pytest.importorskip("paper_2608_11034_amd.c3")


def _declared_functions():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    names = re.findall(r"^\s*(?:const\s+)?[A-Za-z_][\w\s\*]*?\b(c3_\w+)\s*\(", src, flags=re.M)
    return sorted(set(names))


def test_header_declares_the_boundary():
    names = _declared_functions()
    for n in ("c3_signature", "c3_signature_ex", "c3_consensus", "c3_localize", "c3_confirm",
              "c3_tensor_signature", "c3_num_chunks", "c3_signature_workspace_size",
              "c3_localize_workspace_size", "c3_confirm_workspace_size", "c3_status_string",
              "c3_abi_version", "c3_adamw_slice", "c3_optimizer_check",
              "c3_optimizer_check_workspace_size"):
        assert n in names, n


def test_library_exports_every_declared_symbol():
    L = c3.lib()
    for n in _declared_functions():
        assert hasattr(L, n), f"{n} declared in include/c3.h but not exported"
    assert L.c3_abi_version() == 1


def test_struct_sizes_match_the_header():
    assert ctypes.sizeof(c3.TensorMeta) == 72
    assert ctypes.sizeof(c3.LaunchOpts) == 32
    assert ctypes.sizeof(c3.AdamwHparams) == 48
    assert ctypes.sizeof(c3.OptimizerState) == 64
    assert ctypes.sizeof(c3.OptimizerCheckOut) == 64
    assert c3.RECORD_DTYPE.itemsize == 64
    assert c3.OUTLIER_DTYPE.itemsize == 80
    assert c3.VERDICT_DTYPE.itemsize == 24


def _metas(shapes_dtypes):
    metas = (c3.TensorMeta * len(shapes_dtypes))()
    for i, (d, shape) in enumerate(shapes_dtypes):
        metas[i].dtype = d
        metas[i].ndim = len(shape)
        for j, n in enumerate(shape):
            metas[i].shape[j] = n
    return metas


@pytest.mark.parametrize("chunk_bytes", [1024, 3072, 1 << 20])
def test_chunk_plan_matches_oracle(chunk_bytes):
    md = [(c3.F32, (1000,)), (c3.BF16, (0,)), (c3.F16, (3, 5, 7)), (c3.RAW, (4097,)), (c3.BF16, ()),
          (c3.F32, (2048, 1024))]
    L = c3.lib()
    got = L.c3_num_chunks(_metas(md), len(md), chunk_bytes)
    assert got == oracle.num_chunks(md, chunk_bytes)


def test_plan_rejects_bad_arguments():
    L = c3.lib()
    md = _metas([(c3.F32, (1000,))])
    assert L.c3_num_chunks(md, 1, 1000) == -1           # not a multiple of 1024
    assert L.c3_num_chunks(md, 0, 1024) == -1           # no tensors
    assert L.c3_num_chunks(_metas([(7, (10,))]), 1, 1024) == -1     # unknown dtype
    assert L.c3_num_chunks(_metas([(c3.F32, (-1,))]), 1, 1024) == -1
    assert L.c3_signature_workspace_size(md, 1, 0, 1024) == 0        # R = 0
    assert L.c3_signature_workspace_size(md, 1, 1, 1024) > 0         # one replica
    assert L.c3_signature_workspace_size(md, 1, 65, 1024) > 0        # wide peer groups
    assert L.c3_signature_workspace_size(md, 1, 256, 1024) > 0
    assert L.c3_signature_workspace_size(md, 1, 257, 1024) == 0      # R > C3_MAX_PEERS
    assert L.c3_signature_workspace_size(md, 1, 8, 1024) > 0
    assert L.c3_signature_workspace_size_ex(md, 1, 8, 4096, 3072) == 0   # tile not a power of 2
    assert L.c3_signature_workspace_size_ex(md, 1, 8, 4096, 8192) == 0   # tile larger than chunk


def test_argument_errors_return_before_gpu_work():
    L = c3.lib()
    md = _metas([(c3.F32, (1000,))])
    ptrs = (ctypes.c_void_p * 2)(16, 32)
    null = ctypes.c_void_p(0)
    rec = ctypes.c_void_p(64)
    ws = ctypes.c_void_p(256)
    assert L.c3_signature(ptrs, md, 1, 0, 1024, rec, ws, 1 << 20, null) == -1     # R = 0
    assert L.c3_signature(ptrs, md, 1, 257, 1024, rec, ws, 1 << 20, null) == -1   # R > 256
    assert L.c3_signature(ptrs, md, 1, 2, 1000, rec, ws, 1 << 20, null) == -1     # chunk
    assert L.c3_signature(ptrs, md, 1, 2, 1024, rec, null, 1 << 20, null) == -4   # workspace
    assert L.c3_signature(ptrs, md, 1, 2, 1024, rec, ws, 8, null) == -4           # too small
    bad = (ctypes.c_void_p * 2)(16, 40)
    assert L.c3_signature(bad, md, 1, 2, 1024, rec, ws, 1 << 20, null) == -2      # alignment
    assert L.c3_consensus(ctypes.c_void_p(8), c3.EV_U64, 8, 64, 0, 10, c3.EXACT, 1.0,
                          ctypes.c_void_p(8), ctypes.c_void_p(8), ctypes.c_void_p(8), null) == -1
    assert L.c3_consensus(ctypes.c_void_p(8), c3.EV_U64, 8, 64, 4, 10, c3.STATISTICAL, 1.0,
                          ctypes.c_void_p(8), ctypes.c_void_p(8), ctypes.c_void_p(8), null) == -1
    assert L.c3_consensus(ctypes.c_void_p(8), c3.EV_F64, 8, 64, 4, 10, c3.STATISTICAL, -1.0,
                          ctypes.c_void_p(8), ctypes.c_void_p(8), ctypes.c_void_p(8), null) == -1
    assert L.c3_consensus(ctypes.c_void_p(4), c3.EV_U64, 8, 64, 4, 10, c3.EXACT, 1.0,
                          ctypes.c_void_p(8), ctypes.c_void_p(8), ctypes.c_void_p(8), null) == -2
    assert L.c3_consensus(ctypes.c_void_p(8), c3.EV_U64, 8, 64, 4, 0, c3.EXACT, 1.0,
                          null, null, null, null) == 0                          # nothing to do
    assert L.c3_localize(null, null, null, null, 4, 10, null, 0, null, 0, ctypes.c_void_p(8),
                         ctypes.c_void_p(256), 4096, null) == -1
    assert L.c3_consensus(ctypes.c_void_p(8), c3.EV_U64, 8, 64, 257, 10, c3.EXACT, 1.0,
                          ctypes.c_void_p(8), ctypes.c_void_p(8), ctypes.c_void_p(8), null) == -1
    assert L.c3_consensus(ctypes.c_void_p(8), c3.EV_U64, 8, 64, 256, 0, c3.EXACT, 1.0,
                          null, null, null, null) == 0                          # R = 256 valid
    assert L.c3_localize(null, null, null, null, 257, 0, null, 0, null, 0, ctypes.c_void_p(8),
                         ctypes.c_void_p(256), 4096, null) == -1                # R > 256
    assert L.c3_tensor_signature(null, 257, 0, 1, ctypes.c_void_p(8), null) == -1
    assert L.c3_confirm(null, null, 8, 4, 16, 0, ctypes.c_void_p(8), ctypes.c_void_p(256), 4096,
                        null) == -1                                              # window 0
    assert L.c3_tensor_signature(null, 8, 10, 0, ctypes.c_void_p(8), null) == -1
    for code in (0, -1, -2, -3, -4, -5, -99):
        assert isinstance(L.c3_status_string(code), bytes)


def test_singleton_group_is_rejected_before_gpu_work():
    """Sec. 4: one peer provides no comparison.  Every vote, localization
    and confirmation entry point returns C3_E_INVAL for R = 1 (checked before
    any HIP call), while signing one replica stays valid (records are per
    replica; the tests of the emulated sharded protocol sign R = 1)."""
    L = c3.lib()
    null = ctypes.c_void_p(0)
    p8 = ctypes.c_void_p(8)
    for kind, mode in ((c3.EV_U64, c3.EXACT), (c3.EV_F32, c3.STATISTICAL)):
        assert L.c3_consensus(p8, kind, 8, 8, 1, 10, mode, 1.0, p8, p8, p8, null) == -1
        assert L.c3_consensus(p8, kind, 8, 8, 1, 0, mode, 1.0, null, null, null, null) == -1
    assert L.c3_localize(p8, p8, p8, null, 1, 10, p8, 10, p8, 10, p8, ctypes.c_void_p(256),
                         1 << 20, null) == -1
    assert L.c3_confirm(p8, p8, 1, 4, 16, 16, p8, ctypes.c_void_p(256), 1 << 20, null) == -1
    assert L.c3_confirm_workspace_size(1, 4, 16) == 0
    assert L.c3_timing_consensus_workspace_size(1, 4, 16, 16) == 0
    assert L.c3_timing_consensus(p8, p8, c3.EV_F32, 1, 4, 16, 1.0, 16, null, null, null, null,
                                 null, null, p8, ctypes.c_void_p(256), 1 << 20, null) == -1
    md = _metas([(c3.F32, (1000,))])
    assert L.c3_signature_workspace_size(md, 1, 1, 1024) > 0


def test_localize_noalloc_argument_errors_return_before_gpu_work():
    L = c3.lib()
    null = ctypes.c_void_p(0)
    p8 = ctypes.c_void_p(8)
    big = c3.LOCALIZE_NOALLOC_MAX_UNITS + 1
    assert L.c3_localize_noalloc(p8, p8, p8, null, 8, big, p8, 10, p8, 10, p8, null) == -1
    assert L.c3_localize_noalloc(p8, p8, p8, null, 1, 10, p8, 10, p8, 10, p8, null) == -1
    assert L.c3_localize_noalloc(p8, p8, p8, null, 257, 10, p8, 10, p8, 10, p8, null) == -1
    assert L.c3_localize_noalloc(p8, p8, p8, null, 8, 10, p8, 10, p8, 10, null, null) == -1
    assert L.c3_localize_noalloc(p8, ctypes.c_void_p(4), p8, null, 8, 10, p8, 10, p8, 10, p8,
                                 null) == -2


def test_read_probe_argument_errors_return_before_gpu_work():
    L = c3.lib()
    null = ctypes.c_void_p(0)
    p16 = ctypes.c_void_p(256)
    assert L.c3_read_probe(p16, 4096, 3000, p16, null, null, null) == -1      # tile not 2^k
    assert L.c3_read_probe(p16, 4080, 1024, p16, null, null, null) == -1      # bytes % 1024
    assert L.c3_read_probe(p16, 4096, 512, p16, null, null, null) == -1       # tile < 1 KiB
    assert L.c3_read_probe(p16, 4096, 1 << 25, p16, null, null, null) == -1   # tile > 16 MiB
    assert L.c3_read_probe(ctypes.c_void_p(8), 4096, 0, p16, null, null, null) == -2
    assert L.c3_read_probe(null, 0, 0, null, null, null, null) == 0           # nothing to read
    assert L.c3_read_probe(null, 4096, 0, p16, null, null, null) == -1


def test_check_argument_errors_return_before_gpu_work():
    L = c3.lib()
    md = _metas([(c3.F32, (1000,))])
    ptrs = (ctypes.c_void_p * 4)(16, 32, 48, 64)
    null = ctypes.c_void_p(0)
    p8, ws = ctypes.c_void_p(64), ctypes.c_void_p(256)
    need = L.c3_check_workspace_size(md, 1, 2, 1024, 0)
    assert need > L.c3_signature_workspace_size(md, 1, 2, 1024)
    assert L.c3_check_workspace_size(md, 1, 1, 1024, 0) == 0              # a group of one
    args = lambda R, wsb, bm=p8: (ptrs, md, 1, R, 1024, p8, p8, bm, p8, p8, 10, p8, 10, p8, ws,
                                  wsb, null, null)
    assert L.c3_check(*args(1, need)) == -1                               # R = 1
    assert L.c3_check(*args(2, need - 256)) == -4                         # workspace too small
    assert L.c3_check(*args(2, need, ctypes.c_void_p(68))) == -2          # misaligned bitmap
    assert L.c3_check(*args(257, need)) == -1                             # R > 256


def test_binding_has_no_cpu_fallback():
    import torch
    x = torch.zeros(1024)
    with pytest.raises(c3.C3Error):
        c3.signature([[x], [x]], 1024)


def test_adamw_slice_argument_errors_return_before_gpu_work():
    L = c3.lib()
    ptrs = (ctypes.c_void_p * 2)(256, 512)
    out = ctypes.c_void_p(1024)
    null = ctypes.c_void_p(0)
    hp = c3.adamw_hparams(lr=1e-3, betas=(0.9, 0.999), eps=1e-8, weight_decay=0.1, step=1)

    def call(R=2, numel=1000, off=0, n=100, h=hp, o=out, p=ptrs, stride=0):
        return L.c3_adamw_slice(p, p, p, p, R, numel, off, n, ctypes.byref(h), o, stride, null)

    assert call(R=0) == -1 and call(R=65) == -1
    assert call(off=950, n=100) == -1                    # past the end
    assert call(off=-1) == -1 and call(n=-1) == -1
    assert call(o=null) == -1
    assert call(o=ctypes.c_void_p(1026)) == -2           # fp32 alignment
    assert call(p=(ctypes.c_void_p * 2)(256, 514)) == -2
    assert call(p=(ctypes.c_void_p * 2)(256, 0)) == -1
    for bad in (dict(step=0), dict(betas=(1.0, 0.9)), dict(betas=(0.9, -0.1)), dict(eps=0.0),
                dict(lr=-1.0), dict(weight_decay=-0.5)):
        kw = dict(lr=1e-3, betas=(0.9, 0.999), eps=1e-8, weight_decay=0.1, step=1)
        kw.update(bad)
        assert call(h=c3.adamw_hparams(**kw)) == -1, bad
    assert call(stride=99) == -1                         # rows overlap
    assert call(n=0, o=null) == 0                        # nothing to do


def test_optimizer_check_argument_errors_return_before_gpu_work():
    L = c3.lib()
    ptrs = (ctypes.c_void_p * 2)(256, 512)
    null = ctypes.c_void_p(0)
    hp = c3.adamw_hparams(step=1)
    addr = [4096 * (i + 1) for i in range(8)]
    out = c3.OptimizerCheckOut(*addr)

    def state(R=2, numel=10000, S=1024, tile=0):
        p = ctypes.cast(ptrs, ctypes.c_void_p)
        return c3.OptimizerState(p, p, p, p, R, 0, numel, S, tile)

    def ws_size(**kw):
        return L.c3_optimizer_check_workspace_size(ctypes.byref(state(**kw)))

    assert ws_size() > 0 and ws_size(S=768) > 0 and ws_size(tile=1 << 20) > 0
    assert ws_size(R=1) == 0 and ws_size(R=65) == 0 and ws_size(S=100) == 0
    assert ws_size(numel=0) == 0 and ws_size(tile=3000) == 0 and ws_size(tile=512) == 0
    assert L.c3_optimizer_check_workspace_size(null) == 0
    need = ws_size()

    def call(st=None, k=0, o=out, ws=ctypes.c_void_p(1 << 20), nbytes=need):
        st = st or state()
        return L.c3_optimizer_check(ctypes.byref(st), k, ctypes.byref(hp), ctypes.byref(o), ws,
                                    nbytes, null)

    assert call(k=-1) == -1
    assert call(st=state(R=1)) == -1
    assert call(o=c3.OptimizerCheckOut(*(addr[:7] + [0]))) == -1
    assert call(ws=null) == -4 and call(nbytes=need - 1) == -4
    assert call(ws=ctypes.c_void_p((1 << 20) + 8)) == -4
    assert call(o=c3.OptimizerCheckOut(*([4104] + addr[1:]))) == -2
    assert call(o=c3.OptimizerCheckOut(*(addr[:1] + [4100] + addr[2:]))) == -2     # records
    # state bases must be 16-byte aligned and the hyperparameters valid before
    # anything is launched
    bad = (ctypes.c_void_p * 2)(256, 520)
    p = ctypes.cast(bad, ctypes.c_void_p)
    assert call(st=c3.OptimizerState(p, p, p, p, 2, 0, 10000, 1024, 0)) == -2
    zero = (ctypes.c_void_p * 2)(256, 0)
    z = ctypes.cast(zero, ctypes.c_void_p)
    assert call(st=c3.OptimizerState(z, z, z, z, 2, 0, 10000, 1024, 0)) == -1
    for kw in (dict(step=0), dict(betas=(1.0, 0.9)), dict(eps=0.0), dict(lr=-1.0)):
        h = c3.adamw_hparams(**kw)
        assert L.c3_optimizer_check(ctypes.byref(state()), 0, ctypes.byref(h), ctypes.byref(out),
                                    ctypes.c_void_p(1 << 20), need, null) == -1, kw


@pytest.mark.parametrize("numel,S", [(10, 4), (12, 4), (3, 4), (65536 * 3 + 1000, 65536), (0, 8)])
def test_rotating_slice_matches_oracle(numel, S):
    from oracle import adamw
    for k in range(-(-numel // S) * 2 + 1):
        assert c3.optimizer_slice(k, numel, S) == adamw.slice_bounds(k, numel, S)


@pytest.mark.parametrize("header", ["c3.h", "c3_oob.h"])
@pytest.mark.parametrize("compiler", [["gcc", "-x", "c", "-std=c99"], ["g++", "-x", "c++", "-std=c++17"]])
def test_public_headers_compile_alone(header, compiler, tmp_path):
    """Each public header is self-contained plain C (and C++): it needs no
    HIP header, so a C client can include it with any host compiler."""
    import subprocess
    src = tmp_path / "use.c"
    src.write_text(f'#include "{header}"\nint main(void) {{ return 0; }}\n')
    r = subprocess.run(compiler + ["-Wall", "-Wextra", "-Werror", "-pedantic",
                                   "-I", os.path.join(ROOT, "include"), str(src),
                                   "-o", str(tmp_path / "use")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_optimizer_check_tile_limits():
    """The tile that is left after the lowering is at most 16 MiB, as a
    signature's; a larger one is an argument error, not a tile."""
    L = c3.lib()
    ptrs = (ctypes.c_void_p * 2)(256, 512)
    p = ctypes.cast(ptrs, ctypes.c_void_p)

    def state(S, tile):
        return c3.OptimizerState(p, p, p, p, 2, 0, 1 << 24, S, tile)

    def ws_size(S, tile):
        return L.c3_optimizer_check_workspace_size(ctypes.byref(state(S, tile)))
    assert ws_size(1 << 22, 1 << 24) > 0 and ws_size(1 << 23, 1 << 24) > 0
    assert ws_size(1024, 1 << 40) > 0                       # lowered to the slice
    assert ws_size(1 << 23, 1 << 25) == 0 and ws_size(1 << 24, 1 << 30) == 0
    out = c3.OptimizerCheckOut(*[4096 * (i + 1) for i in range(8)])
    hp = c3.adamw_hparams(step=1)
    assert L.c3_optimizer_check(ctypes.byref(state(1 << 23, 1 << 25)), 0, ctypes.byref(hp),
                                ctypes.byref(out), ctypes.c_void_p(1 << 20), 1 << 40,
                                ctypes.c_void_p(0)) == -1


def test_optimizer_check_default_tiles():
    """Tiles of whole KiB whatever the slice divides by: 32 of them, or 256 / R
    where each has 4 KiB, or tiles of 64 KiB; the workspace is R replicas x 7
    slices x 64 bytes a tile."""
    L = c3.lib()
    ptrs = (ctypes.c_void_p * 16)(*[256] * 16)
    p = ctypes.cast(ptrs, ctypes.c_void_p)
    for R, kib, tiles in ((2, 1, 1), (2, 5, 5), (2, 33, 17), (2, 129, 33), (2, 257, 65), (2, 1000, 125),
                          (2, 8200, 129), (3, 512, 74), (8, 1, 1), (8, 32, 32), (8, 33, 17), (8, 64, 32),
                          (8, 257, 29), (8, 500, 32), (16, 2047, 32), (16, 2048, 32), (16, 4097, 65)):
        st = c3.OptimizerState(p, p, p, p, R, 0, 1 << 24, kib * 256, 0)
        need = -(-R * 7 * 64 * tiles // 256) * 256
        assert L.c3_optimizer_check_workspace_size(ctypes.byref(st)) == need, (R, kib)


def test_default_signature_tiles():
    """Equal whole-KiB tiles of at most 256 KiB, and 128 KiB for larger chunks
    that are odd multiples of it: the workspaces are those of that many
    partials of 64 bytes a replica, none where a chunk is one tile."""
    L = c3.lib()
    meta = (c3.TensorMeta * 1)()
    meta[0].dtype, meta[0].ndim = c3.RAW, 1
    for kib, tiles in ((1, 1), (100, 1), (128, 1), (192, 1), (256, 1), (257, 2), (320, 2), (384, 3),
                       (512, 2), (640, 5), (768, 3), (896, 7), (1000, 4), (1152, 9), (1280, 5),
                       (4096, 16), (4224, 33)):
        meta[0].shape[0] = kib * 1024 * 64                 # 64 chunks
        one = L.c3_signature_workspace_size(meta, 1, 1, kib * 1024)
        two = L.c3_signature_workspace_size(meta, 1, 3, kib * 1024)
        assert two - one == (2 * 64 * tiles * 64 if tiles > 1 else 0), kib


def test_timing_workspace_of_wide_groups():
    """Bitmaps of both kinds and the confirmation's workspace; status and
    majority of both kinds too where the votes are separate launches."""
    L = c3.lib()

    def up(n):
        return -(-n // 256) * 256
    for R, G, T, W in ((17, 1, 1, 16), (20, 10, 30, 16), (64, 128, 511, 70), (33, 7, 100, 16)):
        n = G * T
        want = 2 * up(8 * n) + up(L.c3_confirm_workspace_size(R, G, T))
        assert L.c3_timing_consensus_workspace_size(R, G, T, W) == want
    for R, G, T, W in ((8, 10, 100, 70), (17, 16, (1 << 24) + 1, 16)):
        n = G * T
        want = 2 * (up(n) + up(8 * n) + up(4 * n)) + up(L.c3_confirm_workspace_size(R, G, T))
        assert L.c3_timing_consensus_workspace_size(R, G, T, W) == want
