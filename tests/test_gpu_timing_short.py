"""The single-pass timing kernel on few groups and iterations (R * T up to
512), against the CPU oracle: ragged last workgroups, partial steps and mask
segments, and shapes on both sides of the rule."""
import pytest

from test_gpu_timing import _case, _check, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_unit", [False, True])
@pytest.mark.parametrize("R,G,T,W,f64", [
    (4, 1, 1, 16, False), (4, 15, 128, 16, False), (4, 17, 128, 64, True), (4, 16, 129, 16, False),
    (8, 1, 64, 16, True), (8, 33, 63, 33, False), (8, 64, 64, 16, False), (8, 64, 65, 16, False),
    (16, 3, 32, 8, True), (16, 100, 31, 64, False), (16, 16, 33, 16, False), (8, 700, 3, 1, False),
])
def test_short_pass(R, G, T, W, f64, per_unit):
    _case("timing short", R, G, T, W, f64, per_unit)
    fp, tau = _inputs(R, G, T, seed=R * 1000 + G * 7 + T, f64=f64)
    _check(fp, tau, W, per_unit=per_unit)


@pytest.mark.parametrize("R,G,T,f64", [(4, 4096, 900, False), (8, 4096, 600, False), (16, 4096, 240, True),
                                       (8, 4112, 600, False)])
def test_streamed_bitmaps(R, G, T, f64):
    """Passes of over 256 MB, whose bitmaps go past the caches, against the
    separate votes and confirmation."""
    import torch
    from paper_2608_11034_amd import c3
    _case("timing streamed", R, G, T, f64)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(R + T)
    fp = torch.randint(-2**63, 2**63 - 1, (T, G, 1), generator=gen, device="cuda").expand(T, G, R).contiguous()
    fp[T // 3:, 5, R - 1] ^= 77
    tau = torch.randn((T, G, R), generator=gen, device="cuda").mul_(0.02).exp_()
    tau[:, G - 1, 1] *= 1.5
    if f64:
        tau = tau.double()
    ver, fu, tu = c3.timing_consensus(fp, tau)
    for got, ev, mode in ((fu, fp, c3.EXACT), (tu, tau, c3.STATISTICAL)):
        for a, b in zip(got, c3.consensus(ev, mode)):
            assert torch.equal(a, b)
    assert torch.equal(ver, c3.confirm(fu[1].view(T, G), tu[1].view(T, G), R, 16))


@pytest.mark.parametrize("R,G,T,f64", [(4, 4096, 1088, False), (8, 4096, 640, False), (8, 4096, 480, True),
                                       (16, 4096, 336, False), (16, 4096, 256, True)])
@pytest.mark.parametrize("kind", [0, 1])
def test_streamed_bitmaps_of_one_kind(kind, R, G, T, f64):
    """The same with the per-unit results of one kind only."""
    import torch
    from paper_2608_11034_amd import c3
    _case("timing streamed, one kind", kind, R, G, T, f64)
    assert T * G * (R * (16 if f64 else 12) + 13) > 256 << 20
    gen = torch.Generator(device="cuda")
    gen.manual_seed(R + T)
    fp = torch.randint(-2**63, 2**63 - 1, (T, G, 1), generator=gen, device="cuda").expand(T, G, R).contiguous()
    fp[T // 3:, 5, R - 1] ^= 77
    tau = torch.randn((T, G, R), generator=gen, device="cuda").mul_(0.02).exp_()
    tau[:, G - 1, 1] *= 1.5
    if f64:
        tau = tau.double()
    fu, tu = c3.consensus(fp, c3.EXACT), c3.consensus(tau, c3.STATISTICAL)
    want = (fu, tu)[kind]
    got = tuple(torch.full_like(x, 99) for x in want)
    ver = torch.empty((R * G, 24), dtype=torch.uint8, device="cuda")
    c3.timing_consensus(fp, tau, out=(ver, got, None) if kind == 0 else (ver, None, got))
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert torch.equal(ver, c3.confirm(fu[1].view(T, G), tu[1].view(T, G), R, 16))
