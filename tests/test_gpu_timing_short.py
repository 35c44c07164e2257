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
