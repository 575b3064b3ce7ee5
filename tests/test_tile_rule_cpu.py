"""The tile that a level gets without a choice (no GPU needed)."""

import ctypes as C

import pytest

TILES = {1: (8, 8, 4), 2: (8, 8, 8), 3: (32, 8, 4), 4: (32, 8, 4), 5: (8, 8, 16),
         6: (16, 4, 16), 7: (16, 4, 8), 8: (8, 8, 4)}


def _default(dims, precision="fp32", active=False, iterative=False):
    from paper_1603_08161_amd import _lib as L
    return L._lib.vd_debug_default_tile((C.c_int32 * 3)(*dims),
                                        L.VD_FP64 if precision == "fp64" else L.VD_FP32_FP64RED,
                                        (L.VD_FLAG_ACTIVE_SET if active else 0)
                                        | (L.VD_FLAG_ITERATIVE if iterative else 0))


def _blocks(dims, kind):
    n = 1
    for d, t in zip(dims, TILES[kind]):
        n *= -(-d // t)
    return n


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("active", [False, True])
def test_levels_of_one_launch_per_iteration(precision, active):
    """Levels that no kind covers with 256 tiles: 32x8x4 only in float32 without
    the optimised set, else 8x8x8."""
    plain = precision == "fp32" and not active
    for dims in [(65, 64, 64), (72, 72, 72), (70, 66, 73), (96, 96, 96), (110, 110, 110),
                 (200, 64, 64), (64, 200, 90)]:
        assert min(_blocks(dims, k) for k in TILES) > 256
        assert _default(dims, precision, active) == (3 if plain else 2), dims
    assert _default((20, 200, 200), precision, active) == 2  # too narrow for 32 along x


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("active", [False, True])
def test_levels_of_one_launch_solves(precision, active):
    for dims in [(2, 2, 2), (16, 16, 16), (32, 32, 32), (48, 48, 48), (57, 41, 50), (64, 64, 64)]:
        assert _blocks(dims, _default(dims, precision, active)) <= 256


@pytest.mark.parametrize("active", [False, True])
def test_levels_asked_to_run_one_launch_per_iteration(active):
    """In float64 8x8x8 in place of the 1024-node kinds; elsewhere no change."""
    for dims in [(16, 16, 16), (32, 32, 32), (48, 48, 48), (50, 50, 50), (57, 60, 55),
                 (64, 64, 64), (72, 72, 72)]:
        assert _default(dims, "fp32", active, True) == _default(dims, "fp32", active)
        kind = _default(dims, "fp64", active)
        assert _default(dims, "fp64", active, True) == (kind if kind in (7, 8) else 2), dims
