"""The buffer of the weight gradients' partial sums (no GPU needed): large enough
for every batch that a network accepts."""

import ctypes as C
import itertools

import pytest


def _partials(dims, max_batch, batch):
    from paper_1603_08161_amd import _lib as L
    need, have = C.c_int64(), C.c_int64()
    rc = L._lib.vd_debug_net_partials(*dims, max_batch, batch, C.byref(need), C.byref(have))
    assert rc == 0
    return need.value, have.value


def _check(dims, max_batch):
    for batch in range(1, max_batch + 1):
        need, have = _partials(dims, max_batch, batch)
        assert 0 < need <= have, (dims, max_batch, batch)


@pytest.mark.parametrize("dims,max_batch", [((24, 24, 24), 3), ((33, 5, 9), 3)])
def test_partials_of_fewer_samples_than_the_network_holds(dims, max_batch):
    """Cases whose smaller batches take more chunks than the largest one."""
    _check(dims, max_batch)


def test_partials_fit_for_every_batch():
    for n in range(1, 66):
        for max_batch in (1, 2, 3, 4, 5, 7, 8, 13):
            _check((n, n, n), max_batch)
    for dims in itertools.product((1, 2, 5, 16, 33, 57), repeat=3):
        _check(dims, 6)
    _check((5, 4, 3), 400)
    _check((1, 1, 1), 3000)
    _check((700, 3, 2), 9)
