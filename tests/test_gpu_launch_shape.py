"""The launch shape reported is the one that ran: kernels made for a domain
shape set their own workgroups, whatever size was asked for."""
import pytest

pytestmark = pytest.mark.gpu


def lattice_shape(okpz, L, D, C, scheme, threads, p=1.0, q=0.0):
    with okpz.Lattice(L, D, D, C, C, scheme, seed=1, stream=0) as lat:
        assert lat.launch_shape() == {"threads": 0, "cells": 0}
        lat.set_threads(threads)
        lat.run(1, p, q)
        lat.sync()
        got = lat.launch_shape()
        assert got["threads"] * got["cells"] >= (D // C) ** 2
        return got["threads"], got["cells"]


def batch_shape(okpz, n, L, D, scheme, threads, p=1.0, q=0.0, grid=0, C=8):
    b = okpz.Batch()
    for i in range(n):
        b.lattice(L, D, D, C, C, scheme, seed=1, stream=i)
    assert b.launch_shape() == {"threads": 0, "cells": 0, "workgroups": 0, "lds_bytes": 0}
    b.config(threads, grid, True)
    b.run([1] * n, [p] * n, [q] * n)
    b.sync()
    got = b.launch_shape()
    b.close()
    return got["threads"], got["cells"], got["workgroups"]


def test_small_lattice_is_one_wave(okpz):
    assert lattice_shape(okpz, 64, 16, 8, okpz.BLOCK_DT, 0) == (64, 1)
    assert lattice_shape(okpz, 128, 64, 8, okpz.BLOCK_DB, 0) == (64, 1)


@pytest.mark.parametrize("threads,want", [(64, (128, 8)), (128, (128, 8)), (256, (256, 4))])
def test_register_held_step(okpz, threads, want):
    assert lattice_shape(okpz, 512, 256, 8, okpz.BLOCK_DT, threads) == want
    assert batch_shape(okpz, 3, 512, 256, okpz.BLOCK_DT, threads)[:2] == want


def test_generic_and_column_steps(okpz):
    assert lattice_shape(okpz, 256, 64, 8, okpz.BLOCK_DT, 0) == (64, 1)
    assert lattice_shape(okpz, 1024, 256, 16, okpz.BLOCK_DB, 128) == (128, 2)


def test_batch_workgroups(okpz):
    # one tile a step each: no more workgroups than tiles, or as many as asked for
    assert batch_shape(okpz, 5, 128, 64, okpz.BLOCK_DTR, 0, C=16)[2] == 5
    assert batch_shape(okpz, 5, 128, 64, okpz.BLOCK_DTR, 0, C=16, grid=2)[2] == 2
