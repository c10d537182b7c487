"""DT with acceptance draws and few tiles runs the row-paired kernel (two cells
a lane by default, one where a lane per cell is asked for), alone and in
batches, also beside members without draws or with smaller domains: parity
with the oracle's DTr emulation, and the shape that ran."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RATES = [(0.7, 0.3), (0.5, 0.5), (4095 / 4096 + 2.0 ** -22, 1 / 4096 + 2.0 ** -23)]


def emulate(orc, L, D, p, q, stream, n):
    e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DT, p=p, q=q, seed=9, stream=stream)
    ref = orc.init_flat(L)
    for m in range(n):
        e.mcs(ref, m)
    return ref


@pytest.mark.parametrize("L,D,threads,want", [(512, 256, 0, (512, 2)), (1024, 256, 512, (512, 2)),
                                              (256, 128, 0, (128, 2)), (512, 128, 128, (128, 2)),
                                              (512, 128, 256, (256, 1)), (256, 128, 512, (256, 1))])
@pytest.mark.parametrize("pq", RATES)
def test_lattice(okpz, orc, L, D, threads, want, pq):
    print("dt few tiles: L=%d D=%d threads=%d rates %r" % (L, D, threads, pq), flush=True)
    with okpz.Lattice(L, D, D, 8, 8, okpz.BLOCK_DT, 9, 0) as lat:
        lat.set_threads(threads)
        lat.run(5, *pq)
        got = lat.sites()
        shape = lat.launch_shape()
    assert (shape["threads"], shape["cells"]) == want
    assert np.array_equal(got, emulate(orc, L, D, pq[0], pq[1], 0, 5))


def test_lattice_without_draws(okpz, orc):
    with okpz.Lattice(512, 128, 128, 8, 8, okpz.BLOCK_DT, 9, 0) as lat:
        lat.set_threads(256)
        lat.run(4, 1.0, 0.0)
        assert np.array_equal(lat.sites(), emulate(orc, 512, 128, 1.0, 0.0, 0, 4))
        assert lat.launch_shape() == {"threads": 256, "cells": 1}
        lat.set_threads(0)
        lat.run(1, 1.0, 0.0)
        assert lat.launch_shape()["threads"] == 64


@pytest.mark.parametrize("members", [[(256, 128), (512, 128)], [(512, 256), (1024, 256)],
                                     [(256, 128), (512, 256), (512, 128)]])
@pytest.mark.parametrize("threads", [0, 512])
def test_batch(okpz, orc, members, threads):
    rates = [(0.5, 0.5), (1.0, 0.0), (0.9, 0.2)]
    b = okpz.Batch()
    lats = [b.lattice(L, D, D, 8, 8, okpz.BLOCK_DT, seed=9, stream=i) for i, (L, D) in enumerate(members)]
    b.config(threads, 0, True)
    n = [5 - i for i in range(len(members))]
    print("dt few tiles: batch %r threads=%d" % (members, threads), flush=True)
    b.run(n, [rates[i][0] for i in range(len(n))], [rates[i][1] for i in range(len(n))])
    b.sync()
    shape = b.launch_shape()
    big = max(D for _, D in members)
    assert shape["threads"] == (threads or big * big // 128)
    for i, (L, D) in enumerate(members):
        assert np.array_equal(lats[i].sites(), emulate(orc, L, D, rates[i][0], rates[i][1], i, n[i]))
    b.close()
