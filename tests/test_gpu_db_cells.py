"""Parity of the DB device step with one cell per lane with the oracle's DTr
emulation, alone and in a batch: the smallest lattices of both domain sizes
(one tile, whose window wraps onto the lattice's own blocks), rates with and
without acceptance prefixes, thresholds that tie often, and enough MCS that
attempts wait for other waves' (edges and corners) in most rounds; and the
batch's row-paired sweep with two and with four cells per lane."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RATES = [(0.95, 0.05), (1.0, 0.0), (0.0, 1.0), (0.5, 0.5), (1023 / 1024 + 2.0 ** -20, 1 / 1024 + 2.0 ** -21)]


@pytest.mark.parametrize("L,D", [(256, 128), (512, 128), (512, 256), (1024, 256)])
@pytest.mark.parametrize("pq", RATES)
def test_every_mcs(okpz, orc, L, D, pq):
    p, q = pq
    e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DB, p=p, q=q, seed=31, stream=2)
    ref = orc.init_flat(L)
    with okpz.Lattice(L, D, D, 8, 8, okpz.BLOCK_DB, 31, 2) as lat:
        for m in range(8):
            print("db_cells: L=%d D=%d p=%r q=%r MCS %d" % (L, D, p, q, m), flush=True)
            lat.run(1, p, q)
            e.mcs(ref, m)
            assert np.array_equal(lat.sites(), ref)


@pytest.mark.parametrize("D,threads", [(128, 0), (256, 0), (256, 256), (256, 512), (128, 64), (128, 128)])
@pytest.mark.parametrize("pq", [(0.7, 0.3), (1.0, 0.0)])
def test_batch(okpz, orc, D, threads, pq):
    p, q = pq
    Ls = [2 * D, 4 * D, 2 * D]
    b = okpz.Batch()
    lats = [b.lattice(L, D, D, 8, 8, okpz.BLOCK_DB, seed=6, stream=i) for i, L in enumerate(Ls)]
    b.config(threads, 0, True)
    n = [4, 3, 5]
    b.run(n, [p] * 3, [q] * 3)
    b.sync()
    for i, L in enumerate(Ls):
        e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DB, p=p, q=q, seed=6, stream=i)
        ref = orc.init_flat(L)
        for m in range(n[i]):
            e.mcs(ref, m)
        assert np.array_equal(lats[i].sites(), ref)
    b.close()
