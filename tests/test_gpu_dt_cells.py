"""Parity of the register-held DT device step with the oracle's DTr emulation:
the smallest lattices of both domain sizes (one tile, whose window wraps onto
the lattice's own blocks), every number of waves, each way of deciding, and
the same step inside a batch beside larger members."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RATES = [(1.0, 0.0), (0.0, 1.0), (1.0, 1.0), (0.0, 0.0), (0.6, 0.3), (4095 / 4096 + 2.0 ** -22, 1.0)]


@pytest.mark.parametrize("L,D,threads", [(256, 128, 0), (512, 128, 0), (512, 256, 128), (512, 256, 256)])
@pytest.mark.parametrize("pq", RATES)
def test_smallest_lattices(okpz, orc, L, D, threads, pq):
    p, q = pq
    e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DT, p=p, q=q, seed=21, stream=3)
    ref = orc.init_flat(L)
    with okpz.Lattice(L, D, D, 8, 8, okpz.BLOCK_DT, 21, 3) as lat:
        lat.set_threads(threads)
        # rough first, so that the rates without depositions have something to do
        lat.run(4, 0.7, 0.3)
        rough = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DT, p=0.7, q=0.3, seed=21, stream=3)
        for m in range(4):
            rough.mcs(ref, m)
        for m in range(4, 7):
            print("dt_cells: L=%d D=%d threads=%d p=%r q=%r MCS %d" % (L, D, threads, p, q, m), flush=True)
            lat.run(1, p, q)
            e.mcs(ref, m)
            assert np.array_equal(lat.sites(), ref)


@pytest.mark.parametrize("members", [[(256, 128), (512, 128)], [(512, 256), (1024, 256)],
                                     [(256, 128), (512, 256), (512, 128)]])
@pytest.mark.parametrize("threads", [0, 128, 256])
def test_batch_members(okpz, orc, members, threads):
    rates = [(1.0, 0.0), (0.5, 0.5), (0.9, 0.2)]
    b = okpz.Batch()
    lats = [b.lattice(L, D, D, 8, 8, okpz.BLOCK_DT, seed=5, stream=i) for i, (L, D) in enumerate(members)]
    b.config(threads, 0, True)
    n = [3 + i for i in range(len(members))]
    b.run(n, [rates[i][0] for i in range(len(n))], [rates[i][1] for i in range(len(n))])
    b.sync()
    for i, (L, D) in enumerate(members):
        e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DT, p=rates[i][0], q=rates[i][1], seed=5, stream=i)
        ref = orc.init_flat(L)
        for m in range(n[i]):
            e.mcs(ref, m)
        assert np.array_equal(lats[i].sites(), ref)
    b.close()
