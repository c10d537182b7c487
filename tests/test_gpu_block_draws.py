"""The generic DT / DTr step takes its block draws 512 rounds at a time: cells
with fewer rounds than that, two such blocks and eight, alone and in a batch,
against the oracle's DTr emulation."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [4, 16, 32, 64])
@pytest.mark.parametrize("scheme", ["DT", "DTR"])
@pytest.mark.parametrize("pq", [(1.0, 0.0), (0.6, 0.4)])
def test_rounds(okpz, orc, C, scheme, pq):
    p, q = pq
    L, D = 256, 64
    e = orc.Emu(L=L, Dx=D, Dy=D, Cx=C, Cy=C, scheme=getattr(orc, scheme), p=p, q=q, seed=13, stream=4)
    ref = orc.init_flat(L)
    for m in range(3):
        e.mcs(ref, m)
    print("block draws: C=%d %s p=%r q=%r" % (C, scheme, p, q), flush=True)
    with okpz.Lattice(L, D, D, C, C, getattr(okpz, "BLOCK_" + scheme), 13, 4) as lat:
        lat.run(3, p, q)
        assert np.array_equal(lat.sites(), ref)
    b = okpz.Batch()
    lat = b.lattice(L, D, D, C, C, getattr(okpz, "BLOCK_" + scheme), seed=13, stream=4)
    b.run([3], [p], [q])
    b.sync()
    assert np.array_equal(lat.sites(), ref)
    b.close()
