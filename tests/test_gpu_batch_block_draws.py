"""Generic DT / DTr batches with two cells a lane, whose block draws come from the
wave's lanes from 64 rounds on and from the scalar unit below or beside a
member with fewer: parity with the oracle's DTr emulation."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# members (L, Dx, Dy, C); all fill two cells a lane of the largest domain
BATCHES = [[(512, 256, 256, 16), (1024, 256, 256, 16)], [(512, 256, 128, 8), (512, 128, 256, 8)],
           [(512, 256, 128, 8), (256, 64, 64, 4)], [(256, 64, 128, 4)]]


@pytest.mark.parametrize("members", BATCHES)
@pytest.mark.parametrize("scheme", ["DT", "DTR"])
@pytest.mark.parametrize("rates", [[(1.0, 0.0), (1.0, 0.0)], [(0.6, 0.4), (0.3, 0.9)], [(1.0, 0.0), (0.5, 0.5)]])
def test_two_cells(okpz, orc, members, scheme, rates):
    print("batch block draws: %r %s %r" % (members, scheme, rates), flush=True)
    b = okpz.Batch()
    lats = [b.lattice(L, Dx, Dy, C, C, getattr(okpz, "BLOCK_" + scheme), seed=17, stream=i)
            for i, (L, Dx, Dy, C) in enumerate(members)]
    n = [4 - i for i in range(len(members))]
    b.run(n, [rates[i][0] for i in range(len(n))], [rates[i][1] for i in range(len(n))])
    b.sync()
    shape = b.launch_shape()
    assert shape["cells"] == 2
    for i, (L, Dx, Dy, C) in enumerate(members):
        e = orc.Emu(L=L, Dx=Dx, Dy=Dy, Cx=C, Cy=C, scheme=getattr(orc, scheme), p=rates[i][0], q=rates[i][1],
                    seed=17, stream=i)
        ref = orc.init_flat(L)
        for m in range(n[i]):
            e.mcs(ref, m)
        assert np.array_equal(lats[i].sites(), ref)
    b.close()
