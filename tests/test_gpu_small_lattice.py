"""Small lattices: whole MCS in one launch (L <= 128, 8 x 8 cells) against the
oracle's DTr emulation, for every scheme, one to sixteen tiles, square and
oblong domains, each origin mode and runs split at odd places; and the
measurement with one lane a band (up to L = 4096)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RATES = [(1.0, 0.0), (0.7, 0.3), (1023 / 1024 + 2.0 ** -20, 1 / 1024 + 2.0 ** -21)]
SHAPES = [(64, 8, 32), (64, 32, 16), (64, 16, 16), (64, 32, 32), (128, 64, 64), (128, 16, 64), (128, 32, 32)]


@pytest.mark.parametrize("L,Dx,Dy", SHAPES)
@pytest.mark.parametrize("scheme", ["DT", "DB", "DTR"])
@pytest.mark.parametrize("pq", RATES)
def test_runs(okpz, orc, L, Dx, Dy, scheme, pq):
    p, q = pq
    e = orc.Emu(L=L, Dx=Dx, Dy=Dy, Cx=8, Cy=8, scheme=getattr(orc, scheme), p=p, q=q, seed=41, stream=7)
    ref = orc.init_flat(L)
    with okpz.Lattice(L, Dx, Dy, 8, 8, getattr(okpz, "BLOCK_" + scheme), 41, 7) as lat:
        done = 0
        for n in (1, 7, 2):
            print("small: L=%d D=%dx%d %s p=%r q=%r %d MCS" % (L, Dx, Dy, scheme, p, q, n), flush=True)
            lat.run(n, p, q)
            for m in range(done, done + n):
                e.mcs(ref, m)
            done += n
            assert np.array_equal(lat.sites(), ref)
            assert lat.mcs == done


@pytest.mark.parametrize("origin", ["ORIGIN_FIXED", "ORIGIN_COARSE"])
@pytest.mark.parametrize("scheme", ["DT", "DB", "DTR"])
def test_origin_modes_and_launch_limit(okpz, orc, origin, scheme):
    """More MCS than one launch takes, in one call."""
    L, D, n = 64, 16, 4097 + 30
    e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=getattr(orc, scheme), p=0.6, q=0.4, seed=9, stream=1,
                origin_mode=getattr(orc, origin))
    ref = orc.init_flat(L)
    with okpz.Lattice(L, D, D, 8, 8, getattr(okpz, "BLOCK_" + scheme), 9, 1,
                      origin_mode=getattr(okpz, origin)) as lat:
        lat.run(n, 0.6, 0.4)
        for m in range(n):
            e.mcs(ref, m)
        assert np.array_equal(lat.sites(), ref)


@pytest.mark.parametrize("L", [64, 128, 256, 512, 1024, 4096])
def test_measurement(okpz, orc, L):
    e = orc.Emu(L=L, Dx=16, Dy=16, Cx=8, Cy=8, scheme=orc.DT, p=0.9, q=0.1, seed=3, stream=2)
    ref = orc.init_flat(L)
    with okpz.Lattice(L, 16, 16, 8, 8, okpz.BLOCK_DT, 3, 2) as lat:
        for n in range(3):
            lat.run(5, 0.9, 0.1)
            for m in range(5 * n, 5 * n + 5):
                e.mcs(ref, m)
            if n == 0:
                lat.snapshot()
                snap = ref.copy()
            for _ in range(2):
                mo, ac = lat.observe(True)
                want = orc.moments(ref)
                assert all(mo[k] == v for k, v in want.items())
                assert ac["c_h"] == orc.c_h(ref, snap) and ac["c_s"] == orc.c_s(ref, snap)
                assert mo == lat.measure()
