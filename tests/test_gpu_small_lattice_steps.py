"""Small lattices step by step: what a workgroup size or per-launch timing
selects in place of the launch of whole MCS, on narrow domains that share
their edge words, against the oracle's DTr emulation; and both ways in turn
on one lattice."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def pair(okpz, orc, scheme, p=1.0, q=0.0, L=64, D=16, stream=0, origin_mode=0):
    e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=scheme, p=p, q=q, seed=1, stream=stream,
                origin_mode=origin_mode)
    lat = okpz.Lattice(L, D, D, 8, 8, scheme, 1, stream, origin_mode)
    return e, orc.init_flat(L), lat


@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("how", ["threads", "timing"])
def test_every_mcs(okpz, orc, scheme, how):
    e, ref, lat = pair(okpz, orc, scheme)
    with lat:
        lat.set_threads(64) if how == "threads" else lat.timing(True)
        for m in range(400):
            lat.run(1, 1.0, 0.0)
            e.mcs(ref, m)
            assert np.array_equal(lat.sites(), ref), "MCS %d" % m
        if how == "timing":
            assert lat.get_timing()["step_launches"] == 4 * 400


@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("L,D", [(64, 16), (64, 32), (128, 64)])
@pytest.mark.parametrize("pq", [(0.95, 0.05), (0.5, 0.5), (0.3, 0.0), (0.0, 0.6), (1.0, 1.0), (0.0, 0.0)])
def test_rates(okpz, orc, scheme, L, D, pq):
    e, ref, lat = pair(okpz, orc, scheme, *pq, L=L, D=D, stream=3)
    with lat:
        lat.set_threads(64)
        for m in range(20):
            lat.run(1, *pq)
            e.mcs(ref, m)
        assert np.array_equal(lat.sites(), ref)


@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_origins(okpz, orc, scheme, mode):
    e, ref, lat = pair(okpz, orc, scheme, origin_mode=mode)
    with lat:
        lat.set_threads(64)
        for m in range(30):
            lat.run(1, 1.0, 0.0)
            e.mcs(ref, m)
        assert np.array_equal(lat.sites(), ref)


@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("pq", [(1.0, 0.0), (0.7, 0.3)])
def test_both_ways_in_turn(okpz, orc, scheme, pq):
    e, ref, lat = pair(okpz, orc, scheme, *pq, stream=5)
    with lat:
        done = 0
        for i, n in enumerate((3, 2, 5, 1, 4, 7)):
            lat.timing(i % 3 == 1)
            lat.set_threads(128 if i % 3 == 2 else 0)
            lat.run(n, *pq)
            if i % 3 == 1:
                assert lat.get_timing()["step_launches"] == 4 * n
            for m in range(done, done + n):
                e.mcs(ref, m)
            done += n
            assert np.array_equal(lat.sites(), ref) and lat.mcs == done
