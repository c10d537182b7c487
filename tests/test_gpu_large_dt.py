"""The DT step at the full size L = 2^17, where a lattice's last byte is the
last that a 32-bit offset reaches: after one MCS from flat a window across the
lattice's corner equals the oracle's window emulation on every site that the
oracle can determine, for each domain size, number of waves and way of deciding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 1 << 17


@pytest.mark.parametrize("D,threads,p,q", [(256, 0, 1.0, 0.0), (256, 0, 0.95, 0.05), (256, 256, 0.95, 0.05),
                                           (256, 256, 1.0, 1.0), (128, 0, 1.0, 0.0), (128, 0, 0.5, 0.5)])
def test_one_mcs_across_the_corner(okpz, orc, D, threads, p, q):
    print("large DT: D=%d threads=%d p=%r q=%r" % (D, threads, p, q), flush=True)
    window = (L - 1500, L - 1400, 3072, 3072)
    wx0, wy0, W, H = window
    with okpz.Lattice(L, D, D, 8, 8, okpz.BLOCK_DT, seed=1, stream=0) as lat:
        lat.set_threads(threads)
        lat.run(1, p, q)
        got = lat.window(wx0, wy0, W, H)
        shape = lat.launch_shape()
    assert shape["threads"] == {(256, 0): 128, (256, 256): 256, (128, 0): 64}[D, threads]
    emu = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DT, p=p, q=q, seed=1, stream=0)
    ref, valid = orc.init_flat_window(L, window)
    emu.mcs_window(ref, valid, window, 0)
    v = valid.astype(bool)
    assert v.sum() > 0.3 * W * H
    assert np.array_equal(got[v], ref[v])
    flat, _ = orc.init_flat_window(L, window)
    assert (got[v] != flat[v]).any()
