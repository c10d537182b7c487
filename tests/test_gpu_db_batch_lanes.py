"""DB batches on the domains the kernels are made for keep two cells a lane, or
one, with few tiles, whatever workgroup was asked for: the shape that ran and
parity with the oracle's DTr emulation."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def compute_units():
    import torch

    return torch.cuda.get_device_properties(0).multi_processor_count


def run(okpz, orc, n, L, D, threads, p, q, check):
    print("db batch: %d x L=%d D=%d threads=%d p=%r" % (n, L, D, threads, p), flush=True)
    b = okpz.Batch()
    lats = [b.lattice(L, D, D, 8, 8, okpz.BLOCK_DB, seed=8, stream=i) for i in range(n)]
    b.config(threads, 0, True)
    b.run([4] * n, [p] * n, [q] * n)
    b.sync()
    shape = b.launch_shape()
    for i in check:
        e = orc.Emu(L=L, Dx=D, Dy=D, Cx=8, Cy=8, scheme=orc.DB, p=p, q=q, seed=8, stream=i)
        ref = orc.init_flat(L)
        for m in range(4):
            e.mcs(ref, m)
        assert np.array_equal(lats[i].sites(), ref)
    b.close()
    return shape["threads"], shape["cells"]


@pytest.mark.parametrize("p,q", [(1.0, 0.0), (0.7, 0.3)])
def test_two_cells_with_few_tiles(okpz, orc, p, q):
    assert run(okpz, orc, 3, 512, 256, 256, p, q, range(3)) == (512, 2)
    assert run(okpz, orc, 3, 256, 128, 64, p, q, range(3)) == (128, 2)


@pytest.mark.parametrize("p,q", [(1.0, 0.0), (0.7, 0.3)])
def test_four_cells_with_many_tiles(okpz, orc, p, q):
    cus = compute_units()
    n = 4 * cus // 16 + 1  # L = 2048, D = 256: 16 tiles a step each
    assert run(okpz, orc, n, 2048, 256, 256, p, q, (0, n - 1)) == (256, 4)
    assert run(okpz, orc, n // 4 + 1, 2048, 128, 64, p, q, (0,)) == (128, 2)


@pytest.mark.parametrize("p,q", [(1.0, 0.0), (0.7, 0.3)])
def test_one_cell_per_lane(okpz, orc, p, q):
    assert run(okpz, orc, 3, 512, 256, 0, p, q, range(3)) == (1024, 1)
    assert run(okpz, orc, 3, 512, 128, 0, p, q, range(3)) == (256, 1)
    # a lane per cell asked for: the same kernel, not the generic sweep of that shape
    kernel = lambda threads: batch_shape(okpz, 3, 512, 128, threads, p, q)
    assert kernel(256) == kernel(0)
    assert run(okpz, orc, 3, 512, 128, 256, p, q, range(3)) == (256, 1)


def batch_shape(okpz, n, L, D, threads, p, q):
    b = okpz.Batch()
    for i in range(n):
        b.lattice(L, D, D, 8, 8, okpz.BLOCK_DB, seed=8, stream=i)
    b.config(threads, 0, True)
    b.run([1] * n, [p] * n, [q] * n)
    b.sync()
    shape = b.launch_shape()
    b.close()
    return shape


def default_shape(okpz, n, L, Dx, Dy, C):
    b = okpz.Batch()
    for i in range(n):
        b.lattice(L, Dx, Dy, C, C, okpz.BLOCK_DB, seed=8, stream=i)
    print("db batch: %d x L=%d %dx%d cells of %d" % (n, L, Dx, Dy, C), flush=True)
    b.run([1] * n, [0.7] * n, [0.3] * n)
    b.sync()
    shape = b.launch_shape()
    b.close()
    return shape["threads"], shape["cells"]


def test_default_lanes_with_many_tiles(okpz):
    cus = compute_units()
    tiles = lambda per: 4 * cus // per + 1  # lattices for a few more than four tiles per compute unit
    assert default_shape(okpz, tiles(16), 2048, 256, 256, 8) == (256, 4)
    assert default_shape(okpz, tiles(16), 2048, 512, 128, 8) == (256, 4)
    assert default_shape(okpz, tiles(64), 2048, 128, 128, 4) == (256, 4)
    # large domains and eight cells a lane: the larger workgroup
    assert default_shape(okpz, tiles(8), 2048, 512, 256, 8) == (512, 4)
    assert default_shape(okpz, tiles(32), 2048, 256, 128, 4) == (512, 4)
