"""Kernels prepared on the device (kernel planes, compound kernels and their
adjoint, FP64) against the host code of the same library, which runs when the
device code's memory is refused or its limits are passed."""
import ctypes as C

import numpy as np
import pytest

from oracle import mvd_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mvd():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1308_0730_amd import mvd as m
    return m


def problem(dims, exts, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = dims
    views = [rng.uniform(0.5, 2.0, (nz, ny, nx)).astype(np.float32) for _ in exts]
    return views, [rng.uniform(0.05, 1.0, e[::-1]).astype(np.float32) for e in exts]


# PSF extents (x, y, z) per view: equal, different per view and axis, even,
# one point, one view, wider than the 8 outputs and 64 lanes of a thread and
# a wave, as long as the volume, and rows past the LDS of the plane builder
CASES = [((32, 30, 27), [(7, 5, 9)] * 3), ((32, 30, 27), [(3, 9, 5), (11, 1, 7), (5, 7, 1)]),
         ((20, 24, 18), [(4, 6, 8), (5, 3, 2)]), ((16, 16, 16), [(1, 1, 1), (3, 3, 3)]),
         ((30, 20, 18), [(9, 7, 5)]), ((40, 36, 30), [(23, 21, 19), (17, 25, 9)]), ((16, 15, 9), [(15, 15, 9)] * 2),
         ((8, 405, 6), [(3, 301, 3), (3, 5, 5)])]


@pytest.mark.parametrize("i,case", list(enumerate(CASES)))
def test_prepared_kernels_match_oracle(mvd, i, case):
    """One iteration of every variant on a flat start (1e-5, as every
    iteration test)."""
    dims, exts = case
    v, p = problem(dims, exts, 700 + i)
    for variant in (O.RL, O.EFF, O.OPT1, O.OPT2):
        with mvd.Deconvolver(v, p) as d:
            assert O.rel_l2(d.iterate(1, variant).estimate().cpu().numpy(), O.run(v, p, 1, variant)) <= 1e-5, variant


@pytest.mark.parametrize("variant", [O.EFF, O.OPT1])
@pytest.mark.parametrize("exts", [[(5, 7, 3)] * 3, [(3, 9, 5), (11, 1, 7), (5, 7, 1)], [(4, 6, 8), (5, 3, 2)]])
def test_compound_adjoint_on_the_device_is_the_hosts(mvd, variant, exts):
    """The gradients in the PSFs with and without device scratch: the same
    FP64 sums in another order, differing in their rounding only (1e-9, the
    level at which the host adjoint equals the oracle's)."""
    from tests.test_gpu_failures import CappedAllocator, create
    v, p = problem((32, 30, 27), exts, 720)
    L = mvd.lib()

    def grads(cap):
        a = CappedAllocator(mvd, 1 << 40)
        rc, h = create(mvd, v, p, a)
        assert rc == mvd.MVD_OK
        out = [np.zeros(q.shape, np.float64) for q in p]
        ptrs = (C.c_void_p * len(out))(*[o.ctypes.data for o in out])
        loss = C.c_double()
        for step in range(2):
            if step and cap:
                a.cap = a.live  # every buffer exists: only scratch is refused
            assert L.mvd_loss_grad(h, 1, variant, None, 0, C.byref(loss), C.cast(ptrs, C.POINTER(C.c_void_p)), None,
                                   0) == mvd.MVD_OK
        refused = a.refused
        L.mvd_destroy(h)
        return out, refused

    (dev, r0), (host, r1) = grads(False), grads(True)
    assert r0 == 0 and r1 > 0
    for x, y in zip(dev, host):
        np.testing.assert_allclose(x, y, rtol=0, atol=1e-9 * np.abs(y).max())


@pytest.mark.parametrize("dims,exts", [((32, 30, 27), [(7, 5, 9)] * 3), ((40, 36, 30), [(23, 21, 19), (17, 25, 9)]),
                                       ((30, 24, 20), [(5, 4, 7), (5, 3, 2), (1, 1, 1)])])
@pytest.mark.parametrize("variant", [O.RL, O.EFF, O.OPT1, O.OPT2])
def test_device_planes_are_the_hosts(mvd, dims, exts, variant):
    """One iteration with the kernels prepared on the device and by the host
    code (its scratch refused).  The PSFs' own planes have the same bits.  The
    compound kernels' FP64 sums differ in order, 1e-16 of their size, so hardly
    an FP32 rounding of the planes differs and at most a tenth of the voxels,
    by one FP32 step (6e-8): 2e-8 in relative L2, where planes prepared in FP32
    would differ by some 1e-7."""
    from tests.test_gpu_failures import CappedAllocator, create
    v, p = problem(dims, exts, 740)
    q = [x[::-1].copy() for x in p]
    L, P = mvd.lib(), C.POINTER(C.c_void_p)

    def run(refuse):
        a, cfg, out = CappedAllocator(mvd, 1 << 40), (C.c_int * 3)(), np.empty_like(v[0])
        rc, h = create(mvd, v, p, a)
        assert rc == mvd.MVD_OK
        assert L.mvd_get_tiles(h, cfg) == L.mvd_set_tiles(h, *cfg) == mvd.MVD_OK  # four passes: no other memory
        assert L.mvd_iterate(h, 1, variant) == mvd.MVD_OK
        start = np.ones_like(v[0])
        assert L.mvd_set_estimate(h, start.ctypes.data_as(C.c_void_p), mvd.MEM_HOST, 0) == mvd.MVD_OK
        if refuse:
            a.cap = a.live
        ptrs = (C.c_void_p * len(q))(*[x.ctypes.data for x in q])
        dd = (C.c_int * (3 * len(q)))(*sum([list(x.shape[::-1]) for x in q], []))
        assert L.mvd_set_psfs(h, C.cast(ptrs, P), dd, mvd.MEM_HOST) == mvd.MVD_OK
        assert L.mvd_iterate(h, 1, variant) == mvd.MVD_OK
        assert L.mvd_get_estimate(h, out.ctypes.data, mvd.MEM_HOST, 0) == mvd.MVD_OK
        L.mvd_destroy(h)
        return out, a.refused

    (dev, r0), (host, r1) = run(False), run(True)
    assert r0 == 0 and r1 == (1 if variant == O.RL else 2)
    if variant == O.RL:
        np.testing.assert_array_equal(dev, host)
    else:
        assert O.rel_l2(dev, host) <= 2e-8
