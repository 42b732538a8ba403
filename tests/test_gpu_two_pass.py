"""The two-pass form of the convolutions against the FP64 oracle and against
the four passes, at the sizes where its split, its x tiles and its plane
transforms have edges; its batches, its switches and its memory limit."""
import ctypes as C

import numpy as np
import pytest

from oracle import mvd_oracle as O

pytestmark = pytest.mark.gpu

# (nx, ny, nz): the shortest and longest half-rows and lines, ny with every
# split (1 .. 9) and tails in its x tiles, planes of one and several stages
SHAPES = [(8, 4, 2), (10, 5, 3), (16, 8, 9), (30, 27, 25), (32, 36, 15), (48, 45, 16), (54, 40, 27), (64, 64, 64),
          (50, 100, 36), (72, 162, 10), (90, 50, 81), (128, 30, 125), (150, 108, 20), (512, 20, 12), (500, 24, 10),
          (20, 16, 256), (24, 12, 432), (96, 250, 30), (40, 400, 45)]


@pytest.fixture(scope="module")
def mvd():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1308_0730_amd import mvd as m
    return m


def problem(dims, n, seed, weights):
    rng = np.random.default_rng(seed)
    nx, ny, nz = dims
    views = [rng.uniform(0.5, 2.0, (nz, ny, nx)).astype(np.float32) for _ in range(n)]
    ext = [min(d if d % 2 else d - 1, c) for d, c in zip((nz, ny, nx), (5, 7, 9))]
    psfs = [rng.uniform(0.1, 1.0, ext).astype(np.float32) for _ in range(n)]
    ws = [rng.uniform(0, 1, (nz, ny, nx)).astype(np.float32) for _ in range(n)] if weights else None
    return views, psfs, ws


def four_pass(d):
    return d.set_tiles(*d.tiles())


@pytest.mark.parametrize("i,dims", list(enumerate(SHAPES)))
def test_two_pass_matches_oracle(mvd, i, dims):
    weights, lam, variant = bool(i & 1), 0.0006 * (i % 3 == 0), (O.RL, O.EFF, O.OPT1, O.OPT2)[i % 4]
    v, p, w = problem(dims, 2, 900 + i, weights)
    ref = O.run(v, p, 1, variant, lam=lam, weights=w)
    with mvd.Deconvolver(v, p, w, lam=lam) as d:
        start = np.full_like(v[0], d.stats()["scale"])
        d.iterate(2, variant).set_estimate(start)  # the form starts with the second iteration
        d.iterate(1, variant)
        got, st = d.estimate().cpu().numpy(), d.stats()
        four_pass(d).set_estimate(start)
        d.iterate(1, variant)
        old, st4 = d.estimate().cpu().numpy(), d.stats()
        d.default_tiles().set_estimate(start)
        d.iterate(1, variant)
        again = d.estimate().cpu().numpy()
    assert O.rel_l2(got, ref) <= 1e-5 and O.rel_l2(old, ref) <= 1e-5
    np.testing.assert_array_equal(again, got)
    np.testing.assert_allclose(st["flux"], st4["flux"], rtol=1e-6)


def test_two_pass_gives_its_memory_back(mvd):
    """A caller's allocator with room for the four passes only: nothing that
    ran without the two-pass form's memory fails for it."""
    from tests.test_gpu_failures import CappedAllocator, create
    v, p, _ = problem((48, 45, 16), 2, 985, False)
    L = mvd.lib()

    def run(cap, four=False):
        a = CappedAllocator(mvd, cap)
        rc, h = create(mvd, v, p, a)
        assert rc == mvd.MVD_OK
        if four:
            cfg = (C.c_int * 3)()
            assert L.mvd_get_tiles(h, cfg) == L.mvd_set_tiles(h, *cfg) == mvd.MVD_OK
        out = np.empty_like(v[0])
        try:
            for n, variant in ((3, O.RL), (2, O.OPT1), (2, O.EFF)):
                assert L.mvd_iterate(h, n, variant) == mvd.MVD_OK
            assert L.mvd_iterate_combined(h, 2, O.RL, 0) == mvd.MVD_OK
            assert L.mvd_get_estimate(h, out.ctypes.data, mvd.MEM_HOST, 0) == mvd.MVD_OK
            return out, a.live
        finally:
            L.mvd_destroy(h)
            assert a.live == 0

    want, base = run(1 << 40, four=True)
    _, live = run(1 << 40)
    assert live > base
    for cap in (base, base + 4096, live - 256):
        got, used = run(cap)
        assert used <= cap
        assert O.rel_l2(got, want) <= 1e-5


@pytest.mark.parametrize("mean", ["geometric", "arithmetic"])
def test_two_pass_combined(mvd, mean):
    v, p, _ = problem((50, 100, 36), 3, 950, False)
    ref = O.Problem(v, p)
    want = ref.iterate_combined(ref.psi0(), 2, O.EFF, O.GEOMETRIC if mean == "geometric" else O.ARITHMETIC)
    with mvd.Deconvolver(v, p) as d:
        d.iterate_combined(2, "eff", mean)
        assert O.rel_l2(d.estimate().cpu().numpy(), want) <= 1e-5


def test_two_pass_interleaved(mvd):
    """Switching between the forms, single view-updates and the profiler in
    the middle of a run continues from the same estimate."""
    v, p, w = problem((54, 40, 27), 2, 960, True)
    ref = O.run(v, p, 4, O.OPT1, weights=w)
    with mvd.Deconvolver(v, p, w) as d:
        d.iterate(2, "opt1").set_estimate(np.full_like(v[0], d.stats()["scale"]))
        d.iterate(1, "opt1")
        four_pass(d).iterate(1, "opt1")
        d.default_tiles()
        d.profile(1, "opt1")
        for k in range(2):
            d.view_update(k, "opt1")
        assert O.rel_l2(d.estimate().cpu().numpy(), ref) <= 1e-4


def test_two_pass_combined_of_uneven_blocks(mvd):
    """Combined updates of blocks of different extents (one launch per block,
    over the lanes) are each block's own."""
    blocks = [problem(s, 2, 990 + i, False) for i, s in enumerate([(48, 45, 16), (30, 27, 25), (64, 32, 20), (48, 36, 10)])]
    with mvd.Deconvolver.batch(blocks) as b:
        b.iterate_combined(3, "eff", "geometric")
        got, flux = [b.estimate(i).cpu().numpy() for i in range(4)], b.stats()["flux"][1]
    total = 0.0
    for i, (v, p, _) in enumerate(blocks):
        with mvd.Deconvolver(v, p) as d:
            np.testing.assert_array_equal(got[i], d.iterate_combined(3, "eff", "geometric").estimate().cpu().numpy())
            total += d.stats()["flux"][1]
    np.testing.assert_allclose(flux, total, rtol=1e-9)


@pytest.mark.parametrize("graphs", [False, True])
def test_two_pass_batch_is_plain(mvd, graphs):
    """A block gives the same bits alone and in a batch of its extents, under
    every schedule."""
    for dims in ((48, 45, 16), (64, 64, 20)):
        blocks = [problem(dims, 2, 970 + i, False) for i in range(3)]
        refs, scales = [], []
        for v, p, w in blocks:
            with mvd.Deconvolver(v, p, use_graphs=graphs) as d:
                refs.append(d.iterate(2, "eff").estimate().cpu().numpy())
                scales.append(d.stats()["scale"])
        with mvd.Deconvolver.batch(blocks, use_graphs=graphs) as b:
            for sch in ("pass", "block", "run"):
                b.set_schedule(sch)
                for i, (v, _, _) in enumerate(blocks):
                    b.set_estimate(np.full_like(v[0], scales[i]), i)
                b.iterate(2, "eff")
                for i, r in enumerate(refs):
                    np.testing.assert_array_equal(b.estimate(i).cpu().numpy(), r)


def test_new_psfs_reach_the_two_pass_spectra(mvd):
    v, p, _ = problem((48, 45, 16), 2, 980, False)
    q = [x[:, :, ::-1].copy() for x in p]
    with mvd.Deconvolver(v, p) as d, mvd.Deconvolver(v, q) as e:
        d.iterate(2, "eff")
        d.set_psfs(q).set_estimate(np.full_like(v[0], d.stats()["scale"]))
        np.testing.assert_array_equal(d.iterate(2, "eff").estimate().cpu().numpy(),
                                      e.set_estimate(np.full_like(v[0], d.stats()["scale"]))
                                      .iterate(2, "eff").estimate().cpu().numpy())


# (nx, ny, nz), split: volumes past 1.5 Mi spectrum values (every split; the
# largest planes and volumes of the form), then the splits of small ones that
# SHAPES leaves out and both sides of the small rule's line
SPLITS = [((512, 25, 256), 1), ((512, 50, 256), 2), ((400, 162, 50), 3), ((256, 96, 128), 4), ((320, 250, 128), 5),
          ((180, 144, 125), 6), ((216, 240, 200), 8), ((180, 288, 200), 9), ((24, 54, 10), 6), ((24, 48, 8), 6),
          ((400, 243, 32), 3), ((400, 324, 25), 3), ((540, 4, 4), 0), ((512, 250, 64), 2), ((512, 256, 81), 0),
          ((64, 300, 300), 0)]


@pytest.mark.parametrize("i", range(len(SPLITS)))
def test_two_pass_splits(mvd, i):
    """The form runs where its rule says, with every variant with and without
    weights, and gives the oracle's iteration."""
    dims, split = SPLITS[i]
    variant, weights, lam = (O.RL, O.EFF, O.OPT1, O.OPT2)[i % 4], bool(i // 4 & 1), 0.0006 * (i % 3 == 0)
    v, p, w = problem(dims, 2, 1000 + i, weights)
    with mvd.Deconvolver(v, p, w, lam=lam) as d:
        got = d.iterate(1, variant).estimate().cpu().numpy()
        assert d.two_pass_split() == split
    assert O.rel_l2(got, O.run(v, p, 1, variant, lam=lam, weights=w)) <= 1e-5


@pytest.mark.parametrize("dims,variant", [((216, 200, 100), O.OPT1), ((60, 50, 40), O.RL)])
def test_two_pass_of_a_padded_grid(mvd, dims, variant):
    """The linear boundary: the form runs on the padded grid, whose margin
    voxels carry no data."""
    v, p, w = problem(dims, 2, 1030, True)
    ref = O.ProblemLinear(v, p, w, 0.0006)
    with mvd.Deconvolver(v, p, w, lam=0.0006, boundary="linear") as d:
        got = d.iterate(1, variant).estimate().cpu().numpy()
        assert d.two_pass_split() > 0
    assert O.rel_l2(got, ref.interior(ref.iterate(ref.psi0(), 1, variant))) <= 1e-5
