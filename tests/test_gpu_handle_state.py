"""What a handle keeps between calls: the stream its lazily allocated buffers
belong to, the form of its convolutions and the bits of repeated calls."""
import numpy as np
import pytest

from tests.test_gpu_two_pass import mvd, problem  # noqa: F401

pytestmark = pytest.mark.gpu


def test_lazy_buffers_belong_to_the_handles_stream(mvd):
    """Buffers allocated by a later call come from the pool of the handle's
    stream, not of the stream that is current then (whose pending work may
    still use what its pool hands out)."""
    import torch
    v, p, _ = problem((48, 45, 16), 2, 800, False)
    with mvd.Deconvolver(v, p) as d:
        before, other = set(d._bufs), torch.cuda.Stream()
        with torch.cuda.stream(other):
            d.iterate(2, "eff")
        new = set(d._bufs) - before
        assert new
        segs = [(s["address"], s["total_size"], s["stream"]) for s in torch.cuda.memory_snapshot()]
        for a in new:
            assert [st for lo, n, st in segs if lo <= a < lo + n] == [d.stream.cuda_stream]


@pytest.mark.parametrize("dims,variant", [((48, 45, 16), "rl"), ((30, 27, 25), "eff"), ((64, 64, 20), "opt1")])
@pytest.mark.parametrize("graphs", [False, True])
def test_bits_do_not_depend_on_what_ran_before(mvd, dims, variant, graphs):
    """The form of the convolutions comes from the handle's plan alone: the
    first call gives the bits of a repeated one, single iterations and
    view-updates those of one longer run."""
    v, p, w = problem(dims, 2, 810, True)

    def handle():
        return mvd.Deconvolver(v, p, w, use_graphs=graphs)

    with handle() as d:
        start = np.full_like(v[0], d.stats()["scale"])
        first = d.iterate(1, variant).estimate().cpu().numpy()
        flux = d.stats()["flux"]
        assert d.two_pass_split() > 0
        for _ in range(3):
            d.set_estimate(start).iterate(1, variant)
            np.testing.assert_array_equal(d.estimate().cpu().numpy(), first)
            assert d.stats()["flux"] == flux
        steps = d.iterate(1, variant).iterate(1, variant).estimate().cpu().numpy()
    with handle() as d:
        np.testing.assert_array_equal(d.iterate(3, variant).estimate().cpu().numpy(), steps)
    with handle() as d:
        for _ in range(3):
            for k in range(2):
                d.view_update(k, variant)
        np.testing.assert_array_equal(d.estimate().cpu().numpy(), steps)


def test_one_iteration_leaves_no_memory_behind(mvd):
    """After a single iteration a handle holds what it held at create (RL:
    no compound kernel is kept either)."""
    from tests.test_gpu_failures import CappedAllocator, create
    v, p, _ = problem((48, 45, 16), 2, 815, False)
    a = CappedAllocator(mvd, 1 << 40)
    rc, h = create(mvd, v, p, a)
    assert rc == mvd.MVD_OK
    at_create = a.live
    assert mvd.lib().mvd_iterate(h, 1, 0) == mvd.MVD_OK
    assert a.live == at_create and mvd.lib().mvd_two_pass_split(h, 0) > 0
    assert mvd.lib().mvd_iterate(h, 1, 0) == mvd.MVD_OK
    assert a.live > at_create
    mvd.lib().mvd_destroy(h)
    assert a.live == 0


@pytest.mark.parametrize("warm", [0, 1, 2])
@pytest.mark.parametrize("dims", [(48, 45, 16), (64, 300, 300)])
def test_runs_captured_by_the_caller(mvd, warm, dims):
    """A caller's graph of a run, captured on a handle that has run nothing,
    one iteration or two, replayed between eager runs, the profiler, new
    estimates and new PSFs, gives what an eager handle of the same form
    gives.  (64, 300, 300) has four passes only."""
    import torch
    v, p, _ = problem(dims, 2, 830, False)
    q = [x[:, ::-1].copy() for x in p]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        d, e = (mvd.Deconvolver(v, p, use_graphs=False) for _ in range(2))
        start = np.full_like(v[0], d.stats()["scale"])
        if warm:
            d.iterate(warm, "rl").set_estimate(start)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        d.iterate(2, "rl")
    with torch.cuda.stream(s):
        form = d.two_pass_split() > 0
        assert form == (warm == 2 and dims[1] < 300)
        if not form:
            e.set_tiles(*e.tiles())

        def same():
            np.testing.assert_array_equal(d.estimate().cpu().numpy(), e.estimate().cpu().numpy())
            assert d.stats()["flux"] == e.stats()["flux"]

        def replay():
            g.replay()
            e.iterate(2, "rl")
            same()

        replay()
        replay()
        for x in (d, e):
            x.iterate(1, "rl")
        replay()
        for x in (d, e):
            x.profile(1, "rl")
            x.view_update(1, "rl")
        replay()
        for x in (d, e):
            x.set_estimate(start)
        replay()
        for x in (d, e):
            x.set_psfs(q)
        replay()
        d.close()
        e.close()


def test_captured_runs_keep_their_memory(mvd):
    """After a capture the two-pass form's memory is not given back when
    another allocation fails: the graph still reads it."""
    import ctypes as C
    import torch
    from tests.test_gpu_failures import CappedAllocator
    v, p, _ = problem((48, 45, 16), 2, 840, False)
    L, s, a = mvd.lib(), torch.cuda.Stream(), CappedAllocator(mvd, 1 << 40)
    m, h, out = mvd._Marshalled(v, p, None, torch.device("cuda"), False), C.c_void_p(), np.empty_like(v[0])
    with torch.cuda.stream(s):
        opts = a.options(mvd)
        opts.use_graphs = 0
        assert L.mvd_create(C.byref(h), C.byref(m.problem), C.byref(opts)) == mvd.MVD_OK
        assert L.mvd_iterate(h, 2, 0) == mvd.MVD_OK
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        assert L.mvd_iterate(h, 1, 0) == mvd.MVD_OK
    with torch.cuda.stream(s), mvd.Deconvolver(v, p) as e:
        live = a.cap = a.live
        assert L.mvd_iterate(h, 1, 2) == mvd.MVD_ENOMEM and a.live == live
        g.replay()
        assert L.mvd_get_estimate(h, out.ctypes.data, mvd.MEM_HOST, 0) == mvd.MVD_OK
        np.testing.assert_array_equal(out, e.iterate(3, "rl").estimate().cpu().numpy())
        L.mvd_destroy(h)
    assert a.live == 0


# (540, 12, 10) and (16, 3, 8) have no two-pass form: half-rows past its row
# plans, and too few rows for its smallest split; two blocks are equal
UNEVEN = [(48, 45, 16), (540, 12, 10), (30, 27, 25), (16, 3, 8), (64, 32, 20), (30, 27, 25)]


@pytest.mark.parametrize("variant,weights", [("rl", True), ("eff", False)])
@pytest.mark.parametrize("graphs", [False, True])
def test_uneven_blocks_take_their_own_form(mvd, graphs, variant, weights):
    """Every block of a batch of different extents runs in the form that it
    has alone, with its bits, under every schedule, in combined updates and in
    view-updates, with the four-pass blocks beside it."""
    from oracle import mvd_oracle as O
    blocks = [problem(dims, 2, 850 + i, weights) for i, dims in enumerate(UNEVEN)]
    # a run, single iterations and view-updates, a combined update
    steps = [lambda d: d.iterate(3, variant), lambda d: d.iterate(1, variant),
             lambda d: d.view_update(0, variant).view_update(1, variant)]
    if not weights:
        steps += [lambda d: d.iterate_combined(2, variant, "geometric"),
                  lambda d: d.iterate_combined(1, variant, "arithmetic")]
    refs, scales, flux = [], [], np.zeros((len(steps), 2))
    for v, p, w in blocks:
        with mvd.Deconvolver(v, p, w) as d:
            scales.append(d.stats()["scale"])
            out = []
            for i, f in enumerate(steps):
                out.append(f(d).estimate().cpu().numpy())
                flux[i] += d.stats()["flux"]
            refs.append((d.two_pass_split(), out))
    assert [r[0] > 0 for r in refs] == [True, False, True, False, True, True]
    with mvd.Deconvolver.batch(blocks, use_graphs=graphs) as b:
        for sch in ("pass", "block", "run"):
            b.set_schedule(sch)
            for i, (v, _, _) in enumerate(blocks):
                b.set_estimate(np.full_like(v[0], scales[i]), i)
            for j, f in enumerate(steps):
                f(b)
                np.testing.assert_allclose(b.stats()["flux"], flux[j], rtol=1e-6)
                for i, (split, out) in enumerate(refs):
                    assert b.two_pass_split(i) == split
                    got = b.estimate(i).cpu().numpy()
                    if split:
                        np.testing.assert_array_equal(got, out[j])
                    else:
                        assert O.rel_l2(got, out[j]) <= 1e-5
        # set shapes: four passes everywhere, the profiler in between
        b.set_tiles(*b.tiles()).iterate(1, variant)
        assert not any(b.two_pass_split(i) for i in range(len(blocks)))
        b.default_tiles().iterate(1, variant)
        assert [b.two_pass_split(i) for i in range(len(blocks))] == [r[0] for r in refs]


@pytest.mark.parametrize("dims,nb", [((512, 512, 128), 3), ((512, 256, 128), 4)])
def test_job_order_of_the_z_passes(mvd, dims, nb):
    """Equal four-pass blocks whose spectra together exceed the memory-side
    cache (the z passes start on the last block) and do not (they start on
    the first) give the plain handles' bits."""
    import torch
    nx, ny, nz = dims
    g = torch.Generator(device="cuda")
    g.manual_seed(870)
    blocks = [([torch.rand((nz, ny, nx), device="cuda", generator=g) + 0.5],
               [torch.rand((5, 7, 9), device="cuda", generator=g) + 0.1], None) for _ in range(nb)]
    with mvd.Deconvolver.batch(blocks) as b:
        b.iterate(2, "rl")
        for i, (v, p, _) in enumerate(blocks):
            with mvd.Deconvolver(v, p) as d:
                assert b.two_pass_split(i) == d.two_pass_split() == 0
                assert torch.equal(b.estimate(i), d.iterate(2, "rl").estimate())


def test_default_tiles_bring_back_a_form_given_up(mvd):
    """A handle that gave up the two-pass form for want of memory takes it
    again after mvd_default_tiles, with its bits."""
    import ctypes as C
    from tests.test_gpu_failures import CappedAllocator, create
    v, p, _ = problem((48, 45, 16), 2, 880, False)
    L, a, out = mvd.lib(), CappedAllocator(mvd, 1 << 40), np.empty_like(v[0])
    with mvd.Deconvolver(v, p) as e:
        want, start = e.iterate(2, "rl").estimate().cpu().numpy(), np.full_like(v[0], e.stats()["scale"])
    rc, h = create(mvd, v, p, a)
    assert rc == mvd.MVD_OK

    def run():
        assert L.mvd_set_estimate(h, start.ctypes.data_as(C.c_void_p), mvd.MEM_HOST, 0) == mvd.MVD_OK
        assert L.mvd_iterate(h, 2, 0) == mvd.MVD_OK
        assert L.mvd_get_estimate(h, out.ctypes.data, mvd.MEM_HOST, 0) == mvd.MVD_OK
        return L.mvd_two_pass_split(h, 0) > 0

    assert run()
    a.cap = a.live
    assert L.mvd_iterate(h, 1, 2) == mvd.MVD_OK  # its kernel planes take the place of the spectra
    assert not run()
    a.cap = 1 << 40
    assert not run()
    assert L.mvd_default_tiles(h) == mvd.MVD_OK
    assert run()
    np.testing.assert_array_equal(out, want)
    L.mvd_destroy(h)
    assert a.live == 0


@pytest.mark.parametrize("dims", [(48, 45, 16), (512, 16, 12), (512, 3, 8), (540, 12, 10), (720, 10, 8), (864, 12, 10),
                                  (1000, 8, 6), (1024, 8, 6)])
def test_a_saved_estimate_continues_with_the_same_bits(mvd, dims):
    """A run continued from a saved estimate (whose spectrum a forward pass
    computes) gives the bits of the unbroken one (whose update pass left it)."""
    v, p, w = problem(dims, 2, 890, True)
    with mvd.Deconvolver(v, p, w) as d:
        saved = d.iterate(2, "eff").estimate().cpu().numpy()
        went_on = d.iterate(2, "eff").estimate().cpu().numpy()
        d.set_estimate(saved)
        np.testing.assert_array_equal(d.iterate(2, "eff").estimate().cpu().numpy(), went_on)


def test_psfs_that_find_no_memory_leave_the_old_ones(mvd):
    """PSFs with a longer z window than the handle has room for: ENOMEM, and
    the handle runs on with the PSFs it has."""
    import ctypes as C
    from tests.test_gpu_failures import CappedAllocator, create
    v, p, _ = problem((48, 45, 16), 2, 900, False)
    big = [np.ones((15, 7, 9), np.float32) for _ in p]
    L, a, out = mvd.lib(), CappedAllocator(mvd, 1 << 40), np.empty_like(v[0])
    rc, h = create(mvd, v, p, a)
    assert rc == mvd.MVD_OK
    assert L.mvd_iterate(h, 2, 1) == mvd.MVD_OK
    cfg = (C.c_int * 3)()
    assert L.mvd_get_tiles(h, cfg) == mvd.MVD_OK
    for tiles in (False, True):
        if tiles:
            assert L.mvd_set_tiles(h, *cfg) == mvd.MVD_OK
        a.cap = 0
        ptrs = (C.c_void_p * 2)(*[x.ctypes.data for x in big])
        dims = (C.c_int * 6)(*([9, 7, 15] * 2))
        assert L.mvd_set_psfs(h, C.cast(ptrs, C.POINTER(C.c_void_p)), dims, mvd.MEM_HOST) == mvd.MVD_ENOMEM
        a.cap = 1 << 40
        assert L.mvd_iterate(h, 2, 1) == mvd.MVD_OK
    assert L.mvd_get_estimate(h, out.ctypes.data, mvd.MEM_HOST, 0) == mvd.MVD_OK
    L.mvd_destroy(h)
    with mvd.Deconvolver(v, p) as d:
        # the failed call gave the two-pass form's memory back: four passes since
        d.iterate(2, "eff").set_tiles(*cfg).iterate(4, "eff")
        np.testing.assert_array_equal(out, d.estimate().cpu().numpy())


@pytest.mark.parametrize("graphs", [False, True])
def test_lanes_of_several_uneven_blocks(mvd, graphs):
    """More blocks than lanes: a plane pass takes a lane's blocks of all
    extents in one launch, an x pass those of one half-row and workgroup, and
    four-pass blocks follow; every block keeps the bits it has alone."""
    from oracle import mvd_oracle as O
    rng = np.random.default_rng(905)
    dims = [tuple(int(rng.choice(c)) for c in ((16, 20, 24, 32, 40, 48), (8, 12, 15, 24, 30), (9, 16, 25, 32)))
            for _ in range(36)] + [(16, 3, 8), (540, 12, 10), (64, 64, 40)]
    blocks = [problem(d, 2, 910 + i, False) for i, d in enumerate(dims)]
    steps = [lambda d: d.iterate(2, "eff"), lambda d: d.iterate_combined(2, "rl", "geometric"),
             lambda d: d.view_update(1, "eff")]
    refs, flux = [], 0.0
    for v, p, _ in blocks:
        with mvd.Deconvolver(v, p) as d:
            refs.append([f(d).estimate().cpu().numpy() for f in steps] + [d.two_pass_split()])
            flux += np.array(d.stats()["flux"])
    with mvd.Deconvolver.batch(blocks, use_graphs=graphs) as b:
        for j, f in enumerate(steps):
            f(b)
            for i, r in enumerate(refs):
                got = b.estimate(i).cpu().numpy()
                if r[-1]:
                    np.testing.assert_array_equal(got, r[j])
                else:
                    assert O.rel_l2(got, r[j]) <= 1e-5
        np.testing.assert_allclose(b.stats()["flux"], flux, rtol=1e-6)


def test_crowded_lanes_of_four_pass_blocks(mvd):
    """Several small blocks of a lane without a two-pass form: the whole batch
    takes the four passes."""
    dims = [(32, 24, z) for z in (16, 18, 20)]
    dims += [(4, 3, z) for z in (2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 32, 36, 40)]
    blocks = [problem(d, 1, 950 + i, False) for i, d in enumerate(dims)]
    with mvd.Deconvolver.batch(blocks) as b:
        b.iterate(2, "rl")
        assert not any(b.two_pass_split(i) for i in range(len(dims)))
        for i, (v, p, _) in enumerate(blocks):
            with mvd.Deconvolver(v, p) as d:
                np.testing.assert_allclose(b.estimate(i).cpu().numpy(), d.iterate(2, "rl").estimate().cpu().numpy(),
                                           rtol=1e-4)
