"""GPU parity: the HIP path through the C ABI against the FP64 oracle on the
same seeded inputs.  Tolerances (relative L2 over the compared pixels):
1e-5 for float32 storage; 2e-3 for float16 / int16 storage, where the oracle is
fed the same stored values (widened exactly) -- the kernel's own arithmetic is
additionally held to 2e-5 there.  The full-image cases also hold every pixel
to the per-pixel error bound of tests/error_bound.py (delay allowance: the
plan's own float32 delay-error bound)."""
import ctypes
import sys

import numpy as np
import pytest

import error_bound as EB
from oracle import oracle as O
from paper_2203_14906_amd import phantom as ph
from sign_band import plan_eps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL_F32 = 1e-5
TOL_REDUCED = 2e-3
TOL_SAME_VALUES = 2e-5


@pytest.fixture(scope="module")
def hd():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2203_14906_amd import hodmas          # raises if libhodmas.so is missing
    return hodmas


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rel_l2(g, o):
    n = np.linalg.norm(o)
    return np.linalg.norm(g - o) / n if n > 0 else np.linalg.norm(g)


def stored(rf, dtype, seed=0):
    """(stored array, dequant scale) for a storage form."""
    if dtype == "f32":
        return ph.to_fp32(rf), 1.0
    if dtype == "f16":
        return ph.to_fp16(rf), 1.0
    codes, scale = ph.to_int16(rf, seed)
    return codes, float(scale)


def gpu_image(hd, plan, arr, order):
    dev = torch.from_numpy(np.ascontiguousarray(arr)).cuda()
    out = plan.beamform(dev, order)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def oracle_image(arr, scale, geom, grid, order, pixels=None):
    return O.beamform(arr, geom, grid, order, dequant_scale=scale if arr.dtype == np.int16 else None,
                      pixels=pixels)


def check_pixels(g, o, bounds, k, what):
    """Every pixel within its error bound."""
    q = EB.worst_ratio(g, o, bounds[k])
    say("%-48s at most %.3f of the pixel bound" % (what, q))
    assert q <= 1.0, "%s: a pixel reaches %.2f of its error bound" % (what, q)


def check(err, dtype, what):
    say("%-48s rel L2 %.3e" % (what, err))
    if dtype == "f32":
        assert err <= TOL_F32, what
    else:
        assert err <= TOL_REDUCED, what
        assert err <= TOL_SAME_VALUES, what


@pytest.mark.parametrize("cfg", [1, 2])
def test_config_full_image_fp32(hd, cfg):
    f = ph.config_frame(cfg)
    orders = ph.CONFIGS[cfg]["orders"]
    arr = ph.to_fp32(f.rf)
    plan = hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=max(orders))
    say("config %d: %d x %d grid, N=%d, S=%d, tiling %s" % (cfg, f.grid.nx, f.grid.nz, arr.shape[0],
        arr.shape[1], tuple(getattr(plan.info().tiling, n) for n in ("tile_x", "tile_z", "split", "chunk"))))
    bounds = EB.pixel_bounds(arr, f.geometry, f.grid, orders, plan_eps(plan, f.geometry, f.grid))
    for k in orders:
        say("config %d order %d" % (cfg, k))
        g = gpu_image(hd, plan, arr, k)
        o = oracle_image(arr, 1.0, f.geometry, f.grid, k)
        check(rel_l2(g, o), "f32", "config %d f32 order %d" % (cfg, k))
        check_pixels(g, o, bounds, k, "config %d f32 order %d" % (cfg, k))
    plan.close()


@pytest.mark.parametrize("dtype", ["i16", "f16"])
def test_config3_sampled(hd, dtype):
    f = ph.config_frame(3)
    arr, scale = stored(f.rf, dtype, seed=3000)
    plan = hd.Plan(f.geometry, f.grid, arr.shape[1], dtype, max_order=6, dequant_scale=scale)
    rng = np.random.default_rng(33)
    n = 3000
    ix = np.concatenate([rng.integers(0, 1024, n), np.arange(1024), [0, 1023, 0, 1023]]).astype(np.int32)
    iz = np.concatenate([rng.integers(0, 1024, n), np.full(1024, 1023), [0, 0, 1023, 1023]]).astype(np.int32)
    for k in range(1, 7):
        say("config 3 %s order %d" % (dtype, k))
        g = gpu_image(hd, plan, arr, k)
        o = oracle_image(arr, scale, f.geometry, f.grid, k, pixels=(ix, iz))
        check(rel_l2(g[iz, ix], o), dtype, "config 3 %s order %d (sampled)" % (dtype, k))
    plan.close()


def test_config3_full_image_order6_f16(hd):
    f = ph.config_frame(3)
    arr, scale = stored(f.rf, "f16")
    plan = hd.Plan(f.geometry, f.grid, arr.shape[1], "f16", max_order=6)
    say("config 3 f16 order 6, full image")
    g = gpu_image(hd, plan, arr, 6)
    o = oracle_image(arr, 1.0, f.geometry, f.grid, 6)
    check(rel_l2(g, o), "f16", "config 3 f16 order 6 (full image)")
    plan.close()


@pytest.mark.parametrize("tiling", [None, (16, 16, 1, 64), (16, 8, 2, 5), (8, 8, 4, 3), (32, 8, 1, 7),
                                    (16, 16, 2, 5), (32, 16, 1, 7)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "i16"])
def test_small_ragged_frames(hd, tiling, dtype):
    # several tiles plus ragged edges; a deep grid so far pixels run past the record
    f = ph.make_frame(13, 300, 37, 53, n_points=6, n_lines=1, snr_db=15.0, seed=17)
    grid = ph.Grid(nx=37, nz=53, x0_m=-3e-3, dx_m=0.17e-3, z0_m=0.2e-3, dz_m=0.21e-3)
    arr, scale = stored(f.rf, dtype, seed=17)
    plan = hd.Plan(f.geometry, grid, arr.shape[1], dtype, max_order=6, dequant_scale=scale,
                   tiling=tiling)
    bounds = EB.pixel_bounds(arr, f.geometry, grid, range(1, 7), plan_eps(plan, f.geometry, grid),
                             dequant_scale=scale if dtype == "i16" else None)
    for k in range(1, 7):
        say("small frame %s tiling %s order %d" % (dtype, tiling, k))
        g = gpu_image(hd, plan, arr, k)
        o = oracle_image(arr, scale, f.geometry, grid, k)
        check(rel_l2(g, o), dtype, "small %s %s k=%d" % (dtype, tiling, k))
        check_pixels(g, o, bounds, k, "small %s %s k=%d" % (dtype, tiling, k))
    plan.close()


@pytest.mark.parametrize("tiling", [(16, 16, 1, 67), (16, 16, 1, 33), (8, 8, 4, 67)])
@pytest.mark.parametrize("n", [6, 31, 32, 33, 64, 67])
def test_orders_across_blocks_of_elements(hd, n, tiling):
    """Element counts on either side of the groups of 4 and blocks of 32 the
    sums accumulate in, whole and left over at a chunk's end, with and without
    split groups, every pixel within its error bound."""
    f = ph.make_frame(n, 600, 40, 30, n_points=8, snr_db=15.0, seed=23 + n)
    grid = ph.make_grid(40, 30, 4e-3, 9e-3)
    arr = ph.to_fp32(f.rf)
    plan = hd.Plan(f.geometry, grid, 600, "f32", max_order=6, tiling=tiling)
    bounds = EB.pixel_bounds(arr, f.geometry, grid, range(3, 7), plan_eps(plan, f.geometry, grid))
    for k in range(3, 7):
        say("blocks n=%d tiling %s order %d" % (n, tiling, k))
        g = gpu_image(hd, plan, arr, k)
        check_pixels(g, oracle_image(arr, 1.0, f.geometry, grid, k), bounds, k, "blocks n=%d %s k=%d" % (n, tiling, k))
    plan.close()


@pytest.mark.parametrize("mirror", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "f16", "i16"])
def test_waves_that_stage_more_than_64_rows(hd, dtype, mirror):
    """A chunk of 272 rows (68 per wave: more than one vector of table entries),
    a second, ragged chunk, with rows inside the record and, with the record
    test forced, through the clamped copies; the record's own ends as well (the
    grid's last rows lie past them)."""
    n, S, nx, nz = 280, 500, 64, 48
    f = ph.make_frame(n, S, 8, 8, n_points=12, snr_db=15.0, seed=41, pitch=0.04e-3)
    grid = ph.Grid(nx=nx, nz=nz, x0_m=-(nx - 1) * 0.02e-3, dx_m=0.04e-3, z0_m=16.5e-3, dz_m=0.05e-3)
    arr, scale = stored(f.rf, dtype, seed=41)
    fl = hd.FLAG_MIRROR if mirror else 0
    chunk = 136 if mirror else 272
    plans = [hd.Plan(f.geometry, grid, S, dtype, max_order=6, dequant_scale=scale, flags=fl | g,
                     tiling=(16, 16, 1, chunk)) for g in (0, hd.FLAG_FORCE_CHECK)]
    assert plans[0].info().tiling.chunk == chunk
    tested = [t.check for t in plans[0].tables()[0]]
    assert any(tested) and not all(tested)
    bounds = EB.pixel_bounds(arr, f.geometry, grid, (1, 2, 5), plan_eps(plans[0], f.geometry, grid),
                             dequant_scale=scale if dtype == "i16" else None)
    for k in (1, 2, 5):
        say("rows %s mirror %s order %d" % (dtype, mirror, k))
        free, forced = (gpu_image(hd, p, arr, k) for p in plans)
        assert np.array_equal(free, forced)
        check_pixels(free, oracle_image(arr, scale, f.geometry, grid, k), bounds, k, "rows %s k=%d" % (dtype, k))
    for p in plans:
        p.close()


def test_single_element_and_order_above_n(hd):
    f = ph.make_frame(1, 256, 9, 11, n_points=2, seed=4)
    grid = ph.make_grid(9, 11, 3e-3, 5e-3)
    arr = ph.to_fp32(f.rf)
    plan = hd.Plan(f.geometry, grid, 256, "f32", max_order=6)
    o1 = oracle_image(arr, 1.0, f.geometry, grid, 1)
    assert rel_l2(gpu_image(hd, plan, arr, 1), o1) <= TOL_F32
    for k in range(2, 7):                       # k > N: no k-subset exists
        assert np.all(gpu_image(hd, plan, arr, k) == 0.0)
    plan.close()


def test_one_pixel_grids_rows_and_columns(hd):
    # tiles one pixel wide or deep: every other lane of the workgroup is idle
    f = ph.make_frame(16, 400, 24, 24, n_points=4, seed=8)
    arr = ph.to_fp32(f.rf)
    for nx, nz in ((1, 1), (1, 37), (53, 1), (2, 3)):
        grid = ph.Grid(nx=nx, nz=nz, x0_m=-0.3e-3, dx_m=0.2e-3, z0_m=3e-3, dz_m=0.15e-3)
        for tiling in (None, (16, 16, 1, 0), (8, 8, 4, 5)):
            plan = hd.Plan(f.geometry, grid, 400, "f32", max_order=6, tiling=tiling)
            for k in (1, 2, 5, 6):
                g = gpu_image(hd, plan, arr, k)
                o = oracle_image(arr, 1.0, f.geometry, grid, k)
                check(rel_l2(g, o), "f32", "grid %dx%d %s k=%d" % (nx, nz, tiling, k))
            plan.close()


def test_zero_rf_and_out_of_record(hd):
    g = ph.Geometry(16)
    grid = ph.make_grid(20, 20, 4.8e-3, 5e-3)
    plan = hd.Plan(g, grid, 128, "f32", max_order=6)
    zero = np.zeros((16, 128), dtype=np.float32)
    for k in range(1, 7):
        assert np.all(gpu_image(hd, plan, zero, k) == 0.0)
    plan.close()
    # a grid 40 mm deep sees nothing of a 128-sample record
    far = ph.Grid(nx=8, nz=8, x0_m=-1e-3, dx_m=0.3e-3, z0_m=40e-3, dz_m=0.3e-3)
    plan = hd.Plan(g, far, 128, "f32", max_order=3)
    assert plan.info().active_pairs == 0
    ones = np.ones((16, 128), dtype=np.float32)
    for k in (1, 2, 3):
        assert np.all(gpu_image(hd, plan, ones, k) == 0.0)
    plan.close()


def test_t0_irregular_stride_and_scale(hd):
    rng = np.random.default_rng(21)
    ex = np.sort(rng.uniform(-4e-3, 4e-3, 29))
    geom = ph.Geometry(29, t0_s=1.5e-6, element_x_m=ex)
    grid = ph.Grid(nx=45, nz=31, x0_m=-4.5e-3, dx_m=0.2e-3, z0_m=0.3e-3, dz_m=0.25e-3)
    S, stride = 500, 517
    rf = rng.standard_normal((29, S)) * 0.3
    padded = np.full((29, stride), np.nan, dtype=np.float32)   # padding must never be read
    padded[:, :S] = rf
    plan = hd.Plan(geom, grid, S, "f32", max_order=6, channel_stride=stride, frame_max=2.5)
    for k in range(1, 7):
        dev = torch.from_numpy(padded).cuda()
        got = plan.beamform(dev, k).cpu().numpy().astype(np.float64)
        o = O.beamform(padded[:, :S].copy(), geom, grid, k)
        check(rel_l2(got, o), "f32", "t0/irregular/stride k=%d" % k)
    plan.close()


def test_plain_and_forced_check_modes(hd):
    """FORCE_CHECK stages every row through registers and tests every delay;
    the default plan copies the rows of tiles inside the record straight into
    LDS and tests nothing there -- the images agree bit for bit."""
    f = ph.make_frame(24, 400, 33, 29, n_points=5, n_lines=1, seed=8)
    arr = ph.to_fp32(f.rf)
    base = hd.Plan(f.geometry, f.grid, 400, "f32", max_order=6)
    forced = hd.Plan(f.geometry, f.grid, 400, "f32", max_order=6, flags=hd.FLAG_FORCE_CHECK)
    plain = hd.Plan(f.geometry, f.grid, 400, "f32", max_order=6, flags=hd.FLAG_ACC_PLAIN)
    for k in range(1, 7):
        o = oracle_image(arr, 1.0, f.geometry, f.grid, k)
        a = gpu_image(hd, base, arr, k)
        np.testing.assert_array_equal(gpu_image(hd, forced, arr, k), a)
        check(rel_l2(gpu_image(hd, plain, arr, k), o), "f32", "plain accumulation k=%d" % k)
        check(rel_l2(a, o), "f32", "compensated k=%d" % k)
    for p in (base, forced, plain):
        p.close()


def test_repeatable_bitwise(hd):
    f = ph.config_frame(1)
    arr = ph.to_fp32(f.rf)
    plan = hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=6)
    dev = torch.from_numpy(arr).cuda()
    for k in (1, 4, 6):
        first = plan.beamform(dev, k).clone()
        for _ in range(3):
            assert torch.equal(plan.beamform(dev, k), first)
    plan.close()


def test_abi_errors_on_device(hd):
    f = ph.make_frame(8, 128, 8, 8, n_points=1, seed=2)
    plan = hd.Plan(f.geometry, f.grid, 128, "f32", max_order=4)
    dev = torch.from_numpy(ph.to_fp32(f.rf)).cuda()
    out = torch.empty((8, 8), dtype=torch.float32, device="cuda")
    L = hd.lib
    p_rf, p_out = ctypes.c_void_p(dev.data_ptr()), ctypes.c_void_p(out.data_ptr())
    for k in (0, 5, 7, -1):
        assert L.hodmas_beamform(plan.handle, p_rf, k, p_out, None) == hd.EUNSUPPORTED
    assert L.hodmas_beamform(plan.handle, None, 1, p_out, None) == hd.EINVAL
    assert L.hodmas_beamform(plan.handle, p_rf, 1, None, None) == hd.EINVAL
    assert L.hodmas_beamform(plan.handle, p_rf, 4, p_out, None) == hd.OK
    torch.cuda.synchronize()
    with pytest.raises(ValueError):
        plan.beamform(dev.to(torch.float16), 1)
    plan.close()


def test_streams_and_concurrent_plans(hd):
    f1 = ph.make_frame(32, 512, 48, 40, n_points=3, seed=31)
    f2 = ph.make_frame(64, 1024, 40, 64, n_points=3, seed=32)
    a1, a2 = ph.to_fp32(f1.rf), ph.to_fp32(f2.rf)
    p1 = hd.Plan(f1.geometry, f1.grid, 512, "f32", max_order=6)
    p2 = hd.Plan(f2.geometry, f2.grid, 1024, "f32", max_order=6)
    d1, d2 = torch.from_numpy(a1).cuda(), torch.from_numpy(a2).cuda()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    outs = []
    for k in (2, 5):
        with torch.cuda.stream(s1):
            o1 = p1.beamform(d1, k, stream=s1)
        with torch.cuda.stream(s2):
            o2 = p2.beamform(d2, k, stream=s2)
        outs.append((k, o1, o2))
    torch.cuda.synchronize()
    for k, o1, o2 in outs:
        check(rel_l2(o1.cpu().numpy().astype(np.float64), oracle_image(a1, 1.0, f1.geometry, f1.grid, k)),
              "f32", "stream 1 k=%d" % k)
        check(rel_l2(o2.cpu().numpy().astype(np.float64), oracle_image(a2, 1.0, f2.geometry, f2.grid, k)),
              "f32", "stream 2 k=%d" % k)
    p1.close()
    p2.close()


def test_threads_share_a_plan(hd):
    # the plan is immutable: four host threads launch with it at once, each on
    # its own stream and frames, and every image equals the one-thread result
    import threading
    f = ph.make_frame(32, 512, 48, 40, n_points=3, seed=33)
    plan = hd.Plan(f.geometry, f.grid, 512, "f32", max_order=6)
    rfs = [torch.from_numpy(ph.to_fp32(ph.make_frame(32, 512, 48, 40, n_points=3, seed=40 + i).rf)).cuda()
           for i in range(4)]
    ref = {(i, k): plan.beamform(rfs[i], k).clone() for i in range(4) for k in (1, 3, 6)}
    torch.cuda.synchronize()
    got, errors = {}, []

    def work(i):
        try:
            st = torch.cuda.Stream()
            for rep in range(5):
                for k in (1, 3, 6):
                    got[(i, k, rep)] = plan.beamform(rfs[i], k, stream=st)
            hd.sync(st)
        except Exception as e:          # reported below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    hd.sync()
    for (i, k, rep), img in got.items():
        assert torch.equal(img, ref[(i, k)]), "thread %d order %d rep %d" % (i, k, rep)
    plan.close()


def test_maximum_sizes(hd):
    # the element-count limit, a long record and the widest grid side of this
    # build, on phantom RF (band-limited pulses in noise) at the 0.075 mm pixel
    # pitch of the imaging workloads.  The float32 delay error grows with a
    # tile's extent in samples, and for k >= 3 the slope of |v|^(1/k) near 0
    # amplifies it, so coarse grids on white noise are held to the bar at
    # order 1 only (below).
    cases = [
        (4096, 2048, 0.01e-3, ph.Grid(nx=40, nz=24, x0_m=-1.5e-3, dx_m=0.075e-3, z0_m=5e-3, dz_m=0.075e-3)),
        (8, 1 << 20, 0.3e-3, ph.Grid(nx=24, nz=16, x0_m=-1e-3, dx_m=0.075e-3, z0_m=10.0, dz_m=0.075e-3)),
        (8, 512, 0.3e-3, ph.Grid(nx=16384, nz=4, x0_m=-8e-3, dx_m=1e-6, z0_m=2e-3, dz_m=0.075e-3)),
    ]
    for n, S, pitch, grid in cases:
        geom = ph.Geometry(n, pitch_m=pitch)
        arr = ph.to_fp32(ph.make_frame(n, S, 8, 8, n_points=6, n_lines=1, snr_db=10.0, seed=99,
                                       pitch=pitch).rf)
        plan = hd.Plan(geom, grid, S, "f32", max_order=6)
        for k in (1, 3, 6):
            say("max-size case N=%d S=%d grid %dx%d order %d" % (n, S, grid.nx, grid.nz, k))
            g = gpu_image(hd, plan, arr, k)
            o = oracle_image(arr, 1.0, geom, grid, k)
            check(rel_l2(g, o), "f32", "max N=%d S=%d nx=%d k=%d" % (n, S, grid.nx, k))
        plan.close()


def test_white_noise_order1(hd):
    # order 1 is linear in the samples, so the bar holds even for white noise
    # at the element limit on a coarse 0.3 mm grid (higher orders take |v|^(1/k), whose slope is
    # unbounded at 0; band-limited RF is covered above)
    geom = ph.Geometry(4096, pitch_m=0.01e-3)
    grid = ph.Grid(nx=16, nz=8, x0_m=-2.4e-3, dx_m=0.3e-3, z0_m=5e-3, dz_m=0.3e-3)
    arr = np.random.default_rng(99).standard_normal((4096, 2048)).astype(np.float32)
    plan = hd.Plan(geom, grid, 2048, "f32", max_order=1)
    check(rel_l2(gpu_image(hd, plan, arr, 1), oracle_image(arr, 1.0, geom, grid, 1)), "f32",
          "white noise N=4096 k=1")
    plan.close()


@pytest.mark.parametrize("tiling", [None, (16, 8, 2, 5), (8, 8, 4, 3), (32, 16, 1, 7), (16, 16, 2, 64)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "i16"])
def test_all_orders_one_pass(hd, tiling, dtype):
    f = ph.make_frame(13, 300, 37, 53, n_points=6, n_lines=1, snr_db=15.0, seed=17)
    grid = ph.Grid(nx=37, nz=53, x0_m=-3e-3, dx_m=0.17e-3, z0_m=0.2e-3, dz_m=0.21e-3)
    arr, scale = stored(f.rf, dtype, seed=17)
    plan = hd.Plan(f.geometry, grid, arr.shape[1], dtype, max_order=6, dequant_scale=scale,
                   tiling=tiling)
    dev = torch.from_numpy(np.ascontiguousarray(arr)).cuda()
    for kmax in (6, 4, 1):
        say("all orders %s tiling %s kmax %d" % (dtype, tiling, kmax))
        outs = plan.beamform_orders(dev, kmax)
        torch.cuda.synchronize()
        for k in range(1, kmax + 1):
            g = outs[k - 1].cpu().numpy().astype(np.float64)
            o = oracle_image(arr, scale, f.geometry, grid, k)
            check(rel_l2(g, o), dtype, "orders<=%d %s %s k=%d" % (kmax, dtype, tiling, k))
    plan.close()


def test_all_orders_config1_and_degenerate(hd):
    f = ph.config_frame(1)
    arr = ph.to_fp32(f.rf)
    for flags in (0, hd.FLAG_ACC_PLAIN):
        plan = hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=6, flags=flags)
        outs = plan.beamform_orders(torch.from_numpy(arr).cuda(), 6)
        torch.cuda.synchronize()
        for k in range(1, 7):
            o = oracle_image(arr, 1.0, f.geometry, f.grid, k)
            check(rel_l2(outs[k - 1].cpu().numpy().astype(np.float64), o), "f32",
                  "config 1 all orders flags %d k=%d" % (flags, k))
        plan.close()
    # fewer elements than the order: exact zeros, as for the one-order kernel
    g1 = ph.make_frame(3, 256, 9, 11, n_points=2, seed=4)
    grid = ph.make_grid(9, 11, 3e-3, 5e-3)
    a1 = ph.to_fp32(g1.rf)
    plan = hd.Plan(g1.geometry, grid, 256, "f32", max_order=6)
    outs = plan.beamform_orders(torch.from_numpy(a1).cuda(), 6)
    torch.cuda.synchronize()
    for k in range(1, 4):
        check(rel_l2(outs[k - 1].cpu().numpy().astype(np.float64),
                     oracle_image(a1, 1.0, g1.geometry, grid, k)), "f32", "N=3 all orders k=%d" % k)
    for k in range(4, 7):
        assert np.all(outs[k - 1].cpu().numpy() == 0.0)
    # ABI errors
    L = hd.lib
    out = torch.empty((11, 9), dtype=torch.float32, device="cuda")
    ptrs = (ctypes.c_void_p * 6)(*([out.data_ptr()] * 6))
    p_rf = ctypes.c_void_p(torch.from_numpy(a1).cuda().data_ptr())
    assert L.hodmas_beamform_orders(plan.handle, p_rf, 7, ptrs, None) == hd.EUNSUPPORTED
    assert L.hodmas_beamform_orders(plan.handle, p_rf, 0, ptrs, None) == hd.EUNSUPPORTED
    assert L.hodmas_beamform_orders(plan.handle, None, 2, ptrs, None) == hd.EINVAL
    assert L.hodmas_beamform_orders(plan.handle, p_rf, 2, None, None) == hd.EINVAL
    torch.cuda.synchronize()
    plan.close()


@pytest.mark.parametrize("mirror", [False, True])
@pytest.mark.parametrize("stride", [1 << 24, (1 << 25) - 64])
def test_int16_frames_of_2_to_4_gib(hd, stride, mirror):
    """64 records so far apart that the frame takes 2 GiB, or all but 4: row starts
    past 2^31 bytes.  Every image is bitwise that of the same records side by side,
    per order, all orders and in a batch.  (The frame stands in the middle of an
    allocation, so an offset taken for a signed one would still be inside.)"""
    n, S = 64, 700
    f = ph.make_frame(n, S, 256, 48, n_points=8, snr_db=15.0, seed=29)
    codes, scale = ph.to_int16(f.rf, 29)
    near = torch.from_numpy(codes).cuda()
    pool = torch.zeros(3 * n * stride, dtype=torch.int16, device="cuda")
    far = pool[n * stride:2 * n * stride].view(n, stride)
    far[:, :S] = near
    fl = hd.FLAG_MIRROR if mirror else 0
    plans = [hd.Plan(f.geometry, f.grid, S, "i16", max_order=6, dequant_scale=float(scale), flags=fl,
                     channel_stride=s) for s in (S, stride)]
    assert not all(t.check for t in plans[1].tables()[0])
    images = [[p.beamform(r, k) for k in range(1, 7)] for p, r in zip(plans, (near, far))]
    for k, (a, b) in enumerate(zip(*images)):
        say("int16 records %d apart, mirror %s, order %d" % (stride, mirror, k + 1))
        assert torch.equal(a, b), k + 1
    if not mirror:
        for a, b in zip(plans[0].beamform_orders(near, 6), plans[1].beamform_orders(far, 6)):
            assert torch.equal(a, b)
    bt = hd.Batch(6, 6 * plans[1].info().n_tiles, plans[1].info().lds_bytes)
    outs = [torch.empty_like(a) for a in images[0]]
    bt.set([plans[1]] * 6, [far] * 6, list(range(1, 7)), outs)
    bt.launch()
    torch.cuda.synchronize()
    for a, b in zip(images[0], outs):
        assert torch.equal(a, b)
    bt.close()
    for p in plans:
        p.close()
