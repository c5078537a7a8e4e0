"""Batched form on the GPU: a mixed batch in one persistent launch gives every
frame bitwise the image of its own per-frame launch (so parity carries over),
graph replays match the eager launch, and bad work lists are refused."""
import sys

import numpy as np
import pytest

from oracle import oracle as O
from paper_2203_14906_amd import phantom as ph

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hd():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2203_14906_amd import hodmas
    return hodmas


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


SPECS = [  # (N, S, nx, nz, order, dtype)
    (64, 1024, 96, 80, 1, "f32"), (128, 2048, 128, 128, 6, "f16"), (32, 512, 37, 53, 3, "i16"),
    (64, 1024, 64, 64, 4, "f16"), (16, 600, 40, 24, 2, "f32"), (128, 1024, 200, 100, 5, "i16"),
    (256, 2048, 64, 96, 2, "f16"), (8, 300, 17, 19, 6, "f32"), (64, 2048, 150, 150, 3, "f32"),
    (4, 256, 12, 12, 6, "f16"),  # order above the element count: zero image
]


def make_batch_inputs(hd, specs, seed0=500):
    plans, rfs, outs, orders, frames = [], [], [], [], []
    for i, (n, S, nx, nz, k, dt) in enumerate(specs):
        f = ph.make_frame(n, S, nx, nz, n_points=5, n_lines=1, snr_db=15.0, seed=seed0 + i)
        if dt == "f32":
            arr, scale = ph.to_fp32(f.rf), 1.0
        elif dt == "f16":
            arr, scale = ph.to_fp16(f.rf), 1.0
        else:
            arr, scale = ph.to_int16(f.rf, seed0 + i)
        plans.append(hd.Plan(f.geometry, f.grid, S, dt, max_order=6, dequant_scale=float(scale)))
        rfs.append(torch.from_numpy(arr).cuda())
        outs.append(torch.full((nz, nx), float("nan"), dtype=torch.float32, device="cuda"))
        orders.append(k)
        frames.append((f, arr, float(scale)))
    return plans, rfs, outs, orders, frames


def test_mixed_batch_equals_per_frame_launches(hd):
    plans, rfs, outs, orders, frames = make_batch_inputs(hd, SPECS)
    alone = [p.beamform(r, k) for p, r, k in zip(plans, rfs, orders)]
    torch.cuda.synchronize()
    batch = hd.Batch(max_frames=32, max_units=100000)
    batch.set(plans, rfs, orders, outs)
    inf = batch.info()
    say("batch: %d frames, %d units, grid %d, lds %d" % (inf.n_frames, inf.n_units, inf.grid, inf.lds_bytes))
    batch.launch()
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(alone, outs)):
        assert torch.equal(a, b), "frame %d differs between the batch and its own launch" % i
    # spot parity of two members against the oracle
    for i in (1, 5):
        f, arr, scale = frames[i]
        o = O.beamform(arr, f.geometry, f.grid, orders[i], dequant_scale=scale if arr.dtype == np.int16 else None)
        g = outs[i].cpu().numpy().astype(np.float64)
        err = np.linalg.norm(g - o) / np.linalg.norm(o)
        say("batch member %d (order %d, %s) rel L2 %.3e" % (i, orders[i], arr.dtype, err))
        assert err <= 2e-5
    assert torch.all(outs[-1] == 0)
    batch.close()
    for p in plans:
        p.close()


def test_graph_replays_and_reset_work_list(hd):
    plans, rfs, outs, orders, _ = make_batch_inputs(hd, SPECS[:6], seed0=700)
    alone = [p.beamform(r, k).clone() for p, r, k in zip(plans, rfs, orders)]
    batch = hd.Batch(max_frames=16, max_units=50000)
    batch.set(plans, rfs, orders, outs)
    batch.capture()
    for rep in range(4):
        for o in outs:
            o.fill_(float("nan"))
        # unrelated eager work between replays
        junk = torch.randn(1 << 16, device="cuda").sum()
        batch.replay()
        torch.cuda.synchronize()
        assert torch.isfinite(junk)
        for i, (a, b) in enumerate(zip(alone, outs)):
            assert torch.equal(a, b), "replay %d frame %d" % (rep, i)
    # a new work list (other orders, reversed frames) is read by the same graph
    orders2 = [(k % 6) + 1 for k in orders][::-1]
    plans2, rfs2, outs2 = plans[::-1], rfs[::-1], outs[::-1]
    batch.set(plans2, rfs2, orders2, outs2)
    batch.replay()
    torch.cuda.synchronize()
    for p, r, k, o in zip(plans2, rfs2, orders2, outs2):
        assert torch.equal(p.beamform(r, k), o)
    batch.close()
    for p in plans:
        p.close()


def test_graph_replays_follow_changing_kind_mixes(hd):
    """Replays fit the instantiated graph to each work list (absent kinds
    switched off, grids cut to the unit count): a kind that leaves and comes
    back, a single tiny frame, and back-to-back replays without a host wait
    all give every frame its own launch's image."""
    plans, rfs, outs, orders, _ = make_batch_inputs(hd, SPECS, seed0=900)
    alone = [p.beamform(r, k).clone() for p, r, k in zip(plans, rfs, orders)]
    batch = hd.Batch(max_frames=16, max_units=100000)
    batch.set(plans, rfs, orders, outs)
    batch.capture()
    picks = [list(range(len(SPECS))), [2, 8], [9], [4, 0], list(range(len(SPECS))), [7]]
    for step, idx in enumerate(picks):
        for i in idx:
            outs[i].fill_(float("nan"))
        batch.set([plans[i] for i in idx], [rfs[i] for i in idx], [orders[i] for i in idx],
                  [outs[i] for i in idx])
        for _ in range(3):                       # replays queued back to back
            batch.replay()
        torch.cuda.synchronize()
        for i in idx:
            assert torch.equal(alone[i], outs[i]), "step %d frame %d" % (step, i)
        say("replay step %d (frames %s) ok" % (step, idx))
    batch.close()
    for p in plans:
        p.close()


@pytest.mark.parametrize("comp", [True, False])
def test_batch_multi_chunk_split_and_batch_lds(hd, comp):
    # units of several chunks, split tilings (combined through LDS between
    # units) and orders above the element count, one after another in a
    # persistent workgroup
    flags = 0 if comp else hd.FLAG_ACC_PLAIN
    cases = [  # (N, S, nx, nz, order, dtype, tiling, extra flags)
        (32, 512, 40, 36, 3, "f32", (16, 16, 1, 5), 0), (24, 400, 33, 29, 6, "f16", (8, 8, 4, 7), 0),
        (48, 700, 45, 50, 2, "i16", (16, 8, 2, 9), 0), (128, 2048, 96, 96, 5, "f32", (8, 8, 4, 43), 0),
        (256, 2048, 64, 64, 4, "f16", (8, 8, 4, 19), 0), (20, 300, 16, 16, 6, "f32", (16, 16, 1, 3), 0),
        (64, 1024, 48, 48, 1, "i16", (16, 16, 1, 64), 0), (5, 200, 18, 18, 6, "f16", (8, 8, 4, 2), 0),
    ]
    plans, rfs, outs, orders = [], [], [], []
    for i, (n, S, nx, nz, k, dt, til, fl) in enumerate(cases):
        f = ph.make_frame(n, S, nx, nz, n_points=4, n_lines=1, snr_db=15.0, seed=900 + i)
        if dt == "f32":
            arr, scale = ph.to_fp32(f.rf), 1.0
        elif dt == "f16":
            arr, scale = ph.to_fp16(f.rf), 1.0
        else:
            arr, scale = ph.to_int16(f.rf, 900 + i)
        p = hd.Plan(f.geometry, f.grid, S, dt, max_order=6, dequant_scale=float(scale), tiling=til,
                    flags=flags | fl)
        t = p.info().tiling
        say("case %d: N=%d %dx%d k=%d %s tiling %s" % (i, n, nx, nz, k, dt, (t.tile_x, t.tile_z, t.split, t.chunk)))
        plans.append(p)
        rfs.append(torch.from_numpy(arr).cuda())
        outs.append(torch.full((nz, nx), float("nan"), dtype=torch.float32, device="cuda"))
        orders.append(k)
    alone = [p.beamform(r, k).clone() for p, r, k in zip(plans, rfs, orders)]
    lds = max(p.info().lds_bytes for p in plans)
    batch = hd.Batch(max_frames=16, max_units=100000, max_lds_bytes=lds, flags=flags)
    batch.set(plans, rfs, orders, outs)
    batch.launch()
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(alone, outs)):
        assert torch.equal(a, b), "case %d differs between the batch and its own launch" % i
    batch.close()
    for p in plans:
        p.close()


def test_batch_rejects_bad_work_lists(hd):
    f = ph.make_frame(16, 256, 20, 20, n_points=2, seed=3)
    p4 = hd.Plan(f.geometry, f.grid, 256, "f32", max_order=4)
    plain = hd.Plan(f.geometry, f.grid, 256, "f32", max_order=6, flags=hd.FLAG_ACC_PLAIN)
    host = hd.Plan(f.geometry, f.grid, 256, "f32", max_order=6, flags=hd.FLAG_HOST_ONLY)
    rf = torch.from_numpy(ph.to_fp32(f.rf)).cuda()
    out = torch.empty((20, 20), dtype=torch.float32, device="cuda")
    b = hd.Batch(max_frames=2, max_units=10000)
    with pytest.raises(hd.HodmasError) as e:
        b.set([p4], [rf], [5], [out])
    assert e.value.status == hd.EUNSUPPORTED
    with pytest.raises(hd.HodmasError) as e:
        b.set([plain], [rf], [2], [out])
    assert e.value.status == hd.EINVAL
    with pytest.raises(hd.HodmasError) as e:
        b.set([host], [rf], [2], [out])
    assert e.value.status == hd.EINVAL
    with pytest.raises(hd.HodmasError) as e:
        b.set([p4, p4, p4], [rf] * 3, [1] * 3, [out] * 3)
    assert e.value.status == hd.EINVAL
    small = hd.Batch(max_frames=2, max_units=1)
    with pytest.raises(hd.HodmasError) as e:
        small.set([p4], [rf], [1], [out])
    assert e.value.status == hd.EINVAL
    tiny_lds = hd.Batch(max_frames=2, max_units=10000, max_lds_bytes=256)
    with pytest.raises(hd.HodmasError) as e:
        tiny_lds.set([p4], [rf], [1], [out])
    assert e.value.status == hd.EINVAL
    with pytest.raises(hd.HodmasError) as e:
        b.launch()                      # nothing set yet
    assert e.value.status == hd.EINVAL
    pl = hd.Batch(max_frames=2, max_units=10000, flags=hd.FLAG_ACC_PLAIN)
    pl.set([plain], [rf], [3], [out])
    pl.launch()
    torch.cuda.synchronize()
    assert torch.equal(out, plain.beamform(rf, 3))
    for x in (b, small, tiny_lds, pl):
        x.close()
    for x in (p4, plain, host):
        x.close()


def test_each_kind_gets_its_own_lds_and_grid(hd):
    """A kind runs with the LDS of its own largest plan, so a small-LDS work
    list gets a larger persistent grid than a large-LDS one in the same batch;
    graph replays refit the nodes' LDS and grid when the list changes, and
    every image stays bitwise its own launch."""
    f = ph.config_frame(1)
    arr = ph.to_fp32(f.rf)
    dev = torch.from_numpy(arr).cuda()
    S = arr.shape[1]
    big = hd.Plan(f.geometry, f.grid, S, "f32", max_order=4, tiling=(16, 16, 1, 64))
    small = hd.Plan(f.geometry, f.grid, S, "f32", max_order=4, tiling=(16, 16, 1, 4))
    lb, ls = big.info().lds_bytes, small.info().lds_bytes
    assert ls < lb
    bt = hd.Batch(max_frames=4, max_units=4 * big.info().n_tiles, max_lds_bytes=64 * 1024)
    outs = [torch.full((f.grid.nz, f.grid.nx), float("nan"), dtype=torch.float32, device="cuda")
            for _ in range(4)]
    ref = {(id(p), k): p.beamform(dev, k).cpu().numpy() for p in (big, small) for k in (2, 4)}
    captured = False
    for rep, plan in enumerate([big, small, big, small]):
        for o in outs:
            o.fill_(float("nan"))
        bt.set([plan] * 4, [dev] * 4, [2, 4, 2, 4], outs)
        inf = bt.info()
        assert inf.lds_bytes == plan.info().lds_bytes
        if plan is small:
            grid_small = inf.grid
        else:
            grid_big = inf.grid
        if not captured:
            bt.launch()
            bt.capture()
            captured = True
        else:
            bt.replay()
        torch.cuda.synchronize()
        for i, o in enumerate(outs):
            assert np.array_equal(o.cpu().numpy(), ref[(id(plan), [2, 4][i % 2])]), (rep, i)
    say("per-kind LDS: big %d B -> grid %d, small %d B -> grid %d" % (lb, grid_big, ls, grid_small))
    assert grid_small >= grid_big
    bt.close()
    big.close()
    small.close()


def test_graph_gains_kinds_after_capture(hd):
    """A graph captured for one kind holds only that kind's kernel; a later
    work list with other kinds has it rebuilt at the next replay, and every
    frame still gets its own launch's image (also when the list shrinks back)."""
    plans, rfs, outs, orders, _ = make_batch_inputs(hd, SPECS, seed0=950)
    alone = [p.beamform(r, k).clone() for p, r, k in zip(plans, rfs, orders)]
    batch = hd.Batch(max_frames=16, max_units=100000)
    first = [0]
    for step, idx in enumerate([first, list(range(len(SPECS))), first, [len(SPECS) - 1, 1]]):
        for i in idx:
            outs[i].fill_(float("nan"))
        batch.set([plans[i] for i in idx], [rfs[i] for i in idx], [orders[i] for i in idx],
                  [outs[i] for i in idx])
        if step == 0:
            batch.capture()
        for _ in range(2):
            batch.replay()
        torch.cuda.synchronize()
        for i in idx:
            assert torch.equal(alone[i], outs[i]), "step %d frame %d" % (step, i)
    batch.close()
    for p in plans:
        p.close()


@pytest.mark.parametrize("dtype", ["f32", "f16", "i16"])
@pytest.mark.parametrize("tiling,frames", [((8, 8, 4, 0), 150), ((16, 16, 1, 0), 48), (None, 5)])
def test_mixed_orders_in_one_kernel(hd, dtype, tiling, frames):
    """Frames of all orders, paired and unpaired, in one list: short units that
    are drawn several at a time, longer ones, and a list smaller than the
    device.  Every image equals its own launch on each of several launches and
    replays of the same list (the draws start from zero each time) and after
    the list changes."""
    f = ph.make_frame(24, 500, 64, 64, n_points=5, snr_db=15.0, seed=71)
    grid = ph.make_grid(64, 64, 24 * 0.3e-3, 9e-3)
    arr = {"f32": ph.to_fp32, "f16": ph.to_fp16}.get(dtype, lambda r: ph.to_int16(r, 71)[0])(f.rf)
    scale = float(ph.to_int16(f.rf, 71)[1]) if dtype == "i16" else 1.0
    rf = torch.from_numpy(np.ascontiguousarray(arr)).cuda()
    two = [hd.Plan(f.geometry, grid, 500, dtype, max_order=6, dequant_scale=scale, tiling=tiling, flags=fl)
           for fl in (0, hd.FLAG_MIRROR)]
    own = {(i, k): two[i].beamform(rf, k).clone() for i in (0, 1) for k in range(1, 7)}
    picks = [(i % 2, i // 2 % 6 + 1) for i in range(frames)]
    outs = [torch.empty((64, 64), device="cuda") for _ in picks]
    units = sum(p.info().n_tiles for p in two) * frames
    bt = hd.Batch(frames, units, max(p.info().lds_bytes for p in two))
    for part in (picks, picks[: frames // 2], picks):
        bt.set([two[i] for i, _ in part], [rf] * len(part), [k for _, k in part], outs[: len(part)])
        bt.capture()
        for go in (bt.launch, bt.replay, bt.launch, bt.replay):
            for o in outs:
                o.fill_(float("nan"))
            go()
            torch.cuda.synchronize()
            for o, p in zip(outs, part):
                assert torch.equal(o, own[p]), (p, go.__name__)
    bt.close()
    for p in two:
        p.close()


@pytest.mark.parametrize("extra", [0, 1, 3000])
def test_more_units_than_the_largest_grid(hd, extra):
    """A kind's grid ends at 65536 workgroups: units beyond it are taken by a
    second step of the first workgroups (65536 units exactly, a few more, and
    a part of a second round), every image bitwise its own launch."""
    f = ph.config_frame(1)
    arr = ph.to_fp32(f.rf)
    rfs = [torch.from_numpy(np.ascontiguousarray(arr * s)).cuda() for s in (1.0, -0.5, 0.25)]
    plan = hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=1, tiling=(16, 8, 2, 16))
    tiles = plan.info().n_tiles
    n = -(-65536 // tiles) + -(-extra // tiles)
    alone = [plan.beamform(r, 1) for r in rfs]
    out = torch.full((n, f.grid.nz, f.grid.nx), float("nan"), dtype=torch.float32, device="cuda")
    bt = hd.Batch(max_frames=n, max_units=n * tiles)
    bt.set([plan] * n, [rfs[i % 3] for i in range(n)], [1] * n, list(out.unbind(0)))
    assert bt.info().n_units == n * tiles >= 65536 + extra
    bt.launch()
    torch.cuda.synchronize()
    for j in range(3):
        assert bool((out[j::3] == alone[j]).all())
    bt.close()
    plan.close()


@pytest.mark.parametrize("frames", [127, 128, 130])
def test_long_lists_of_short_units_at_several_orders(hd, frames):
    """Three orders whose units fill the device several times: up to 8191 units
    an order in one kernel, from 8192 on in their own, paired ones mixed in
    both cases; every image bitwise its own launch, launched and replayed, and
    the list may change between the two."""
    f = ph.make_frame(8, 300, 64, 64, n_points=5, snr_db=15.0, seed=72)
    grid = ph.make_grid(64, 64, 8 * 0.3e-3, 9e-3)
    rf = torch.from_numpy(ph.to_fp32(f.rf)).cuda()
    orders = (1, 3, 6)
    for flags in (0, hd.FLAG_MIRROR):
        plan = hd.Plan(f.geometry, grid, 300, "f32", max_order=6, tiling=(8, 8, 4, 0), flags=flags)
        assert plan.info().n_tiles == 64
        own = [plan.beamform(rf, k) for k in orders]
        out = torch.empty((3, frames, 64, 64), device="cuda")
        bt = hd.Batch(3 * frames, 3 * frames * 64, plan.info().lds_bytes)
        for used in (frames, 20, frames):
            bt.set([plan] * (3 * used), [rf] * (3 * used), [k for k in orders for _ in range(used)],
                   [out[i, j] for i in range(3) for j in range(used)])
            bt.capture()
            for go in (bt.launch, bt.replay, bt.replay):
                out.fill_(float("nan"))
                go()
                torch.cuda.synchronize()
                for i in range(3):
                    assert bool((out[i, :used] == own[i]).all()), (flags, used, orders[i])
        bt.close()
        plan.close()


def test_launches_of_one_list_overlap_on_several_streams(hd):
    """Launches and replays of one list of several orders, each on its own
    stream and none waiting for another, between products that leave them a part
    of the device; then launches and replays alone: every one forms every unit
    (a launch only reads the list)."""
    f = ph.config_frame(1)
    arr = ph.to_fp32(f.rf)
    rf = torch.from_numpy(arr).cuda()
    plan = hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=6, tiling=(16, 16, 1, 16), flags=hd.FLAG_MIRROR)
    own = {k: plan.beamform(rf, k).clone() for k in range(1, 7)}
    orders = [i % 6 + 1 for i in range(240)]
    outs = [torch.empty((f.grid.nz, f.grid.nx), device="cuda") for _ in orders]
    bt = hd.Batch(len(orders), len(orders) * plan.info().n_tiles, plan.info().lds_bytes)
    bt.set([plan] * len(orders), [rf] * len(orders), orders, outs)
    bt.capture()
    streams = [torch.cuda.Stream() for _ in range(3)]
    busy = torch.randn((4096, 4096), device="cuda")

    def check(what, *runs):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        for go, stream in runs:
            go(stream=stream)
        torch.cuda.synchronize()
        for i, (o, k) in enumerate(zip(outs, orders)):
            assert torch.equal(o, own[k]), (what, i)

    for rep in range(4):
        say("overlapping launches, round %d" % rep)
        torch.cuda.synchronize()
        busy @ busy
        for i in range(6):
            (bt.replay if i == 3 else bt.launch)(stream=streams[i % 3])
        torch.cuda.synchronize()
        check("launch", (bt.launch, streams[0]))
        check("replay", (bt.replay, streams[1]))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bt.launch()

    def captured(stream):
        with torch.cuda.stream(stream):
            graph.replay()

    for rep in range(4):
        say("a captured launch beside others, round %d" % rep)
        torch.cuda.synchronize()
        busy @ busy
        for i in range(6):
            (captured if i % 2 else bt.launch)(stream=streams[i % 3])
        torch.cuda.synchronize()
        check("captured", (captured, streams[2]))
        check("launch after it", (bt.launch, streams[0]))
    bt.close()
    plan.close()


def test_one_large_plan_leaves_the_others_their_workgroups(hd):
    """A long list of small plans at all orders and one plan of 36 KB tiles: the
    large one's order runs by itself, so the device holds as many workgroups of
    the others as their own LDS allows; every image is bitwise its own launch,
    launched and replayed, also in a short list, where all orders run as one."""
    f = ph.make_frame(64, 2048, 128, 128, n_points=5, snr_db=15.0, seed=73)
    arr = ph.to_fp32(f.rf)
    rf = torch.from_numpy(arr).cuda()
    small, big = (hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=6, tiling=(16, 16, 1, c))
                  for c in (4, 64))
    own = {(p, k): p.beamform(rf, k).clone() for p in (small, big) for k in range(1, 7)}
    bt = hd.Batch(400, 400 * small.info().n_tiles, big.info().lds_bytes)
    bt.set([big], [rf], [3], [torch.empty((f.grid.nz, f.grid.nx), device="cuda")])
    alone = bt.info().grid
    bt.set([small], [rf], [3], [torch.empty((f.grid.nz, f.grid.nx), device="cuda")])
    assert bt.info().grid > alone
    for frames in (330, 30):
        use = [(small, i % 6 + 1) for i in range(frames)] + [(big, 3)]
        outs = [torch.empty((f.grid.nz, f.grid.nx), device="cuda") for _ in use]
        bt.set([p for p, _ in use], [rf] * len(use), [k for _, k in use], outs)
        say("%d frames: %d workgroups at once, %d of the large plan alone" % (frames, bt.info().grid, alone))
        assert (bt.info().grid > alone) == (frames == 330)
        bt.capture()
        for go in (bt.launch, bt.replay, bt.replay):
            for o in outs:
                o.fill_(float("nan"))
            go()
            torch.cuda.synchronize()
            for i, (o, u) in enumerate(zip(outs, use)):
                assert torch.equal(o, own[u]), (frames, go.__name__, i)
    bt.close()
    small.close()
    big.close()


@pytest.mark.parametrize("first,then", [(4, 40), (40, 4)])
def test_a_captured_launch_forms_later_lists(hd, first, then):
    """A launch captured into a graph of the caller's reads the list from device
    memory: after a set of more or fewer frames at the same orders, few enough to
    run as one kernel or enough for one per order, its replays form that list."""
    f = ph.config_frame(1)
    arr = ph.to_fp32(f.rf)
    rf = torch.from_numpy(arr).cuda()
    plan = hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=3, tiling=(16, 16, 1, 16))
    own = {k: plan.beamform(rf, k).clone() for k in (2, 3)}
    outs = [torch.empty((f.grid.nz, f.grid.nx), device="cuda") for _ in range(40)]
    bt = hd.Batch(40, 40 * plan.info().n_tiles, plan.info().lds_bytes)

    def put(n):
        bt.set([plan] * n, [rf] * n, [2 + i % 2 for i in range(n)], outs[:n])

    put(first)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        bt.launch()
    for n in (first, then, first):
        put(n)
        for go in (graph.replay, bt.launch, graph.replay):
            for o in outs:
                o.fill_(float("nan"))
            go()
            torch.cuda.synchronize()
            for i in range(n):
                assert torch.equal(outs[i], own[2 + i % 2]), (n, i)
    bt.close()
    plan.close()


def test_set_and_replay_in_turn_do_not_wait(hd):
    """Replays of lists that differ in length, order, LDS and kinds while the one
    before still waits for the GPU: none waits on the host, and each forms its own
    list; a list replayed again is fitted into the graph."""
    f = ph.config_frame(1)
    arr = ph.to_fp32(f.rf)
    rf = torch.from_numpy(arr).cuda()
    a, b = (hd.Plan(f.geometry, f.grid, arr.shape[1], "f32", max_order=4, tiling=(16, 16, 1, c)) for c in (16, 64))
    own = {(p, k): p.beamform(rf, k).clone() for p in (a, b) for k in (2, 4)}
    outs = [torch.empty((f.grid.nz, f.grid.nx), device="cuda") for _ in range(60)]
    bt = hd.Batch(60, 60 * a.info().n_tiles, b.info().lds_bytes)
    busy = torch.randn((8192, 8192), device="cuda")
    lists = [[(a, 2)] * 60, [(a, 2)] * 31, [(b, 2)] * 60, [(a, 4)] * 7, [(a, 2), (b, 4)] * 30]

    def put(use):
        bt.set([p for p, _ in use], [rf] * len(use), [k for _, k in use], outs[: len(use)])

    def check(use):
        torch.cuda.synchronize()
        for i, u in enumerate(use):
            assert torch.equal(outs[i], own[u]), i

    put(lists[0])
    bt.capture()
    bt.replay()
    for before, use in zip(lists, lists[1:]):
        say("%d frames after %d" % (len(use), len(before)))
        put(before)
        bt.replay()
        bt.replay()
        check(before)
        for o in outs:
            o.fill_(float("nan"))
        done = torch.cuda.Event()
        for _ in range(20):
            busy @ busy
        done.record()
        bt.replay()                     # `before`, unchanged: behind the products
        put(use)
        bt.replay()
        assert not done.query(), "waited for the GPU"
        check(use)
        for o in outs:
            o.fill_(float("nan"))
        bt.replay()
        check(use)
    bt.close()
    a.close()
    b.close()
