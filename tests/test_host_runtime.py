"""Host code of the library on a runtime without a device (``host_runtime``): launch
geometry at sizes that no test allocates, and failing allocations."""

import ctypes as C

import pytest

import host_runtime


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("host_runtime")
    return lambda function: host_runtime.run(folder, "test_host_runtime", function)


def shape_survives_failed_tuning(h):
    """A tuner that runs out of memory leaves a batch that still runs: a schedule and
    rows of one shape, none of them null or released."""
    h.watch("k_tiles", 8)
    m, s = h.map(1000), h.source(20_000)
    for fail_at in range(6):
        b = h.batch([s] * 40, [m] * 40, tile_points=1024)
        chosen = (C.c_int32 * 4)()
        h.fake.fake_fail_at(fail_at)
        rc = h.call("vg_batch_tune", b, h.poses(40), 1, chosen)
        assert rc == (h.OOM if h.fake.fake_failed() else 0)
        h.fake.fake_fail_at(-1)
        h.fake.fake_reset()
        i = h.info(b)
        d = C.c_void_p(1 << 45)
        h.check("vg_linearize_async", b, d, d, None)
        (_, grid, block, (fac, units, u0, n_units, tc, poses, posef, partials)), = h.launches("k_tiles")
        assert units and partials and poses
        u0, n_units, tc = (x & 0xFFFFFFFF for x in (u0, n_units, tc))
        assert (grid, block, 64 * tc) == (i["grid"], i["block"], i["tile"]) and u0 == 0
        fresh = h.batch([s] * 40, [m] * 40, tile_points=i["tile"], block_threads=i["block"], tile_order=i["order"])
        assert h.info(fresh)["tiles"] == i["tiles"]
        h.check("vg_batch_destroy", fresh)
        h.check("vg_batch_destroy", b)
        assert h.fake.fake_bad_frees() == 0


def test_batch_survives_a_tuner_out_of_memory(run):
    run("shape_survives_failed_tuning")


def preprocessing_launches_fit_the_device(h):
    """Sizes around the powers of two at which 16 or 32 lanes a point, or the cell table's
    entries, reach 2^32 threads; beyond the cell table's reach the call is refused."""
    xyz, sensor = (C.c_double * 16)(), (C.c_double * 3)()
    h.watch("k_knnILi", 4)
    for m, k in ((1, 1), (1000, 10), ((1 << 27) + 77, 10), ((1 << 27) + 77, 17), ((1 << 28) + 77, 16),
                 ((1 << 28) + 77, 32), ((1 << 29) + 77, 1), (715_000_000, 1)):
        h.fake.fake_reset()
        h.set("downsampled", m)
        cloud = h.make("vg_preprocess", h.ctx, xyz, m, C.c_double(0.5), k, sensor)
        for name, grid, block, _ in h.launches():
            assert 0 < grid * block < 1 << 32, (name, grid, block)
        # the searches take every query once
        lanes = 16 if k <= 16 else 32
        done = 0
        for name, grid, block, args in h.launches("k_knnILi"):
            assert "k_knnILi%dE" % lanes in name
            assert args[3] == done
            done += grid * block // lanes
        assert m <= done < m + 256 // lanes
        h.check("vg_cloud_destroy", cloud)
    h.fake.fake_reset()
    h.set("downsampled", 720_000_000)
    out = C.c_void_p()
    assert h.call("vg_preprocess", h.ctx, xyz, 720_000_000, C.c_double(0.5), 1, sensor, C.byref(out)) == -5
    assert out.value is None and not h.launches("k_knn")
    assert h.fake.fake_bad_frees() == 0


def test_preprocessing_launches_at_the_largest_frames(run):
    run("preprocessing_launches_fit_the_device")


def launches_per_factor_stay_bounded(h):
    """2^20 + 3 factors (2^30 are accepted): no launch grows with the factors beyond 2^28
    threads, and the reductions take every factor once."""
    F = (1 << 20) + 3
    h.watch("k_reduce", 3)
    s, m = h.source(0), h.map(0)
    b = h.batch([s] * F, [m] * F)
    d = C.c_void_p(1 << 45)
    for name, args in (("vg_linearize_async", (d, d, None)), ("vg_evaluate_async", (d, d)),
                       ("vg_backward_async", (d, d, None, d, None, 0)), ("vg_lm_step_async", (d, d, d, d))):
        h.fake.fake_reset()
        h.check(name, b, *args)
        for kernel, grid, block, _ in h.launches():
            assert 0 < grid * block <= 1 << 28, (kernel, grid, block)
        done = 0
        for kernel, grid, block, (_, _, f0) in h.launches("k_reduce"):
            assert f0 & 0xFFFFFFFF == done % F
            done += grid
        assert done == (2 * F if name == "vg_lm_step_async" else F)


def test_launches_of_very_many_factors(run):
    run("launches_per_factor_stay_bounded")


def tuner_times_what_it_installs(h):
    """Every shape that the tuner times is launched with the workgroups of a batch created
    with that shape, and so is the shape that it leaves."""
    h.watch("k_tiles", 13)
    s, m = h.source(200_000), h.map(1000)
    expect = {}

    def launched():
        out = set()
        for _, grid, block, args in h.launches("k_tiles"):
            n_units, tc, interleave = (args[k] & 0xFFFFFFFF for k in (3, 4, 12))
            out.add((block, 64 * tc, 2 if interleave else 1, n_units, grid))
        return out

    for plain in (0, 1):
        F = 1 if plain else 50
        b = h.batch([s] * F, [m] * F, plain_per_factor=plain)
        chosen = (C.c_int32 * 4)()
        h.fake.fake_reset()
        h.check("vg_batch_tune", b, h.poses(F), 1, chosen)
        timed = launched()
        assert len({t[:3] for t in timed}) == (10 if plain else 48)
        for block, tile, order, n_units, grid in timed:
            key = (F, block, tile, order)
            if key not in expect:
                fresh = h.batch([s] * F, [m] * F, block_threads=block, tile_points=tile, tile_order=order)
                expect[key] = h.info(fresh)["grid"]
                h.check("vg_batch_destroy", fresh)
            assert grid == expect[key], (key, grid, expect[key])
        h.fake.fake_reset()
        d = C.c_void_p(1 << 45)
        h.check("vg_linearize_async", b, d, d, None)
        (block, tile, order, _, grid), = launched()
        assert [block, tile, order] == [chosen[0], chosen[1], chosen[3]] and grid == expect[(F, block, tile, order)]


def test_tuner_times_the_schedules_it_installs(run):
    run("tuner_times_what_it_installs")


def plain_factors_are_not_grouped(h):
    """The per-factor loop launches one factor at a time: as many workgroups as the factor has
    tiles, however many factors the batch has."""
    h.watch("k_tiles", 5)
    s, m = h.source(200_000), h.map(1000)
    F = 100
    b = h.batch([s] * F, [m] * F, plain_per_factor=1)
    h.fake.fake_reset()
    e, H, g = (C.c_double * F)(), (C.c_double * (36 * F))(), (C.c_double * (6 * F))()
    h.check("vg_linearize", b, h.poses(F), e, H, g, None)
    units = [args[3] & 0xFFFFFFFF for _, _, _, args in h.launches("k_tiles")]
    assert units == [-(-200_000 // h.info(b)["tile"])] * F
    # the same factors in one launch share prologues
    c = h.batch([s] * F, [m] * F)
    h.fake.fake_reset()
    h.check("vg_linearize", c, h.poses(F), e, H, g, None)
    (_, _, _, args), = h.launches("k_tiles")
    assert args[3] & 0xFFFFFFFF < sum(units)


def test_plain_factors_are_not_grouped(run):
    run("plain_factors_are_not_grouped")


def kept_memory_is_given_back(h):
    """Blocks and workspaces kept idle, of any context on the device, never make a call fail
    for want of memory; a call that does fail leaves no error behind in the runtime."""
    m, s = h.map(1000), h.source(30_000)
    b = h.batch([s] * 40, [m] * 40)
    d = C.c_void_p(1 << 45)
    F, iters = 40, 10_000
    ni, nj = (C.c_int64 * 2000)(*range(2000)), (C.c_int64 * 2000)(*range(1, 2001))
    keys, found = (C.c_int64 * (3 * 30_000))(), (C.c_int32 * 30_000)()
    out, acc, eh = (C.c_double * (12 * F))(), (C.c_int32 * (F * iters))(), (C.c_double * (F * iters))()
    chosen = (C.c_int32 * 4)()
    cloud_xyz, sensor = (C.c_double * 16)(), (C.c_double * 3)()
    other = h.make("vg_context_create", 0, None)
    calls = {
        "graph": lambda: h.call("vg_create_graph", h.ctx, 2001, 2000, ni, nj, C.byref(C.c_void_p())),
        "gradients": lambda: h.call("vg_backward_async", b, d, d, None, d, d, 1),
        "correspondences": lambda: h.call("vg_correspondences", b, h.poses(1), 3, keys, found),
        "histories": lambda: h.call("vg_lm_run", b, h.poses(F), iters, C.c_double(1e-4), out, acc, eh),
        "tuner": lambda: h.call("vg_batch_tune", b, h.poses(F), 1, chosen),
        "small source": lambda: h.call("vg_create_source", other, cloud_xyz, cloud_xyz, None, 100, C.byref(C.c_void_p())),
        "large source": lambda: h.call("vg_create_source", other, cloud_xyz, cloud_xyz, None, 900_000,
                                       C.byref(C.c_void_p())),
        "frame": lambda: h.call("vg_preprocess", other, cloud_xyz, 100_000, C.c_double(0.5), 10, sensor,
                                C.byref(C.c_void_p())),
    }
    for keeper in (h.ctx, h.make("vg_context_create", 0, None)):
        for name, call in calls.items():
            # a source of a million points leaves 160 MB of blocks and 90 MB of workspace
            src = h.make("vg_create_source", keeper, cloud_xyz, cloud_xyz, None, 1_000_000)
            before = h.fake.fake_used()
            h.check("vg_source_destroy", src)
            assert h.fake.fake_used() == before
            h.fake.fake_reset()
            h.fake.fake_budget(h.fake.fake_used() + 512)
            rc = call()
            assert rc == 0, (name, rc, h.lib.vg_last_error())
            assert h.fake.fake_last_error() == 0
            # nothing left to give back: the call fails, and leaves no error behind
            h.fake.fake_budget(0)
            assert h.call("vg_create_source", other, cloud_xyz, cloud_xyz, None, 50_000_000, C.byref(C.c_void_p())) == h.OOM
            assert h.call("vg_create_graph", h.ctx, 2001, 2000, ni, nj, C.byref(C.c_void_p())) == h.OOM
            assert h.fake.fake_last_error() == 0
            h.fake.fake_budget(-1)
    assert h.fake.fake_bad_frees() == 0


def test_kept_memory_never_fails_a_call(run):
    run("kept_memory_is_given_back")


def everything_is_freed(h):
    """A context gives back all that it kept."""
    base = h.fake.fake_used()
    for _ in range(2):
        h.ctx = h.make("vg_context_create", 0, None)
        m, s = h.map(100_000, (0.5, 1.0)), h.source(300_000)
        b = h.batch([s] * 40, [m] * 40)
        h.check("vg_batch_tune", b, h.poses(40), 1, None)
        h.check("vg_batch_destroy", b)
        for call in (("vg_source_destroy", s), ("vg_voxelmap_destroy", m)):
            h.check(*call)
        h.check("vg_context_destroy", h.ctx)
        assert h.fake.fake_used() == base and h.fake.fake_bad_frees() == 0


def test_contexts_give_back_what_they_kept(run):
    run("everything_is_freed")


def tuned_batches_hold_one_schedule(h):
    """A batch that was given another launch shape holds the rows of that shape only."""
    s, m = h.source(1_000_000), h.map(1000)

    def used():   # without what is kept idle: a failing call gives that back
        h.fake.fake_budget(0)
        a = (C.c_double * 16)()
        assert h.call("vg_create_source", h.ctx, a, a, None, 50_000_000, C.byref(C.c_void_p())) == h.OOM
        h.fake.fake_budget(-1)
        return h.fake.fake_used()

    for F, tile in ((1, 64), (40, 256), (40, 2048)):
        base = used()
        large = h.batch([s] * F, [m] * F, tile_points=16384)
        lean = used() - base
        h.check("vg_batch_destroy", large)
        b = h.batch([s] * F, [m] * F, tile_points=tile)
        chosen = (C.c_int32 * 4)()
        h.check("vg_batch_tune", b, h.poses(F), 1, chosen)
        # rows of 320 bytes a tile and less than 32 of tables, those of the first shape too
        tiles, first = (F * -(-1_000_000 // t) for t in (chosen[1], tile))
        assert used() - base <= lean + 1.125 * (tiles * 352 + 4096) + first * 32, (F, tile, chosen[1])
        h.check("vg_batch_destroy", b)
        assert used() == base


def test_tuned_batches_hold_one_schedule(run):
    run("tuned_batches_hold_one_schedule")


def maps_build_level_by_level_when_short_of_memory(h):
    """The levels of a map are built together, with the temporaries of all of them; where these
    do not fit, one after the other, with those of one."""
    n, res = 20_000_000, (0.25, 0.5, 1.0, 2.0)

    def peak(resolutions, budget=-1):
        h.check("vg_context_destroy", h.ctx)
        h.ctx = h.make("vg_context_create", 0, None)
        h.fake.fake_reset()
        base = h.fake.fake_used()
        h.fake.fake_budget(base + budget if budget >= 0 else -1)
        m = h.map(n, resolutions)
        assert h.lib.vg_last_error() == b""
        top = h.fake.fake_peak() - base
        h.fake.fake_budget(-1)
        for level in range(len(resolutions)):
            v, cap = C.c_int64(), C.c_int64()
            h.check("vg_voxelmap_info", m, level, C.byref(v), C.byref(cap))
            assert (v.value, cap.value) == (100, 64)
        assert len(h.launches("k_map_stats")) == (1 if budget < 0 else len(resolutions))
        h.check("vg_voxelmap_destroy", m)
        return top

    one, together = peak(res[:1]), peak(res)
    assert together > 2 * one
    for budget in (one + 100_000, (one + together) // 2):
        assert peak(res, budget) <= budget
    h.fake.fake_budget(h.fake.fake_used() + one // 2)
    out = C.c_void_p()
    a, r = (C.c_double * 16)(), (C.c_double * 4)(*res)
    assert h.call("vg_build_voxelmap", h.ctx, a, a, n, r, 4, C.byref(out)) == h.OOM
    assert h.fake.fake_bad_frees() == 0


def test_maps_build_level_by_level_when_short_of_memory(run):
    run("maps_build_level_by_level_when_short_of_memory")


def repeated_calls_allocate_nothing(h):
    """Temporaries come from the workspace and large objects from kept blocks once a call of
    that size has been made."""
    xyz, sensor, res = (C.c_double * 16)(), (C.c_double * 3)(), (C.c_double * 2)(0.5, 1.0)
    h.set("voxels", 20_000)
    h.set("blocks", 5000)

    def frame():
        h.set("downsampled", 40_000)
        cloud = h.make("vg_preprocess", h.ctx, xyz, 100_000, C.c_double(0.5), 10, sensor)
        objects = [("vg_source_destroy", h.make("vg_create_source_from_cloud", h.ctx, cloud)),
                   ("vg_voxelmap_destroy", h.make("vg_build_voxelmap_from_cloud", h.ctx, cloud, res, 2)),
                   ("vg_voxelmap_destroy", h.map(150_000, (0.25, 0.5, 1.0))), ("vg_source_destroy", h.source(150_000)),
                   ("vg_cloud_destroy", cloud)]
        for name, handle in objects:
            h.check(name, handle)

    for call in range(4):
        h.fake.fake_reset()
        frame()
        assert call == 0 or h.fake.fake_allocations() == 0, (call, h.fake.fake_allocations())


def test_repeated_calls_allocate_nothing(run):
    run("repeated_calls_allocate_nothing")


def waves_follow_the_blocks_of_a_graph(h):
    """A graph of many blocks for the length of its lists is assembled by one wave a block (most
    blocks have one contribution), another by four."""
    d = C.c_void_p(1 << 45)
    path = [(i, i + 1) for i in range(7999)]            # 24,000 blocks
    for N, edges, waves in ((100, [(0, i) for i in range(1, 100)], 4), (8000, path, 1),
                            (8000, path + [(0, 9)] * 36, 1), (8000, path + [(0, 9)] * 40, 4)):
        F = len(edges)
        ni, nj = (C.c_int64 * F)(*[e[0] for e in edges]), (C.c_int64 * F)(*[e[1] for e in edges])
        g = h.make("vg_create_graph", h.ctx, N, F, ni, nj)
        blocks = C.c_int64()
        h.check("vg_graph_structure", g, C.byref(blocks), None, None)
        h.fake.fake_reset()
        h.check("vg_graph_assemble_async", g, d, d, d, d)
        (_, grid, block, _), = h.launches("k_graph_assemble")
        assert (grid, block) == (blocks.value, 64 * waves), (N, F, grid, block)
        h.check("vg_graph_destroy", g)


def test_waves_follow_the_blocks_of_a_graph(run):
    run("waves_follow_the_blocks_of_a_graph")


def poses_alone_take_a_thread_each(h):
    """Retractions without their Jacobians: a thread per factor; with them a wave."""
    d = C.c_void_p(1 << 45)
    for F in (1, 64, 65, 1_000_000):
        for jr, threads in ((None, -(-F // 64) * 64), (d, 64 * F)):
            h.fake.fake_reset()
            h.check("vg_se3_retract_async", h.ctx, F, d, d, d, jr)
            (_, grid, block, _), = h.launches("k_se3")
            assert grid * block == threads


def test_poses_alone_take_a_thread_each(run):
    run("poses_alone_take_a_thread_each")


def small_levels_are_ordered_on_the_host(h):
    """Exporting a level launches nothing up to 16,384 voxels."""
    for voxels, launches in ((1, 0), (16_384, 0), (16_385, 2)):
        h.set("voxels", voxels)
        m = h.map(20_000)
        h.fake.fake_reset()
        n = C.c_int64(voxels)
        k, f, c = (C.c_int64 * (3 * voxels))(), (C.c_double * (6 * voxels))(), (C.c_int64 * voxels)()
        h.check("vg_voxelmap_export", m, 0, C.byref(n), k, f, f, c)
        assert n.value == voxels and min(len(h.launches()), 2) == launches
        h.check("vg_voxelmap_destroy", m)


def test_small_levels_are_ordered_on_the_host(run):
    run("small_levels_are_ordered_on_the_host")


def host_memory_runs_out(h):
    """Calls that run out of host memory return VG_ERR_OOM, hold nothing afterwards and leave
    their handles usable; no exception leaves the library."""
    import resource

    s, m = h.source(1000), h.map(1000)
    F, n = 60_000, 60_000
    src, tgt = (C.c_void_p * F)(*[s.value] * F), (C.c_void_p * F)(*[m.value] * F)
    o = host_runtime.Options()
    nodes = [(C.c_int64 * n)(*range(k, n + k)) for k in (0, 1)]
    keep = h.batch([s] * 4000, [s_ for s_ in [m] * 4000], tile_points=64)
    poses = h.poses(4000)
    iters = 200
    out, acc, eh = (C.c_double * (12 * 4000))(), (C.c_int32 * (iters * 4000))(), (C.c_double * (iters * 4000))()
    h.set("voxels", 400_000)
    big = h.map(600_000)
    voxels = C.c_int64(400_000)
    rows = [(C.c_int64 * (3 * 400_000))(), (C.c_double * (3 * 400_000))(), (C.c_double * (6 * 400_000))(),
            (C.c_int64 * 400_000)()]
    made = C.c_void_p()
    # (in this order: the small pieces of a graph's lists stay with the host's allocator)
    calls = {"lm": ("vg_lm_run", keep, poses, iters, C.c_double(1e-4), out, acc, eh),
             "tuner": ("vg_batch_tune", keep, poses, 1, None),
             "export": ("vg_voxelmap_export", big, 0, C.byref(voxels), *rows),
             "batch": ("vg_create_factor_batch", h.ctx, F, src, tgt, None, C.byref(o), C.byref(made)),
             "graph": ("vg_create_graph", h.ctx, n + 1, n, *nodes, C.byref(made))}
    undo = {"batch": "vg_batch_destroy", "graph": "vg_graph_destroy"}
    soft, hard = resource.getrlimit(resource.RLIMIT_AS)
    refused = dict.fromkeys(calls, 0)
    for name, call in calls.items():
        for _ in range(2):   # shapes and kept blocks as after a call
            assert h.call(*call) == 0
            if name in undo:
                h.check(undo[name], made)
        for step in range(24):
            base, shape = h.fake.fake_used(), h.info(keep)
            with open("/proc/self/statm") as f:
                now = int(f.read().split()[0]) * 4096
            resource.setrlimit(resource.RLIMIT_AS, (now + (step * step << 18), hard))
            rc = h.call(*call)
            resource.setrlimit(resource.RLIMIT_AS, (soft, hard))
            assert rc in (0, h.OOM), (name, step, rc)
            if rc == 0 and name in undo:
                h.check(undo[name], made)
            if rc != 0:
                refused[name] += 1
                assert h.lib.vg_last_error()
            if name != "tuner":
                assert h.fake.fake_used() == base, (name, step, base, h.fake.fake_used())
            d = C.c_void_p(1 << 45)
            h.check("vg_linearize_async", keep, d, d, None)
            assert h.info(keep)["tile"] == shape["tile"] or name == "tuner"
    assert all(refused.values()), refused
    assert h.fake.fake_bad_frees() == 0


def test_host_memory_running_out(run):
    run("host_memory_runs_out")
