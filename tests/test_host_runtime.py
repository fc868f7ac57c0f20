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
