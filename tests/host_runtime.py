"""The built library on a HIP runtime without a device (``host_runtime.cpp``), for
tests of its host code: which launches a call makes, with which grids and
arguments, and what it does when an allocation fails.  Nothing is computed.

``run`` executes a function of a test module in a process of its own, whose only
HIP runtime is that one.
"""

import ctypes as C
import functools
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2407_10344_amd", "libvgicp.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@functools.lru_cache(maxsize=None)
def build(folder):
    out = os.path.join(folder, "host_runtime.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + ROCM + "/include",
                    os.path.join(HERE, "host_runtime.cpp"), "-o", out], check=True)
    return out


def run(folder, module, function):
    """``module.function(Host())`` in a process of its own."""
    if not os.path.exists(LIB):
        from paper_2407_10344_amd import build as b
        b.build()
    code = ("import sys; sys.path[:0] = [%r, %r]; import host_runtime, %s as m; m.%s(host_runtime.Host(%r)); print('done')"
            % (HERE, ROOT, module, function, build(str(folder))))
    # large allocations of the host are mapped, and unmapped when they are freed
    env = dict(os.environ, MALLOC_MMAP_THRESHOLD_="131072")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), (r.returncode, r.stdout[-3000:], r.stderr[-6000:])


class Options(C.Structure):
    _fields_ = [("precision", C.c_int32), ("surface_validation", C.c_int32), ("use_graph", C.c_int32),
                ("plain_per_factor", C.c_int32), ("block_threads", C.c_int32), ("tile_points", C.c_int32),
                ("blocks_per_cu", C.c_int32), ("lane_kahan", C.c_int32), ("tune_cache", C.c_char_p),
                ("tile_order", C.c_int32)]


class Host:
    OOM = -3

    def __init__(self, runtime):
        self.fake = C.CDLL(runtime, mode=C.RTLD_GLOBAL)
        self.lib = C.CDLL(LIB)
        f = self.fake
        for name in ("used", "peak", "failed", "bad_frees", "last_error", "launches", "allocations"):
            getattr(f, "fake_" + name).restype = C.c_int64
        f.fake_name.restype, f.fake_name.argtypes = C.c_char_p, [C.c_int64]
        f.fake_grid.restype, f.fake_grid.argtypes = C.c_uint32, [C.c_int64]
        f.fake_block.restype, f.fake_block.argtypes = C.c_uint32, [C.c_int64]
        f.fake_arg.restype, f.fake_arg.argtypes = C.c_uint64, [C.c_int64, C.c_int]
        f.fake_args.argtypes = [C.c_int64]
        f.fake_budget.argtypes = f.fake_fail_at.argtypes = [C.c_int64]
        f.fake_set.argtypes = [C.c_char_p, C.c_int64]
        f.fake_watch.argtypes = [C.c_char_p, C.c_int]
        self.lib.vg_last_error.restype = C.c_char_p
        self.ctx = self.make("vg_context_create", 0, None)

    def set(self, key, value):
        self.fake.fake_set(key.encode(), value)

    def watch(self, kernel, n_args):
        self.fake.fake_watch(kernel.encode(), n_args)

    def call(self, name, *args):
        conv = [C.c_int64(a) if isinstance(a, int) and not isinstance(a, bool) else a for a in args]
        return getattr(self.lib, name)(*conv)

    def check(self, name, *args):
        rc = self.call(name, *args)
        assert rc == 0, (name, rc, self.lib.vg_last_error())

    def make(self, name, *args):
        h = C.c_void_p()
        self.check(name, *args, C.byref(h))
        return h

    def launches(self, part=""):
        """(name, grid, block, recorded arguments) of the launches whose kernel's name holds ``part``."""
        f, out = self.fake, []
        for k in range(f.fake_launches()):
            name = f.fake_name(k).decode()
            if part in name:
                out.append((name, f.fake_grid(k), f.fake_block(k), [f.fake_arg(k, i) for i in range(f.fake_args(k))]))
        return out

    # a cloud's arrays are only handed to copies, which do nothing: no memory behind them, but point 0
    def source(self, n):
        a = (C.c_double * 16)()
        return self.make("vg_create_source", self.ctx, a, a, None, n)

    def map(self, n, resolutions=(0.5,)):
        a, r = (C.c_double * 16)(), (C.c_double * len(resolutions))(*resolutions)
        return self.make("vg_build_voxelmap", self.ctx, a, a, n, r, len(resolutions))

    def batch(self, sources, maps, **options):
        F = len(sources)
        o = Options(**options)
        src = (C.c_void_p * F)(*[s.value for s in sources])
        tgt = (C.c_void_p * F)(*[m.value for m in maps])
        return self.make("vg_create_factor_batch", self.ctx, F, src, tgt, None, C.byref(o))

    def info(self, batch):
        v = [C.c_int64(), C.c_int64()] + [C.c_int32() for _ in range(4)]
        self.check("vg_batch_info", batch, *[C.byref(x) for x in v])
        return dict(zip(("points", "tiles", "block", "tile", "grid", "order"), [x.value for x in v]))

    @staticmethod
    def poses(F):
        return (C.c_double * (12 * F))(*([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0] * F))
