"""The library's host code without a GPU: reads, and the launch that a problem statement
leaves to the library. Each test runs in a process of its own, where stand-ins for the HIP
runtime calls (aux/hip_host_shim.cpp) are loaded before the library."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
import numpy as np
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2309_10292_amd import gs
L = gs.load()
DP = ctypes.POINTER(ctypes.c_double)

def aligned(nbytes):
    raw = np.zeros(nbytes + 256, np.uint8)
    o = -raw.ctypes.data % 256
    return raw[o:o + nbytes]

class HostSim:
    "A simulation over host memory (no steps)."
    def __init__(self, nx, ny, nz, buffers=None, **kw):
        self.p = gs.make_params(nx, ny, nz, init="none", **kw)
        self.fields = buffers or [aligned(256) for _ in range(4)]
        self.ws = aligned(256)
        self.h = ctypes.c_void_p()
        gs.check(L.gs_init(ctypes.byref(self.p), *[f.ctypes.data for f in self.fields], self.ws.ctypes.data, None,
                           ctypes.byref(self.h)))
    def config(self):
        c = [ctypes.c_int32() for _ in range(3)]
        gs.check(L.gs_get_config(self.h, *[ctypes.byref(x) for x in c]))
        return tuple(x.value for x in c)
    def read(self, u, v):
        gs.check(L.gs_read(self.h, u.ctypes.data_as(DP), v.ctypes.data_as(DP)))
    def close(self):
        gs.check(L.gs_destroy(self.h))

class HostBatch:
    "A batch of cubes (no steps, and no fields: the library does not touch them)."
    def __init__(self, sides, **kw):
        p, n = gs.make_params(8, 8, 8, init="none", **kw), len(sides)
        d, r = (ctypes.c_int32 * n)(*sides), (ctypes.c_double * n)(*[0.03] * n)
        nbytes = int(L.gs_batch_workspace_bytes(n, d, d, d))
        self.ws, self.h = aligned(nbytes), ctypes.c_void_p()
        gs.check(L.gs_batch_init(ctypes.byref(p), n, d, d, d, r, r, 1 << 40, 1 << 60, self.ws.ctypes.data, nbytes, None,
                                 ctypes.byref(self.h)))
    def config(self, i=0):
        c = [ctypes.c_int32() for _ in range(3)]
        gs.check(L.gs_batch_get_config(self.h, i, *[ctypes.byref(x) for x in c]))
        return tuple(x.value for x in c)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("shim") / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "aux", "hip_host_shim.cpp"), "-o", so], check=True)

    def go(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), so], cwd=ROOT, capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return go


@pytest.mark.parametrize("flush", [0, 1])
@pytest.mark.parametrize("times", [1, 8])
def test_half_precision_reads_in_either_denormal_mode(run, times, flush):
    """All 65536 FP16 patterns, in a plain copy and through the ring, whatever the calling
    thread does with denormals: every half is a normal FP32 number."""
    run(f"""
    bits = np.tile(np.arange(65536, dtype=np.uint16), {times})
    want = bits.view(np.float16).astype(np.float64)
    fields = [aligned(bits.nbytes) for _ in range(4)]
    fields[0][:] = bits.view(np.uint8)
    fields[1][:] = bits[::-1].copy().view(np.uint8)
    s = HostSim(64, 32, 32 * {times}, fields, storage="f16")
    u, v = np.empty(bits.size), np.empty(bits.size)
    shim.shim_flush_denormals({flush})
    s.read(u, v)
    shim.shim_flush_denormals(0)
    for got, w in ((u, want), (v, want[::-1])):
        assert np.array_equal(np.isnan(got), np.isnan(w))
        ok = ~np.isnan(w)
        assert np.array_equal(got[ok].view(np.int64), w[ok].view(np.int64))
    """)


def test_library_tile_fuses_the_callers_steps(run):
    """tile = 0 with tblock set: the library's tile runs that depth in every size class and storage type."""
    run("""
    for shape in [(32, 32, 32), (64, 64, 64), (88, 88, 88), (16, 600, 600), (168, 168, 168), (512, 512, 512)]:
        for storage in ("f64", "f32", "bf16", "f16", "bf16c"):
            for noise in (0.0, 1e-3):
                for tblock in (0, 1, 2, 3, 4):
                    tile, depth, _ = HostSim(*shape, storage=storage, noise=noise, tblock=tblock).config()
                    assert (depth == tblock or not tblock) and 1 <= depth <= gs.max_tblock(tile, storage), \
                        (shape, storage, noise, tblock, tile, depth)
    """)


def test_callers_z_chunk_is_used(run):
    """tile = 0 with zchunk set: a kernel that streams along z, with that chunk, also on the grids that the block
    kernel takes otherwise (tiles 10 to 12, which have planes of their own)."""
    run("""
    for shape in [(16, 20, 24), (32, 32, 32), (48, 48, 48), (64, 64, 64), (80, 80, 80), (16, 600, 600), (192, 192, 192)]:
        for storage in ("f64", "f32", "bf16c"):
            for tblock in (0, 1, 4):
                tile, depth, zchunk = HostSim(*shape, storage=storage, tblock=tblock, zchunk=9).config()
                assert not 10 <= tile <= 12 and zchunk == 9, (shape, storage, tblock, tile, zchunk)
                assert 1 <= depth <= gs.max_tblock(tile, storage)
    assert 10 <= HostSim(32, 32, 32).config()[0] <= 12
    """)


@pytest.mark.parametrize("tile, tblock", [(0, 1), (0, 4), (6, 4), (7, 3), (8, 0)])
def test_batch_chunk_for_the_callers_depth(run, tile, tblock):
    """A batch with tile or tblock set and no zchunk: the chunk of least estimated makespan at that depth (FP64, one
    workgroup of more than 256 lanes per CU)."""
    run(f"""
    shim.shim_device(256, 512)
    for sides in ([72, 88, 96, 96, 104, 112, 120, 120], [24] * 24, [128] * 32, [64, 192] * 8):
        t, T, zchunk = HostBatch(sides, tile={tile}, tblock={tblock}).config()
        assert t == ({tile} or 6) and T == ({tblock} or 1), (t, T)
        tx, ty = gs.tile_info(t, "f64", T)
        def cost(zc):
            n = planes = longest = 0
            for L in sides:
                cols = -(-L // tx) * -(-L // ty)
                if t == 6 and T <= 3: # narrow tiles where they are 10 % fewer
                    c = cols
                    for wx, wy in ((32, 51 - 2 * T), (48, 36 - 2 * T)):
                        k = 1.1 * -(-L // wx) * -(-L // wy)
                        if k <= c: c, cols = k, -(-L // wx) * -(-L // wy)
                n += cols * -(-L // zc)
                planes += cols * (L + 2 * T * -(-L // zc))
                longest = max(longest, min(zc, L) + 2 * T)
            return longest if n <= 256 else planes / 256 + 0.5 * longest
        # configurations report chunks cut to the grid
        want = min((8, 16, 32, 64), key=cost)
        assert zchunk == min(want, sides[0]), (sides, zchunk, want)
    """)


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
def test_reads_into_one_array(run, storage):
    """u and v read into the same or overlapping arrays: u first, then v, at every size."""
    run(f"""
    ny, nz = 64, 128
    n = 64 * ny * nz
    dtype = dict(f64=np.float64, f32=np.float32, bf16=np.uint16)["{storage}"]
    bits = [(np.arange(n) % 251 + 251 * f).astype(np.float32) for f in range(2)]
    want = [(b.view(np.uint32) >> 16 << 16).view(np.float32).astype(np.float64) if "{storage}" == "bf16" else b.astype(np.float64) for b in bits]
    fields = [aligned(n * dtype().itemsize) for _ in range(4)]
    for f in range(2):
        x = (bits[f].view(np.uint32) >> 16).astype(np.uint16) if "{storage}" == "bf16" else bits[f].astype(dtype)
        fields[f][:] = x.view(np.uint8)
    s = HostSim(64, ny, nz, fields, storage="{storage}")
    for shift in (0, 100, n // 2):
        for first in (0, 1): # which of the two arrays begins earlier
            for _ in range(20):
                got = np.full(n + shift, -1.0)
                at = [shift, 0] if first else [0, shift]
                s.read(got[at[0]:], got[at[1]:])
                model = np.full(n + shift, -1.0)
                for f in range(2):
                    model[at[f]:at[f] + n] = want[f]
                assert np.array_equal(got, model), (shift, first, np.flatnonzero(got != model)[:4])
    """)


@pytest.mark.parametrize("known", [0, 1])
def test_fp64_reads_into_memory_of_the_runtime(run, known):
    """FP64 goes to memory that the runtime knows (pinned, managed, a device's) in plain copies, whichever of the two
    arrays that is."""
    run(f"""
    n = 64 * 64 * 128
    fields = [aligned(8 * n) for _ in range(4)]
    for f in range(2):
        fields[f].view(np.float64)[:] = np.arange(n) + f
    s = HostSim(64, 64, 128, fields)
    out = [np.empty(n), np.empty(n)]
    shim.shim_known(ctypes.c_void_p(out[{known}].ctypes.data))
    s.read(*out)
    assert shim.shim_pinned() == 0 and all(np.array_equal(out[f], np.arange(n) + f) for f in range(2))
    shim.shim_known(None)
    s.read(*out)
    assert shim.shim_pinned() == 1 and all(np.array_equal(out[f], np.arange(n) + f) for f in range(2))
    """)


def test_tune_on_grids_of_more_blocks_than_a_launch_takes(run):
    """The autotuner passes over the candidates whose launch would have 2^32 threads or more (the block kernel's on
    a grid of 1.3 G cells) and measures the others."""
    run("""
    s = HostSim(2048, 1024, 640, storage="bf16")
    table, n = (gs.gs_tune_entry * 256)(), ctypes.c_int32()
    gs.check(L.gs_tune(s.h, 1, ctypes.cast(table, ctypes.c_void_p), 256, ctypes.byref(n)))
    tried = {(e.tile, e.tblock) for e in table[:n.value]}
    every = {(tile, T) for tile in range(1, 15) for T in range(1, gs.max_tblock(tile, "bf16") + 1)}
    # 10.5 M blocks of 8 x 4 x 4 cells in workgroups of 64, 192, 256 and, at four steps, 448 lanes
    assert every - tried == {(10, 4)}, every - tried
    """)


def test_pinned_memory_of_many_handles_is_bounded(run):
    """Forty simulations that have each read a large field hold 16 rings, and none when they are closed; all of them
    read what they should, again and again."""
    run("""
    n = 64 * 64 * 128
    def make(i):
        fields = [aligned(4 * n) for _ in range(2)] * 2
        for f in range(2):
            fields[f].view(np.float32)[:] = np.arange(n) % 1000 + i + f
        return HostSim(64, 64, 128, fields[:2] + [aligned(256), aligned(256)], storage="f32")
    sims, u, v = [make(i) for i in range(40)], np.empty(n), np.empty(n)
    for turn in range(2):
        for i, s in enumerate(sims):
            s.read(u, v)
            assert np.array_equal(u, np.arange(n) % 1000 + i) and np.array_equal(v, u + 1)
            assert shim.shim_pinned() <= 16 and shim.shim_events() == 4 * shim.shim_pinned()
    assert shim.shim_pinned() == 16
    sims[3].close()
    sims[30].read(u, v)
    assert shim.shim_pinned() == 16 # the place goes to the next that reads
    for i, s in enumerate(sims):
        if i != 3: s.close()
    assert shim.shim_pinned() == 0 and shim.shim_events() == 0
    """)


def test_launches_fit_the_devices_compute_units(run):
    """A device with an eighth of the compute units takes, for an eighth of the work, the launch that the whole one
    takes for all of it: single grids (192 cells of x are whole tiles of every width), batches and the surrogate."""
    run("""
    got = []
    for cus, scale in ((256, 8), (32, 1)):
        shim.shim_device(cus, 1024)
        c = []
        for storage in ("f64", "f32", "bf16"):
            for noise in (0.0, 1e-3):
                for ny, nz in ((20, 20), (10, 61), (40, 40), (55, 90), (120, 110), (200, 190)):
                    c.append(HostSim(192 * scale, ny, nz, storage=storage, noise=noise).config())
                for sides in ([24, 40], [56, 64, 72], [96, 128, 192], [160]):
                    c.append(HostBatch(sides * scale, storage=storage, noise=noise).config())
        got.append(c)
    differ = [(a, b) for a, b in zip(*got) if a != b]
    assert not differ, (len(differ), len(got[0]), differ[:5])
    """)


def test_surrogate_launches_fit_the_devices_compute_units(run):
    """The same for the surrogate's kernels: the workgroups of a prediction of eight samples are eight times those of
    one on an eighth of the compute units."""
    run("""
    nx, ny, nz = 32, 40, 30
    n = nx * ny * nz
    grids = []
    for cus, batch in ((256, 8), (32, 1)):
        shim.shim_device(cus, 1024)
        need = int(L.gs_surrogate_workspace_bytes(nx, ny, nz, batch))
        ws, p, h = aligned(need), np.zeros(60578, np.float32), ctypes.c_void_p()
        gs.check(L.gs_surrogate_init(nx, ny, nz, batch, p.ctypes.data, ws.ctypes.data, need, None, ctypes.byref(h)))
        x, fk = [aligned(4 * n * batch) for _ in range(4)], np.full(batch, 0.05)
        first = shim.shim_launches()
        gs.check(L.gs_surrogate_predict(h, batch, 1, x[0].ctypes.data, x[1].ctypes.data, fk.ctypes.data, fk.ctypes.data,
                                        x[2].ctypes.data, x[3].ctypes.data))
        grids.append([shim.shim_grid(i) for i in range(first, shim.shim_launches())])
    # the input's packing, and four layers
    assert len(grids[1]) == 5 and grids[0] == [8 * g for g in grids[1]], grids
    """)
