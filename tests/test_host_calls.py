"""CPU checks of what the library's host code asks of the device: its sources
(csrc/*.cpp) are built with the host compiler against a device that computes
nothing and records every launch (tests/host_calls/recording_device.cpp), with
a limit on its memory and allocations that fail on request."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

import synth
from paper_2608_07307_amd import _lib as L
from paper_2608_07307_amd import _mesh_arrays, params

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_07307_amd", "csrc")
DEVICE = os.path.join(ROOT, "tests", "host_calls", "recording_device.cpp")
HIP_INC = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP_INC),
                                reason="needs g++ and the HIP headers")

KINDS = {1: "upload", 2: "articulate", 3: "window", 4: "primary", 5: "trace", 6: "fans", 7: "adjoint", 8: "reduce"}


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("host_calls")
    jobs, objs = [], []
    for s in [os.path.join(CSRC, f) for f in ("capi.cpp", "scene.cpp", "nplate.cpp", "propagate.cpp", "spad.cpp")] + [DEVICE]:
        o = tmp / (os.path.basename(s) + ".o")
        objs.append(str(o))
        jobs.append(subprocess.Popen(["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INC,
                                      "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", s, "-o", str(o)]))
    assert [j.wait() for j in jobs] == [0] * len(jobs)
    out = tmp / "libcalls.so"
    # (its own HIP calls, not those of a runtime that the process has loaded)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *objs, "-o", str(out)], check=True)
    return out


class Device:
    """One fresh copy of the library and its recording device."""

    def __init__(self, path):
        self.lib = lib = C.CDLL(str(path))
        lib.srp_last_error.restype = C.c_char_p
        lib.dev_used.restype = lib.dev_faults.restype = lib.dev_log.restype = C.c_int64
        lib.dev_limit.argtypes = [C.c_int64]
        lib.dev_log.argtypes = [C.c_void_p, C.c_int64]
        V, I32, I64 = C.c_void_p, C.c_int32, C.c_int64
        lib.srp_build_scene.argtypes = [V, I64, V, I64, V, V, V, I32, V, I32, C.POINTER(V)]
        lib.srp_eval.argtypes = [V, V, V, V, V]
        lib.srp_eval_batch.argtypes = lib.srp_eval_batch_noalloc.argtypes = [V, I64, V, V]
        lib.srp_eval_grad_batch.argtypes = [V, I64, V, V, I64, V]
        lib.srp_eval_grad.argtypes = [V] * 7
        lib.srp_plan_create.argtypes = [V, I64, I32, V, V, I64, C.POINTER(V)]
        lib.srp_plan_update.argtypes = [V, V, I64]
        lib.srp_set_schedule.argtypes = [I32, I32]

    def error(self):
        return self.lib.srp_last_error().decode()

    def scene(self, mesh):
        verts, tris, tm, tn, mats, nodes = _mesh_arrays(mesh)
        h = C.c_void_p()
        rc = self.lib.srp_build_scene(L.ptr(verts), len(verts), L.ptr(tris), len(tris), L.ptr(tm), L.ptr(tn), mats,
                                      len(mesh.mats), nodes, len(nodes), C.byref(h))
        assert rc == 0, self.error()
        return h

    def items(self, entries):
        """entries: (scene, params[, angles]) per item; angles are kept alive with the array."""
        arr = (L.srp_batch_item * len(entries))()
        arr.keep = []
        for k, (sc, p, *ang) in enumerate(entries):
            arr[k].scene, arr[k].angles, arr[k].p = sc, None, p
            if ang:
                a = np.ascontiguousarray(ang[0], np.float64)
                arr.keep.append(a)
                arr[k].angles = a.ctypes.data
        return arr

    def log(self):
        n = self.lib.dev_log(None, 0)
        a = np.zeros((n, 8), np.int64)
        self.lib.dev_log(a.ctypes.data, n)
        self.lib.dev_clear()
        return [(KINDS[r[0]], *r[1:].tolist()) for r in a]

    def batch(self, entries, grad=False, noalloc=False):
        arr, n = self.items(entries), len(entries)
        self.lib.dev_clear()
        if grad:
            return self.lib.srp_eval_grad_batch(arr, n, 1 << 20, 1 << 20, 1 << 20, None)
        return (self.lib.srp_eval_batch_noalloc if noalloc else self.lib.srp_eval_batch)(arr, n, 1 << 20, None)


@pytest.fixture
def devices(so, tmp_path):
    def fresh():
        fresh.n += 1
        p = tmp_path / f"lib{fresh.n}.so"
        shutil.copy(so, p)   # (a library of another path is loaded, and starts, anew)
        return Device(p)
    fresh.n = 0
    return fresh


@pytest.fixture
def dev(devices):
    return devices()


SUN = (0.3, -0.5, 0.8)


def test_a_failed_result_allocation_does_not_launch_without_a_result(dev):
    """A scene's first evaluation allocates its result; when that fails, the next
    one must not launch with the half that succeeded."""
    sc = dev.scene(synth.box_wing())
    p, r = params(SUN, 64, 1), L.srp_result()
    dev.lib.dev_fail_host(1)
    assert dev.lib.srp_eval(sc, C.byref(p), C.byref(r), None, None) == L.SRP_ERR_OOM
    assert dev.lib.srp_eval(sc, C.byref(p), C.byref(r), None, None) == 0, dev.error()
    assert dev.lib.dev_faults() == 0 and dev.log()[-1][0] == "reduce"


def _grid_mesh(n_tris):
    """A plate of at least n_tris triangles."""
    k = int(np.ceil(np.sqrt(n_tris / 2)))
    return synth.plate((-1, -1, 0), (2, 0, 0), (0, 2, 0), nu=k, nv=k)


def test_large_diffuse_batches_of_expensive_scenes_are_taken(dev):
    """130 evaluations at 8192^2 with 16 diffuse rays hold 2.2e9 fan passes, more
    than a unit list can number: they run as sub-batches, as any batch beyond
    the workspace cap, and the choice between fans in the trace kernel and a
    list must not refuse them.  A captured plan of that many is not split, and
    traces its fans without a list."""
    sc = dev.scene(_grid_mesh(40000))
    entries = [(sc, params(SUN, 8192, 2, diffuse=16))] * 130
    assert 130 * 1024 * 1024 * 2 * 8 > 2 ** 31
    assert dev.batch(entries) == 0, dev.error()
    log = dev.log()
    assert sum(r[1] for r in log if r[0] == "reduce") == 130
    assert all(r[4] for r in log if r[0] == "trace")       # (sub-batches keep their lists)
    h = C.c_void_p()
    arr = dev.items(entries)
    assert dev.lib.srp_plan_create(arr, 130, 0, 1 << 20, None, 0, C.byref(h)) == 0, dev.error()
    trace = [r for r in dev.log() if r[0] == "trace"]
    assert len(trace) == 1 and trace[0][3] == 1 and trace[0][4] == 0


@pytest.mark.parametrize("schedule", [(0, 0), (1, 4), (5, 2)])
def test_large_gradient_batches_are_taken_at_any_schedule(dev, schedule):
    """8,200 evaluations at 8192^2 hold 8.6e9 patches.  A gradient batch's trace is
    handed out in the schedule's chunks, whose counters are 32-bit; its size
    alone, and patches per chunk set for forward batches, must not refuse it."""
    sc = dev.scene(synth.box_wing())
    dev.lib.srp_set_schedule(*schedule)
    assert dev.batch([(sc, params(SUN, 8192, 0))] * 8200, grad=True) == 0, dev.error()
    assert sum(r[1] for r in dev.log() if r[0] == "reduce") == 8200


def _tiles(n, px):
    return (-(-(16 * -(-n // 16)) // px)) ** 2


@pytest.mark.parametrize("small", [0, 1, 500, 3000])
def test_launches_are_numbered_through_uneven_batches(dev, small):
    """One fine image beside many coarse ones: the rasteriser's and the adjoint's
    blocks are those of the images themselves, not the largest one's for every
    evaluation, and every block finds its own evaluation."""
    fine, coarse = dev.scene(_grid_mesh(2000)), dev.scene(synth.box_wing())
    entries = [(coarse, params(SUN, 64, 1))] * small
    entries.insert(small // 3, (fine, params(SUN, 2048, 1)))
    if small > 1:   # another rasterised size behind the others
        entries.append((fine, params(SUN, 300, 1)))
    assert dev.batch(entries, grad=True) == 0, dev.error()
    log = dev.log()
    primary = [r for r in log if r[0] == "primary"]
    adjoint = [r for r in log if r[0] == "adjoint"]
    px = primary[0][3]
    with_vis = [e for e in entries if e[0] is fine]
    assert primary[0][2] == len(with_vis) and primary[0][4] == sum(_tiles(p.n, px) for _, p in with_vis)
    patches = [4 * (-(-p.n // 16)) ** 2 for _, p in entries]
    assert adjoint[0][2] <= sum(-(-k // 8) for k in patches) and dev.lib.dev_faults() == 0


def _patches(n):
    return 4 * (-(-n // 16)) ** 2


@pytest.mark.parametrize("plan", [False, True])
@pytest.mark.parametrize("bounces,ppc", [(0, 1), (2, 5), (4, 64)])
def test_gradients_without_room_for_their_chains(devices, plan, bounces, ppc):
    """A gradient batch whose hit chains do not fit the device's free memory runs
    them a window after the other, eager and captured: evaluations are cut at gradient
    groups (of 8 to 64 patches here), every group is swept once, from the chains of its
    own patches, and no chain lies outside the workspace."""
    many = synth.greebled_spacecraft(seed=3, bus_n=8, n_greebles=20, seg_nx=3, seg_ny=4)
    sizes = [(many, 2000), (synth.box_wing(), 33), (many, 1000), (synth.box_wing(), 700), (many, 100), (many, 1)]
    chains = sum(256 * (bounces + 1) * _patches(n) for _, n in sizes)
    hits = sum(520 * _patches(n) for m, n in sizes if m is many and n > 100)

    def run(limit):
        dev = devices()
        scenes = {id(m): dev.scene(m) for m, _ in sizes}
        entries = [(scenes[id(m)], params(SUN, n, bounces)) for m, n in sizes]
        dev.lib.srp_set_schedule(ppc, 4)
        dev.lib.dev_limit(limit)
        before = dev.lib.dev_used()
        if plan:
            arr, h = dev.items(entries), C.c_void_p()
            assert dev.lib.srp_plan_create(arr, len(arr), L.SRP_PLAN_GRAD, 1 << 20, 1 << 20, 1 << 20, C.byref(h)) == 0, \
                dev.error()
            assert dev.lib.srp_plan_update(h, arr, len(arr)) == 0, dev.error()
        else:
            assert dev.batch(entries, grad=True) == 0, dev.error()
        assert dev.lib.dev_faults() == 0
        return dev.lib.dev_used() - before, sum(r[0] == "adjoint" for r in dev.log())

    need, sweeps = run(-1)
    assert sweeps == 1
    need, sweeps = run(need - chains - hits + (6 << 20))
    assert sweeps >= chains // (4 << 20) > 1


def test_large_captured_gradient_batches_hold_a_part_of_their_chains(devices):
    """A captured batch is not split at the workspace cap: beyond it the rasterised hits
    are left out, and at most 1 GiB of chains is held at a time."""
    dev = devices()
    sc = dev.scene(synth.icosphere(subdiv=2))
    entries = [(sc, params(SUN, 2048, 4))] * 150
    arr, h = dev.items(entries), C.c_void_p()
    before = dev.lib.dev_used()
    assert dev.lib.srp_plan_create(arr, len(arr), L.SRP_PLAN_GRAD, 1 << 20, 1 << 20, 1 << 20, C.byref(h)) == 0, dev.error()
    log = dev.log()
    chains = 150 * 65536 * 256 * 5
    assert sum(r[0] == "adjoint" for r in log) == -(-chains // (1 << 30)) and dev.lib.dev_faults() == 0
    assert sum(r[1] for r in log if r[0] == "trace") == 150 + -(-chains // (1 << 30)) - 1   # (cut where a window ends)
    assert dev.lib.dev_used() - before < 4 << 30


@pytest.mark.parametrize("sizes,bounces,diffuse", [((112, 688), 3, 19), ((368, 592), 3, 20), ((400, 480), 3, 37),
                                                   ((144, 608), 3, 38)])
def test_the_fixed_workspace_holds_what_patch_counted_range_sums_left(dev, sizes, bounces, diffuse):
    """Diffuse batches within a few hundred bytes of the fixed workspace, which
    held them with one range sum per 1,024 patches: those counted by fan passes
    as well (16 here) must not push them out."""
    sc = dev.scene(synth.box_wing())
    entries = [(sc, params(SUN, n, bounces, diffuse=diffuse)) for n in sizes]
    assert dev.batch(entries, noalloc=True) == 0, dev.error()
    log = dev.log()
    assert log[-1][0] == "reduce" and log[-1][2] > sum(max(1, _patches(n) // 1024) for n in sizes)


def test_queues_hold_every_item_and_nothing_else(dev):
    """Every item of a launch is at exactly one position of one queue, no queue counts
    a position without an item (a wave would ask it in vain), and where waves have
    items of their own every item has its wave."""
    totals = list(range(300)) + [64 * k + d for k in (16, 64, 1000) for d in (-1, 0, 1, 37, 63)]
    assert [t for t in totals if dev.lib.queue_faults(t, 1)] == []
    for blocks in (255, 256, 257, 300, 511, 512, 1024):
        for total in (1, 255, 256, 1000, 1024, 4 * blocks - 1, 4 * blocks, 4 * blocks + 1):
            assert dev.lib.queue_faults(total, blocks) == 0, (total, blocks)


def _merged(parts):
    """One rigid body of several meshes."""
    m = synth.icosphere(subdiv=0)
    at = np.cumsum([0] + [len(p.verts) for p in parts])
    m.tris = np.concatenate([p.tris + a for p, a in zip(parts, at)]).astype(np.int32)
    m.verts = np.concatenate([p.verts for p in parts])
    m.tri_mat, m.tri_node = np.zeros(len(m.tris), np.int32), np.zeros(len(m.tris), np.int32)
    return m


def _on_booms(subdiv, length):
    """A sphere of 20 x 4^subdiv triangles and six bare booms of `length` times its radius."""
    s = synth.icosphere(subdiv=subdiv)
    L, w = length, 0.02
    parts = [s] + [synth.plate(o, u, v, nu=4, nv=1) for o, u, v in (
        ((-L, -w, 0), (2 * L, 0, 0), (0, 2 * w, 0)), ((-w, 0, -L), (0, 0, 2 * L), (2 * w, 0, 0)),
        ((0, -L, -w), (0, 2 * L, 0), (0, 0, 2 * w)))]
    return _merged(parts)


@pytest.mark.parametrize("mesh,n,items,rasterised", [
    ("crowded", 512, 32, False),     # 81,920 triangles on a few tiles, 0.31 per pixel of the whole image
    ("crowded", 1024, 64, True),     # the same body over some dozen tiles of a launch of a million patches
    ("crowded", 2048, 1, True),      # and over more of them in one fine image
    ("crowded", 1024, 8, True),
    ("crowded", 1040, 8, True),
    ("even", 512, 64, True),         # as many triangles all over the image
    ("even", 400, 53, True),         # 0.51 per pixel: only in launches of 131,072 patches
    ("even", 372, 60, True),
    ("even", 368, 62, False),        # 0.605
    ("craft", 300, 648, True),
    ("craft", 1024, 64, True),
    ("craft", 512, 8, True),
    ("small craft", 128, 64, True),
    ("plates", 512, 64, False),      # 200 layers, few triangles in any tile
])
def test_images_with_crowded_tiles_keep_the_traversal(dev, mesh, n, items, rasterised):
    m = {"crowded": lambda: _on_booms(6, 20), "even": lambda: synth.icosphere(subdiv=6),
         "plates": lambda: _merged([synth.plate((-1, -1, k / 100 - 1), (2, 0, 0), (0, 2, 0), nu=4, nv=4) for k in range(200)]),
         "craft": lambda: synth.procedural_sized(3, 50000), "small craft": lambda: synth.procedural_sized(3, 3000)}[mesh]()
    sc, other = dev.scene(m), dev.scene(_grid_mesh(2000))
    rng = np.random.default_rng(1)
    assert dev.batch([(sc, params(s, n, 1)) for s in rng.normal(size=(items, 3))]) == 0, dev.error()
    got = [r for r in dev.log() if r[0] == "primary"]
    assert [r[2] for r in got] == ([items] if rasterised else [])
    # an image beside it that is not crowded is rasterised in either case
    assert dev.batch([(sc, params(SUN, n, 1))] * items + [(other, params(SUN, 1024, 1))]) == 0, dev.error()
    got = [r for r in dev.log() if r[0] == "primary"]
    assert [r[2] for r in got] == [items + 1 if rasterised else 1] and dev.lib.dev_faults() == 0


def test_long_items_are_taken_one_at_a_time(dev):
    """Chunks that trace a craft's diffuse fans are long beside a request: runs of them end
    a launch on the waves that took the last ones.  Others go in runs of at most a
    fourth of what is left, whatever the launch."""
    craft, small = dev.scene(synth.procedural_sized(3, 8000)), dev.scene(synth.box_wing())
    for sc, diffuse, single in ((craft, 16, 1), (craft, 1, 0), (small, 1, 0), (small, 16, 0), (craft, 0, 0)):
        assert dev.batch([(sc, params(SUN, 400, 1, diffuse=diffuse))] * 24) == 0, dev.error()
        assert [r[5] for r in dev.log() if r[0] == "trace"] == [single]
    dev.lib.run_of.restype = C.c_uint32
    for blocks in (1, 16, 256, 512, 1024):
        for left in (1, 2, 100, 4096, 1 << 25):
            assert dev.lib.run_of(left, blocks, 1) == 1
            assert 1 <= dev.lib.run_of(left, blocks, 0) <= max(1, left // 4)
    assert dev.lib.run_of(4096, 1024, 0) > 1


@pytest.mark.parametrize("mesh,n,items,bounces,diffuse,listed", [
    ("box-wing", 256, 2, 4, 4, True),       # a small launch: always
    ("box-wing", 256, 30, 4, 4, False),
    ("box-wing", 256, 30, 2, 16, False),
    ("box-wing", 256, 30, 2, 31, True),
    ("80 triangles", 256, 30, 2, 8, False),
    ("80 triangles", 256, 30, 1, 16, True),
    ("craft", 256, 30, 2, 8, True),
    ("craft", 256, 64, 2, 16, False),       # a big launch of cheap rays
])
def test_fans_of_few_rays_from_few_triangles_have_no_launch_of_their_own(dev, mesh, n, items, bounces, diffuse, listed):
    m = {"box-wing": synth.box_wing, "80 triangles": lambda: synth.icosphere(subdiv=1),
         "craft": lambda: synth.procedural_sized(3, 8000)}[mesh]()
    assert dev.batch([(dev.scene(m), params(SUN, n, bounces, diffuse=diffuse))] * items) == 0, dev.error()
    trace = [r for r in dev.log() if r[0] == "trace"]
    assert len(trace) == 1 and trace[0][3] != trace[0][4] and trace[0][4] == listed


def test_rasterised_hits_in_the_fixed_workspace_and_across_the_cap(dev):
    """The hits of 16 images at 256^2 fit beside the whole grid's stacks in the fixed
    workspace, those of 30 at 512^2 do not and are left out; a batch whose hits pass
    the workspace cap runs as rasterised sub-batches.  (And 130,000 patches at 0.51
    triangles per pixel are too few.)"""
    dense = dev.scene(synth.icosphere(subdiv=6))
    assert dev.batch([(dense, params(SUN, 400, 1))] * 52) == 0 and not [r for r in dev.log() if r[0] == "primary"]
    sc = dev.scene(synth.procedural_sized(7, 4000))
    for n, items, rasterised in ((256, 16, [16]), (512, 30, [])):
        assert dev.batch([(sc, params(SUN, n, 2))] * items, noalloc=True) == 0, dev.error()
        assert [r[2] for r in dev.log() if r[0] == "primary"] == rasterised
    assert dev.batch([(sc, params(SUN, 8192, 0))] * 30) == 0, dev.error()
    assert [r[2] for r in dev.log() if r[0] == "primary"] == [15, 15]
