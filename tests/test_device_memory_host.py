"""CPU checks of the library's device memory, on a HIP runtime without a device
(host_hip/device.c, loaded before the real one: allocations are numbers with a
limit, copies and fills are checked against them, kernels do nothing). Memory
kept from a destroyed forest never makes a later call fail, stays within its
bounds and goes back on request; every case leaves nothing allocated."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GB = 1 << 30


@pytest.fixture(scope="module")
def device(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host_hip") / "device.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "host_hip", "device.c"), "-o", so,
                           "-lpthread"])
    return so


def run(device, case, *args):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), case, *map(str, args)], capture_output=True, text=True,
                       env=dict(os.environ, LD_PRELOAD=device), cwd=ROOT)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]


# -- what the subprocesses run ---------------------------------------------------

class Dev:
    def __init__(self):
        import paper_1801_08361_amd as rl
        self.rl, self.L, self.d = rl, rl.lib(), C.CDLL(None)
        self.d.dev_used.restype = C.c_uint64
        for f in ("dev_limit", "dev_total"):
            getattr(self.d, f).argtypes = [C.c_uint64]
        self.d.dev_skip.argtypes = [C.c_long]
        self.d.hipMalloc.argtypes = [C.c_void_p, C.c_size_t]
        self.d.hipFree.argtypes = [C.c_void_p]

    used = property(lambda self: self.d.dev_used())

    def malloc(self, n):
        p = C.c_void_p()
        assert self.d.hipMalloc(C.byref(p), n) == 0
        return p

    def forest(self, **kw):
        h = C.c_void_p()
        rc = self.L.reloc_forest_create(C.byref(self.rl.params_default(**kw)), None, C.byref(h))
        assert rc == 0, rc
        return h

    def frame(self, w=640, h=480):
        return [self.malloc(2 * w * h), self.malloc(3 * w * h), self.rl.reloc_intrinsics(w, h, 500.0, 500.0, w / 2, h / 2)]

    def adapt(self, f, fr):
        return self.L.reloc_adapt_frame(f, fr[0], fr[1], C.byref(fr[2]), np.eye(4).ctypes.data, None)

    def destroy(self, f):
        assert self.L.reloc_forest_destroy(f) == 0


LARGE = dict(n_trees=5, depth=13, reservoir_size=1024)     # 0.85 GB
OTHER = dict(n_trees=3, depth=9, reservoir_size=128)


def calls(D, f, fr):
    """every call that allocates device memory, as (name, function)"""
    L, rl = D.L, D.rl
    x, y, pix = D.malloc(64 * 8192), D.malloc(8192), D.malloc(4 * 640 * 480)
    mlp, batch = C.c_void_p(), C.c_void_p()
    assert L.reloc_mlp_create(1, None, C.byref(mlp)) == 0 and L.reloc_batch_create(C.byref(batch)) == 0
    res = (rl.reloc_result * 1)()
    grad, loss, host = np.zeros(5825, np.float32), np.zeros(4, np.float32), np.zeros((480, 640, 8), np.int32)
    out = [np.zeros(1), np.zeros(1), np.zeros(1, np.int32)]
    pts, m, n = np.zeros(8, rl.ENTRY_DTYPE), np.zeros(64, rl.MODE_DTYPE), C.c_int32()
    tr = (rl.reloc_train_frame * 1)()
    tr[0].depth_dev, tr[0].rgb_dev, tr[0].K = fr[0], fr[1], fr[2]
    tr[0].pose_c2w[:] = [float(v) for v in np.eye(4).ravel()]
    at = (rl.reloc_attempt * 1)()
    at[0].forest, at[0].depth_dev, at[0].rgb_dev, at[0].K = f, fr[0], fr[1], fr[2]
    K = C.byref(fr[2])

    def create(**kw):
        h = C.c_void_p()
        rc = L.reloc_forest_create(C.byref(rl.params_default(**kw)), None, C.byref(h))
        return rc if rc else L.reloc_forest_destroy(h)

    def new_mlp():
        h = C.c_void_p()
        rc = L.reloc_mlp_create(1, None, C.byref(h))
        return rc if rc else L.reloc_mlp_destroy(h)

    def relocalise():
        rc = L.reloc_relocalise_ex(f, fr[0], fr[1], K, 0, 0, None, C.byref(res[0]), None)
        return min(rc, 0)

    todo = [("forest of another size", lambda: create(**OTHER)),
            ("adapt", lambda: D.adapt(f, fr)),
            ("relocalise", relocalise),
            ("batch", lambda: L.reloc_relocalise_batch(batch, at, 1, C.byref(res[0]), None)),
            ("split training", lambda: L.reloc_forest_train(f, tr, 1, 4, 64, None)),
            ("network", new_mlp),
            ("gradient", lambda: L.reloc_mlp_gradient(mlp, x, y, 4096, grad.ctypes.data, loss.ctypes.data, None)),
            ("network training", lambda: L.reloc_mlp_train(mlp, x, y, 8192, 3, 8192, C.c_float(1e-3), 0, loss.ctypes.data, None)),
            ("valid pixels", lambda: L.reloc_valid_pixels(f, fr[0], fr[1], K, pix, C.byref(n), None)),
            ("verification", lambda: L.reloc_verify(fr[0], fr[0], 640, 480, *[a.ctypes.data for a in out], None)),
            ("features", lambda: L.reloc_debug_features8(f, fr[0], fr[1], K, host.ctypes.data, None)),
            ("modes of points", lambda: L.reloc_debug_modes_from_points(f, pts.ctypes.data, 8, m.ctypes.data, C.byref(n)))]
    done = [lambda: L.reloc_mlp_destroy(mlp), lambda: L.reloc_batch_destroy(batch),
            *[lambda p=p: D.d.hipFree(p) for p in (x, y, pix)]]
    return todo, done


def case_full_device():
    """with the device full but for what destroyed forests left, each call gets
    its memory from there; a full device without that still refuses"""
    D = Dev()
    f, fr = D.forest(**OTHER), D.frame()
    todo, done = calls(D, f, fr)
    names = [name for name, _ in todo]
    for d in done:
        d()
    for name in names:
        # (a new forest and network, whose scratch is not there yet)
        D.destroy(f)
        f = D.forest(**OTHER)
        todo, done = calls(D, f, fr)
        D.destroy(D.forest(**LARGE))
        assert D.used > GB // 2, (name, "nothing was kept: the case shows nothing")
        D.d.dev_limit(D.used)
        rc = dict(todo)[name]()
        assert rc == 0, (name, rc)
        D.d.dev_limit(288 * GB)
        assert D.L.reloc_trim() == 0
        for d in done:
            d()
    D.destroy(f)
    assert D.L.reloc_trim() == 0
    for p in fr[:2]:
        D.d.hipFree(p)
    assert D.used == 0
    D.d.dev_limit(GB // 2)
    h = C.c_void_p()
    assert D.L.reloc_forest_create(C.byref(D.rl.params_default(**LARGE)), None, C.byref(h)) == D.rl.E_NOMEM
    assert D.used == 0 and h.value is None


def case_bounds():
    """at most 4 GiB, and past 1 GiB an eighth of what the device has free"""
    D = Dev()
    fs = [D.forest(**LARGE) for _ in range(8)]
    for f in fs:
        D.destroy(f)
        assert D.used <= sum(1 for g in fs[fs.index(f) + 1:]) * GB + 4 * GB
    assert 3 * GB < D.used <= 4 * GB
    assert D.L.reloc_trim() == 0 and D.used == 0
    for total in (22 * GB, 14 * GB, 6 * GB):
        D.d.dev_total(total)
        D.d.dev_skip(2)      # (what is free is asked once a second)
        for f in [D.forest(**LARGE) for _ in range(5)]:
            D.destroy(f)
        assert D.used <= max((total - D.used) // 8 + GB // 8, GB)
        assert D.used > GB // 2
        assert D.L.reloc_trim() == 0
    assert D.L.reloc_trim() == 0 and D.used == 0


def case_time():
    """what nobody takes for 10 s goes back at the next allocation, what is
    taken again in time does not"""
    D = Dev()
    D.destroy(D.forest(**LARGE))
    kept = D.used
    D.d.dev_skip(8)
    D.destroy(D.forest(**LARGE))
    assert D.used == kept
    D.d.dev_skip(11)
    h = C.c_void_p()
    assert D.L.reloc_mlp_create(1, None, C.byref(h)) == 0
    assert D.used < GB // 8
    assert D.L.reloc_mlp_destroy(h) == 0
    assert D.used == 0


def case_busy():
    """while the runtime refuses the device-wide wait (another thread captures
    a graph) a destroyed forest leaves nothing, and kept blocks that it refuses
    to free are not lost"""
    D = Dev()
    f = D.forest(**LARGE)
    D.d.dev_refuse(1)
    D.destroy(f)
    assert D.used == 0
    D.d.dev_refuse(0)
    D.destroy(D.forest(**LARGE))
    kept = D.used
    assert kept > GB // 2
    D.d.dev_refuse(2)
    assert D.L.reloc_trim() == 0 and D.used == kept
    D.d.dev_refuse(0)
    assert D.L.reloc_trim() == 0 and D.used == 0


def case_no_scratch():
    """a frame whose scratch does not fit, whichever of its allocations is the
    first that fails: nothing of it stays, the forest's memory is what it was,
    and the frame is accepted once there is room"""
    D = Dev()

    def memory(f):
        b = C.c_uint64()
        assert D.L.reloc_forest_memory(f, C.byref(b)) == 0
        return b.value

    fr, small = D.frame(), D.frame(64, 48)
    f = D.forest(**OTHER)
    own = memory(f)
    assert D.adapt(f, fr) == 0
    need, own_after = memory(f) - own, memory(f)
    D.destroy(f)
    for first in (0, 1):            # a forest without scratch, and one with a smaller frame's
        for k in range(24):
            assert D.L.reloc_trim() == 0
            f = D.forest(**OTHER)
            if first:
                assert D.adapt(f, small) == 0
            had, used = memory(f), D.used
            D.d.dev_limit(used + need * k // 24)
            rc = D.adapt(f, fr)
            assert rc == D.rl.E_NOMEM or (first and k == 23), (k, rc)
            if rc:
                assert own <= memory(f) <= had, (k, own, memory(f), had)
                assert D.used - used <= 8192 * 24 and D.used >= memory(f), (k, D.used - used)
            D.d.dev_limit(288 * GB)
            assert D.adapt(f, fr) == 0 and memory(f) == own_after, k
            before = D.used
            D.destroy(f)
            assert D.used == before, "all of it is kept, at its size"
    assert D.L.reloc_trim() == 0
    for p in fr[:2] + small[:2]:
        D.d.hipFree(p)
    assert D.used == 0


def case_network_training():
    """training that asks for no losses allocates nothing once its minibatch
    has run, however many epochs follow, so that a capture can hold it; the
    losses go straight to the caller's array"""
    D = Dev()
    x, y, h = D.malloc(64 * 8192), D.malloc(8192), C.c_void_p()
    assert D.L.reloc_mlp_create(1, None, C.byref(h)) == 0

    def train(epochs, loss=None):
        return D.L.reloc_mlp_train(h, x, y, 8192, epochs, 512, C.c_float(1e-3), 0, loss, None)

    assert train(1) == 0
    used = D.used
    D.d.dev_refuse(2)
    assert train(64) == 0
    D.d.dev_refuse(0)
    assert D.used == used
    loss = np.full(10, -1.0, np.float32)
    assert train(8, loss.ctypes.data) == 0
    assert not loss[:8].any() and (loss[8:] == -1.0).all()
    assert D.L.reloc_mlp_destroy(h) == 0
    D.d.hipFree(x)
    D.d.hipFree(y)
    assert D.used == 0


def case_train_planes():
    """every training frame's planes begin where its 8-byte stores may, whatever
    the sizes of the frames before"""
    D = Dev()
    f, sizes = D.forest(**OTHER), [(163, 121), (4, 1), (1, 1), (65, 3), (640, 480), (7, 5), (5, 4)]
    frames = [D.frame(*s) for s in sizes]
    tr = (D.rl.reloc_train_frame * len(sizes))()
    for x, fr in zip(tr, frames):
        x.depth_dev, x.rgb_dev, x.K = fr
        x.pose_c2w[:] = [float(v) for v in np.eye(4).ravel()]
    assert D.L.reloc_forest_train(f, tr, len(sizes), 1, 8, None) == 0
    got = np.zeros(4096, np.uint8)
    D.d.dev_upload.restype = C.c_uint64
    n = D.d.dev_upload(C.c_void_p(got.ctypes.data), C.c_uint64(got.size))
    size = n // len(sizes)      # the frames' descriptors; the last word of each is its planes' offset
    assert n == size * len(sizes) and n <= got.size
    at = [int(got[(i + 1) * size - 8: (i + 1) * size].view(np.int64)[0]) for i in range(len(sizes))]
    assert at[0] == 0 and all(a % 8 == 0 for a in at), at
    # 5 bytes a pixel: 16-bit depths and three planes of colours, none over the next frame's
    assert all(b - a >= 5 * w * h for a, b, (w, h) in zip(at, at[1:], sizes)), at


def case_capture():
    """what needs new memory while its stream records a graph is refused, as
    without kept memory, and the recording goes on"""
    D = Dev()
    fr = D.frame()
    f = D.forest(**OTHER)
    assert D.adapt(f, fr) == 0
    D.destroy(f)
    f = D.forest(**OTHER)
    h = C.c_void_p()
    D.d.dev_capture(1)
    assert D.adapt(f, fr) == D.rl.E_NOMEM
    assert D.L.reloc_forest_create(C.byref(D.rl.params_default(**OTHER)), None, C.byref(h)) == D.rl.E_NOMEM
    assert D.d.dev_capturing() == 1
    D.d.dev_capture(0)
    assert D.adapt(f, fr) == 0
    D.d.dev_capture(1)
    assert D.adapt(f, fr) == 0     # its scratch is there
    D.d.dev_capture(0)
    D.destroy(f)
    assert D.L.reloc_trim() == 0
    for p in fr[:2]:
        D.d.hipFree(p)
    assert D.used == 0


# -- the tests ---------------------------------------------------------------------

@pytest.mark.parametrize("case", ["full_device", "bounds", "time", "busy", "no_scratch", "network_training", "train_planes", "capture"])
def test_kept_memory(device, case):
    run(device, case)


if __name__ == "__main__":
    sys.path.insert(0, ROOT)
    globals()["case_" + sys.argv[1]](*map(int, sys.argv[2:]))
    print("ok")
