"""GPU parity of host swapping (Sec. 5): the same small device budget with
swapping after every frame, oracle vs HIP path.  Visible and device-resident
sets must agree frame by frame and the final voxels (device or host copy) by
position.  The transfer buffer is larger than any frame's candidate set, so
the selection of which blocks move does not depend on entry indices (those
differ between the two tables: excess slots are taken in a different order)."""
import numpy as np
import pytest

from gpu_helpers import to_device
from synth.configs import VolumeParams

pytestmark = pytest.mark.gpu


def _walk():
    import test_oracle_swap as S
    return S.walk_frames(40), S.K_SMALL, S.VP


def _state(vol_o=None, vol_g=None):
    res = {}
    if vol_o is not None:
        pos, _, ptr = vol_o.entries()
        dev = np.flatnonzero(ptr >= 0)
        sdf, w = vol_o.block_voxels(dev)
        for k, i in enumerate(dev):
            res[tuple(pos[i])] = (sdf[k], w[k])
        for i in np.flatnonzero(ptr == -1):
            res[tuple(pos[i])] = vol_o.host_block(i)
    else:
        pos, _, ptr = vol_g.entries()
        dev = np.flatnonzero(ptr >= 0)
        sdf, w = vol_g.block_voxels(dev)
        for k, i in enumerate(dev):
            res[tuple(pos[i])] = (sdf[k], w[k])
        out = np.flatnonzero(ptr == -1)
        hs, hw, has = vol_g.host_voxels(out)
        assert has.all()
        for k, i in enumerate(out):
            res[tuple(pos[i])] = (hs[k], hw[k])
    return res


# 2^21 buckets: the ordered swap-out selection scans 513 chunks of 4096
# entries, so its single-workgroup scan carries offsets across two passes of
# 256 chunks (the entries of the walk's blocks spread over all of them)
@pytest.mark.parametrize("n_buckets", [None, 1 << 21])
def test_swapping_parity_walk(n_buckets):
    from oracle import oracle as O
    import paper_1708_00783_amd as T
    frames, K, VP = _walk()
    nb = n_buckets or VP.n_buckets
    print(f"case swap walk, {nb} buckets", flush=True)
    budget = VolumeParams(VP.voxel_size, VP.mu, VP.max_w, nb, VP.n_excess, 5000)
    o = O.Volume.from_params(budget)
    o.enable_swap(4096)
    g = T.Volume(budget, K.width, K.height, swap_transfer_blocks=4096)
    tot_in = tot_out = 0
    for f, (depth, P) in enumerate(frames):
        o.alloc_and_visible(depth, K.as_array(), P)
        o.integrate(depth, K.as_array(), P)
        dd = to_device(depth)
        g.alloc_and_visible(dd, K, P)
        g.integrate(dd, P)
        st = g.stats()
        assert st["n_swapped_in"] == o.n_swapped_in, f
        tot_in += st["n_swapped_in"]
        mo = o.swap_out()
        g.swap_out()
        st = g.stats()
        assert st["n_swapped_out"] == mo, f
        tot_out += mo
        gp, _, gptr = g.entries()
        op, _, optr = o.entries()
        assert {tuple(x) for x in gp[gptr >= 0]} == {tuple(x) for x in op[optr >= 0]}, f
        assert {tuple(x) for x in gp[gptr == -1]} == {tuple(x) for x in op[optr == -1]}, f
        assert {tuple(x) for x in gp[g.visible()]} == {tuple(x) for x in op[o.visible()]}, f
    assert tot_out > 500 and tot_in > 50
    assert g.stats()["flags"] == 0 and o.flags == 0
    a = _state(vol_o=o)
    b = _state(vol_g=g)
    assert a.keys() == b.keys()
    for key in a:
        assert np.array_equal(a[key][1], b[key][1]), key
        assert np.abs(a[key][0].astype(int) - b[key][0].astype(int)).max() <= 1, key


def test_transfer_overflow_merge_parity():
    """tiny transfer buffer: host data waits while the device keeps fusing,
    then merges (secondary integration) -- same weights, SDF within 1 LSB"""
    from oracle import oracle as O
    import paper_1708_00783_amd as T
    from synth import configs, look_at
    vp = configs.C1_VOLUME
    K = configs.C1_INTR
    pose = np.eye(4, dtype=np.float32)
    plane = lambda z: np.full((K.height, K.width), z, np.float32)
    sky = look_at([0.0, 0.0, 0.0], [0.0, 0.0, -5.0], up=(0.0, 1.0, 0.0)).astype(np.float32)
    o = O.Volume.from_params(vp)
    o.enable_swap(40)
    g = T.Volume(vp, K.width, K.height, swap_transfer_blocks=40)
    seq = [(plane(1.0), pose, True)] * 3 + [(plane(0.0), sky, False)] + [(plane(1.02), pose, True)] * 2 + \
          [(plane(0.0), pose, False)] * 60
    for k, (d, P, integ) in enumerate(seq):
        o.alloc_and_visible(d, K.as_array(), P)
        dd = to_device(d)
        g.alloc_and_visible(dd, K, P)
        assert g.stats()["n_swapped_in"] == o.n_swapped_in, k
        if integ:
            o.integrate(d, K.as_array(), P)
            g.integrate(dd, P)
        if k == 3:
            while o.swap_out():
                pass
            for _ in range(200):
                g.swap_out()
                if g.stats()["n_swapped_out"] == 0:
                    break
    assert g.stats()["flags"] & 8 and o.flags & 8
    a = _state(vol_o=o)
    b = _state(vol_g=g)
    assert a.keys() == b.keys()
    for key in a:
        assert np.array_equal(a[key][1], b[key][1]), key
        assert np.abs(a[key][0].astype(int) - b[key][0].astype(int)).max() <= 1, key


def test_swap_out_merges_pending_host_copies():
    """Blocks swapped out, then touched again: they get fresh device blocks
    at once while their host copies come back at most 40 per frame.  Swapping
    everything out again two frames later catches most of them with the host
    copy still pending: the secondary integration (Sec. 5) then fuses the
    device copy into the store copy on the device.  Final voxels by position
    (device or host copy): weights bit-exact, SDF within 1 LSB of the oracle."""
    from oracle import oracle as O
    import paper_1708_00783_amd as T
    from synth import configs, look_at
    vp = configs.C1_VOLUME
    K = configs.C1_INTR
    pose = np.eye(4, dtype=np.float32)
    plane = lambda z: np.full((K.height, K.width), z, np.float32)
    sky = look_at([0.0, 0.0, 0.0], [0.0, 0.0, -5.0], up=(0.0, 1.0, 0.0)).astype(np.float32)
    o = O.Volume.from_params(vp)
    o.enable_swap(40)
    g = T.Volume(vp, K.width, K.height, swap_transfer_blocks=40)
    seq = [(plane(1.0), pose, True)] * 3 + [(plane(0.0), sky, False)] + [(plane(1.02), pose, True)] * 2 + \
          [(plane(0.0), sky, False)] + [(plane(0.0), pose, False)] * 3
    pending_at_swap = 0
    for k, (d, P, integ) in enumerate(seq):
        o.alloc_and_visible(d, K.as_array(), P)
        dd = to_device(d)
        g.alloc_and_visible(dd, K, P)
        assert g.stats()["n_swapped_in"] == o.n_swapped_in, k
        if integ:
            o.integrate(d, K.as_array(), P)
            g.integrate(dd, P)
        if k in (3, 6):
            if k == 6:
                _, _, ptr = g.entries()
                dev = np.flatnonzero(ptr >= 0).astype(np.int32)
                pending_at_swap = int(g.host_voxels(dev)[2].sum())
            while o.swap_out():
                pass
            for _ in range(500):
                g.swap_out()
                if g.stats()["n_swapped_out"] == 0:
                    break
            _, _, ptr = g.entries()
            assert (ptr >= 0).sum() == 0, k
    assert pending_at_swap > 100, pending_at_swap
    a = _state(vol_o=o)
    b = _state(vol_g=g)
    assert a.keys() == b.keys()
    n_lsb = 0
    for key in a:
        assert np.array_equal(a[key][1], b[key][1]), key
        dsdf = np.abs(a[key][0].astype(int) - b[key][0].astype(int))
        assert dsdf.max() <= 1, key
        n_lsb += int((dsdf > 0).sum())
    print(f"pending host copies merged at swap-out: {pending_at_swap}; blocks {len(a)}; "
          f"1-LSB SDF differences {n_lsb}", flush=True)


@pytest.mark.parametrize("buffer", ["pageable", "odd"])
def test_transfer_buffers_the_device_cannot_use_as_given(buffer):
    """a pageable transfer buffer, and a pinned one four bytes off alignment,
    swap as Volume's own does: several hundred blocks out, back in, and out
    again onto their host copies"""
    import ctypes
    import torch
    import paper_1708_00783_amd as T
    from synth import configs
    cap = 4096
    d, p, K, _ = configs.c1_frames(8)
    a = T.Volume(configs.C1_VOLUME, K.width, K.height, swap_transfer_blocks=cap)
    L, par = T.lib(), a.params
    ws = torch.empty(T.tf_workspace_bytes(par), dtype=torch.uint8, device="cuda")
    store = np.zeros(int(L.tf_host_store_bytes(ctypes.byref(par))), np.uint8)
    n = int(L.tf_host_transfer_bytes(ctypes.byref(par)))
    if buffer == "pageable":
        held = np.zeros(n, np.uint8)
        xfer = held.ctypes.data
    else:
        held = torch.empty(n + 64, dtype=torch.uint8, pin_memory=True)
        xfer = held.data_ptr() + 4
    ctx = T.tf_create(par, ws.data_ptr(), ws.numel(), ctypes.c_void_p(store.ctypes.data), ctypes.c_void_p(xfer), None)
    b = T.Volume.borrowed(ctx, par, (ws, store, held))
    try:
        out = inn = 0
        for k in (0, 1, 0, 7, 0, 1):
            for g in (a, b):
                g.frame(to_device(d[k]), K, p[k])
            sa, sb = a.stats(), b.stats()
            assert sa["n_swapped_in"] == sb["n_swapped_in"]
            inn += sa["n_swapped_in"]
            for g in (a, b):
                g.alloc_and_visible(to_device(np.zeros_like(d[k])), T.make_intrinsics(K), _away(p[k]))
                g.swap_out()
            sa, sb = a.stats(), b.stats()
            assert sa["n_swapped_out"] == sb["n_swapped_out"]
            out += sa["n_swapped_out"]
            ra, rb = _state(vol_g=a), _state(vol_g=b)   # by position: excess slots differ
            assert ra.keys() == rb.keys()
            for q in ra:
                assert all(np.array_equal(x, y) for x, y in zip(ra[q], rb[q]))
        print(f"{buffer}: {out} blocks out, {inn} in", flush=True)
        assert out > 6 * 128 and inn > 128
    finally:
        L.tf_destroy(ctx)


def _away(P):
    """the same camera turned around: it sees none of what it saw"""
    return (np.diag([-1.0, 1.0, -1.0, 1.0]) @ np.asarray(P, np.float64)).astype(np.float32)


_FAILING = r"""
import ctypes, os, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before anything that uses the HIP runtime
sys.path[:0] = [sys.argv[2], os.path.join(sys.argv[2], "tests")]
import numpy as np
import torch
torch.zeros(1, device="cuda")
hip = [l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l][0]
assert shim.shim_init(hip.encode()) == 0
import paper_1708_00783_amd as T
from synth import configs
from test_gpu_swap import _away, _state
from gpu_helpers import to_device

nth, cap = int(sys.argv[3]), int(sys.argv[4])
d, p, K, _ = configs.c1_frames(3)
vols = [T.Volume(configs.C1_VOLUME, K.width, K.height, swap_transfer_blocks=cap) for _ in range(2)]
failed = 0

def out_all(g, fail):
    global failed
    for _ in range(500):
        if fail:
            pos, off, ptr = g.entries()
            host = g.host_voxels(np.arange(g.n_entries, dtype=np.int32)[ptr != -2])
            st = g.stats()
            shim.shim_fail(nth)
            try:
                g.swap_out()
            except T.TsdfError:
                failed += 1
                pos2, off2, ptr2 = g.entries()
                host2 = g.host_voxels(np.arange(g.n_entries, dtype=np.int32)[ptr2 != -2])
                assert np.array_equal(ptr, ptr2), "a failed call moved blocks"
                assert all(np.array_equal(a, b) for a, b in zip(host, host2)), "a failed call changed the store"
                assert g.stats()["n_allocated"] == st["n_allocated"]
            shim.shim_fail(0)
        g.swap_out()
        if g.stats()["n_swapped_out"] == 0:
            return
    raise AssertionError("blocks stay on the device")

# Both volumes start as one map and see only what is in it: two runs of the same
# frames give the blocks of a bucket their entries in the order of a race, and a
# small transfer takes blocks by entry, so that they would be fused at other times.
for k in range(3):
    vols[0].alloc_and_visible(to_device(d[k]), K, p[k])
    vols[0].integrate(to_device(d[k]), p[k])
vols[0].save(sys.argv[5])
vols[1].load(sys.argv[5])
for k, away in ((1, False), (1, True), (2, False), (2, False), (2, True)):
    for i, g in enumerate(vols):
        pose = _away(p[k]) if away else p[k]
        g.alloc_and_visible(to_device(np.zeros_like(d[k]) if away else d[k]), K, pose)
        if away:
            out_all(g, i == 1)
        else:
            g.integrate(to_device(d[k]), pose)
a, b = (_state(vol_g=g) for g in vols)
assert a.keys() == b.keys() and len(a) > 500
for q in a:
    assert all(np.array_equal(x, y) for x, y in zip(a[q], b[q])), q
print("failed calls", failed, "blocks", len(a), flush=True)
assert failed >= 2
"""

_SHIM = r"""
#include <dlfcn.h>
static int (*real)(void *);
static int left;
extern "C" int shim_init(const char *path)
{
    real = (int (*)(void *))dlsym(dlopen(path, RTLD_NOLOAD | RTLD_LAZY), "hipStreamSynchronize");
    return real ? 0 : 1;
}
extern "C" void shim_fail(int nth) { left = nth; }
extern "C" int hipStreamSynchronize(void *s)
{
    if (!real) real = (int (*)(void *))dlsym(RTLD_NEXT, "hipStreamSynchronize");
    const int e = real(s);
    return left && --left == 0 ? 999 : e;
}
"""


@pytest.mark.parametrize("nth,cap", [(1, 4096), (1, 100), (2, 100)])
def test_a_failed_swap_out_leaves_the_map(nth, cap, tmp_path):
    """tf_swap_out whose first wait (for the blocks) or second (for pending
    host copies fused with them) reports an error: no block has left the
    device, the store is unchanged, and the calls that follow end in the map of
    a volume without failures.  The error comes from a stand-in for
    hipStreamSynchronize, which waits and then reports it, in a process of its own."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src, so, script = tmp_path / "shim.cpp", tmp_path / "shim.so", tmp_path / "failing.py"
    src.write_text(_SHIM)
    script.write_text(_FAILING)
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-o", str(so), str(src), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-u", str(script), str(so), root, str(nth), str(cap),
                        str(tmp_path / "map")], timeout=100, capture_output=True, text=True)
    print(r.stdout, flush=True)
    assert r.returncode == 0, r.stderr[-2000:]


def test_waits_for_the_stream_keep_the_helpers_asleep():
    """Swap calls that move nothing behind some 150 ms of work on their stream:
    beside the caller's own wait, no thread spins.  (The calls before moved
    hundreds of blocks each way, for which the copy threads were woken.)"""
    import time
    import torch
    import paper_1708_00783_amd as T
    from synth import configs
    d, p, K, _ = configs.c1_frames(2)
    g = T.Volume(configs.C1_VOLUME, K.width, K.height, swap_transfer_blocks=4096)
    dd, zero = to_device(d[0]), to_device(np.zeros_like(d[0]))
    a = torch.zeros((4096, 4096), dtype=torch.float32, device="cuda")

    def busy():
        for _ in range(100):
            torch.mm(a, a)

    def timed(call):
        torch.cuda.synchronize()
        busy()
        t0, c0 = time.perf_counter(), time.process_time()
        call()
        return time.perf_counter() - t0, time.process_time() - c0

    busy()
    for _ in range(2):                     # out, in, and out again
        g.alloc_and_visible(dd, K, p[0])
        g.integrate(dd, p[0])
        g.alloc_and_visible(zero, K, _away(p[0]))
        g.swap_out()
    assert g.stats()["n_swapped_out"] > 128
    w, c = timed(g.swap_out)
    print(f"swap_out behind busy stream: wall {w * 1e3:.1f} ms, CPU {c * 1e3:.1f} ms", flush=True)
    assert w > 0.02 and c < 2 * w + 0.01
    g.alloc_and_visible(dd, K, p[0])
    assert g.stats()["n_swapped_in"] > 128
    w, c = timed(lambda: g.alloc_and_visible(dd, K, p[0]))
    print(f"alloc_and_visible behind busy stream: wall {w * 1e3:.1f} ms, CPU {c * 1e3:.1f} ms", flush=True)
    assert w > 0.02 and c < 2 * w + 0.01


def test_a_transfer_buffer_that_is_not_coherent_is_left_alone():
    """The host reads and writes parts of the transfer buffer while kernels use
    others, which only coherent memory allows: a buffer pinned as non-coherent
    is not touched, and blocks swap out, in and out again as with Volume's own."""
    import ctypes
    import torch
    import paper_1708_00783_amd as T
    from synth import configs
    d, p, K, _ = configs.c1_frames(8)
    a = T.Volume(configs.C1_VOLUME, K.width, K.height, swap_transfer_blocks=4096)
    L, par = T.lib(), a.params
    hip = ctypes.CDLL([x.split()[-1] for x in open("/proc/self/maps") if "libamdhip64" in x][0])
    ws = torch.empty(T.tf_workspace_bytes(par), dtype=torch.uint8, device="cuda")
    store = np.zeros(int(L.tf_host_store_bytes(ctypes.byref(par))), np.uint8)
    n = int(L.tf_host_transfer_bytes(ctypes.byref(par)))
    xfer = ctypes.c_void_p()
    assert hip.hipHostMalloc(ctypes.byref(xfer), ctypes.c_size_t(n), ctypes.c_uint(0x80000000)) == 0
    held = np.ctypeslib.as_array((ctypes.c_uint8 * n).from_address(xfer.value))
    held[:] = 0xa5
    ctx = T.tf_create(par, ws.data_ptr(), ws.numel(), ctypes.c_void_p(store.ctypes.data), xfer, None)
    b = T.Volume.borrowed(ctx, par, (ws, store))
    try:
        for k in (0, 1, 0, 7):
            for g in (a, b):
                g.frame(to_device(d[k]), K, p[k])
                g.alloc_and_visible(to_device(np.zeros_like(d[k])), T.make_intrinsics(K), _away(p[k]))
                g.swap_out()
            assert b.stats()["n_swapped_out"] == a.stats()["n_swapped_out"] > 128
            ra, rb = _state(vol_g=a), _state(vol_g=b)
            assert ra.keys() == rb.keys()
            for q in ra:
                assert all(np.array_equal(x, y) for x, y in zip(ra[q], rb[q]))
        torch.cuda.synchronize()
        assert (held == 0xa5).all()
    finally:
        L.tf_destroy(ctx)
        hip.hipHostFree(xfer)
