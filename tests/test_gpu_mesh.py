"""GPU parity of marching-cubes meshing against the oracle, through the C
ABI.  The oracle meshes the GPU volume's own voxels (exported), so both sides
see the same input; the bar: the same triangles, each as the same ordered
triple of edge keys (integer decisions: observed corners, signs, the case
table, orientation), and every vertex within 1e-5 m of the oracle's float64
position (float32 arithmetic on coordinates below ~10^3 voxels).  The mesh of
a noiseless fused scene lies on the analytic surface (a second surface-error
metric); calls are deterministic; a short output buffer keeps the count and
the leading triangles."""
import numpy as np
import pytest

from gpu_helpers import to_device
from synth import analytic_sdf, configs

pytestmark = pytest.mark.gpu

POS_TOL = 1e-5


def _fused(vp, frames, poses, K):
    import paper_1708_00783_amd as T
    g = T.Volume(vp, K.width, K.height)
    for k in range(len(frames)):
        g.frame(to_device(frames[k]), K, poses[k])
    return g


def _compare(g, voxel, tag):
    from oracle import mesh as M
    pos, sdf, w = g.voxels_by_position()
    oV, oK = M.mesh(pos, sdf, w, voxel)
    gV, gK = g.mesh()
    assert len(gV) == len(oV), f"{tag}: {len(gV)} gpu vs {len(oV)} oracle triangles"
    gs = sorted(map(tuple, gK.tolist()))
    os_ = sorted(map(tuple, oK.tolist()))
    assert gs == os_, f"{tag}: triangle sets differ"
    gp = dict(zip(gK.reshape(-1).tolist(), gV.reshape(-1, 3)))
    op = dict(zip(oK.reshape(-1).tolist(), oV.reshape(-1, 3)))
    err = max(float(np.abs(gp[k] - op[k]).max()) for k in op)
    assert err <= POS_TOL, f"{tag}: vertex error {err}"
    return gV, gK, err


def test_c1_mesh_matches_oracle_and_lies_on_the_scene():
    d, p, K, scene = configs.c1_frames(10)
    g = _fused(configs.C1_VOLUME, d, p, K)
    gV, gK, err = _compare(g, configs.C1_VOLUME.voxel_size, "c1")
    e = analytic_sdf(scene, gV.reshape(-1, 3).astype(np.float64))
    rms = float(np.sqrt(np.mean(e * e)))
    print(f"c1 mesh: {len(gV)} triangles, vertex error {err:.2e} m, surface RMS {rms * 1e3:.3f} mm", flush=True)
    assert len(gV) > 10000
    assert rms < 0.5 * configs.C1_VOLUME.voxel_size
    # counter-clockwise seen from free space: the normals of the floor's triangles point up
    n = np.cross(gV[:, 1] - gV[:, 0], gV[:, 2] - gV[:, 0])
    floor = np.all(np.abs(gV[..., 2]) < 0.003, axis=1)
    assert floor.sum() > 1000 and np.mean(n[floor][:, 2] > 0) > 0.99


def test_c2_frames_mesh_matches_oracle():
    frames = np.stack([configs.c2_frame(k) for k in range(3)])
    poses = np.stack(configs.c2_poses(300)[:3]).astype(np.float32)
    g = _fused(configs.C2_VOLUME, frames, poses, configs.KINECT_INTR)
    gV, _, err = _compare(g, configs.C2_VOLUME.voxel_size, "c2 3 frames")
    print(f"c2 mesh after 3 frames: {len(gV)} triangles, vertex error {err:.2e} m", flush=True)


def test_mesh_is_deterministic_and_respects_the_buffer():
    import ctypes
    import torch
    import paper_1708_00783_amd as T
    d, p, K, _ = configs.c1_frames(4)
    g = _fused(configs.C1_VOLUME, d, p, K)
    a = g.mesh()
    b = g.mesh()
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    n = len(a[0])
    cap = n // 3
    nbytes = int(T.lib().tf_mesh_workspace_bytes(ctypes.byref(g.params)))
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    verts = torch.full((cap, 3, 3), 7.0, dtype=torch.float32, device="cuda")
    T.check(T.lib().tf_mesh(g.ctx, ctypes.c_void_p(verts.data_ptr()), None, cap, ctypes.c_void_p(cnt.data_ptr()),
                            ctypes.c_void_p(ws.data_ptr()), nbytes, T._stream_ptr(None)), "tf_mesh")
    assert int(cnt.item()) == n
    assert np.array_equal(verts.cpu().numpy(), a[0][:cap])
    with pytest.raises(T.TsdfError):
        T.check(T.lib().tf_mesh(g.ctx, None, None, 0, ctypes.c_void_p(cnt.data_ptr()),
                                ctypes.c_void_p(ws.data_ptr()), nbytes - 8, T._stream_ptr(None)), "tf_mesh")


def test_empty_volume_has_no_triangles():
    import paper_1708_00783_amd as T
    g = T.Volume(configs.C1_VOLUME, 160, 120)
    V, Kk = g.mesh()
    assert len(V) == 0 and len(Kk) == 0


@pytest.mark.parametrize("n_buckets,n_excess", [(16, 40), (1 << 12, 1 << 10), (1 << 18, 1 << 12)])
def test_rough_blocks_and_table_sizes_match_oracle(n_buckets, n_excess):
    """One chunk of 64 entries, one scan group and two (the counts' offsets
    take another path in each), on blocks whose signs change from voxel to
    voxel: more triangles in a block than the 256 that emission lists at a time."""
    from synth.scenes import Intrinsics
    rng = np.random.default_rng(n_buckets)
    K = Intrinsics(200.0, 200.0, 23.5, 19.5, 48, 40)
    vp = configs.VolumeParams(0.01, 0.08, 100, n_buckets, n_excess, 4096)
    P = np.eye(4, dtype=np.float32)
    frames = (0.52 + 0.035 * rng.choice([-1.0, 1.0], size=(1, 40, 48))).astype(np.float32)
    g = _fused(vp, frames, [P], K)
    gV, gK, err = _compare(g, vp.voxel_size, f"rough {n_buckets}")
    cell = np.floor(gV.reshape(-1, 3, 3).mean(axis=1) / (8 * vp.voxel_size)).astype(int)
    most = np.unique(cell, axis=0, return_counts=True)[1].max()
    print(f"rough mesh, {n_buckets} buckets: {len(gV)} triangles, at most {most} in a block, error {err:.2e}", flush=True)
    assert most > 256
