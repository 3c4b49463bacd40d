"""revo_op_unproject and revo_op_render_view against the FP64 oracle
(oracle.render).

Unprojection is float32 per element: X = ((u - cx) Z) / fx is good to about
3 ulp (asserted at 1e-6 relative).  Rendering decides integers in float32
(which pixel a point lands on, which point is nearest), so it is compared on
what is unique: the identity view must reproduce the frame bit-exactly (every
point lands on its own pixel centre, far from a rounding boundary), and for a
moved view every pixel where the kernel and the oracle pick different points
(or one of them none) must be explained by float32 rounding: a point within
1e-3 pixel of a rounding boundary, or two candidate depths within 1e-5
relative.  Where both pick the same point the colour is exact and the depth
is Z' rounded to mm (+-1 where Z' is within float32 error of a half)."""
import math

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(808)


def _lib():
    import paper_2604_27441_amd as pkg
    return pkg.lib


def _f32ptr(a):
    a = np.ascontiguousarray(a, dtype=np.float32)
    return a, a.ctypes.data


def _unproject(depth, intr):
    B, H, W = depth.shape
    d = torch.from_numpy(np.ascontiguousarray(depth).view(np.int16)).cuda()
    pts = torch.zeros((B, H, W, 4), dtype=torch.float32, device="cuda")
    k, kp = _f32ptr(intr)
    assert _lib().revo_op_unproject(d.data_ptr(), B, H, W, kp, pts.data_ptr(), None) == 0
    torch.cuda.synchronize()
    return pts


def _render(pts, rgb, pose, intr, Ho, Wo):
    B, H, W = rgb.shape[:3]
    assert pts.shape == (B, H, W, 4)
    c = torch.from_numpy(np.ascontiguousarray(rgb)).cuda()
    zbuf = torch.zeros((B, Ho, Wo), dtype=torch.int64, device="cuda")
    co = torch.zeros((B, Ho, Wo, 3), dtype=torch.uint8, device="cuda")
    do = torch.zeros((B, Ho, Wo), dtype=torch.int16, device="cuda")
    P, pp = _f32ptr(np.asarray(pose).reshape(-1))
    k, kp = _f32ptr(intr)
    assert _lib().revo_op_render_view(pts.data_ptr(), c.data_ptr(), B, H, W, pp, kp, Ho, Wo, zbuf.data_ptr(),
                                      co.data_ptr(), do.data_ptr(), None) == 0
    torch.cuda.synchronize()
    key = zbuf.cpu().numpy().view(np.uint64)
    win = np.where(key == np.uint64(0xFFFFFFFFFFFFFFFF), -1, (key & np.uint64(0xFFFFFFFF)).astype(np.int64))
    return co.cpu().numpy(), do.cpu().numpy().view(np.uint16), win


def _pose(yaw, pitch, t):
    cy, sy, cp, sp = math.cos(yaw), math.sin(yaw), math.cos(pitch), math.sin(pitch)
    Ry = np.array([[cy, 0, sy], [0, 1, 0], [-sy, 0, cy]])
    Rx = np.array([[1, 0, 0], [0, cp, -sp], [0, sp, cp]])
    return np.hstack([Ry @ Rx, np.asarray(t, dtype=np.float64).reshape(3, 1)])


@pytest.mark.parametrize("B,H,W", [(2, 48, 64), (1, 37, 300)])
def test_unproject(B, H, W):
    depth = RNG.integers(0, 4000, (B, H, W)).astype(np.uint16)
    intr = (float(W), float(W), (W - 1) / 2, (H - 1) / 2)
    got = _unproject(depth, intr).cpu().numpy().astype(np.float64)
    for b in range(B):
        ref = oracle.unproject(depth[b], intr)
        assert np.array_equal(got[b, ..., 2:], ref[..., 2:])
        assert np.all(np.abs(got[b, ..., :2] - ref[..., :2]) <= 1e-6 * np.abs(ref[..., :2]) + 1e-9)


def test_identity_view_is_bit_exact():
    rgb, depth = synth.scene_frames(1005, 96, 128, [3, 4])
    depth = depth.copy()
    depth[:, ::7, ::5] = 0  # holes
    intr = (128.0, 128.0, 63.5, 47.5)
    pts = _unproject(depth, intr)
    c, d, w = _render(pts, rgb, np.hstack([np.eye(3), np.zeros((3, 1))]), intr, 96, 128)
    for b in range(2):
        rc, rd, rw = oracle.render_view(oracle.unproject(depth[b], intr), rgb[b], np.hstack([np.eye(3), np.zeros((3, 1))]),
                                        intr, 96, 128)
        assert np.array_equal(w[b], rw) and np.array_equal(c[b], rc) and np.array_equal(d[b], rd)


def _check_moved_view(depth, rgb, pose, intr, Ho, Wo):
    pts = _unproject(depth, intr)
    c, d, w = _render(pts, rgb, pose, intr, Ho, Wo)
    B = depth.shape[0]
    mismatched = 0
    for b in range(B):
        P = oracle.unproject(depth[b], intr)
        rc, rd, rw = oracle.render_view(P, rgb[b], pose, intr, Ho, Wo)
        u, v, z = oracle.project(P, pose, intr)
        valid = (P[..., 3].reshape(-1) > 0) & (z > 0)
        fu, fv = u + 0.5, v + 0.5
        near_edge = valid & ((np.abs(fu - np.rint(fu)) < 1e-3) | (np.abs(fv - np.rint(fv)) < 1e-3))
        same = w[b] == rw
        hit = same & (rw >= 0)
        cols = rgb[b].reshape(-1, 3)
        assert np.array_equal(c[b][hit], cols[rw[hit]]) and not c[b][~(w[b] >= 0)].any()
        zt = z[rw[hit]]
        half = np.abs(zt - np.floor(zt) - 0.5) < 1e-3 * np.maximum(1.0, zt) * 1e-3
        dd = np.abs(d[b][hit].astype(np.int64) - np.rint(zt).astype(np.int64))
        assert np.all((dd == 0) | ((dd == 1) & half))
        for iv, iu in zip(*np.nonzero(~same)):
            mismatched += 1
            g, o = w[b][iv, iu], rw[iv, iu]
            # each side's choice must be a point that can land here under float32 rounding
            cand = []
            for n in (g, o):
                if n >= 0:
                    lands = (math.floor(fu[n]) == iu and math.floor(fv[n]) == iv)
                    assert lands or near_edge[n], (b, iv, iu, n)
                    cand.append(z[n])
            if g >= 0 and o >= 0:
                assert near_edge[g] or near_edge[o] or abs(z[g] - z[o]) <= 1e-5 * z[o], (b, iv, iu, z[g], z[o])
            else:
                n = g if g >= 0 else o
                assert near_edge[n], (b, iv, iu, n)
    assert mismatched <= 1e-3 * B * Ho * Wo, mismatched


@pytest.mark.parametrize("yaw,pitch,t", [(0.05, 0.0, (40.0, 0.0, 0.0)), (-0.12, 0.06, (-150.0, 60.0, 300.0))])
def test_moved_view_small(yaw, pitch, t):
    rgb, depth = synth.scene_frames(1006, 96, 128, [2, 3])
    intr = (128.0, 128.0, 63.5, 47.5)
    _check_moved_view(depth, rgb, _pose(yaw, pitch, t), intr, 96, 128)


@pytest.mark.parametrize("zoom", [4.0, 2.0, 1.0, 0.5])
@pytest.mark.parametrize("H,W", [(17, 65), (35, 130)])
def test_zoomed_view(zoom, H, W):
    """A view through intrinsics scaled by `zoom`, pixel centres well inside
    their targets, so the winners are exact: at 4 the target boxes of whole
    source tiles (64 x 16) are too tall for the LDS z-buffer and points go to
    the z-buffer one by one, at 2 only the boxes' middle columns fit, at 0.5 four
    points meet on a target."""
    B = 2
    depth = RNG.integers(500, 3000, (B, H, W)).astype(np.uint16)
    depth[:, ::5, ::3] = 0
    rgb = RNG.integers(0, 256, (B, H, W, 3)).astype(np.uint8)
    intr = (float(W), float(W), 0.0, 0.0)
    Ho, Wo = int(H * zoom) + 3, int(W * zoom) - 2   # the last columns fall outside
    view = (W * zoom, W * zoom, 0.25 - 0.5 * (zoom < 1), 0.25 - 0.5 * (zoom < 1))
    pose = np.hstack([np.eye(3), np.zeros((3, 1))])
    c, d, w = _render(_unproject(depth, intr), rgb, pose, view, Ho, Wo)
    for b in range(B):
        rc, rd, rw = oracle.render_view(oracle.unproject(depth[b], intr), rgb[b], pose, view, Ho, Wo)
        assert np.array_equal(w[b], rw) and np.array_equal(c[b], rc) and np.array_equal(d[b], rd)


# calls of at most 400 000 points (one row per wave) and of more (two)
@pytest.mark.parametrize("B,H,W", [(2, 35, 130), (2, 330, 611)])
@pytest.mark.parametrize("zoom", [8.0, 2.0, 1.0, 0.5, 0.25])
def test_zoomed_view_of_mixed_rows(B, H, W, zoom):
    """As test_zoomed_view, with every other row thinned to one pixel in eight:
    waves of one workgroup whose points go to the z-buffer themselves beside
    waves whose points meet in LDS (at 0.25 four of a row on every pixel)."""
    depth = RNG.integers(500, 3000, (B, H, W)).astype(np.uint16)
    depth[:, ::2, np.arange(W) % 8 != 3] = 0
    rgb = RNG.integers(0, 256, (B, H, W, 3)).astype(np.uint8)
    intr = (float(W), float(W), 0.0, 0.0)
    Ho, Wo = int(H * zoom) + 3, int(W * zoom) - 2
    c0 = {0.5: -0.25, 0.25: -0.375}.get(zoom, 0.25)
    view = (W * zoom, W * zoom, c0, c0)
    pose = np.hstack([np.eye(3), np.zeros((3, 1))])
    c, d, w = _render(_unproject(depth, intr), rgb, pose, view, Ho, Wo)
    for b in range(B):
        rc, rd, rw = oracle.render_view(oracle.unproject(depth[b], intr), rgb[b], pose, view, Ho, Wo)
        assert np.array_equal(w[b], rw) and np.array_equal(c[b], rc) and np.array_equal(d[b], rd)


def test_moved_view_720p():
    rgb, depth = synth.scene_frames(1003, 720, 1280, [4, 5])
    intr = (1280.0, 1280.0, 639.5, 359.5)
    _check_moved_view(depth, rgb, _pose(0.08, -0.03, (120.0, -40.0, 150.0)), intr, 720, 1280)


def test_rejects_bad_arguments():
    pts = torch.zeros((1, 4, 4, 4), dtype=torch.float32, device="cuda")
    z = torch.zeros((1, 4, 4), dtype=torch.int64, device="cuda")
    k, kp = _f32ptr((4.0, 4.0, 1.5, 1.5))
    P, pp = _f32ptr(np.hstack([np.eye(3), np.zeros((3, 1))]).reshape(-1))
    c = torch.zeros((1, 4, 4, 3), dtype=torch.uint8, device="cuda")
    d = torch.zeros((1, 4, 4), dtype=torch.int16, device="cuda")
    assert _lib().revo_op_render_view(pts.data_ptr(), c.data_ptr(), 1, 4, 4, pp, kp, 0, 4, z.data_ptr(), c.data_ptr(),
                                      d.data_ptr(), None) != 0
    assert _lib().revo_op_unproject(d.data_ptr(), 1, 4, 4, kp, pts.data_ptr() + 4, None) != 0
