"""Penetration of realised sets at the edges of its launch: fewer and more sets than
a wave takes, hands of one to eight fingers (one to 64 links), SDF grids from a
single cell up, objects inside, at the border of and away from the grid, links of
zero length (no depth of their own), ids outside the batch, and the hand's
self-collision.  Joint values are the launch's own; the depth is compared with the
oracle's FP64 walk of the same joints (capsule axes sampled per mm) at the IK bar of
1e-5 m, and validity must follow from the launch's own errors and depth."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _hand(F, dof, zero_len):
    X, Y = synth.X_AX, synth.Y_AX
    rng = np.random.default_rng(F * 10 + dof)
    fingers = []
    for f in range(F):
        a = 2 * np.pi * f / F
        joints = [((X if t % 2 else Y), 0.0 if zero_len and t == 0 else float(rng.uniform(0.01, 0.04)),
                   0.008, -0.5, 1.2) for t in range(dof)]
        fingers.append({"base": (synth._finger_base_rotation(a, 0.9),
                                 np.array([0.03 * np.cos(a), 0.03 * np.sin(a), 0.0])), "joints": joints})
    return synth._build_hand(fingers, 8)


@pytest.mark.parametrize("F,dof,n_sets,dims,k,shift,sc,zero_len", [
    (1, 1, 1, 2, 1, 0.0, 0, False),
    (1, 8, 65, 17, 1, 0.0, 0, True),
    (3, 3, 22, 64, 2, 0.05, 1, False),
    (5, 5, 12, 33, 5, 0.0, 1, False),
    (5, 4, 13, 64, 3, 0.3, 0, True),     # the object's grid away from most links
    (8, 8, 9, 64, 8, 0.0, 1, True),
    (8, 8, 700, 64, 4, 0.02, 0, False),
])
def test_penetration_of_realised_sets(F, dof, n_sets, dims, k, shift, sc, zero_len):
    from paper_2511_07418_amd import lg
    print(f"[penetrate] F={F} dof={dof} sets={n_sets} dims={dims} sc={sc}", flush=True)
    hand = _hand(F, dof, zero_len)
    fp = synth.FieldParams(samples=64, seed=1, grid=16, h=0.012, bins=32, grid_frame=synth.grid_frames(hand, 16, 0.012))
    field = lg.lg_build_field(hand, fp)
    obj = synth.sphere_object(0.04, 96)
    sdf = synth.sdf_sphere(0.04, dims=dims)
    P, D = 7, (n_sets + 6) // 7
    poses = synth.palm_poses(P, seed=F).reshape(P, 3, 4)
    poses[:, 0, 3] += shift
    poses = poses.reshape(P, 12)
    rng = np.random.default_rng(n_sets)
    fing = np.sort(np.stack([rng.permutation(F)[:k] for _ in range(P * D)]), axis=1)
    link = (fing * dof + rng.integers(0, dof, size=fing.shape)).astype(np.int8)
    pt = rng.integers(0, obj.n, size=fing.shape).astype(np.int32)
    ids = rng.permutation(P * D)[:n_sets].astype(np.int32)
    bad = ids.copy()
    if n_sets > 5:
        bad[3], bad[5] = -1, P * D
    ik = synth.IKParams(iters=3, self_collision=sc)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    vals = dev(sdf.values)
    pts, nrm = (dev(a) for a in obj.soa())
    r = lg.lg_realize(field, lg.sdf_struct(sdf, vals), pts, nrm, dev(poses), dev(pt.reshape(P, D, k)),
                      dev(link.reshape(P, D, k)), k, D, dev(bad), dev(np.array([n_sets], np.int32)), n_sets + 3, ik)
    torch.cuda.synchronize()
    q, depth, valid = (t.cpu().numpy()[:n_sets] for t in (r.q, r.depth, r.valid))
    err, ang = r.contact_err.cpu().numpy()[:n_sets], r.contact_ang.cpu().numpy()[:n_sets]
    for i in range(n_sets):
        if bad[i] < 0 or bad[i] >= P * D:
            assert np.isnan(depth[i]) and valid[i] == 0
            continue
        ref = oracle.penetration(hand, q[i], sdf, poses[bad[i] // D])
        if sc:
            ref = max(ref, oracle.self_penetration(hand, q[i]))
        if np.isinf(ref):
            assert depth[i] == ref
        else:
            assert abs(depth[i] - ref) <= 1e-5, (i, depth[i], ref)
        want = err[i].max() <= np.float32(ik.tol_pos) and ang[i].max() <= np.float32(ik.tol_ang) \
            and depth[i] <= np.float32(ik.margin)
        assert bool(valid[i]) == bool(want), i
    field.release()
