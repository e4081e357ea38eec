"""The batched server's kernel forms against the per-stream server (count, valid count
and hash of the accepted ids): the compaction over chunks and with a scan between, for
poses and for sets, beside members of a few flags; the 22-joint hand's query, joint
steps and penetration, with and without self-collision, beside smaller hands; and one
mix in which every kernel class has members (fingers, bin words, windows, contacts,
cone edges, joints per finger, self-collision), so that a batch needs as many member
lists as its table may hold."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.test_gpu_penetrate import _hand

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _serve(lg, specs, batched, chunk_poses):
    """specs: (field, points, normals, poses, search, ik or None, sdf); results in order, stats"""
    srv = lg.Server(budget_bytes=16 << 30, max_active=64, chunk_poses=chunk_poses, batched=batched, batch_slots=1)
    keep, tickets = [], []
    for i, (f, p, n, poses, sp, ik, sdf) in enumerate(specs):
        kw = dict(ik=ik, sdf=sdf) if ik is not None else {}
        keep.append(srv.make_request(f, p, n, poses, sp, request_id=40 + i, **kw))
        tickets.append(srv.submit(keep[-1][0]))
    out = [srv.wait(t, 100.0) for t in tickets]
    st = srv.stats()
    srv.destroy()
    assert all(r["state"] == lg.LG_REQ_DONE for r in out), [r["status"] for r in out]
    return [(r["n_acc"], r["n_valid"], r["acc_hash"]) for r in out], st


def _both(lg, specs, chunk_poses):
    # a first request of some milliseconds: the others wait for the one batch slot and share the next batch
    w = synth.workload("c1", n_poses=1024, n_points=64)
    field = lg.lg_build_field(w.hand, w.field, keep_witness=False)
    first = (field, w.obj.pts, w.obj.nrm, w.poses, dataclasses.replace(w.search, draws=16384), None, None)
    want, _ = _serve(lg, [first] + specs, False, chunk_poses)
    got, st = _serve(lg, [first] + specs, True, chunk_poses)
    field.release()
    assert got == want
    assert st["batches"] < st["batched_chunks"]
    return got[1:]


@pytest.mark.parametrize("P,D,chunk_poses", [
    (4096, 16, 4096),             # 65,536 sets: count and scatter; the poses in one block
    (33000, 3, 40000),            # poses and sets by count and scatter
    (1025, 16384, 4096),          # 2,050 chunks of 8,192 flags: a scan between
])
def test_compaction_forms(P, D, chunk_poses):
    from paper_2511_07418_amd import lg
    print(f"[serve forms] P={P} D={D}", flush=True)
    w = synth.workload("c1", n_poses=4096, n_points=64)
    field = lg.lg_build_field(w.hand, w.field, keep_witness=False)
    big = np.tile(w.poses, ((P + 4095) // 4096, 1))[:P]
    sp = dataclasses.replace(w.search, draws=D)
    small = dataclasses.replace(w.search, draws=7)
    specs = [(field, w.obj.pts, w.obj.nrm, big, sp, None, None),
             (field, w.obj.pts, w.obj.nrm, w.poses[:300], small, None, None),
             (field, w.obj.pts[:33], w.obj.nrm[:33], w.poses[:1], w.search, None, None)]
    got = _both(lg, specs, chunk_poses)
    assert got[0][0] > 0 and got[1][0] > 0
    field.release()


def test_22_joint_hand_beside_smaller_ones():
    from paper_2511_07418_amd import lg
    print("[serve forms] 22 joints", flush=True)
    w3 = synth.workload("c3", n_poses=3000, n_points=20011, samples=65536)
    w2 = synth.workload("c2", n_poses=700, n_points=5003, samples=65536, with_sdf=True)
    w1 = synth.workload("c1", n_poses=500, with_sdf=True)
    f3, f2, f1 = (lg.lg_build_field(w.hand, w.field) for w in (w3, w2, w1))
    specs = []
    for w, f, d in ((w3, f3, 32), (w1, f1, 16), (w3, f3, 5), (w2, f2, 32)):
        for sc in (0, 1):
            specs.append((f, w.obj.pts, w.obj.nrm, w.poses, dataclasses.replace(w.search, draws=d),
                          dataclasses.replace(w.ik, self_collision=sc, margin=0.004), w.sdf))
    got = _both(lg, specs, 4096)
    assert all(g[0] > 0 for g in got)
    assert got[0][1] > got[1][1] > 0      # self-collision rejects grasps
    for f in (f1, f2, f3):
        f.release()


def test_every_kernel_class_in_one_mix():
    from paper_2511_07418_amd import lg
    print("[serve forms] every class", flush=True)
    obj = synth.sphere_object(0.04, 500)
    sdf = synth.sdf_sphere(0.04, dims=33)
    poses = synth.palm_poses(64, seed=3).reshape(-1, 3, 4).copy()
    poses[:, :, 3] *= 0.5
    poses = poses.reshape(-1, 12).astype(np.float32)
    base = synth.workload("c1", n_poses=1).search
    fields, specs = [], []
    for i, (F, dof) in enumerate(((3, 4), (4, 5), (5, 6), (8, 8))):
        hand = _hand(F, dof, False)
        for bins in (32, 64):
            for frames in (synth.grid_frames, synth.grid_frames_finger_aligned):
                fp = synth.FieldParams(samples=4096, seed=1, grid=32, h=0.006, bins=bins,
                                       grid_frame=frames(hand, 32, 0.006))
                field = lg.lg_build_field(hand, fp)
                fields.append(field)
                j = len(fields)
                for sc, m in ((j & 1, 8), (1 - (j & 1), 6)):
                    k = (min(F, 3), min(F, 4), min(F, 5), (6, 8)[sc] if F == 8 else F)[(j + i) % 4]
                    sp = dataclasses.replace(base, draws=6, k=k, m_edges=m)
                    specs.append((field, obj.pts, obj.nrm, poses, sp, synth.IKParams(iters=3, self_collision=sc), sdf))
    assert len(specs) <= 64
    assert {s[4].k for s in specs} >= {3, 4, 5, 6, 8}
    got = _both(lg, specs, 64)
    assert sum(g[0] for g in got) > 0
    for f in fields:
        f.release()
