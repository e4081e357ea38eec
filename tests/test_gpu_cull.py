"""The bounded queries against the unbounded ones, bit for bit, where the culling
by occupied voxels and the launch's split can go wrong: point counts at the edges
of chunks and of the waves' units, every block size (few poses), windows whose
rows of voxels fill one word, part of one or several, chunks from a voxel to the
whole window across (ordered and shuffled points), poses at and beyond the
windows' faces, scaled and sheared poses, and points or normals that are not
finite.  The unbounded query is held to the oracle by the parity tests."""
import dataclasses

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _poses(P, kind):
    p = synth.palm_poses(P, seed=5).reshape(P, 3, 4).copy()
    rng = np.random.default_rng(3)
    if kind == "scaled":
        p[:, :, :3] *= rng.uniform(0.3, 4.0, size=(P, 1, 1))
    elif kind == "sheared":
        p[:, :, :3] += rng.normal(scale=0.7, size=(P, 3, 3))
    elif kind == "faces":
        p[:, :, 3] += rng.uniform(-0.12, 0.12, size=(P, 3))
    return p.reshape(P, 12).astype(np.float32)


@pytest.mark.parametrize("name,G,h,N,P,kind,order", [
    ("c1", 32, 0.004, 1, 3, "rigid", True),
    ("c1", 32, 0.004, 63, 256, "faces", True),
    ("c1", 36, 0.004, 65, 257, "rigid", True),
    ("c1", 32, 0.004, 2048, 600, "faces", False),   # shuffled: chunks as large as the object
    ("c2", 64, 0.003, 4097, 300, "rigid", True),
    ("c2", 40, 0.005, 16385, 130, "faces", True),
    ("c3", 128, 0.0015, 8191, 96, "rigid", True),
    ("c3", 64, 0.003, 20000, 64, "scaled", True),
    ("c3", 64, 0.003, 3000, 64, "sheared", True),
    ("c2", 64, 0.003, 5000, 64, "nonfinite", True),
])
def test_bounded_queries_equal_unbounded(name, G, h, N, P, kind, order):
    from paper_2511_07418_amd import lg
    print(f"[cull] {name} G={G} N={N} P={P} {kind}", flush=True)
    w = synth.workload(name, n_poses=1, n_points=N, samples=4096, with_sdf=False)
    fp = dataclasses.replace(w.field, grid=G, h=h, grid_frame=synth.grid_frames(w.hand, G, h))
    pts, nrm = (a.copy() for a in w.obj.soa())
    rng = np.random.default_rng(1)
    if not order:
        perm = rng.permutation(N)
        pts, nrm = np.ascontiguousarray(pts[:, perm]), np.ascontiguousarray(nrm[:, perm])
    if kind == "nonfinite":
        for a in (pts, nrm):
            for v in (np.nan, np.inf, -np.inf):
                a[rng.integers(0, 3, 40), rng.integers(0, N, 40)] = v
        nrm[:, rng.integers(0, N, 40)] = 0.0
    for frames in (fp.grid_frame, synth.grid_frames_finger_aligned(w.hand, G, h)):
        field = lg.lg_build_field(w.hand, dataclasses.replace(fp, grid_frame=frames), keep_witness=False)
        tp, tn, po = (torch.from_numpy(a).cuda() for a in (pts, nrm, _poses(P, kind)))
        b = lg.lg_chunk_bounds(tp)
        for got, ref in ((lg.lg_query_domains_bounded(field, tp, tn, po, b), lg.lg_query_domains(field, tp, tn, po)),
                         (lg.lg_query_domains_cone(field, tp, tn, po, 0.97, bounds=b),
                          lg.lg_query_domains_cone(field, tp, tn, po, 0.97))):
            torch.cuda.synchronize()
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
            words = ref[0].cpu().numpy().view(np.uint32)
            pop = np.unpackbits(words.view(np.uint8), axis=-1).sum(axis=-1)
            assert (pop == ref[1].cpu().numpy()).all()
            if kind not in ("scaled", "sheared") and P > 100:
                assert int(ref[1].sum()) > 0
        field.release()
