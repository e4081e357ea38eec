"""Penetration with many sets per wave (several side by side) against the same sets in
a short list (one after another, held to the oracle by the penetration test): hands of
one to eight fingers, numbers of sets that leave the last wave or its last group
short, ids outside the batch, with and without the hand's self-collision.  The same
bits."""
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


@pytest.mark.parametrize("F,dof,n_sets", [(1, 8, 40001), (2, 6, 40003), (3, 3, 131072), (5, 4, 40001), (7, 2, 33001),
                                          (8, 8, 32769)])
@pytest.mark.parametrize("sc", [0, 1])
def test_many_sets_give_the_bits_of_few(F, dof, n_sets, sc):
    from paper_2511_07418_amd import lg
    print(f"[penetrate many] F={F} dof={dof} sets={n_sets} sc={sc}", flush=True)
    hand = _hand(F, dof, False)
    fp = synth.FieldParams(samples=64, seed=1, grid=16, h=0.012, bins=32, grid_frame=synth.grid_frames(hand, 16, 0.012))
    field = lg.lg_build_field(hand, fp)
    obj = synth.sphere_object(0.04, 96)
    sdf = synth.sdf_sphere(0.04, dims=33)
    P, D, few = 11, 16, 150
    poses = synth.palm_poses(P, seed=F).reshape(P, 3, 4)
    poses[:, 0, 3] += np.linspace(0.0, 0.2, P)   # some sets away from the grid
    rng = np.random.default_rng(F)
    fing = np.sort(np.stack([rng.permutation(F)[:min(F, 3)] for _ in range(P * D)]), axis=1)
    k = fing.shape[1]
    link = (fing * dof + rng.integers(0, dof, size=fing.shape)).astype(np.int8)
    pt = rng.integers(0, obj.n, size=fing.shape).astype(np.int32)
    ids = rng.permutation(P * D)[:few].astype(np.int32)
    ids[[3, 77]] = -1, P * D
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    vals = dev(sdf.values)
    pts, nrm = (dev(a) for a in obj.soa())

    def run(lst):
        n = len(lst)
        r = lg.lg_realize(field, lg.sdf_struct(sdf, vals), pts, nrm, dev(poses.reshape(P, 12)), dev(pt.reshape(P, D, k)),
                          dev(link.reshape(P, D, k)), k, D, dev(lst), dev(np.array([n], np.int32)), n,
                          synth.IKParams(iters=3, self_collision=sc))
        torch.cuda.synchronize()
        return [t.view(torch.uint8 if t.dtype == torch.uint8 else torch.int32).cpu().numpy()
                for t in (r.q, r.depth, r.valid)]

    want = run(ids)
    at = np.arange(n_sets) % few
    got = run(ids[at])
    for g, w in zip(got, want):
        assert np.array_equal(g, w[at])
    assert np.isfinite(want[1].view(np.float32)).sum() > few // 4
    field.release()
