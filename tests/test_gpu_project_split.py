"""The projections' split over waves (Alg. 2): several sets per wave, one set, and
parts of a set's candidates give each pose the same points.  The first poses of a large
batch, run alone in batches that take each form, must get the batch's sets, verdicts
and t*; candidate counts that are and are not multiples of a group's eight."""
import dataclasses

import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("name,k,inner,draws", [("c1", 3, 5, 64), ("c1", 2, 4, 33), ("c1", 1, 1, 64), ("c2", 4, 16, 64)])
def test_small_batches_give_the_points_of_a_large_one(name, k, inner, draws):
    from paper_2511_07418_amd import lg
    print(f"[project split] {name} k={k} inner={inner} draws={draws}", flush=True)
    w = synth.workload(name, n_poses=12000, n_points=2048, samples=16384, with_sdf=False)
    sp = dataclasses.replace(w.search, k=k, draws=draws, opt_outer=1, opt_inner=inner, opt_sigma=0.004)
    field = lg.lg_build_field(w.hand, w.field, keep_witness=False)
    pts, nrm = (torch.from_numpy(a).cuda() for a in w.obj.soa())
    poses = torch.from_numpy(w.poses).cuda()
    bits, count = lg.lg_query_domains(field, pts, nrm, poses)
    torch.cuda.synchronize()
    # poses that draw sets, so that the batch's size is the launch's
    use = torch.nonzero((count > 0).sum(dim=1) >= k).flatten()[:1200]
    assert use.numel() >= 600, use.numel()
    poses, bits, count = (t[use].contiguous() for t in (poses, bits, count))

    def run(P):
        b = lg.lg_search(field, pts, nrm, poses[:P].contiguous(), bits[:P].contiguous(), count[:P].contiguous(), sp)
        torch.cuda.synchronize()
        return b.set_pt, b.set_link, b.verdict, b.tstar

    want = run(len(poses))
    assert int((want[0] >= 0).sum()) > 0
    for P in (1, 3, 29, 113, 300, 449):
        for g, v in zip(run(P), want):
            assert torch.equal(torch.nan_to_num(g, nan=-1.0) if g.dtype == torch.float64 else g,
                               torch.nan_to_num(v[:P], nan=-1.0) if v.dtype == torch.float64 else v[:P]), P
    field.release()
