"""The queries' block sizes and forms: pose counts at the edges of each block size
give the rows that 16 poses at a time give, with and without chunk bounds (kernels of
their own on lattice windows), for hands of one to eight fingers and both bin counts.
The small queries are held to the oracle by the parity tests."""
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


@pytest.mark.parametrize("F,bins,N", [(1, 64, 700), (3, 32, 1029), (4, 64, 64), (5, 64, 1029), (8, 32, 333)])
@pytest.mark.parametrize("lattice", [True, False])
def test_rows_do_not_depend_on_the_block_size(F, bins, N, lattice):
    from paper_2511_07418_amd import lg
    print(f"[query blocks] F={F} bins={bins} N={N} lattice={lattice}", flush=True)
    hand = _hand(F, 3, False)
    frames = (synth.grid_frames if lattice else synth.grid_frames_finger_aligned)(hand, 32, 0.006)
    fp = synth.FieldParams(samples=8192, seed=1, grid=32, h=0.006, bins=bins, grid_frame=frames)
    field = lg.lg_build_field(hand, fp, keep_witness=False)
    obj = synth.sphere_object(0.04, N)
    pts, nrm = (torch.from_numpy(a).cuda() for a in obj.soa())
    bounds = lg.lg_chunk_bounds(pts)
    poses = synth.palm_poses(1025, seed=4).reshape(-1, 3, 4).copy()
    poses[:, :, 3] *= np.linspace(0.2, 1.0, 1025)[:, None]
    poses = torch.from_numpy(poses.reshape(-1, 12).astype(np.float32)).cuda()
    want = [lg.lg_query_domains(field, pts, nrm, poses[i:i + 16].contiguous()) for i in range(0, 1025, 16)]
    want = [torch.cat([w[j] for w in want]) for j in range(2)]
    assert int(want[1].sum()) > 0
    for P in (255, 256, 257, 1023, 1024, 1025):
        po = poses[:P].contiguous()
        for got in (lg.lg_query_domains(field, pts, nrm, po), lg.lg_query_domains_bounded(field, pts, nrm, po, bounds)):
            torch.cuda.synchronize()
            assert torch.equal(got[0], want[0][:P]) and torch.equal(got[1], want[1][:P]), P
    field.release()
