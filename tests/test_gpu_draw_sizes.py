"""More contacts of one pose than 32 bits count (draws x contacts above 2^31), and as
many sets as there may be: every set's points and links are written, for a pose
without usable domains and for one whose domains hold no bit (each draw looks one up
and finds none)."""
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


@pytest.mark.parametrize("D,k,count", [((1 << 28) + 1, 8, 0), ((1 << 28) + 1, 8, 1), ((1 << 31) - 1, 1, 0)])
def test_every_contact_of_a_huge_draw_is_written(D, k, count):
    from paper_2511_07418_amd import lg
    from tests.test_gpu_penetrate import _hand
    F, N = 8, 32
    print(f"[draw sizes] D={D} k={k} count={count}", flush=True)
    hand = _hand(F, 1, False)
    fp = synth.FieldParams(samples=64, seed=1, grid=16, h=0.012, bins=32, grid_frame=synth.grid_frames(hand, 16, 0.012))
    field = lg.lg_build_field(hand, fp, keep_witness=False)
    obj = synth.sphere_object(0.04, N)
    pts, nrm = (torch.from_numpy(a).cuda() for a in obj.soa())
    sp = dataclasses.replace(synth.workload("c1", n_poses=1).search, draws=D, k=k)
    bits = torch.zeros((1, F, 1), dtype=torch.int32, device="cuda")
    counts = torch.full((1, F), count, dtype=torch.int32, device="cuda")
    b = lg.SearchBuffers(1, sp, "cuda", n_points=N)
    b.set_pt.fill_(5)
    b.set_link.fill_(5)
    lg.lg_search(field, pts, nrm, torch.from_numpy(synth.palm_poses(1, seed=2)).cuda(), bits, counts, sp, bufs=b)
    torch.cuda.synchronize()
    for name in ("set_pt", "set_link"):
        v = getattr(b, name).flatten()
        assert v.numel() == D * k
        assert all(bool((v[i:i + (1 << 28)] == -1).all()) for i in range(0, v.numel(), 1 << 28)), name
    assert not bool(b.verdict.any()) and bool(b.tstar.isnan().all()) and int(b.n_acc) == 0
    field.release()
