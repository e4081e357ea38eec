"""The force-closure LPs of a launch against the oracle's tableau simplex at the
edges of the launch's work split: one LP, fewer LPs than waves, waves whose lanes
take several LPs each, every cone kind (the 8-edge closed-form pricing, the
general edge loop), frictionless cones, and contacts drawn twice (degenerate
bases).  Domains hold every object point, so the sets are arbitrary point tuples.
Bars as for every search: verdicts exact outside |t* - eps| <= 1e-6, t* within
1e-9."""
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


@pytest.mark.parametrize("name,P,D,N,m,mu", [
    ("c1", 1, 1, 64, 8, 0.5),
    ("c1", 3, 7, 97, 8, 0.5),
    ("c2", 17, 16, 300, 16, 0.5),
    ("c3", 9, 64, 257, 3, 0.3),
    ("c3", 5, 33, 65, 8, 0.0),
    ("c3", 40, 64, 3, 8, 0.8),       # three points: contacts repeat within a set
    ("c1", 300, 512, 2048, 8, 0.5),  # 75 LPs per wave
])
def test_lp_launch_against_the_oracle(name, P, D, N, m, mu):
    from paper_2511_07418_amd import lg
    print(f"[lp] {name} P={P} D={D} N={N} m={m} mu={mu}", flush=True)
    w = synth.workload(name, n_poses=P, n_points=N, samples=256, draws=D, with_sdf=False)
    sp = dataclasses.replace(w.search, m_edges=m, mu=mu)
    F, NW = w.hand.n_fingers, (N + 31) // 32
    words = np.full((P, F, NW), 0xFFFFFFFF, np.uint32)
    if N % 32:
        words[..., -1] = (1 << (N % 32)) - 1
    field = lg.lg_build_field(w.hand, w.field, keep_witness=False)
    soa = [torch.from_numpy(a).cuda() for a in w.obj.soa()]
    bufs = lg.lg_search(field, soa[0], soa[1], torch.from_numpy(w.poses).cuda(),
                        torch.from_numpy(words.view(np.int32)).cuda(),
                        torch.full((P, F), N, dtype=torch.int32, device="cuda"), sp)
    torch.cuda.synchronize()
    spt = bufs.set_pt.cpu().numpy()
    assert spt.min() >= 0 and spt.max() < N
    V = oracle.verdicts(w.obj.pts, w.obj.nrm, spt, sp)
    ver, ts = bufs.verdict.cpu().numpy().reshape(-1), bufs.tstar.cpu().numpy().reshape(-1)
    assert np.abs(ts - V["tstar"]).max() <= 1e-9
    assert ((ver != V["verdict"]) & (V["vflag"] == 0)).sum() == 0
    n = int(bufs.n_acc.item())
    assert (bufs.acc_list[:n].cpu().numpy() == np.flatnonzero(ver)).all()
    field.release()
