"""More poses than one launch takes (a grid holds fewer than 2^32 threads; a pose is a
block of up to 256): the rows of every part of such a batch equal those of a small batch
of the same poses, for the queries, the draws with their verdicts, the second contact
round, and both servers."""
import dataclasses

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

P = (1 << 24) + 77


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2511_07418_amd import lg
    w = synth.workload("c1", n_poses=2048, n_points=32)
    field = lg.lg_build_field(w.hand, w.field, keep_witness=False)
    pts, nrm = (torch.from_numpy(a).cuda() for a in w.obj.soa())
    some = torch.from_numpy(w.poses).cuda()
    poses = some.repeat((P + 2047) // 2048, 1)[:P].contiguous()
    yield lg, w, field, pts, nrm, some, poses
    field.release()


def _same_rows(big, small):
    """row i of big is row i % len(small) of small"""
    n = len(small)
    full = P // n * n
    return bool((big[:full].view(-1, *small.shape) == small).all()) and torch.equal(big[full:], small[:P - full])


@pytest.mark.parametrize("form", ["plain", "bounded", "cone"])
def test_queries(env, form):
    lg, w, field, pts, nrm, some, poses = env
    print(f"[many poses] {form}", flush=True)
    bounds = lg.lg_chunk_bounds(pts)

    def query(po, b, c):
        if form == "plain":
            return lg.lg_query_domains(field, pts, nrm, po, b, c)
        if form == "bounded":
            return lg.lg_query_domains_bounded(field, pts, nrm, po, bounds, b, c)
        return lg.lg_query_domains_cone(field, pts, nrm, po, 0.9, b, c)

    want = query(some, None, None)
    bits = torch.full((P, field.n_fingers, 1), -5, dtype=torch.int32, device="cuda")
    count = torch.full((P, field.n_fingers), -5, dtype=torch.int32, device="cuda")
    query(poses, bits, count)
    torch.cuda.synchronize()
    assert int(want[1].sum()) > 0
    assert _same_rows(bits, want[0]) and _same_rows(count, want[1])


def test_draws_and_second_round(env):
    lg, w, field, pts, nrm, some, poses = env
    print("[many poses] draws", flush=True)
    bits, count = lg.lg_query_domains(field, pts, nrm, poses)
    sp = dataclasses.replace(w.search, draws=1, k=2)
    b = lg.lg_search(field, pts, nrm, poses, bits, count, sp)
    e = lg.lg_search_extend(field, pts, nrm, poses, bits, count, sp, b, 1, request_id=7)
    torch.cuda.synchronize()
    for i in (0, (1 << 23) - 100, (1 << 24) - 1000, P - 1000):   # each launch's part and their borders
        s = slice(i, i + 1000)
        part = dataclasses.replace(sp, pose_offset=i)
        args = (field, pts, nrm, poses[s].contiguous(), bits[s].contiguous(), count[s].contiguous(), part)
        b1 = lg.lg_search(*args)
        e1 = lg.lg_search_extend(*args, b1, 1, request_id=7)
        torch.cuda.synchronize()
        for big, small in ((b, b1), (e, e1)):
            assert int((small.set_pt >= 0).sum()) > 0
            for n in ("set_pt", "set_link", "verdict"):
                assert torch.equal(getattr(big, n)[s], getattr(small, n)), (i, n)
            assert torch.equal(torch.nan_to_num(big.tstar[s], nan=-1.0), torch.nan_to_num(small.tstar, nan=-1.0))
    for x in (b, e):
        n = int(x.n_acc)
        assert n > 0 and torch.equal(x.acc_list[:n].long(), torch.nonzero(x.verdict.flatten()).flatten())


def test_servers(env):
    lg, w, field, pts, nrm, some, poses = env
    print("[many poses] servers", flush=True)
    sp = dataclasses.replace(w.search, draws=1, k=2)
    pipe_bits, pipe_count = lg.lg_query_domains(field, pts, nrm, poses)
    b = lg.lg_search(field, pts, nrm, poses, pipe_bits, pipe_count, dataclasses.replace(sp, request_id=3))
    torch.cuda.synchronize()
    n = int(b.n_acc)
    want = (n, lg.accepted_hash(3, b.acc_list[:n].cpu().numpy()))
    assert n > 0
    host = poses.cpu().numpy()
    for batched in (False, True):
        srv = lg.Server(budget_bytes=12 << 30, max_active=2, chunk_poses=1 << 25, batched=batched)
        req, keep = srv.make_request(field, w.obj.pts, w.obj.nrm, host, sp, request_id=3)
        r = srv.wait(srv.submit(req), 100.0)
        srv.destroy()
        assert r["state"] == lg.LG_REQ_DONE
        assert (r["n_acc"], r["acc_hash"]) == want, batched
