"""Draws and reverse lookups against the oracle on random domains: point counts at
the edges of words, superblocks (8 words) and scans (64 superblocks), single-point
and almost empty domains, sets that are not a multiple of the block, fewer contacts
than fingers, and windows with and without a common lattice.  Points must be
identical; links outside the oracle's rounding flags."""
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


@pytest.mark.parametrize("name,N,P,D,k,density,lattice", [
    ("c1", 1, 4, 5, 3, 1.0, True),
    ("c1", 31, 9, 100, 2, 0.2, True),
    ("c2", 33, 20, 16, 4, 0.1, False),
    ("c2", 257, 20, 33, 3, 0.02, True),
    ("c3", 2049, 12, 64, 5, 0.004, True),
    ("c3", 16384, 8, 77, 4, 0.0005, False),
    ("c3", 16415, 8, 64, 5, 0.5, True),
])
def test_draws_on_random_domains(name, N, P, D, k, density, lattice):
    from paper_2511_07418_amd import lg
    print(f"[draw] {name} N={N} P={P} D={D} k={k}", flush=True)
    w = synth.workload(name, n_poses=P, n_points=N, samples=2048, draws=D, with_sdf=False)
    if not lattice:
        w.field.grid_frame = synth.grid_frames_finger_aligned(w.hand, w.field.grid, w.field.h)
    sp = dataclasses.replace(w.search, k=k)
    F, NW = w.hand.n_fingers, (N + 31) // 32
    rng = np.random.default_rng(N)
    bits = rng.uniform(size=(P, F, N)) < density
    bits[0, :, :] = False
    bits[0, :, N - 1] = True                       # one point, the last
    words = np.zeros((P, F, NW * 32), np.uint8)
    words[:, :, :N] = bits
    words = np.packbits(words, axis=2, bitorder="little").view(np.uint32).reshape(P, F, NW)
    count = bits.sum(axis=2).astype(np.uint32)
    ref = oracle.build_field(w.hand, w.field, flags=False)
    field = lg.lg_field_import(w.hand, w.field, ref["bits"])
    pts, nrm = (torch.from_numpy(a).cuda() for a in w.obj.soa())
    b = lg.lg_search(field, pts, nrm, torch.from_numpy(w.poses).cuda(), torch.from_numpy(words.view(np.int32)).cuda(),
                     torch.from_numpy(count.view(np.int32)).cuda(), sp)
    torch.cuda.synchronize()
    o_pt, o_ln, flag = oracle.draw(w.hand, w.field, ref["bits"], w.obj.pts, w.obj.nrm, w.poses, words, count, sp,
                                   link_flags=True)
    assert np.array_equal(b.set_pt.cpu().numpy(), o_pt)
    mis = b.set_link.cpu().numpy().astype(np.int32) != o_ln
    assert (mis & (flag == 0)).sum() == 0 and mis.sum() <= max(1, 1e-3 * mis.size)
    assert (o_pt >= 0).any()
    field.release()
