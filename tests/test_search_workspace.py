"""The workspace that a search with contact-point optimisation asks for grows with the
sets by what its kernels use: the verdict's lists, the candidate ids (4 bytes per set,
contact and candidate), 36 bytes per set and 36 per candidate, and nothing beyond."""
import ctypes as C
import dataclasses

import pytest

import synth


@pytest.mark.parametrize("draws,k,inner", [(64, 5, 8), (33, 3, 1), (16, 8, 16)])
def test_growth_per_set(draws, k, inner):
    lg = pytest.importorskip("paper_2511_07418_amd.lg")
    base = dataclasses.replace(synth.workload("c1", n_poses=1).search, draws=draws, k=k, opt_inner=inner)
    p0 = lg.search_params(base)
    p1 = lg.search_params(dataclasses.replace(base, opt_outer=1))
    P = 8192

    def grown(p):
        return [lg.lib().lg_search_workspace_bytes(4096, n, C.byref(p)) for n in (P, 2 * P)]

    (a0, b0), (a1, b1) = grown(p0), grown(p1)
    sets = P * draws
    used = sets * (4 * k * inner + 36 + 36 * inner)
    assert 0 <= (b1 - a1) - (b0 - a0) - used <= 8 * 256     # the pieces' alignment
