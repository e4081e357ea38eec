"""The candidates' projection onto the domains (Alg. 2) at the edges of its cell
grid and its searches, against the oracle, which reads every point: mutations far
shorter than the point spacing (one cell's points), of several millimetres over
sparse and over dense points (own row, rows around it, the wave's rings), and as
large as the object (candidates outside the grid, rings up to the limit); point
counts that are not multiples of a wave, and one point per cell row.  The same
points, up to the outcomes of near-ties that the oracle lists."""
import dataclasses

import pytest

import synth
from tests.test_gpu_optimize import _opt_check

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("sigma,n_points", [(5e-4, 2048), (5e-4, 40001), (0.003, 40001), (0.02, 2048), (0.02, 333),
                                            (0.15, 2048), (1e-6, 333)])
def test_projection(sigma, n_points):
    print(f"[project] sigma={sigma} n_points={n_points}", flush=True)
    w = synth.workload("c1", n_poses=24, n_points=n_points)
    _opt_check(w, dataclasses.replace(w.search, opt_outer=1, opt_inner=5, opt_sigma=sigma), max_flag_frac=1.0)
