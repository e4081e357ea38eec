"""Penetration of hands whose link segments limit a wave's sets (fewer than one per
finger's lane): lists around whole waves, fewer sets per wave, several grids' worth,
against the same sets in a short list (held to the oracle by the penetration test).  The
same bits."""
import pytest

from tests.test_gpu_penetrate_many import _gpu, test_many_sets_give_the_bits_of_few as _same_bits  # noqa: F401

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# sets per wave: 1 x 8 39, 2 x 6 26, 2 x 8 19, 6 x 7 7, 8 x 8 4 (4,096 waves)
@pytest.mark.parametrize("F,dof,n_sets", [(1, 8, 4096 * 39 + 40), (2, 6, 4096 * 26 - 1), (2, 8, 4096 * 19 + 1),
                                          (6, 7, 4096 * 7 + 8), (6, 7, 4096 * 5 + 1), (8, 8, 4096 * 4),
                                          (8, 8, 4096 * 3 - 1)])
@pytest.mark.parametrize("sc", [0, 1])
def test_wave_of_fewer_sets(F, dof, n_sets, sc):
    _same_bits(F, dof, n_sets, sc)
