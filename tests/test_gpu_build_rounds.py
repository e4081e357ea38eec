"""Field builds at the edges of their rounds and parts: one sample, counts around a
block, around the first round (4,096) and its doublings, link surfaces that do not
divide into the parts, and windows per finger.  Bars of the field build: bits sure
subset of GPU subset of sure | maybe, witnesses between the oracle's bounds and
present exactly where a bit is set; a build without witnesses has the same bits."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import _check_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("name,samples,n_surf,G,h", [
    ("c1", 1, 256, 32, 0.004),
    ("c1", 255, 7, 36, 0.004),
    ("c1", 4096, 256, 32, 0.004),
    ("c1", 4097, 33, 32, 0.004),
    ("c2", 8193, 17, 64, 0.003),
    ("c3", 16641, 5, 40, 0.005),
])
def test_build_rounds(name, samples, n_surf, G, h):
    from paper_2511_07418_amd import lg
    print(f"[build] {name} S={samples} n_surf={n_surf} G={G}", flush=True)
    w = synth.workload(name, n_poses=1, n_points=64, samples=samples, with_sdf=False)
    hand = {"c1": synth.hand_c1, "c2": synth.hand_c2, "c3": synth.hand_c3}[name](n_surf=n_surf)
    frames = (synth.grid_frames if samples % 2 else synth.grid_frames_finger_aligned)(hand, G, h)
    w = dataclasses.replace(w, hand=hand, field=dataclasses.replace(w.field, grid=G, h=h, grid_frame=frames))
    field = lg.lg_build_field(hand, w.field, keep_witness=True)
    _check_field(w, field)
    bits, _ = field.export()
    plain = lg.lg_build_field(hand, w.field, keep_witness=False)
    assert np.array_equal(plain.export()[0], bits)
    a, b = field.info(), plain.info()
    assert a["dropped"] == b["dropped"] and a["bits_set"] == b["bits_set"]
    assert a["bits_set"] == int(np.unpackbits(bits.view(np.uint8)).sum())
    field.release()
    plain.release()
