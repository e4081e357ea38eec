"""The proposer at the edges of its launches: batches around the 32 objects a
workgroup takes through the head, point counts around a workgroup's steps, and
objects with no targets, with more than the 64 a workgroup holds at a time, and
with one.

Forward: an object's outputs do not depend on its batch or on how the encoder's
points are split over workgroups (the same products in the same order, a maximum
with the lowest point on ties), so every batch equals the objects one at a time,
bit for bit.  Backward: the loss and the gradient of a batch are the target-count-
weighted means of the objects' own; the chain rounds two operands of each of its
three products to bfloat16 (at most 2^-9 each, of values that scale with the
batch), 6 * 2^-9 = 1.2 % of the summed terms, held to the backward's bar of 3e-2
of each tensor's largest entry; the loss to 1e-5 (FP32 sums)."""
import numpy as np
import pytest

from oracle import proposer as op

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2511_07418_amd import lg as _lg
    return _lg


def _clouds(B, Np, seed):
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(B, Np, 3))
    v /= np.linalg.norm(v, axis=2, keepdims=True)
    ax = rng.uniform(0.02, 0.08, size=(B, 1, 3))
    n = v / ax
    n /= np.linalg.norm(n, axis=2, keepdims=True)
    return torch.from_numpy(np.concatenate([ax * v, n], axis=2).astype(np.float32)).cuda()


@pytest.mark.parametrize("B,Np", [(1, 1), (31, 511), (32, 512), (33, 513), (65, 1025), (300, 2049)])
def test_forward_of_a_batch_is_that_of_its_objects(lg, B, Np):
    prop = lg.Proposer(max_batch=B, max_points=Np, max_targets=1, seed=3)
    x = _clouds(B, Np, seed=B)
    whole = prop.forward(x)
    for b in sorted({0, B // 2, B - 1}):
        one = prop.forward(x[b:b + 1].contiguous())
        torch.cuda.synchronize()
        for k in ("out", "feat", "arg"):
            assert torch.equal(whole[k][b], one[k][0]), (b, k)
    prop.release()


@pytest.mark.parametrize("counts", [[1], [64, 65, 0, 200], [7] * 31 + [0, 130] + [3] * 2])
def test_backward_of_a_batch_is_the_mean_of_its_objects(lg, counts):
    B, Np, T = len(counts), 300, sum(counts)
    prop = lg.Proposer(max_batch=B, max_points=Np, max_targets=T, seed=4)
    x = _clouds(B, Np, seed=9)
    y = torch.from_numpy(np.random.default_rng(2).normal(0, 0.7, size=(T, 9)).astype(np.float32)).cuda()
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    loss, grad = prop.backward(x, y, torch.from_numpy(off).cuda())
    ref, ref_loss = np.zeros(prop.n_params), 0.0
    for b in range(B):
        if counts[b] == 0:
            continue
        lb, gb = prop.backward(x[b:b + 1].contiguous(), y[off[b]:off[b + 1]].contiguous(),
                               torch.tensor([0, counts[b]], dtype=torch.int32, device="cuda"))
        ref += gb.cpu().numpy().astype(np.float64) * counts[b] / T
        ref_loss += float(lb) * counts[b] / T
    torch.cuda.synchronize()
    assert float(loss) == pytest.approx(ref_loss, rel=1e-5)
    got, want = op.unflatten(grad.cpu().numpy().astype(np.float64)), op.unflatten(ref)
    for t, _ in op.LAYERS:
        assert np.abs(got[t] - want[t]).max() <= 3e-2 * np.abs(want[t]).max() + 1e-9, t
    prop.release()
