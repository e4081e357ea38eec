"""Compactions against NumPy at the edges of their forms: one block (up to 32,768
flags), count and scatter over chunks of 8,192 with the blocks adding up the counts
themselves (up to 2,048 chunks), and with a scan between; counts around each limit,
all, no and few flags, and flag arrays at a 4-byte alignment.  Through the
list of unstable sets (whole draw, verdict 0), which compacts an arbitrary flag."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("n,share", [
    (1, 1.0), (1, 0.0), (15, 0.5), (16, 1.0), (1025, 0.3), (16385, 0.5), (32768, 1.0), (32769, 0.01),
    (40961, 0.5), (8192 * 12, 0.0), (2048 * 8192, 0.02), (2048 * 8192 + 1, 0.02),
])
@pytest.mark.parametrize("shift", [0, 4])
def test_compaction(n, share, shift):
    from paper_2511_07418_amd import lg
    print(f"[compact] n={n} share={share} shift={shift}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    keep = torch.rand(n, generator=g, device="cuda") < share
    set_pt = torch.where(keep, 0, -1).to(torch.int32)
    set_link = torch.zeros(n, dtype=torch.int8, device="cuda")
    verdict = torch.zeros(n, dtype=torch.uint8, device="cuda")
    L = lg.lib()
    nb = int(L.lg_compact_unstable_workspace_bytes(n, 1))
    ws = torch.empty(nb + 256, dtype=torch.uint8, device="cuda")[shift:]
    lst = torch.full((n + 8,), -5, dtype=torch.int32, device="cuda")
    tot = torch.full((1,), -5, dtype=torch.int32, device="cuda")
    st = L.lg_compact_unstable(lg._ptr(set_pt), lg._ptr(set_link), lg._ptr(verdict), n, 1, 1, lg._ptr(lst),
                               lg._ptr(tot), lg._ptr(ws), nb, None)
    assert st == lg.LG_OK
    torch.cuda.synchronize()
    want = torch.nonzero(keep).flatten().to(torch.int32)
    assert int(tot) == want.numel()
    assert torch.equal(lst[:want.numel()], want) and bool((lst[want.numel():] == -5).all())
