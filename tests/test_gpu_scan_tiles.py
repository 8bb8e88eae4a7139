"""The single-pass MFMA scan over its instantiations (K steps of d = 384, 512,
768 and 1,024, also dimensions that round up to them; one, two, four and eight
query tiles, full and ragged) against the dot4 scan: the same ranks and
scores, bit for bit, over deleted rows, a resumed read, and enough rows that
every wavefront takes several half-blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

D = [384, 500, 512, 768, 1000, 1024]


@pytest.fixture(scope="module", params=D)
def index(request):
    import torch
    from paper_2608_07152_amd import eahr as E
    d = request.param
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    n = 300_007
    centers = torch.randn(40, d, device="cuda", generator=g)
    lab = torch.randint(0, 40, (n,), device="cuda", generator=g)
    x = torch.randn(n, d, device="cuda", generator=g).mul_(0.6).add_(centers[lab])
    x /= x.norm(dim=1, keepdim=True)
    idx = E.pvs_build(x)
    gone = torch.randperm(n, device="cuda", generator=g)[: n // 10].cpu().numpy()
    E.pvs_delete(idx, gone)
    e = E.pvs_snapshot(idx)
    q = (centers[torch.randint(0, 40, (256,), device="cuda", generator=g)]
         + 0.6 * torch.randn(256, d, device="cuda", generator=g))
    return idx, e, q / q.norm(dim=1, keepdim=True)


@pytest.mark.parametrize("B", [9, 32, 33, 64, 65, 128, 129, 256])
def test_mfma_equals_dot4(index, monkeypatch, B):
    from paper_2608_07152_amd import eahr as E
    idx, e, q = index

    def read(path):
        monkeypatch.setenv("EAHR_SCAN_PATH", path)
        st = E.pvs_open(idx, q[:B].contiguous(), e)
        parts = [E.pvs_next(st, m) for m in (20, 200, 1500)]
        E.pvs_close(st)
        return [np.concatenate([p[i] for p in parts], axis=1) for i in (0, 1)]

    ids, sc = read("mfma")
    want_ids, want_sc = read("gemv")
    assert np.array_equal(ids, want_ids)
    assert np.array_equal(sc.view(np.int32), want_sc.view(np.int32))
