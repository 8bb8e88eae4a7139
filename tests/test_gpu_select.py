"""Threshold selection from the sample (histogram windows over 16-bit codes): the
prefix stays exact and the scans stay selective where the k-th value lies in
the first window, far below it (one row of a huge norm, also where the codes
are bfloat16's), below zero (every score negative), at zero, and where every
value is the same; for the
one-query, small-batch, one-, four- and eight-tile sample passes and for
samples of every block (small n) and of some (large n)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(E, x, q, m, max_candidates):
    idx = E.pvs_build(x)
    st = E.pvs_open(idx, q)
    ids, sc, cnt, _ = E.pvs_next(st, m)
    assert np.all(cnt == min(m, len(x)))
    rows = np.arange(len(x))
    for b in range(0, len(q), max(1, len(q) // 5)):
        s = E.pvs_scores(st, b, rows)
        want = np.lexsort((rows, -s.astype(np.float64)))[:m]
        assert np.array_equal(ids[b], want)
        assert np.array_equal(sc[b] + 0.0, s[want] + 0.0)
    st_ = E.pvs_stats(st)
    assert st_["candidates"] <= max_candidates * len(q), st_


@pytest.mark.parametrize("n,d,B", [(5000, 48, 1), (5000, 48, 20), (300_001, 16, 1), (300_001, 16, 7),
                                   (290_000, 64, 40), (270_000, 384, 40), (270_000, 384, 200), (262_144, 64, 140)])
@pytest.mark.parametrize("kind", ["plain", "outlier", "sentinel", "tiny", "negative", "zero", "same"])
def test_selected_threshold(n, d, B, kind):
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(n + d + B)
    x = rng.standard_normal((n, d), dtype=np.float32)
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    q = rng.standard_normal((B, d), dtype=np.float32)
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    m = 300
    # the first scan certifies the request or min(2^17, n / 16) ranks over its
    # queries, 1.25 times or five standard deviations above that, and the widest
    # intervals here (d = 384) reach 2.5 times as many rows: at most 4.4 times
    # the larger of the two in all
    limit = 6 * max(m, min(1 << 17, n // 16) // B)
    if kind == "outlier":
        x[n // 2] *= 1e4       # the k-th score is below 1e-4 of the index's largest bound
    elif kind == "sentinel":
        x[n // 2] *= 1e15
    elif kind == "tiny":
        x *= 1e-12
        x[n // 2] *= 1e27
    elif kind == "negative":
        x = np.abs(x)
        q = -np.abs(q)
        limit *= 4             # wider intervals: the scores are larger than their spread
    elif kind == "zero":
        limit = n
        x[:, 0] = 0
        x[: n - 50, :] = 0     # nearly every score is exactly 0
    elif kind == "same":
        x[:] = x[0]
        m, limit = 40, 7 * n   # every scan takes them all
    _check(E, x, q, m, limit)


def test_selection_scale_extremes():
    """Rows and queries near the ends of the float range."""
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(5)
    for rs, qs in ((1e-18, 1e-18), (1e18, 1e15), (1e-30, 1.0), (1e15, 1e-30)):
        x = (rng.standard_normal((6000, 32)) * rs).astype(np.float32)
        q = (rng.standard_normal((3, 32)) * qs).astype(np.float32)
        _check(E, x, q, 200, 6 * (6000 // 16))


@pytest.fixture(scope="module", params=[(64, 270_001), (384, 270_001), (512, 270_001), (768, 270_001), (1024, 270_001),
                                        (64, 393_275), (384, 393_275)])
def sampled_index(request):
    """Rows of which one in two or three runs is sampled (with three the sample
    ends in positions that hold no row), a tenth of them deleted."""
    import torch
    from paper_2608_07152_amd import eahr as E
    d, n = request.param
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    x = torch.randn(n, d, device="cuda", generator=g)
    idx = E.pvs_build(x)
    E.pvs_delete(idx, torch.randperm(n, device="cuda", generator=g)[: n // 10].cpu().numpy())
    e = E.pvs_snapshot(idx)
    yield E, idx, e, torch.randn(256, d, device="cuda", generator=g)
    E.pvs_free(idx)


@pytest.mark.parametrize("B", [9, 32, 40, 100, 200, 256])
def test_the_sample_passes_agree(sampled_index, monkeypatch, B):
    """The dot4 and the MFMA sample passes keep the same codes, so tau and with
    it every count of the scans is the same: one, two, four and eight tiles of
    the single-pass kernel (d = 384 up) and of the block kernel (d = 64); a
    first scan, and one past the certified ranks."""
    E, idx, e, q = sampled_index

    def counts(path):
        monkeypatch.setenv("EAHR_SCAN_PATH", path)
        st = E.pvs_open(idx, q[:B].contiguous(), e)
        out = []
        for m in (100, 20_000):   # a first scan certifies at most about 1.25 n / 4 / 9 = 13,700
            E.pvs_next(st, m)
            s = E.pvs_stats(st)
            out.append({k: s[k] for k in ("scans", "candidates", "certified", "rescans", "overflows")})
        E.pvs_close(st)
        return out

    counts("mfma")   # whatever the index expects of its readers, for both alike
    got, want = counts("mfma"), counts("gemv")
    assert got == want
    assert got[0]["candidates"] > 0 and got[1]["scans"] > got[0]["scans"] > 0


@pytest.mark.parametrize("n,d", [(4_000_000, 16), (1_200_000, 384)])
def test_neighbours_stored_side_by_side_take_one_scan(n, d):
    """Near-duplicates next to each other: the rows asked for fall into the
    sample by whole runs, and the request still takes one scan."""
    import torch
    from paper_2608_07152_amd import eahr as E
    B, m = 256, 100
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    centers = torch.randn(n // m, d, device="cuda", generator=g)
    centers /= centers.norm(dim=1, keepdim=True)
    x = centers.repeat_interleave(m, dim=0)
    x += 1e-3 * torch.randn(n, d, device="cuda", generator=g)
    idx = E.pvs_build(x)
    del x
    for _ in range(3):
        pick = torch.randperm(n // m, device="cuda", generator=g)[:B]
        st = E.pvs_open(idx, centers[pick].contiguous())
        ids, _, cnt, _ = E.pvs_next(st, m)
        assert list(cnt) == [m] * B
        assert np.array_equal(np.sort(ids, axis=1), pick.cpu().numpy()[:, None] * m + np.arange(m))
        s = E.pvs_stats(st)
        E.pvs_close(st)
        assert s["scans"] == 1 and s["rescans"] == 0, s
    E.pvs_free(idx)
