"""The segmented key sort at the edges of its tiles (512, 2,048 and 4,096 keys)
and merge levels: complete rankings, read through the interval scans (sorted
into the pinned copy, query after query) and through the exhaustive generator
(sorted in place), against numpy's order of the authoritative scores.  Integer
vectors give many equal scores, so the id order inside a tie is checked too."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 63, 511, 512, 513, 2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193, 16383, 16384, 16385, 32769, 70001]


@pytest.mark.parametrize("n", EDGES)
@pytest.mark.parametrize("generator", ["intervals", "full_scan"])
def test_complete_ranking_is_sorted(n, generator):
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(n)
    x = rng.integers(-3, 4, size=(n, 8)).astype(np.float32)
    q = rng.integers(-3, 4, size=(3, 8)).astype(np.float32)
    q[1] = 0                                  # every score equal: id order
    idx = E.pvs_build(x)
    st = E.pvs_open(idx, q, generator=generator)
    ids, sc, cnt, stt = E.pvs_next(st, n)
    assert list(cnt) == [n] * 3 and list(stt) == [E.LIST_EXHAUSTED] * 3
    rows = np.arange(n)
    for b in range(3):
        s = E.pvs_scores(st, b, rows) + 0.0
        want = np.lexsort((rows, -s.astype(np.float64)))
        assert np.array_equal(ids[b], want)
        assert np.array_equal(sc[b] + 0.0, s[want])


def test_lists_of_different_lengths_pack_next_to_each_other():
    """Queries whose certified lists end in different tiles, one of them short."""
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(3)
    n, d = 40_000, 16
    x = rng.standard_normal((n, d)).astype(np.float32)
    x[:30_000] *= np.linspace(0.01, 1.0, 30_000, dtype=np.float32)[:, None]
    q = rng.standard_normal((9, d)).astype(np.float32)
    idx = E.pvs_build(x)
    st = E.pvs_open(idx, q)
    parts = [E.pvs_next(st, m)[0] for m in (7, 600, 9000)]
    got = np.concatenate(parts, axis=1)
    rows = np.arange(n)
    for b in range(len(q)):
        s = E.pvs_scores(st, b, rows).astype(np.float64)
        assert np.array_equal(got[b], np.lexsort((rows, -s))[:got.shape[1]])


@pytest.mark.parametrize("B", [256, 257, 1000])
def test_large_batches_pack(B):
    """More queries than one workgroup of the offsets takes, their lists of
    different lengths."""
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(B)
    n, d = 6000, 8
    x = rng.standard_normal((n, d)).astype(np.float32)
    x[: n // 2] *= 0.1
    q = rng.standard_normal((B, d)).astype(np.float32)
    idx = E.pvs_build(x)
    st = E.pvs_open(idx, q)
    got = np.concatenate([E.pvs_next(st, m)[0] for m in (3, 700)], axis=1)
    rows = np.arange(n)
    for b in list(range(0, B, 17)) + [255, B - 1]:
        s = E.pvs_scores(st, b, rows).astype(np.float64)
        assert np.array_equal(got[b], np.lexsort((rows, -s))[:got.shape[1]]), b
