"""Memory of closed handles is reused, bounded and given back; results do not
depend on whose memory a handle reuses, from one thread or several."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _first_ids(E, x, q, m):
    idx = E.pvs_build(x)
    st = E.pvs_open(idx, q)
    ids, sc, _, _ = E.pvs_next(st, m)
    E.pvs_close(st)
    E.pvs_free(idx)
    return ids, sc


def _want(x, q, m):
    return np.argsort(-(q.astype(np.float64) @ x.astype(np.float64).T), axis=1, kind="stable")[:, :m]


def test_segments_built_and_freed_in_turn():
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(0)
    for i in range(12):
        n, d = int(rng.integers(100, 30_000)), int(rng.integers(8, 300))
        x = rng.standard_normal((n, d)).astype(np.float32)
        q = rng.standard_normal((int(rng.integers(1, 40)), d)).astype(np.float32)
        ids, _ = _first_ids(E, x, q, 10)
        assert np.array_equal(ids, _want(x, q, 10)), (i, n, d)


def test_threads_with_streams_of_their_own():
    import torch
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(1)
    xs = [rng.standard_normal((20_000, 64)).astype(np.float32) for _ in range(4)]
    qs = [rng.standard_normal((5, 64)).astype(np.float32) for _ in range(4)]
    bad = []

    def work(t):
        try:
            s = torch.cuda.Stream()
            for _ in range(10):
                idx = E.pvs_build(xs[t], stream=s)
                st = E.pvs_open(idx, qs[t])
                ids = E.pvs_next(st, 20)[0]
                E.pvs_close(st)
                E.pvs_free(idx)
                if not np.array_equal(ids, _want(xs[t], qs[t], 20)):
                    bad.append(t)
        except Exception as e:   # noqa: BLE001
            bad.append((t, repr(e)))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad


def test_memory_is_given_back():
    import torch
    from paper_2608_07152_amd import eahr as E
    q = np.ones((1, 256), np.float32)
    small = np.ones((64, 256), np.float32)
    _first_ids(E, small, q, 5)
    for _ in range(4):      # whatever earlier work left
        E.pvs_free(E.pvs_build(small))
    before = torch.cuda.mem_get_info()[0]
    big = torch.ones(1_000_000, 256, device="cuda")
    idx = E.pvs_build(big)                      # 1.3 GB
    torch.cuda.synchronize()
    built = torch.cuda.mem_get_info()[0]
    E.pvs_free(idx)                             # kept ...
    assert abs(built - torch.cuda.mem_get_info()[0]) <= 64 << 20
    idx = E.pvs_build(big)                      # ... and used again
    assert abs(built - torch.cuda.mem_get_info()[0]) <= 64 << 20
    del big
    torch.cuda.empty_cache()
    E.pvs_free(idx)
    held = before - torch.cuda.mem_get_info()[0]
    assert (1 << 30) <= held <= (3 << 29), held   # this index and no more
    huge = torch.ones(5_000_000, 256, device="cuda")
    idx = E.pvs_build(huge)                     # 6.4 GB: more than is ever kept
    del huge
    torch.cuda.empty_cache()
    E.pvs_free(idx)
    assert before - torch.cuda.mem_get_info()[0] <= (4 << 30) + (64 << 20)
    for _ in range(4):
        E.pvs_free(E.pvs_build(small))
    assert before - torch.cuda.mem_get_info()[0] <= 64 << 20


def test_many_states_open_at_once():
    """More blocks than the pool keeps, closed together and opened again."""
    from paper_2608_07152_amd import eahr as E
    rng = np.random.default_rng(2)
    x = rng.standard_normal((5000, 32)).astype(np.float32)
    q = rng.standard_normal((3, 32)).astype(np.float32)
    idx = E.pvs_build(x)
    want = _want(x, q, 10)
    for _ in range(2):
        states = [E.pvs_open(idx, q) for _ in range(150)]
        for st in states[::10]:
            assert np.array_equal(E.pvs_next(st, 10)[0], want)
        for st in states:
            E.pvs_close(st)


def test_release_memory():
    """What closed handles left is free after the call; open handles go on."""
    import torch
    from paper_2608_07152_amd import eahr as E
    q = np.ones((1, 256), np.float32)
    _first_ids(E, np.ones((64, 256), np.float32), q, 5)
    E.eahr_release_memory()
    rng = np.random.default_rng(3)
    x = rng.standard_normal((3000, 256)).astype(np.float32)
    held = E.pvs_build(x)
    st = E.pvs_open(held, x[:2])
    first = E.pvs_next(st, 10)[0]
    before = torch.cuda.mem_get_info()[0]
    big = torch.ones(1_000_000, 256, device="cuda")
    E.pvs_free(E.pvs_build(big))                # 1.3 GB kept
    del big
    torch.cuda.empty_cache()
    assert before - torch.cuda.mem_get_info()[0] > 1 << 30
    E.eahr_release_memory()
    assert before - torch.cuda.mem_get_info()[0] <= 64 << 20
    ids = np.concatenate([first, E.pvs_next(st, 40)[0]], axis=1)
    assert np.array_equal(ids, _want(x, x[:2], 50))
    E.pvs_close(st)
    E.pvs_free(held)
