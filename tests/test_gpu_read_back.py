"""Read-backs through the pinned mailboxes: every value that comes back must be the one on
the device -- the bytes that a checkpoint (which takes the runtime's copies) holds -- whatever
handles, streams and threads share the pool, for the smallest and the largest read-back, and
for more handles at once than the pool keeps."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    return P, torch


def make(P, cfg, n, **kw):
    return P.Integrator(cfg["process"], cfg["ndim"], cfg["nbins"], cfg["seed"], cfg["alpha"], cfg["params"],
                        max_events=n, **kw)


def run(P, cfg, n, iters, **kw):
    g = make(P, cfg, n, **kw)
    out = []
    for _ in range(iters):
        r = g.iterate(n)
        d, s = g.get_hist()
        g.refine()
        e = g.get_grid()
        res = g.result()
        assert e.tobytes() in g.get_state()  # the checkpoint holds the grid as the runtime copied it
        assert np.array([r["I"], r["var"]]).tobytes() in g.get_state()
        out.append(np.array([r["I"], r["var"], res["I"], res["sigma"], res["chi2_dof"]]).tobytes() + d.tobytes()
                   + s.tobytes() + e.tobytes())
    g.close()
    return out


SMALL = dict(process=W.GAUSS, ndim=1, nbins=2, seed=3, alpha=1.5, params=[0.5, 0.2])
LARGE = dict(process=W.GAUSS, ndim=16, nbins=255, seed=3, alpha=1.5, params=[0.5, 0.2])


@pytest.mark.parametrize("cfg", [SMALL, LARGE, W.config("dy_z")], ids=["small", "large", "dy_z"])
def test_threads_and_streams_share_the_pool(env, cfg):
    P, torch = env
    ref = run(P, cfg, 2000, 4)
    got, errors = [], []

    def work(stream):
        try:
            for _ in range(3):
                got.append(run(P, cfg, 2000, 4, stream=stream))
        except Exception as e:  # reported below
            errors.append(e)

    streams = [torch.cuda.Stream() for _ in range(4)]
    threads = [threading.Thread(target=work, args=(s,)) for s in streams]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert len(got) == 12 and all(x == ref for x in got)


def test_more_handles_than_the_pool_keeps(env):
    P, _ = env
    cfg = W.config("dy_z")
    ref = run(P, cfg, 500, 1)
    for _ in range(2):
        hs = [make(P, cfg, 500) for _ in range(20)]
        res = [h.iterate(500)["I"] for h in hs]
        assert len(set(res)) == 1
        for h in hs:
            h.close()
    assert run(P, cfg, 500, 1) == ref


def test_result_over_more_iterations_than_a_wave(env):
    P, _ = env
    g = make(P, SMALL, 64)
    it = [g.iterate(64) for _ in range(131)]
    for first in (0, 64, 130):
        r = g.result(first=first)
        w = np.array([1.0 / x["var"] for x in it[first:]])
        I = np.array([x["I"] for x in it[first:]])
        m = (w * I).sum() / w.sum()
        assert r["n_iter"] == 131 - first
        assert abs(r["I"] / m - 1) < 1e-13 and abs(r["sigma"] * np.sqrt(w.sum()) - 1) < 1e-13
        chi = (w * (I - m) ** 2).sum() / (130 - first) if first < 130 else 0.0
        assert abs(r["chi2_dof"] - chi) <= 1e-11 * max(chi, 1.0)


def test_checkpoints_with_short_and_long_histories(env):
    """A checkpoint goes in through the mailbox while the grid and the history fit it (4,000
    doubles), by the runtime's copies beyond: either way it comes out as it went in."""
    P, _ = env
    g, k = make(P, SMALL, 64), make(P, SMALL, 64)
    for it in range(2100):
        if it in (0, 1, 7, 2045, 2046, 2047, 2099):
            blob = g.get_state()
            k.set_state(blob)
            assert k.get_state() == blob, it
        g.iterate(64, sync=False)
    assert k.iterate(64)["I"] == _second(g, k)


def _second(g, k):
    """g's last iteration, run again from the checkpoint before it (2,099 iterations)."""
    blob = g.get_state()
    return np.frombuffer(blob[-16:], dtype=np.float64)[0]
