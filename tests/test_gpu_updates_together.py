"""Runs on one stream, which issue the updates of several stages in one launch: bit for bit those of K streams, which do not; more stages than a launch takes,
both types, one mini-batch and several, with kept versions (whose updates stay launches of their own)."""
import numpy as np
import pytest

from workloads import Config, init_params, make_batch
from workloads.configs import linear, softmax_ce

pytestmark = pytest.mark.gpu


def _mlp(K, N, dtype):
    layers = [linear(24, 24, True) for _ in range(K - 1)] + [linear(24, 10, False), softmax_ce(10)]
    return Config(name="t", dtype=dtype, M=4 * N, N=N, stages=[[l] for l in layers[:K - 1]] + [layers[K - 1:]], in_shape=(24,), classes=10, seed=3, lr=0.005)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("K,N,batches,vertical_sync", [(1, 2, 2, False), (2, 4, 5, False), (3, 1, 4, False), (4, 4, 6, False), (4, 2, 6, True), (19, 2, 3, False), (35, 3, 2, False)])
def test_updates_together(monkeypatch, K, N, batches, vertical_sync, dtype):
    from paper_2410_14312_amd import Pipeline
    cfg = _mlp(K, N, dtype)
    params = init_params(cfg)
    data = [make_batch(cfg, i) for i in range(batches)]
    res = []
    for one in (False, True):
        monkeypatch.setenv("TMPS_ISSUE_THREADS", "1")
        pipe = Pipeline(cfg, params, one_stream=one, vertical_sync=vertical_sync)
        losses, log = pipe.run(data)
        res.append((losses, log, [pipe.get_params(s) for s in range(K)], [pipe.stages[s].version() for s in range(K)]))
    assert res[0][0] == res[1][0] and np.array_equal(res[0][1], res[1][1]) and res[0][3] == res[1][3] == [batches] * K
    for a, b in zip(res[0][2], res[1][2]):
        for la, lb in zip(a, b):
            for k in la:
                assert np.array_equal(la[k], lb[k]), k


@pytest.mark.parametrize("one,K", [(True, 1), (True, 4), (True, 19), (False, 4)])
def test_every_launch_of_updates_has_an_empty_bracket(one, K):
    """What a pair of timing events costs is measured beside every launch that is bracketed so, on one stream as on K."""
    import paper_2410_14312_amd as T
    cfg = _mlp(K, 2, "f32")
    pipe = T.Pipeline(cfg, init_params(cfg), one_stream=one)
    data = [make_batch(cfg, i) for i in range(2)]
    pipe.run(data)
    T.profile_enable(True)
    try:
        pipe.run(data)
        prof = T.profile_read()
    finally:
        T.profile_enable(False)
    assert prof["event_pair"][1] == prof["update"][1] > 0
