"""Pipeline runs in the form with K streams and a host thread per stage (TMPS_ISSUE_THREADS=1; short runs are otherwise issued
on one stream): against the oracle, and bit for bit against the same run issued by one thread and on one stream."""
import numpy as np
import pytest

from tests.test_gpu_baseline_1f1b import _compare as compare_1f1b
from tests.test_gpu_pipeline import _compare
from workloads import Config, get_config, init_params, make_batch
from workloads.configs import linear, softmax_ce

pytestmark = pytest.mark.gpu


@pytest.fixture
def k_streams(monkeypatch):
    monkeypatch.setenv("TMPS_ISSUE_THREADS", "1")


def _deep(W):
    layers = [linear(32, 32, True) for _ in range(W - 1)] + [linear(32, 10, False), softmax_ce(10)]
    return Config(name="t", dtype="f32", M=8, N=2, stages=[[l] for l in layers[:W - 1]] + [layers[W - 1:]], in_shape=(32,), classes=10,
                  seed=3, lr=0.005)


@pytest.mark.parametrize("vertical_sync", [False, True])
@pytest.mark.parametrize("name", ["tiny_mlp_f32", "tiny_transformer_f32", "tiny_transformer_bf16", "tiny_resnet_f32", "tiny_resnet_bf16"])
def test_small_networks(k_streams, name, vertical_sync):
    _compare(get_config(name), 6, bias_std=0.05, vertical_sync=vertical_sync)


@pytest.mark.parametrize("W,vertical_sync", [(4, False), (4, True), (7, False)])
def test_deep_pipelines(k_streams, W, vertical_sync):
    _compare(_deep(W), 12, bias_std=0.05, vertical_sync=vertical_sync)


@pytest.mark.parametrize("name,batch", [("tiny_mlp_f32", 8), ("tiny_transformer_bf16", 2)])
def test_1f1b(k_streams, name, batch):
    compare_1f1b(get_config(name), 9, batch)


@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("name", ["tiny_mlp_f32", "mlp4x1024_bf16", "tiny_transformer_bf16", "tiny_resnet_bf16"])
def test_forms_of_a_run_agree_bit_for_bit(monkeypatch, name, graphs):
    from paper_2410_14312_amd import Pipeline
    cfg = get_config(name)
    params = init_params(cfg)
    forms = [("1", False), ("0", False), ("0", True)]
    pipes = [Pipeline(cfg, params, one_stream=one, graphs=graphs) for _, one in forms]
    for rnd in range(3):   # (graphs: direct, captured, replayed)
        batches = [make_batch(cfg, 5 * rnd + i) for i in range(5)]
        res = []
        for pipe, (threads, _) in zip(pipes, forms):
            monkeypatch.setenv("TMPS_ISSUE_THREADS", threads)
            res.append(pipe.run(batches))
        for pipe, r in zip(pipes[1:], res[1:]):
            assert r[0] == res[0][0], "losses of run %d" % rnd
            assert np.array_equal(r[1], res[0][1]), "version log of run %d" % rnd
            for s in range(cfg.K):
                for a, b in zip(pipe.get_params(s), pipes[0].get_params(s)):
                    for k in a:
                        assert np.array_equal(a[k], b[k]), (rnd, s, k)
