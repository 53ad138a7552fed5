"""The gradient that a worker of a run hands to one whose result passed through a ReLU leaves already masked.  One mini-batch of one
micro-batch through the pipeline runner against the same passes called one by one (there the worker below masks what it is given):
the same kernels on the same numbers, so every parameter must be equal bit for bit."""
import numpy as np
import pytest

from workloads.configs import Config, affine, avgpool, bottleneck, conv, linear, maxpool, softmax_ce
from workloads import init_params, make_batch

pytestmark = pytest.mark.gpu


def _residual():
    below, h, c = bottleneck(8, 16, 8, 1, True)
    above, h, c2 = bottleneck(h, c, 16, 2, True)      # two layers read the stage input: the first convolution and the projection
    return (8, 8, 16), [below, above + [avgpool(h, h, c2), linear(c2, 10, False), softmax_ce(10)]]


NETS = {
    "linear": lambda: ((40,), [[linear(40, 48, True)], [linear(48, 24, True)], [linear(24, 10, False), softmax_ce(10)]]),
    "ragged": lambda: ((37,), [[linear(37, 53, True)], [linear(53, 10, False), softmax_ce(10)]]),
    "conv": lambda: ((8, 8, 8), [[conv(8, 8, 8, 16)], [conv(8, 8, 16, 64), maxpool(8, 8, 64)], [conv(4, 4, 64, 64)],
                                 [linear(4 * 4 * 64, 10, False), softmax_ce(10)]]),
    "pool above": lambda: ((8, 8, 8), [[conv(8, 8, 8, 16)], [maxpool(8, 8, 16), linear(4 * 4 * 16, 10, False), softmax_ce(10)]]),
    "residual": _residual,
    "join above": lambda: ((8, 8, 16), [[conv(8, 8, 16, 64)], bottleneck(8, 64, 16, 1, False)[0] + [avgpool(8, 8, 64), linear(64, 10, False), softmax_ce(10)]]),
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("net", sorted(NETS))
def test_runner_and_single_passes_agree_bit_for_bit(net, dtype):
    import torch
    from paper_2410_14312_amd import Pipeline, Stage

    shape, stages = NETS[net]()
    M = 12
    cfg = Config(name=net, dtype=dtype, M=M, N=1, stages=stages, in_shape=shape, classes=10, seed=7, lr=0.05, momentum=0.9)
    params = init_params(cfg)
    x, labels = make_batch(cfg, 0)
    pipe = Pipeline(cfg, params)
    pipe.run([(x, labels)])

    mine = [Stage(specs, dtype, M, 1, 1, cfg.lr, cfg.momentum, borrow_input=True) for specs in stages]
    for st, p in zip(mine, params):
        st.set_params(p)
    act, ld = mine[0].prepare_input(x).contiguous(), torch.from_numpy(np.asarray(labels, np.int32)).to(mine[0].device)
    kept = []
    for st in mine:
        kept.append(act)
        y = torch.empty(M * st.out_elems, dtype=torch.float32 if st.is_last else st.act_dtype, device=st.device)
        st.forward_micro(0, act, y=y, labels=ld if st.is_last else None)
        act = y
    dy = None
    for k in reversed(range(len(mine))):
        st = mine[k]
        dx = torch.empty(M * st.in_elems, dtype=st.act_dtype, device=st.device) if k else None
        st.backward([0], dy=dy, dx=dx)
        st.update()
        dy = dx
    torch.cuda.synchronize()
    for k, st in enumerate(mine):
        assert torch.equal(st.regions[0], pipe.stages[k].regions[0]), "parameters of stage %d" % k
        n = 4 * st.P
        assert torch.equal(st.regions[1][:n], pipe.stages[k].regions[1][:n]), "momentum of stage %d" % k
