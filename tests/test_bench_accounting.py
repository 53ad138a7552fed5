"""The FLOP accounting of bench.py (what its MFMA fractions are computed from) against counts written out by hand
from the layer shapes of the benchmark configurations, and the per-stage split against the whole."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402
from workloads import get_config  # noqa: E402

NAMES = ("tiny_mlp_f32", "mlp4x1024_bf16", "vgg16_bf16", "resnet50_bf16", "gpt2_small_bf16")


def forward_macs_per_sample(cfg):
    w = bench.algorithmic_work(cfg)
    return sum(v[1] for k, v in w.items() if k.endswith("_fwd")) / 2.0 / cfg.M


def test_tiny_mlp_forward_macs():
    # 64-128-128-10
    assert forward_macs_per_sample(get_config("tiny_mlp_f32")) == 64 * 128 + 128 * 128 + 128 * 10


def test_mlp_forward_macs():
    # 3072-1024-1024-1024-1024-10
    assert forward_macs_per_sample(get_config("mlp4x1024_bf16")) == 3072 * 1024 + 3 * 1024 * 1024 + 1024 * 10


def test_vgg16_forward_macs():
    # 13 3x3 convolutions on 32x32 images (channels 64,64 | 128,128 | 256 x3 | 512 x3 | 512 x3, a 2x2 pooling after each
    # block) and the 512-4096-4096-10 classifier
    macs, hw, cin = 0, 32, 3
    for block in ((64, 64), (128, 128), (256, 256, 256), (512, 512, 512), (512, 512, 512)):
        for cout in block:
            macs += hw * hw * 9 * cin * cout
            cin = cout
        hw //= 2
    macs += 512 * 4096 + 4096 * 4096 + 4096 * 10
    assert forward_macs_per_sample(get_config("vgg16_bf16")) == macs


def test_resnet50_forward_macs():
    # stem 7x7/2 to 112x112x64, then bottleneck groups of 3/4/6/3 blocks (widths 64/128/256/512, outputs 4x as wide,
    # stride on the 3x3 convolution of a group's first block, projection shortcut on that block), 1000-way classifier
    macs = 112 * 112 * 49 * 3 * 64
    hw, cin = 56, 64
    for gi, (blocks, width) in enumerate(((3, 64), (4, 128), (6, 256), (3, 512))):
        for b in range(blocks):
            stride = 2 if (b == 0 and gi > 0) else 1
            out_hw = hw // stride
            macs += hw * hw * cin * width                       # 1x1 reduce, at the input resolution
            macs += out_hw * out_hw * 9 * width * width         # 3x3, carries the stride
            macs += out_hw * out_hw * width * 4 * width         # 1x1 expand
            if b == 0:
                macs += out_hw * out_hw * cin * 4 * width       # projection shortcut
            cin, hw = 4 * width, out_hw
    macs += 2048 * 1000
    got = forward_macs_per_sample(get_config("resnet50_bf16"))
    assert got == macs
    assert abs(got - 4.09e9) < 0.01 * 4.09e9                    # the usual figure for this network at 224x224


def test_gpt2_forward_macs():
    # per token and layer: d x 3d, d x d, d x 4d, 4d x d; causal attention: a query at position i sees i + 1 keys,
    # two products of the head size per (query, key) pair; output layer d x vocabulary
    d, layers, s, vocab = 768, 12, 512, 32000
    linear = layers * (d * 3 * d + d * d + 2 * d * 4 * d) + d * vocab
    attention = layers * 2 * d * (s + 1) / 2.0
    assert forward_macs_per_sample(get_config("gpt2_small_bf16")) == pytest.approx((linear + attention) * s, rel=1e-12)


@pytest.mark.parametrize("name", NAMES)
def test_stages_add_up_to_the_whole(name):
    cfg = get_config(name)
    whole = bench.algorithmic_work(cfg)
    parts = [bench.algorithmic_work(cfg, only_stage=s) for s in range(cfg.K)]
    for klass, (launches, flops, nbytes) in whole.items():
        assert sum(p.get(klass, [0, 0.0, 0.0])[0] for p in parts) == launches
        assert sum(p.get(klass, [0, 0.0, 0.0])[1] for p in parts) == pytest.approx(flops, rel=1e-12)
        assert sum(p.get(klass, [0, 0.0, 0.0])[2] for p in parts) == pytest.approx(nbytes, rel=1e-12)


@pytest.mark.parametrize("name", NAMES[1:])
def test_training_flops_are_three_forward_passes_minus_the_first_input_gradient(name):
    cfg = get_config(name)
    w = bench.algorithmic_work(cfg)
    fwd = sum(v[1] for k, v in w.items() if k in ("dense_fwd", "conv_fwd"))
    dgrad = sum(v[1] for k, v in w.items() if k in ("dense_dgrad", "conv_dgrad"))
    wgrad = sum(v[1] for k, v in w.items() if k in ("dense_wgrad", "conv_wgrad"))
    assert wgrad == pytest.approx(fwd, rel=1e-12)
    if name == "gpt2_small_bf16":
        assert dgrad == pytest.approx(fwd, rel=1e-12)   # its first layer is an embedding: every contraction has an input gradient
    else:
        assert dgrad < fwd                              # the first layer has no input gradient
        assert dgrad > 0.9 * fwd or name == "mlp4x1024_bf16"   # (the MLP's first layer is half of its work)


@pytest.mark.parametrize("name", NAMES)
def test_rates_do_not_depend_on_how_micro_batches_are_grouped(name):
    """A forward pass over several micro-batches is one launch per layer: the same FLOPs in the same time are the same rate,
    and only the weights are read less often."""
    cfg = get_config(name)
    for klass, (launches, flops, nbytes) in bench.algorithmic_work(cfg).items():
        apart = bench.class_entry(cfg, klass, 2.0, launches)
        assert apart["gbs"] == pytest.approx(nbytes / 2e-3 / 1e9, rel=1e-12)
        for merged in (launches / 2, launches / 1.5, launches / cfg.N):
            e = bench.class_entry(cfg, klass, 2.0, merged)
            assert e["tflops"] == pytest.approx(flops / 2e-3 / 1e12, rel=1e-12)
            assert e["gflop_per_launch"] * merged == pytest.approx(flops / 1e9, rel=1e-12)
            assert e["gbs"] <= apart["gbs"] * (1 + 1e-12)
            if klass not in ("dense_fwd", "conv_fwd"):
                assert e["gbs"] == pytest.approx(apart["gbs"], rel=1e-12)


def test_weights_are_read_once_by_every_pass():
    cfg = get_config("tiny_mlp_f32")
    weights = (64 * 128 + 128 * 128 + 128 * 10) * 4
    by_pass = [bench.algorithmic_work(cfg, passes=p)["dense_fwd"][2] for p in (1, 2, 4)]
    assert by_pass[1] - by_pass[0] == weights and by_pass[2] - by_pass[0] == 3 * weights


@pytest.mark.parametrize("name", NAMES)
def test_both_gradients_of_a_layer_in_one_launch_count_together(name):
    """What the library launches together is moved to a class of its own, with all of its work: at the batch sizes of the two smaller networks' layers
    and of two of VGG-16's classifier, and nowhere for the transformer, whose weight gradients wait for the end of a pass."""
    from paper_2410_14312_amd import dense_gradients_joint

    cfg = get_config(name)
    apart, got = bench.algorithmic_work(cfg), bench.algorithmic_work(cfg, joint=dense_gradients_joint)
    classes = ("dense_dgrad", "dense_wgrad", "dense_backward")
    for i in (1, 2):
        assert sum(got.get(k, [0] * 3)[i] for k in classes) == pytest.approx(sum(apart.get(k, [0] * 3)[i] for k in classes), rel=1e-12)
    layers = {"tiny_mlp_f32": 2, "mlp4x1024_bf16": 4, "vgg16_bf16": 2, "resnet50_bf16": 0, "gpt2_small_bf16": 0}[name]
    both = got.get("dense_backward", [0, 0.0, 0.0])
    assert both[0] == layers
    assert both[0] + got.get("dense_wgrad", [0])[0] == apart["dense_wgrad"][0] and both[0] + got.get("dense_dgrad", [0])[0] == apart["dense_dgrad"][0]
    if layers:
        e = bench.class_entry(cfg, "dense_backward", 2.0, layers, dense_gradients_joint)
        assert e["tflops"] == pytest.approx(both[1] / 2e-3 / 1e12, rel=1e-12)
    assert "dense_dgrad" not in got if name == "mlp4x1024_bf16" else True


def test_gradients_of_a_convolution_in_one_launch_with_the_affine_layer_behind_count_there():
    """Seven of the first group's 1 x 1 convolutions (the second group's have more outputs than a workgroup's accumulators), with all of their products and
    with the bytes of one launch: the result's gradient, the result and the input read once, what a later reader of the input contributed, the input's gradient written."""
    from paper_2410_14312_amd import pointwise_gradients_joint

    cfg = get_config("resnet50_bf16")
    apart, got = bench.algorithmic_work(cfg), bench.algorithmic_work(cfg, joint_pointwise=pointwise_gradients_joint)
    classes = ("conv_dgrad", "conv_wgrad", "affine")
    assert sum(got[k][1] for k in classes) == pytest.approx(sum(apart[k][1] for k in classes), rel=1e-12)
    assert apart["conv_dgrad"][0] - got["conv_dgrad"][0] == 7 and apart["conv_wgrad"][0] - got["conv_wgrad"][0] == 7 and apart["affine"][0] == got["affine"][0]
    # (inputs, outputs, a joined gradient): the first block's reduction, expansion and projection, two more blocks' reductions and expansions
    P, layers = cfg.M * 56 * 56, [(64, 64, 1), (64, 256, 0), (64, 256, 0), (256, 64, 1), (64, 256, 0), (256, 64, 1), (64, 256, 0)]
    one = sum(P * (2 * o + (2 + j) * i) * 2 + i * o * 6 for i, o, j in layers)
    assert got["affine"][2] - (apart["affine"][2] - sum(P * 3 * o * 2 for _, o, _ in layers)) == pytest.approx(one, rel=1e-12)
    moved = sum(2 * P * (i + o) * 2 + i * o * 6 for i, o, _ in layers)
    assert sum(apart[k][2] - got[k][2] for k in classes[:2]) == pytest.approx(moved, rel=1e-12)


def test_the_stem_s_pooling_counts_with_the_affine_layer_below_where_both_are_one_launch():
    from paper_2410_14312_amd import pool_affine_gradients_joint

    cfg = get_config("resnet50_bf16")
    apart, got = bench.algorithmic_work(cfg), bench.algorithmic_work(cfg, joint_pool=pool_affine_gradients_joint)
    z, y = cfg.M * 112 * 112 * 64, cfg.M * 56 * 56 * 64
    assert apart["affine"][0] - got["affine"][0] == 1 and apart["affine"][2] - got["affine"][2] == 3 * z * 2
    assert got["pool_bwd"][0] == apart["pool_bwd"][0] and got["pool_bwd"][2] - apart["pool_bwd"][2] == z * 2
    rest = cfg.M * (2 * 7 * 7 * 2048 + 2048) * 2   # (the global average pooling)
    assert got["pool_bwd"][2] - rest == 2 * z * 2 + y * 3   # read z, dy and a byte for each winner, write dz
    # 2 x 2 windows without an affine layer: winners and dy read, dx written
    vgg = get_config("vgg16_bf16")
    maps = vgg.M * sum(hw * hw * c for hw, c in ((32, 64), (16, 128), (8, 256), (4, 512), (2, 512)))
    assert bench.algorithmic_work(vgg, joint_pool=pool_affine_gradients_joint)["pool_bwd"][2] == maps * 2 + maps // 4 * 3


def test_a_join_and_the_next_block_s_first_convolution_count_as_one_launch():
    """Two of the first group's, where the join's result is not read again."""
    from paper_2410_14312_amd import pointwise_forward_joint

    cfg = get_config("resnet50_bf16")
    apart, got = bench.algorithmic_work(cfg), bench.algorithmic_work(cfg, joint_forward=pointwise_forward_joint)
    pairs = 2
    assert apart["conv_fwd"][0] - got["conv_fwd"][0] == pairs * cfg.N and apart["conv_fwd"][1] == pytest.approx(got["conv_fwd"][1], rel=1e-12)
    assert apart["conv_fwd"][2] - got["conv_fwd"][2] == pytest.approx(pairs * cfg.M * 56 * 56 * 256 * 2, rel=1e-12)
    # as many launches as passes over one micro-batch each make
    e = bench.class_entry(cfg, "conv_fwd", 2.0, got["conv_fwd"][0], joint_forward=pointwise_forward_joint)
    assert e["gbs"] == pytest.approx(got["conv_fwd"][2] / 2e-3 / 1e9, rel=1e-12)


def test_classes_that_hold_no_event_pair_are_those_that_are_launched_with_stamps():
    """An empty pair of events is subtracted from every class but these: a class is either launched with its kernels' own stamps (launch_timed) or bracketed."""
    import re

    from paper_2410_14312_amd import KERNEL_CLASSES

    root = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_14312_amd", "csrc")
    text = "\n".join(open(os.path.join(root, f)).read() for f in sorted(os.listdir(root)))
    enum = re.findall(r"\bkc\w+", re.search(r"enum KernelClass \{(.*?)\};", open(os.path.join(root, "profile.h")).read(), re.S).group(1))
    names = dict(zip(enum, KERNEL_CLASSES))
    assert len(enum) == len(KERNEL_CLASSES) + 1 and enum[-1] == "kcCount"
    bracketed = {names[k] for k in re.findall(r"(?:TMPS_RUN\(|ProfileScope \w+\()(kc\w+)", text)}
    assert bracketed == {"softmax_ce", "update", "relu_mask", "reduce", "copy", "event_pair"}
    assert set(bench.KERNEL_STAMPED) == set(KERNEL_CLASSES) - bracketed
    stamped = {names[k] for k in re.findall(r"launch_timed\((kc\w+)", text)}
    assert stamped and not stamped & bracketed
