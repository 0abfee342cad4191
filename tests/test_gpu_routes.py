"""Parity of kernels and dispatch branches at the sizes where they can go wrong: edges of tiles, remainders, the
smallest and the largest of their ranges.  Same oracle and bars as tests/test_gpu_parity.py."""
import numpy as np
import pytest

import dp_workloads as W
from tests.test_gpu_parity import _check_all_regimes

pytestmark = pytest.mark.gpu


def _tokens(batch, seq, vocab, rng, kind):
    if kind == "same":  # one token throughout: every step of an example adds up to one row
        return np.full((batch, seq), vocab - 1, dtype=np.int32)
    if kind == "uniform":  # as many distinct tokens as there can be
        return rng.integers(0, vocab, size=(batch, seq)).astype(np.int32)
    return W.zipf_tokens(rng, vocab, 1.1, (batch, seq))


@pytest.mark.parametrize("vocab,dim,seq,classes,batch,kind", [
    (1, 1, 1, 2, 1, "same"),              # the smallest of everything
    (300, 3, 255, 2, 70, "zipf"),         # scalar rows; one key per thread, one short of the sort's size
    (256, 127, 256, 15, 9, "uniform"),    # a row per workgroup; the widest scalar rows
    (257, 128, 257, 16, 9, "same"),       # the widest rows and the most classes; two keys per thread
    (2000, 20, 1024, 4, 70, "uniform"),   # four keys per thread; more pairs than a workgroup's list holds at a time
    (5000, 8, 40, 3, 1100, "zipf"),       # more examples than a pass takes; tokens of several chunks
    (70000, 36, 12, 2, 33, "uniform"),    # a table too large for 256 workgroups' LDS
    (300, 129, 40, 3, 9, "zipf"),         # rows wider than the kernel of the whole network takes: pairs with rows of their own
    (90, 132, 300, 16, 5, "zipf"),
])
def test_embedding_mean_classifier_network(vocab, dim, seq, classes, batch, kind):
    from paper_2010_09063_amd import DpStep
    m = W.model(W.token_input(seq), [W.embedding(vocab, dim), W.seq_mean(), W.dense(dim, classes)], classes)
    rng = np.random.default_rng(seq)
    x = _tokens(batch, seq, vocab, rng, kind)
    y = rng.integers(0, classes, size=batch).astype(np.int32)
    theta = W.init_params(m, rng, bias_scale=0.2) * np.float32(4)
    st = DpStep(m, batch)
    assert _routes(st, 1) == ["fused - fused pairs" if dim <= 128 else "gather - pairs pairs"]
    _check_all_regimes(m, x, y, theta, f"embedding V{vocab} D{dim} T{seq} N{classes} B{batch} {kind}", stepper=st)


@pytest.mark.parametrize("d_in,hidden,classes,batch", [
    (1, 1, 2, 1), (1, 4, 7, 8), (1, 130, 15, 33), (5, 31, 3, 33), (33, 32, 2, 31), (257, 129, 15, 65), (104, 50, 10, 1025), (1023, 639, 7, 96)])
def test_two_layer_networks_of_widths_off_the_vector_size(d_in, hidden, classes, batch):
    """Widths that are no multiples of four floats: one short of, at and past a 32-wide tile or slice."""
    m = W.model(W.image_input(d_in), [W.dense(d_in, hidden, act="tanh"), W.dense(hidden, classes)], classes)
    rng = np.random.default_rng(hidden)
    x, y = W.make_inputs(m, batch, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    _check_all_regimes(m, x, y, theta, f"dense {d_in}->{hidden}->{classes}/B{batch}")


@pytest.mark.parametrize("d_in,hidden,classes,batch,small", [
    (104, 50, 10, 1024, True), (104, 50, 10, 1025, False),  # few tiles of weights
    (513, 449, 3, 2048, True), (513, 449, 3, 2049, False),  # 270 of them
    (63, 511, 3, 1024, True), (252, 1000, 3, 2048, True),   # more tiles in the second product than in the first
    (104, 52, 10, 4096, True)])                             # whole groups of four floats: any batch
def test_two_layer_networks_where_the_batch_is_a_long_k(d_in, hidden, classes, batch, small):
    """Off the vector size the clipped sums leave the kernel whose workgroups take the whole batch as their K (which also
    makes the final write) before it falls behind; the two routes on both sides of the line."""
    import torch
    from paper_2010_09063_amd import DpStep
    m = W.model(W.image_input(d_in), [W.dense(d_in, hidden, act="tanh"), W.dense(hidden, classes)], classes)
    rng = np.random.default_rng(hidden)
    x, y = W.make_inputs(m, batch, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    st = DpStep(m, batch)
    assert (st.dp_step_describe_plan()[1]["sum"] == "joint") == small
    _check_all_regimes(m, x, y, theta, f"dense {d_in}->{hidden}->{classes}/B{batch}", stepper=st)
    dev = torch.device("cuda")
    tt, tx, ty = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (theta, x, y))
    st.dp_step_profile(True)
    st.dp_step(tt, tx, ty, batch, 1.0, 1.0, 1, torch.empty_like(tt))
    labels = [r[0] for r in st.dp_step_profile_read()]
    st.dp_step_free()
    assert ("finalize_noise" not in labels) == small, labels


def _routes(st, layers):
    plan = st.dp_step_describe_plan()
    return [" ".join(plan[l][k] for k in ("fwd", "bwd", "norm", "sum")) for l in range(layers)]


# the last column: the kernels of each convolution (forward, backward-data, norm, clipped sum)
@pytest.mark.parametrize("cin,widths,plane,act,pool,batch,routes", [
    (3, (16, 48), (32, 32), "tanh", "max", 3,      # one and two blocks of output channels, the second half empty
     ["first - direct+store weighted", "split+maxpool split split+store weighted"]),
    (3, (48, 100, 20), (4, 32), "relu", "avg", 5,  # the fewest rows of a 32-wide plane; ragged blocks on both sides
     ["direct - generic+store weighted", "split split split+store weighted", "split+avgpool split split+store weighted"]),
    (4, (40, 12), (16, 16), "tanh", "avg", 9,      # few columns: split norms, general batch sums (with stored rows: without weights)
     ["direct - split+store weighted", "split+avgpool direct split+store weighted"]),
    (16, (96, 33), (16, 16), "tanh", "max", 4,     # three blocks; one channel past a block
     ["split - split+store weighted", "split+maxpool split split+store weighted"]),
    (17, (20, 70), (4, 16), "relu", "avg", 3,      # a chunk of sixteen input channels and one more
     ["split - split split", "split+avgpool split split split"]),
    (16, (40, 130), (8, 8), "tanh", "avg", 9,
     ["split - split split", "split+avgpool split split split"]),
    (24, (64, 16), (4, 8), "relu", "max", 7,       # two images of a tile, a ragged last tile
     ["split - direct direct", "split+maxpool split generic generic"]),
    (32, (64, 10), (4, 4), "relu", "avg", 13,      # four images of a tile; batch sums over a ragged last run
     ["split - gram split", "split+avgpool direct split split"]),
    (16, (160, 32), (8, 4), "tanh", "max", 1,
     ["split - ws ws", "split+maxpool split generic generic"]),
    # norms with two blocks of output channels per workgroup (from 512 workgroups on), a plane of each width
    (130, (60,), (8, 8), "tanh", "avg", 104, ["split+avgpool - split split"]),
    (64, (128,), (16, 16), "tanh", "avg", 128, ["mf64+avgpool - split+store weighted"]),
    (40, (128,), (8, 32), "tanh", "avg", 128, ["mf64+avgpool - split+store weighted"]),
])
def test_convolutions_on_the_bf16_matrix_units(cin, widths, plane, act, pool, batch, routes):
    from paper_2010_09063_amd import DpStep
    h, w = plane
    layers, c = [], cin
    for d in widths:
        layers.append(W.conv2d(c, d, 3, stride=1, pad=1, act=act))
        c = d
    layers += [W.maxpool2d(2, 2) if pool == "max" else W.avgpool2d(2, 2), W.dense(c * (h // 2) * (w // 2), 3)]
    m = W.model(W.image_input(cin, h, w), layers, 3)
    rng = np.random.default_rng(h * w + cin)
    x, y = W.make_inputs(m, batch, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    st = DpStep(m, batch)
    assert _routes(st, len(widths)) == routes
    _check_all_regimes(m, x, y, theta, f"conv {cin}->{widths} {plane} {act} {pool} B{batch}", stepper=st)
    st = DpStep(m, batch, no_stored_gradients=1)
    recomputed = [r.replace("direct+store weighted", "direct direct").replace("generic+store weighted", "generic generic")
                  .replace("split+store weighted", "split split") for r in routes]
    if widths[0] > 32 and 9 * cin + 1 <= 64:
        recomputed[0] = recomputed[0].replace("split split", "split generic")
    assert _routes(st, len(widths)) == recomputed
    _check_all_regimes(m, x, y, theta, f"conv {cin}->{widths} {plane} recomputed", stepper=st)


@pytest.mark.parametrize("cin,cout,max_batch,norm", [
    (64, 128, 128, "split"), (64, 128, 160, "gram"), (96, 96, 120, "split"), (128, 128, 128, "split"), (128, 128, 160, "gram"),
    (192, 192, 90, "split"), (192, 192, 128, "gram"), (256, 256, 64, "split"), (256, 256, 90, "gram"), (128, 128, 257, "gram")])
def test_norms_of_8x8_planes_take_the_faster_kernel(cin, cout, max_batch, norm):
    from paper_2010_09063_amd import DpStep
    m = W.model(W.image_input(cin, 8, 8), [W.conv2d(cin, cout, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(2, 2), W.dense(16 * cout, 3)], 3)
    rng = np.random.default_rng(cin)
    x, y = W.make_inputs(m, 5, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    st = DpStep(m, max_batch)
    assert st.dp_step_describe_plan()[0]["norm"] == norm
    _check_all_regimes(m, x, y, theta, f"8x8 {cin}->{cout} {norm}", stepper=st)
    st.dp_step_free()


@pytest.mark.parametrize("cin,cout,plane,batch,options", [
    (48, 100, (24, 24), 5, {}), (33, 65, (16, 24), 9, {}), (16, 128, (28, 28), 2, {}),
    (20, 96, (16, 16), 3, dict(no_minimal_filtering=1, no_specialised_waves=1))])
def test_stored_gradients_of_wide_layers_on_the_direct_kernel(cin, cout, plane, batch, options):
    """More than 64 output channels on planes that the specialised-wave kernel does not take: four wave groups of nine taps
    a block of channels.  (Rows laid out for groups of five taps were too short: examples overwrote each other and the last one
    what lies behind the buffer.)"""
    from paper_2010_09063_amd import DpStep
    h, w = plane
    m = W.model(W.image_input(cin, h, w), [W.conv2d(cin, cout, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(4, 4),
                                           W.dense(cout * (h // 4) * (w // 4), 3)], 3)
    rng = np.random.default_rng(cout)
    x, y = W.make_inputs(m, batch, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    st = DpStep(m, batch, **options)
    assert _routes(st, 1)[0].endswith("direct+store weighted")
    _check_all_regimes(m, x, y, theta, f"conv {cin}->{cout} {plane} stored rows", stepper=st)


@pytest.mark.parametrize("cin,cout,plane,options", [
    (40, 14, (15, 32), {}), (90, 7, (16, 32), dict(no_minimal_filtering=1)), (33, 32, (32, 32), dict(no_minimal_filtering=1, no_stored_gradients=1))])
def test_direct_norms_of_several_examples_per_workgroup(cin, cout, plane, options):
    """Input channels that are no multiple of 32, at most 32 output channels and more examples than resident workgroups: the
    waves add up through the staging area, and what they leave in the planes of channels that do not exist must not reach the
    next example's norm (it was off by 4e-6 to 1.6e-4; the bar is ten times what is left)."""
    from oracle import dpsgd_oracle as O
    from paper_2010_09063_amd import DpStep
    from tests.gpu_util import run_gpu
    h, w = plane
    m = W.model(W.image_input(cin, h, w), [W.conv2d(cin, cout, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(3, 3),
                                           W.dense(cout * (h // 3) * (w // 3), 3)], 3)
    rng = np.random.default_rng(cin)
    x, y = W.make_inputs(m, 7, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    n = 120
    st = DpStep(m, 7 * n, **options)
    assert st.dp_step_describe_plan()[0]["norm"].startswith("direct")
    norms = run_gpu(m, theta, np.tile(x, (n, 1, 1, 1)), np.tile(y, n), 0.5, 0.0, 0, stepper=st)[1]
    st.dp_step_free()
    err = np.abs(norms.reshape(n, 7) / np.asarray(O.dp_step(m, theta, x, y, 0.5, 0.0, 0)["norms"]) - 1)
    print(f"{cin}->{cout} {plane}: norms off by up to {err.max():.1e}", flush=True)
    assert err.max() <= 2e-6


def test_norm_kernel_above_65535_examples():
    """One workgroup per example, in a dimension of the grid that goes that far.  Six examples 11,000 times over: the sum
    is 11,000 times theirs."""
    from oracle import dpsgd_oracle as O
    from paper_2010_09063_amd import DpStep
    from tests.gpu_util import assert_parity, run_gpu
    m = W.model(W.image_input(16, 8, 8), [W.conv2d(16, 20, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(4, 4), W.dense(80, 3)], 3)
    rng = np.random.default_rng(7)
    x, y = W.make_inputs(m, 6, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    n = 11000
    st = DpStep(m, 6 * n)
    assert st.dp_step_describe_plan()[0]["norm"] == "split"
    st_out, norms = run_gpu(m, theta, np.tile(x, (n,) + (1,) * (x.ndim - 1)), np.tile(y, n), 0.5, 0.0, 0, stepper=st)
    st.dp_step_free()
    ref = O.dp_step(m, theta, x, y, 0.5, 0.0, 0)
    assert_parity(m, st_out, n * np.asarray(ref["clipped_sum"]), "66,000 examples", n * np.asarray(ref["abs_sum"]))
    assert np.allclose(norms.reshape(n, 6), np.asarray(ref["norms"])[None], rtol=1e-4)


# Few input channels, whose padding to blocks of 32 costs more than the faster unit gives: norms and sums, each by its rule.
@pytest.mark.parametrize("cin,cout,plane,batch,norm,total", [
    (7, 97, (16, 16), 61, "generic", "generic"), (8, 97, (16, 16), 61, "split", "split"),  # one column of 64, a second one
    (7, 64, (16, 16), 61, "split", "generic"), (7, 65, (16, 16), 61, "generic", "generic"),
    (3, 63, (16, 16), 61, "split", "generic"), (3, 64, (16, 16), 61, "generic", "generic"),
    (7, 64, (16, 16), 257, "generic", "generic"), (7, 64, (8, 16), 61, "generic", "generic"), (7, 64, (6, 32), 61, "split", "generic"),
    (14, 9, (4, 4), 61, "generic", "generic"), (15, 9, (4, 4), 61, "split", "split"),
    (15, 32, (8, 8), 128, "generic", "generic"), (15, 32, (8, 8), 129, "split", "split"), (15, 33, (8, 8), 9, "split", "split"),
    (8, 32, (8, 16), 128, "split", "generic"), (8, 32, (8, 16), 129, "split", "split"), (8, 32, (6, 32), 9, "split", "split"),
    (5, 8, (16, 16), 511, "split", "split"), (5, 8, (16, 16), 512, "generic", "split"), (6, 8, (16, 16), 512, "split", "split")])
def test_weight_gradients_of_few_channels_take_the_faster_kernel(cin, cout, plane, batch, norm, total):
    from paper_2010_09063_amd import DpStep
    m = W.model(W.image_input(cin, *plane), [W.conv2d(cin, cout, 3, stride=1, pad=1, act="relu"), W.avgpool2d(2, 2),
                                             W.dense(cout * plane[0] * plane[1] // 4, 3)], 3)
    st = DpStep(m, batch, no_stored_gradients=1)
    plan = st.dp_step_describe_plan()[0]
    st.dp_step_free()
    assert (plan["norm"], plan["sum"]) == (norm, total)


def test_split_convolutions_add_no_bias():
    """The bf16 instruction rounds its sums downwards.  A bias gradient adds up 32,768 backprops here: an error of 2**-24 of
    each with one sign shows as 1e-5 of the tensor's size (1.1e-5 with all six products in one accumulator); with random
    signs the two routes differ by up to 2.6e-6.  The bar is twice that."""
    import torch
    from paper_2010_09063_amd import DpStep
    m = W.model(W.image_input(48, 16, 16), [W.conv2d(48, 48, 3, stride=1, pad=1, act="tanh") for _ in range(4)] +
                [W.maxpool2d(2, 2), W.dense(48 * 64, 3)], 3)
    rng = np.random.default_rng(1)
    x, y = W.make_inputs(m, 128, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.05)
    dev = torch.device("cuda")
    tt, tx, ty = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (theta, x, y))
    out = []
    for opt in ({}, {"generic_conv": 1}):
        st = DpStep(m, 128, **opt)
        g = torch.empty_like(tt)
        st.dp_step_nonprivate(tt, tx, ty, 128, g)
        out.append(g.double())
        st.dp_step_free()
    d = out[0] - out[1]
    at = 0
    for l in range(4):
        n = 48 * 48 * 9
        b = slice(at + n, at + n + 48)
        rms = out[1][at:at + n + 48].norm() / (n + 48) ** 0.5
        print(f"layer {l}: bias differs by up to {float(d[b].abs().max() / rms):.2e}, on average {float(d[b].mean() / rms):.2e}", flush=True)
        assert float(d[b].abs().max() / rms) <= 6e-6
        at += n + 48


def _split_case(kind):
    if kind == "lstm":
        m = W.model(W.token_input(256), [W.embedding(300, 100), W.lstm_last(100, 100), W.dense(100, 2)], 2)
        rng, batch = np.random.default_rng(3), 128
        x, y = W.make_inputs(m, batch, rng, zipf_exponent=1.1)
        return m, x, y, W.init_params(m, rng, bias_scale=0.05)
    m = W.model(W.image_input(16, 32, 32), [W.conv2d(16, 16, 3, stride=1, pad=1, act="tanh") for _ in range(2)] +
                [W.avgpool2d(2, 2), W.dense(16 * 256, 3)], 3)
    rng, batch = np.random.default_rng(4), 256
    x, y = W.make_inputs(m, batch, rng, x_dist="normal")
    return m, x, y, W.init_params(m, rng, bias_scale=0.05)


@pytest.mark.parametrize("kind,private", [("lstm", True), ("lstm", False), ("conv", True), ("conv", False)])
def test_split_products_have_no_one_sided_error(kind, private):
    """The bf16 instruction rounds its sums downwards, and gradients add up many of its results: per-example gradients
    (private) and partial sums over the batch, a frequent token's rows over all steps.  The mean error of a tensor
    against 64 bits, over its root mean square: random errors of 2e-7 to 6e-7 average to 1e-9 to 3e-9 (40,000 weights),
    6e-9 (2,304) and 1e-8 (800 coordinates of frequent tokens), somewhat more as they are not independent; the fp32
    kernels gave up to 5e-9, 1.2e-8 and 1.8e-8.  With every product of one sign it was -5e-8, -4.6e-7 and -7.5e-8."""
    import torch
    from oracle import dpsgd_oracle as O
    from paper_2010_09063_amd import DpStep
    m, x, y, theta = _split_case(kind)
    ref = np.asarray(O.dp_step(m, theta, x, y, 0.5 if private else 1e30, 0.0, 0)["clipped_sum"])
    dev = torch.device("cuda")
    tt, tx, ty = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (theta, x, y))
    st, g = DpStep(m, len(y)), torch.empty_like(tt)
    if private:
        st.dp_step(tt, tx, ty, len(y), 0.5, 0.0, 0, g)
    else:
        st.dp_step_nonprivate(tt, tx, ty, len(y), g)
    err = g.double().cpu().numpy() - ref
    st.dp_step_free()
    bars = {"E": 6e-8, "W_ih": 1.5e-8, "W_hh": 1.5e-8, "W": 8e-8}
    for li, name, shape, off in W.param_tensors(m):
        if name == "b" or m["layers"][li]["kind"] == "dense":
            continue
        s = slice(off, off + (8 * shape[1] if name == "E" else int(np.prod(shape))))  # (the embedding: its eight most frequent tokens)
        rms = np.sqrt(np.mean(ref[s] ** 2))
        print(f"layer {li} {name}: mean error {err[s].mean() / rms:+.2e}, rms {np.sqrt(np.mean(err[s] ** 2)) / rms:.2e}", flush=True)
        assert abs(err[s].mean() / rms) <= bars[name], (li, name)


@pytest.mark.parametrize("out", ["last", "seq"])
@pytest.mark.parametrize("dim,hidden,seq,batch,projection,dx", [
    (1, 1, 1, 1, "split", "split"),           # the smallest of everything
    (17, 33, 5, 7, "split", "split"),         # rows that start on 4 bytes; K one past a step, N past a block of columns
    (112, 104, 33, 3, "split", "split"),      # the widest that the projection's and the input gradient's waves hold; a ragged last tile of rows
    (113, 105, 3, 5, "generic", "generic"),   # one past both: the tiled contraction
    (128, 16, 4, 9, "split", "split"),        # the projection with its K in two halves
    (9, 100, 2, 6, "split", "split"),         # the recurrence's narrower padding filled, an even number of steps
    (12, 128, 2, 3, "split", "generic"),      # its wider padding filled
    (128, 128, 37, 5, "generic", "generic"),  # nine blocks of rows: three staged blocks per wave in the weight gradient
    (64, 56, 140, 3, "split", "split"),       # several tiles per workgroup's run would need more rows: stored per-example gradients
])
def test_lstm_products_with_weights_in_registers(dim, hidden, seq, batch, projection, dx, out):
    from paper_2010_09063_amd import DpStep
    layers = [W.embedding(40, dim), (W.lstm_last if out == "last" else W.lstm_seq)(dim, hidden)]
    layers += ([W.seq_mean()] if out == "seq" else []) + [W.dense(hidden, 3)]
    m = W.model(W.token_input(seq), layers, 3)
    rng = np.random.default_rng(dim + hidden)
    x, y = W.make_inputs(m, batch, rng, zipf_exponent=0.8)
    theta = W.init_params(m, rng, bias_scale=0.3) * np.float32(2)
    st = DpStep(m, batch)
    assert _routes(st, 2) == ["gather - pairs pairs", f"{projection}+recurrence recurrence+{dx} " +
                              ("split+store weighted" if seq >= 128 else "split split")]
    _check_all_regimes(m, x, y, theta, f"lstm {out} D{dim} H{hidden} T{seq} B{batch}", stepper=st)


def test_sequence_mean_holds_one_hidden_sequence():
    """The network with a mean over the hidden states needs no [batch][steps][hidden] buffer that the one on the last state
    does without: the recurrence takes the mean's gradient, and hidden states are there for the weight gradient anyway."""
    from paper_2010_09063_amd import DpStep
    ws = []
    for lstm, mean in ((W.lstm_last, []), (W.lstm_seq, [W.seq_mean()])):
        m = W.model(W.token_input(64), [W.embedding(50, 8), lstm(8, 100)] + mean + [W.dense(100, 2)], 2)
        st = DpStep(m, 64)
        ws.append(st.workspace_bytes)
        st.dp_step_free()
    assert ws[1] - ws[0] < 4 * 64 * 64 * 100 // 4, ws


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 1e30, float(np.finfo(np.float32).max), float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("kind", ["conv", "conv4", "lstm"])
def test_an_example_out_of_range_stays_its_own(kind, value):
    """One input value (a token's embedding for the LSTM) that is infinite, not a number, huge or the type's largest or
    lowest, as a mask is (a bf16 rounds that to infinity): the other examples' norms do not change, and the example's own is as finite as on the fp32 kernels (1e30 squared is not, in a Gram matrix)."""
    import torch
    from paper_2010_09063_amd import DpStep
    rng = np.random.default_rng(3)
    if kind == "lstm":
        m = W.model(W.token_input(12), [W.embedding(30, 16), W.lstm_last(16, 20), W.dense(20, 3)], 3)
        x, y = W.make_inputs(m, 7, rng, zipf_exponent=0.5)
        x[x == 29] = 3
    else:
        cin, cout, p = (16, 48, 16) if kind == "conv" else (24, 20, 4)
        m = W.model(W.image_input(cin, p, p), [W.conv2d(cin, cout, 3, stride=1, pad=1, act="tanh"),
                                               W.conv2d(cout, cout, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(2, 2), W.dense(cout * p * p // 4, 3)], 3)
        x, y = W.make_inputs(m, 7, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    dev = torch.device("cuda")

    def norms(theta, x, **options):
        st, out = DpStep(m, 7, **options), torch.empty(7, device=dev)
        tt, tx, ty = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (theta, x, y))
        st.dp_step(tt, tx, ty, 7, 1.0, 0.0, 0, torch.empty_like(tt))
        st.dp_step_last_norms(out)
        out = out.cpu().numpy()
        st.dp_step_free()
        return out

    clean, bad_x, bad_theta = norms(theta, x), x.copy(), theta.copy()
    if kind == "lstm":
        bad_x[2, 5] = 29
        bad_theta[29 * 16 + 4] = value
    else:
        bad_x.reshape(7, -1)[2, 77] = value
    here = norms(bad_theta, bad_x)
    plain = norms(bad_theta, bad_x, no_minimal_filtering=1, no_lstm_wgrad=1, no_rows_gemm=1, no_side_stream=1)
    others = [0, 1, 3, 4, 5, 6]
    assert np.array_equal(here[others], clean[others])
    assert np.isfinite(here[2]) == np.isfinite(plain[2]), (here[2], plain[2])


# rows of the pairs below a hidden layer: one coordinate per lane, four 32 apart (a last group of each size), four in line
@pytest.mark.parametrize("dim,seq,vocab", [(31, 40, 7), (33, 40, 7), (65, 300, 400), (129, 600, 90), (251, 40, 3000), (132, 300, 25)])
def test_embedding_rows_of_each_width_below_a_hidden_layer(dim, seq, vocab):
    from paper_2010_09063_amd import DpStep
    m = W.model(W.token_input(seq), [W.embedding(vocab, dim), W.seq_mean(), W.dense(dim, 12, "tanh"), W.dense(12, 5)], 5)
    rng = np.random.default_rng(dim)
    x, y = W.make_inputs(m, 9, rng)
    x[0, :] = vocab - 1  # one token throughout
    theta = W.init_params(m, rng, bias_scale=0.3)
    _check_all_regimes(m, x, y, theta, f"embedding {vocab}x{dim} T{seq} below a hidden layer", stepper=DpStep(m, 9))


# Large batches take the convolutions on the fp16 units; the routes go by the largest batch, so a few examples reach them, but for
# layers whose weights can be resident, which go by the batch.
@pytest.mark.parametrize("cin,widths,plane,act,pool,max_batch,batch,routes", [
    (32, (48, 33), (32, 32), "tanh", "max", 65, 3, ["f16 -", "f16+maxpool f16"]),   # two blocks of output channels; bands of one image
    (36, (33, 100), (8, 32), "relu", "avg", 257, 3, ["f16 -", "f16+avgpool f16"]),  # ragged chunks of sixteen; one image per two waves, an odd image over
    (49, (34, 130), (4, 32), "tanh", "avg", 513, 5, ["f16 -", "f16+avgpool f16"]),  # images of one strip; two and five blocks
    (48, (64, 40), (16, 16), "tanh", "max", 257, 2, ["f16 -", "f16+maxpool f16"]),
    (32, (128, 34), (4, 16), "relu", "max", 1025, 7, ["f16 -", "f16+maxpool f16"]), # four images of a tile, a ragged last one
    (33, (70, 36), (32, 16), "tanh", "avg", 129, 2, ["f16 -", "f16+avgpool f16"]),
    (130, (128, 34), (8, 8), "relu", "avg", 1025, 3, ["f16 -", "f16+avgpool f16"]), # four waves along the output channels; nine chunks
    (41, (130, 34), (16, 8), "tanh", "max", 513, 3, ["f16 -", "f16+maxpool f16"]),
    (56, (256, 64), (4, 4), "tanh", "max", 4097, 19, ["f16 -", "f16+maxpool f16"]),
    (35, (260, 34), (8, 4), "relu", "avg", 2049, 9, ["f16 -", "f16+avgpool f16"]),
    (32, (48, 36), (64, 32), "relu", "avg", 33, 1, ["f16 -", "f16+avgpool f16"]),
    (32, (32, 64), (32, 32), "tanh", "max", 65, 65, ["f16 -", "f16+maxpool split"]), # one block; three pieces stay three; the smallest batch that is not left to resident weights
    (32, (32, 64), (32, 32), "tanh", "max", 65, 64, ["f16 -", "f16+maxpool split"]), # the largest that is
    (32, (32, 64), (32, 32), "tanh", "max", 64, 3, ["mf32 -", "f16+maxpool split"]),
    (32, (48, 33), (32, 32), "tanh", "max", 65, 33, ["f16 -", "f16+maxpool f16"]),
    (40, (32, 64, 32), (16, 16), "relu", "avg", 140, 129, ["split -", "f16 split", "split+avgpool f16"]),  # 32 -> 64 each way, above the line and on it
    (40, (32, 64, 32), (16, 16), "relu", "avg", 140, 128, ["split -", "f16 split", "split+avgpool f16"]),
    (40, (32, 64, 32), (16, 16), "relu", "avg", 128, 5, ["split -", "mf32 split", "split+avgpool mf32"]),
    (64, (128, 128), (8, 8), "relu", "avg", 513, 3, ["f16 -", "f16+avgpool f16"]),   # one tile over the line, and on it
    (64, (128, 128), (8, 8), "relu", "avg", 512, 3, ["mf64 -", "mf64+avgpool mf64"]),
])
def test_convolutions_on_the_fp16_matrix_units(cin, widths, plane, act, pool, max_batch, batch, routes):
    from paper_2010_09063_amd import DpStep
    h, w = plane
    layers, c = [], cin
    for d in widths:
        layers.append(W.conv2d(c, d, 3, stride=1, pad=1, act=act))
        c = d
    layers += [W.maxpool2d(2, 2) if pool == "max" else W.avgpool2d(2, 2), W.dense(c * (h // 2) * (w // 2), 3)]
    m = W.model(W.image_input(cin, h, w), layers, 3)
    rng = np.random.default_rng(h * w + cin)
    x, y = W.make_inputs(m, batch, rng, x_dist="normal")
    x *= np.exp(rng.standard_normal((batch,) + (1,) * (x.ndim - 1))).astype(np.float32)  # every example has a scale of its own
    x.reshape(batch, cin, -1)[:, : cin // 2] *= np.float32(1e-3)  # and grows over the chunks of channels
    theta = W.init_params(m, rng, bias_scale=0.3)
    st = DpStep(m, max_batch)
    plan = st.dp_step_describe_plan()
    assert [plan[l]["fwd"] + " " + plan[l]["bwd"] for l in range(len(widths))] == routes
    _check_all_regimes(m, x, y, theta, f"conv {cin}->{widths} {plane} {act} {pool} B{batch} of {max_batch}", stepper=st)


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 1e30, -1e-30, float(np.finfo(np.float32).max), float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("where", ["value", "column"])
@pytest.mark.parametrize("plane,max_batch", [(32, 65), (16, 257), (8, 513), (4, 2049)])
def test_an_example_out_of_range_stays_its_own_on_the_fp16_units(plane, max_batch, where, value):
    """Scales go by example: one value or a column of every channel that is infinite, not a number, huge or tiny leaves the other
    examples as they are, and where the units behind it saturate the rest of its own example counts as it does in fp32."""
    import torch
    from paper_2010_09063_amd import DpStep
    rng = np.random.default_rng(3)
    c = max(36, 1024 // plane)
    m = W.model(W.image_input(40, plane, plane), [W.conv2d(40, c, 3, stride=1, pad=1, act="tanh"), W.conv2d(c, c, 3, stride=1, pad=1, act="relu"),
                                                  W.avgpool2d(2, 2), W.dense(c * plane * plane // 4, 3)], 3)
    x, y = W.make_inputs(m, 7, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    dev = torch.device("cuda")

    def step(x, max_batch, **options):
        """norms, clipped sum, plain sum"""
        st, out = DpStep(m, max_batch, **options), torch.empty(7, device=dev)
        plan = st.dp_step_describe_plan()
        assert all(plan[l]["fwd"].startswith("direct" if options else "f16") for l in (0, 1)), plan
        tt, tx, ty = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (theta, x, y))
        clipped, summed = torch.empty_like(tt), torch.empty_like(tt)
        st.dp_step(tt, tx, ty, 7, 1.0, 0.0, 0, clipped)
        st.dp_step_last_norms(out)
        st.dp_step_nonprivate(tt, tx, ty, 7, summed)
        got = [v.cpu().numpy() for v in (out, clipped, summed)]
        st.dp_step_free()
        return got

    bad = x.copy()
    if where == "value":
        bad.reshape(7, -1)[2, 77] = value
    else:
        bad.reshape(7, 40, plane, plane)[2, :, :, plane // 2] = value
    clean, here = step(x, max_batch)[0], step(bad, max_batch)
    plain = step(bad, 7, no_minimal_filtering=1)
    others = [0, 1, 3, 4, 5, 6]
    assert np.array_equal(here[0][others], clean[others])
    assert np.isfinite(here[0][2]) == np.isfinite(plain[0][2]), (here[0][2], plain[0][2])
    if np.isfinite(plain[0]).all():
        assert np.allclose(here[0], plain[0], rtol=1e-4)
        # the sums of both routes, tensor by tensor: 1.2e-6 apart at most without such values, about four times that
        for got, ref in zip(here[1:], plain[1:]):
            for li, name, shape, off in W.param_tensors(m):
                a, b = (v[off:off + int(np.prod(shape))].astype(np.float64) for v in (got, ref))
                assert np.linalg.norm(a - b) <= 5e-6 * np.linalg.norm(b), (li, name, np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("cin,widths,rows,batch", [(3, (33, 8), 32, 5), (1, (48, 8), 16, 3), (2, (64, 8), 32, 4), (3, (100, 8), 16, 2), (3, (64, 8), 16, 300)])
def test_first_layers_of_more_than_32_output_channels(cin, widths, rows, batch):
    """Forward pass and weight gradients of a first layer on up to three channels, blocks of 32 output channels and a last one that is not full; rows
    stored and not, and the same from an input that starts on 4 bytes, which the split kernel takes."""
    import torch
    from paper_2010_09063_amd import DpStep
    layers = [W.conv2d(cin, widths[0], 3, stride=1, pad=1, act="tanh"), W.maxpool2d(2, 2), W.conv2d(widths[0], widths[1], 3, stride=1, pad=1, act="tanh"),
              W.avgpool2d(2, 2), W.dense(widths[1] * 8 * rows // 4, 3)]
    m = W.model(W.image_input(cin, rows, 32), layers, 3)
    rng = np.random.default_rng(widths[0])
    x, y = W.make_inputs(m, batch, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.3)
    for options, norm in (({}, "first+store"), (dict(no_stored_gradients=1), "first")):
        st = DpStep(m, batch, **options)
        plan = st.dp_step_describe_plan()[0]
        assert (plan["fwd"], plan["norm"]) == ("first", norm)
        if batch < 100:
            _check_all_regimes(m, x, y, theta, f"first layer {cin}->{widths[0]} {rows}x32 {norm}", stepper=st)
        dev, out = torch.device("cuda"), []
        for shift in (0, 1):
            flat = torch.empty(x.size + 4, device=dev)
            tx = flat[shift:shift + x.size].view(*x.shape)
            tx.copy_(torch.from_numpy(x))
            tt, ty = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (theta, y))
            g, n = torch.empty_like(tt), torch.empty(batch, device=dev)
            st.dp_step(tt, tx, ty, batch, 1.0, 0.0, 0, g)
            st.dp_step_last_norms(n)
            out.append((g.double().cpu().numpy(), n.cpu().numpy()))
        st.dp_step_free()
        assert np.allclose(out[0][1], out[1][1], rtol=1e-5)
        assert np.linalg.norm(out[0][0] - out[1][0]) <= 1e-5 * np.linalg.norm(out[0][0])


@pytest.mark.parametrize("out", ["last", "seq"])
@pytest.mark.parametrize("hidden,seq,batch,scale", [
    (33, 5, 257, 2), (56, 2, 258, 2), (57, 1, 257, 2), (80, 7, 300, 2), (100, 6, 257, 2), (105, 3, 259, 2), (128, 9, 257, 2),
    (64, 12, 261, 4), (64, 3, 261, 30),  # gradients that grow or die by more than a scale allows for: written twice (as the first ones always are)
    (48, 40, 7, 2), (33, 3, 1, 2), (16, 6, 257, 2)])  # fewer examples: two per workgroup going forward only, or not at all
def test_lstm_recurrences_of_two_examples_per_workgroup(hidden, seq, batch, scale, out):
    """Above 256 examples, an odd one left over; the padded widths of the kernels filled and one past them."""
    layers = [W.embedding(40, 9), (W.lstm_last if out == "last" else W.lstm_seq)(9, hidden)]
    m = W.model(W.token_input(seq), layers + ([W.seq_mean()] if out == "seq" else []) + [W.dense(hidden, 3)], 3)
    rng = np.random.default_rng(hidden + seq)
    x, y = W.make_inputs(m, batch, rng, zipf_exponent=0.8)
    theta = W.init_params(m, rng, bias_scale=0.3) * np.float32(2)
    for li, name, shape, off in W.param_tensors(m):
        if name == "W_hh":
            theta[off:off + int(np.prod(shape))] *= np.float32(scale / 2)
    _check_all_regimes(m, x, y, theta, f"lstm {out} H{hidden} T{seq} B{batch}")
