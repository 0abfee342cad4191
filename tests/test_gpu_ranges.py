"""Operands of very different sizes on the routes that split fp32 operands into pieces: masks, outliers, wide weights.  The direct
fp32 kernels are the reference."""
import numpy as np
import pytest

import dp_workloads as W

pytestmark = pytest.mark.gpu


def _both_gradients(m, theta, x, y, max_batch, **options):
    """(plan, norms, clipped sum at C = 1, plain sum) of one step without noise."""
    import torch
    from paper_2010_09063_amd import DpStep
    dev = torch.device("cuda")
    st = DpStep(m, max_batch, **options)
    tt, tx, ty = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in (theta, x, y))
    n, g, p = torch.empty(len(y), device=dev), torch.empty_like(tt), torch.empty_like(tt)
    st.dp_step(tt, tx, ty, len(y), 1.0, 0.0, 0, g)
    st.dp_step_last_norms(n)
    st.dp_step_nonprivate(tt, tx, ty, len(y), p)
    out = (st.dp_step_describe_plan(), *(v.double().cpu().numpy() for v in (n, g, p)))
    st.dp_step_free()
    return out


def _by_tensor(m, got, ref, bar, label):
    for li, name, shape, off in W.param_tensors(m):
        a, b = got[off:off + int(np.prod(shape))], ref[off:off + int(np.prod(shape))]
        assert np.linalg.norm(a - b) <= bar * np.linalg.norm(b), (label, li, name, np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("columns,value", [(1, 1e9), (2, 1e9), (4, -1e9), (2, 1e30), (4, 1e30)])
@pytest.mark.parametrize("stored", [True, False])
@pytest.mark.parametrize("plane,max_batch", [(32, 7), (16, 7), (8, 7)])
def test_weight_gradients_behind_a_mask(plane, max_batch, stored, columns, value):
    """Columns of every channel of one example hold a huge value.  The units behind it saturate, so the gradient comes from the rest of
    the example alone, and the sums over the batch from the others too: 2e-5 is a tenth of what fp16 pieces under one scale lost."""
    rng = np.random.default_rng(plane + columns)
    m = W.model(W.image_input(40, plane, plane), [W.conv2d(40, 36, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(2, 2),
                                                  W.dense(36 * plane * plane // 4, 3)], 3)
    x, y = W.make_inputs(m, 7, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    x.reshape(7, 40, plane, plane)[2, :, :, plane // 2:plane // 2 + columns] = value
    plan, norms, clipped, plain = _both_gradients(m, theta, x, y, max_batch, **({} if stored else dict(no_stored_gradients=1)))
    assert (plan[0]["norm"], plan[0]["sum"]) == (("split+store", "weighted") if stored and plane > 8 else ("split", "split")), plan[0]
    _, norms0, clipped0, plain0 = _both_gradients(m, theta, x, y, max_batch, no_minimal_filtering=1)
    assert np.isfinite(norms0).all() and np.allclose(norms, norms0, rtol=2e-5)
    _by_tensor(m, clipped, clipped0, 2e-5, "clipped")
    _by_tensor(m, plain, plain0, 2e-5, "plain")


@pytest.mark.parametrize("power", [16, 18, 24])
@pytest.mark.parametrize("plane", [32, 16, 8])
def test_weight_gradient_sums_beside_a_large_example(plane, power):
    """A workgroup's share of the batch holds an example that is 2^power larger, saturates its units and adds nothing to the first layer's
    gradient: the others' sum is what it is without it.  All but twelve examples are empty, so that its neighbours are the sum."""
    rng = np.random.default_rng(plane)
    m = W.model(W.image_input(40, plane, plane), [W.conv2d(40, 36, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(2, 2),
                                                  W.dense(36 * plane * plane // 4, 3)], 3)
    x, y = W.make_inputs(m, 600, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    x[12:] = 0
    x[5] = np.abs(x[5]).max() * np.float32(2.0 ** power)
    keep = np.arange(600) != 5
    plan, _, _, plain = _both_gradients(m, theta, x, y, 600)
    assert plan[0]["sum"] in ("split", "weighted")
    _, _, _, one = _both_gradients(m, theta, x[~keep], y[~keep], 600, no_minimal_filtering=1)
    _, _, _, rest = _both_gradients(m, theta, x[keep], y[keep], 600, no_minimal_filtering=1)
    conv = 40 * 36 * 9
    assert np.abs(one[:conv]).max() == 0  # (an fp32 tanh of such a sum has a slope of zero)
    # fp32 sums over the rest in two orders: 1.1e-6 at most, four times that
    assert np.linalg.norm(plain[:conv] - rest[:conv]) <= 4.4e-6 * np.linalg.norm(rest[:conv])


@pytest.mark.parametrize("groups", [1, 2])
@pytest.mark.parametrize("plane", [32, 16, 8])
def test_weight_gradients_take_no_longer_for_small_values(plane, groups):
    """A few values 2^-40 of the others': no kernel goes another, slower way for them (the launches differ by the box's noise; a factor of two is asked)."""
    import torch
    from paper_2010_09063_amd import DpStep
    rng = np.random.default_rng(plane)
    m = W.model(W.image_input(40, plane, plane), [W.conv2d(40, 36, 3, stride=1, pad=1, act="tanh"), W.avgpool2d(2, 2),
                                                  W.dense(36 * plane * plane // 4, 3)], 3)
    x, y = W.make_inputs(m, 64, rng, x_dist="normal")
    x = 1 + np.abs(x)
    theta = W.init_params(m, rng, bias_scale=0.1)
    small = x.copy()
    for g in range(groups):
        small.reshape(64, 40, plane, plane)[3, 7 + g, 5, ::max(plane // 8, 2)] *= np.float32(2.0 ** -40)
    dev = torch.device("cuda")
    st = DpStep(m, 64, no_stored_gradients=1)
    tt, ty, g = torch.from_numpy(theta).to(dev), torch.from_numpy(y).to(dev), torch.empty(len(theta), device=dev)
    times = []
    for v in (x, small):
        tx, best = torch.from_numpy(np.ascontiguousarray(v)).to(dev), {}
        for _ in range(8):
            st.dp_step_profile(True)
            st.dp_step(tt, tx, ty, 64, 1.0, 0.0, 0, g)
            st.dp_step_nonprivate(tt, tx, ty, 64, g)
            for label, n, ms in st.dp_step_profile_read():
                best[label] = min(best.get(label, 1e9), ms / n)
        times.append(best)
    st.dp_step_free()
    assert "conv_wgrad_norm#0" in times[0] and "conv_clipped_sum#0" in times[0], times[0]
    assert all(times[1][k] <= 2 * times[0][k] for k in times[0]), times


def _fp16_network(plane, act="tanh"):
    c = max(33, 1024 // plane)  # (33: a block of 32 output channels and one of one)
    return c, W.model(W.image_input(40, plane, plane), [W.conv2d(40, c, 3, stride=1, pad=1, act=act), W.conv2d(c, c, 3, stride=1, pad=1, act="tanh"),
                                                        W.avgpool2d(2, 2), W.dense(c * plane * plane // 4, 3)], 3)


FP16_PLANES = [(32, 65), (16, 257), (8, 513), (4, 2049)]  # (plane, largest batch): more than 256 tiles of 128 pixels


def _same_as_direct(m, theta, x, y, max_batch, label):
    plan, norms, clipped, plain = _both_gradients(m, theta, x, y, max_batch)
    assert all(plan[l]["fwd"].startswith("f16") for l in (0, 1)) and plan[1]["bwd"] == "f16", plan
    _, norms0, clipped0, plain0 = _both_gradients(m, theta, x, y, len(y), no_minimal_filtering=1)
    # the two routes' rounding: 1.2e-6 at most in a tensor, 5.5e-7 in a norm; about four times that
    assert np.isfinite(norms0).all() and np.allclose(norms, norms0, rtol=2e-6), (label, norms / norms0 - 1)
    _by_tensor(m, clipped, clipped0, 5e-6, label + " clipped")
    _by_tensor(m, plain, plain0, 5e-6, label + " plain")


@pytest.mark.parametrize("kind", ["columns", "all but two columns", "all but three rows", "channels", "channels of half the filters"])
@pytest.mark.parametrize("value", [2.0 ** 18, 2.0 ** 21, 1e9, -1e15])
@pytest.mark.parametrize("plane,max_batch", FP16_PLANES)
def test_forward_pass_beside_a_mask(plane, max_batch, value, kind):
    """Huge inputs of one example saturate the units that see them; what the other units see of the image keeps its bits, whatever
    share of it that is."""
    c, m = _fp16_network(plane)
    rng = np.random.default_rng(plane)
    x, y = W.make_inputs(m, 5, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    v, w = x.reshape(5, 40, plane, plane), theta[:c * 40 * 9].reshape(c, 40, 9)
    if kind == "columns":
        v[2, :, :, plane // 2:] = value
    elif kind == "all but two columns":
        v[2, :, :, 2:] = value
    elif kind == "all but three rows":
        v[2, :, 3:] = value
    else:
        v[2, ::4] = value
        w[(slice(1, None, 2) if kind[8:] else slice(None)), ::4] = 0  # filters that do not look at these channels
    _same_as_direct(m, theta, x, y, max_batch, f"{kind} {value}")


@pytest.mark.parametrize("power", [15, 18, 21, 30, 60])
@pytest.mark.parametrize("plane,max_batch", FP16_PLANES)
def test_backprops_beside_a_large_part_that_does_not_count(plane, max_batch, power):
    """Half of every plane has backprops 2^power larger than the rest, and the layer before is saturated there: its gradient is the other half's."""
    c, m = _fp16_network(plane)
    rng = np.random.default_rng(plane)
    x, y = W.make_inputs(m, 5, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    x.reshape(5, 40, plane, plane)[:, :, :, plane // 2:] = 1e6
    last = theta[-(c * plane * plane // 4 * 3 + 3):-3].reshape(c, plane // 2, plane // 2, 3)
    last[:, :, :max(plane // 4 - 1, 1)] *= np.float32(2.0 ** -power)  # (the columns between see both)
    _same_as_direct(m, theta, x, y, max_batch, f"2^{power}")


@pytest.mark.parametrize("power", [12, 16, 20, 27, 60])
@pytest.mark.parametrize("plane,max_batch", FP16_PLANES)
def test_filters_of_very_different_sizes(plane, max_batch, power):
    """Three filters of four are 2^power smaller than the fourth, and the next layer makes up for it (no activation between: a tanh of a
    small value is good to 2^-24, not to its own size)."""
    c, m = _fp16_network(plane, "none")
    rng = np.random.default_rng(plane)
    x, y = W.make_inputs(m, 5, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    n = c * 40 * 9
    small = np.arange(c) % 4 != 0
    theta[:n].reshape(c, 360)[small] *= np.float32(2.0 ** -power)
    theta[n:n + c][small] *= np.float32(2.0 ** -power)
    theta[n + c:n + c + c * c * 9].reshape(c, c, 9)[:, small] *= np.float32(2.0 ** power)
    _same_as_direct(m, theta, x, y, max_batch, f"2^{power}")


@pytest.mark.parametrize("plane,max_batch", FP16_PLANES)
def test_forward_passes_take_no_longer_for_small_values(plane, max_batch):
    """Two pixels of an image, all channels, 2^-40 of the rest: a sum that sees others besides is as exact as any, and no other way is gone."""
    import torch
    from paper_2010_09063_amd import DpStep
    c, m = _fp16_network(plane)
    rng = np.random.default_rng(plane)
    x, y = W.make_inputs(m, 64, rng, x_dist="normal")
    theta = W.init_params(m, rng, bias_scale=0.1)
    small = x.copy()
    small.reshape(64, 40, plane, plane)[3, :, 1, :2] *= np.float32(2.0 ** -40)
    dev = torch.device("cuda")
    st = DpStep(m, max_batch)
    assert st.dp_step_describe_plan()[0]["fwd"] == "f16"
    tt, ty, g = torch.from_numpy(theta).to(dev), torch.from_numpy(y).to(dev), torch.empty(len(theta), device=dev)
    times = []
    for v in (x, small):
        tx, best = torch.from_numpy(np.ascontiguousarray(v)).to(dev), 1e9
        for _ in range(8):
            st.dp_step_profile(True)
            st.dp_step(tt, tx, ty, 64, 1.0, 0.0, 0, g)
            best = min([best] + [ms for label, _, ms in st.dp_step_profile_read() if label == "conv_fwd#0"])
        times.append(best)
    st.dp_step_free()
    assert times[1] <= 2 * times[0], times


@pytest.mark.parametrize("out", ["last", "seq"])
@pytest.mark.parametrize("where", ["into a saturated gate", "from a unit that is off"])
@pytest.mark.parametrize("hidden,power", [(48, 10), (48, 16), (48, 30), (100, 22), (100, 120), (128, 30)])
def test_lstm_weights_of_very_different_sizes(hidden, power, where, out):
    """Weights 2^power larger than the others that add nothing: those that lead into a gate which they saturate have no part in
    the gradient of the unit they come from, those that come from a unit which is always zero none in the state.  Two examples per
    workgroup against one, which is fp32 throughout."""
    layers = [W.embedding(40, 9), (W.lstm_last if out == "last" else W.lstm_seq)(9, hidden)]
    m = W.model(W.token_input(12), layers + ([W.seq_mean()] if out == "seq" else []) + [W.dense(hidden, 3)], 3)
    rng = np.random.default_rng(hidden)
    x, y = W.make_inputs(m, 258, rng, zipf_exponent=0.8)
    theta = W.init_params(m, rng, bias_scale=0.3) * np.float32(2)
    t = {name: theta[off:off + int(np.prod(shape))].reshape(shape) for li, name, shape, off in W.param_tensors(m) if li == 1}
    if where == "into a saturated gate":  # unit 7's output gate, from every unit, the same sign: far from zero from the second step on
        t["W_hh"][:, 3 * hidden + 7] = 2.0 ** power
        t["b"][3 * hidden + 7] = 2.0 ** power * hidden * 1.5  # (whatever the state)
    else:
        t["b"][3 * hidden + 5] = -1e4
        t["W_hh"][5, :] = 2.0 ** power
    _, norms, clipped, plain = _both_gradients(m, theta, x, y, 258)
    parts = [_both_gradients(m, theta, x[i:i + 129], y[i:i + 129], 129) for i in (0, 129)]
    norms0 = np.concatenate([p[1] for p in parts])
    assert np.isfinite(norms0).all() and np.allclose(norms, norms0, rtol=4e-6), np.abs(norms / norms0 - 1).max()
    _by_tensor(m, clipped, parts[0][2] + parts[1][2], 4e-6, "clipped")
    _by_tensor(m, plain, parts[0][3] + parts[1][3], 4e-6, "plain")


@pytest.mark.parametrize("out", ["last", "seq"])
@pytest.mark.parametrize("hidden", [48, 64, 100, 128])
@pytest.mark.parametrize("power,between", [(12, 2.0 ** -25), (18, 2.0 ** -25), (23, 2.0 ** -25), (30, 0.0)])
def test_lstm_gate_gradients_of_very_different_sizes(hidden, power, between, out):
    """Half of the units count 2^power less and hardly look at the other half's gates: their part of the gradient comes from themselves.
    Two examples per workgroup against one, which is fp32 throughout."""
    layers = [W.embedding(40, 9), (W.lstm_last if out == "last" else W.lstm_seq)(9, hidden)]
    m = W.model(W.token_input(12), layers + ([W.seq_mean()] if out == "seq" else []) + [W.dense(hidden, 3)], 3)
    rng = np.random.default_rng(hidden + power)
    x, y = W.make_inputs(m, 258, rng, zipf_exponent=0.8)
    theta = W.init_params(m, rng, bias_scale=0.3) * np.float32(2)
    at = {(li, name): slice(off, off + int(np.prod(shape))) for li, name, shape, off in W.param_tensors(m)}
    last = max(li for li, _ in at)
    half = np.arange(hidden) < hidden // 2  # the units that count
    gates = np.tile(half, 4)
    w = theta[at[1, "W_hh"]].reshape(hidden, 4 * hidden)
    w[np.ix_(~half, gates)] = np.sign(w[np.ix_(~half, gates)]) * np.abs(w).max() * np.float32(between)
    theta[at[last, "W"]].reshape(hidden, 3)[~half] *= np.float32(2.0 ** -power)
    _, norms, clipped, plain = _both_gradients(m, theta, x, y, 258)
    parts = [_both_gradients(m, theta, x[i:i + 129], y[i:i + 129], 129) for i in (0, 129)]
    assert np.allclose(norms, np.concatenate([p[1] for p in parts]), rtol=4e-6)
    for got, ref, label in ((clipped, parts[0][2] + parts[1][2], "clipped"), (plain, parts[0][3] + parts[1][3], "plain")):
        _by_tensor(m, got, ref, 4e-6, label)
        for name in ("W_ih", "W_hh", "b"):
            a, b = (v[at[1, name]].reshape(-1, 4 * hidden)[:, ~gates] for v in (got, ref))
            # the two routes' rounding: 3.1e-7 at most at 2^12, 9.2e-7 at 2^23; about four times that
            assert np.linalg.norm(a - b) <= 4e-6 * np.linalg.norm(b), (label, name, np.linalg.norm(a - b) / np.linalg.norm(b))
