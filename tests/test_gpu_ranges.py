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
