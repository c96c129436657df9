"""Host-only checks of the driver's buffers and of what its training step launches (no kernel runs: the device calls
of the binding are replaced by recorders, the buffers lie in host memory)."""
import types

import numpy as np
import pytest

from ggnn_synth import backbone_graph, draw_candidates, draw_params, draw_readout

torch = pytest.importorskip("torch")
from paper_1906_11786_amd import capi, driver  # noqa: E402

E, H, N = 3, 32, 200


@pytest.fixture
def calls(monkeypatch):
    """Names of the binding's device calls with their arguments, in order."""
    log = []
    for name in ("ggnn_transpose_weights", "ggnn_gru_pack_weights", "ggnn_forward", "ggnn_backward", "ggnn_readout_loss",
                 "ggnn_readout_loss_bwd", "ggnn_sgd_momentum"):
        monkeypatch.setattr(capi, name, lambda *a, _n=name: log.append((_n, a)))
    return log


def _model(dt, params=None):
    comp = driver.compile_graphs([backbone_graph(5, 0, N, E, span_mean=4.0, max_span=30)], 32, E, reorder=False)
    params = draw_params(5, N, comp.n_pad, H, E, dt, with_bias=True) if params is None else params(comp)
    return driver.BandedGGNN(comp, H, 1, dt, params, device="cpu"), params, comp


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_parameters_of_more_types_than_the_graphs_have(dt, calls):
    def more(comp):
        p = draw_params(5, N, comp.n_pad, H, E + 2, dt, with_bias=True)
        return types.SimpleNamespace(**{k: getattr(p, k) for k in ("X", "G", "W", "bias", "Wi", "U", "b")})
    m, p, _ = _model(dt, more)
    np.testing.assert_array_equal(m.W.float().numpy(), np.asarray(p.W[:E], np.float32))
    np.testing.assert_array_equal(m.bias.numpy(), np.asarray(p.bias[:E], np.float32))
    np.testing.assert_array_equal(m.U.float().numpy(), np.asarray(p.U, np.float32))


@pytest.mark.parametrize("name", ["W", "bias", "Wi", "U", "b"])
def test_parameters_of_too_few_values_are_refused(name, calls):
    def fewer(comp):
        p = draw_params(5, N, comp.n_pad, H, E, "f32", with_bias=True)
        d = {k: getattr(p, k) for k in ("X", "G", "W", "bias", "Wi", "U", "b")}
        d[name] = np.ones(1)
        return types.SimpleNamespace(**d)
    with pytest.raises(ValueError, match=name):
        _model("f32", fewer)


@pytest.mark.parametrize("shape", [(H,), (H, 1), (1, H)])
def test_readout_weights_of_any_shape_with_h_values(shape, calls):
    m, _, comp = _model("f32")
    w, b = draw_readout(5, H)
    m.setup_training(draw_candidates(5, comp.offsets), np.reshape(w, shape), b)
    np.testing.assert_array_equal(m.w_out.numpy(), np.asarray(w, np.float32))


@pytest.mark.parametrize("count", [0, 1, H - 1, H + 1])
def test_readout_weights_of_another_count_are_refused(count, calls):
    m, _, comp = _model("f32")
    with pytest.raises(ValueError, match="w_out"):
        m.setup_training(draw_candidates(5, comp.offsets), np.ones(count), 0.0)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_a_second_setup_leaves_the_tensors_of_the_first(dt, calls):
    m, _, comp = _model(dt)
    cands = draw_candidates(5, comp.offsets)
    m.setup_training(cands, np.full(H, 2.0), 3.0)
    held = [m.w_out, m.b_out] + [st[0] for st in m.param_state if st[3] is not None] + [st[1] for st in m.param_state]
    for t in held:
        t.add_(0.25)   # as training does
    want = [t.clone() for t in held]
    m.setup_training(cands, np.full(H, 5.0), 7.0)
    assert all(torch.equal(a, b) for a, b in zip(held, want))
    assert (m.w_out == 5).all() and m.b_out.item() == 7 and not any(st[1].any() for st in m.param_state)
    # the parameters of the model itself stay where they are, and the masters hold their values
    assert m.param_state[3][0] is m.b and m.model.b == m.b.data_ptr()
    for i, t in enumerate((m.W, m.Wi, m.U, m.b)):
        assert torch.equal(m.param_state[i][0].to(t.dtype), t)
    del calls[:]
    m.train_step()
    updates = [a for n, a in calls if n == "ggnn_sgd_momentum"]
    assert len(updates) == len(m.param_state)
    assert {a[1].data_ptr() for a in updates} == {st[0].data_ptr() for st in m.param_state}


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_train_step_updates_what_param_state_holds(dt, calls):
    """One launch for the parameters as set up; without an entry (a parameter that is to stay as it is), or with
    another in its place, one launch per entry that is left."""
    m, _, comp = _model(dt)
    m.setup_training(draw_candidates(5, comp.offsets), *draw_readout(5, H))

    def updated():
        del calls[:]
        m.train_step()
        return [(a[1].data_ptr(), a[2].data_ptr(), a[3].data_ptr()) for n, a in calls if n == "ggnn_sgd_momentum"]
    assert updated() == [(m.master.data_ptr(), m.velocity.data_ptr(), m.grad_buf.data_ptr())]
    full = list(m.param_state)
    for state in (full[1:], full[:2] + [tuple(t.clone() if isinstance(t, torch.Tensor) else t for t in full[2])] + full[3:],
                  []):
        m.param_state = state
        assert updated() == [tuple(t.data_ptr() for t in st[:3]) for st in state]
    m.param_state = full
    assert len(updated()) == 1
