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
