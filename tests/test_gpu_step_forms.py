"""Launch forms of the device kernels at the sizes where their choice changes,
against the CPU oracle: integer-valued inputs, where every partial sum is exact,
are compared bitwise."""
import numpy as np
import pytest

import oracle as O
from gpu_helpers import TOL, relerr, say, dev, host, round_to, torch_dt

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
capi = pytest.importorskip("paper_1906_11786_amd.capi")


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    yield
    torch.cuda.synchronize()


def _edges(rng, n, m, E, span):
    src = rng.integers(0, n, m)
    dst = np.clip(src + rng.integers(-span, span + 1, m), 0, n - 1)
    return src, dst, rng.integers(0, E, m)


def _step_case(dt, B, H, E, nb, seed, bias):
    """One forward and one reverse step (ggnn_step_bits_gru's aggregate, with and without W^T, and
    ggnn_banded_step_bits_bwd), integers."""
    rng = np.random.default_rng(seed)
    n = B * nb
    src, dst, et = _edges(rng, n, 3 * n, E, min(2 * B, 70))
    bits, bits_t, _, _, _ = capi.ggnn_banded_pack_bits(n, E, B, src, dst, et)
    s, d, e, _, _ = O.kept_edges(src, dst, et, B)
    X = rng.integers(-2, 3, (n, H)).astype(np.float64)
    W = rng.integers(-1, 2, (E, H, H)).astype(np.float64)
    b = rng.integers(-2, 3, (E, H)).astype(np.float64) if bias else None
    want = O.aggregate(n, s, d, e, O.msg_transform(X, W, b))
    tb, tbt = torch.from_numpy(bits).cuda(), torch.from_numpy(bits_t).cuda()
    Xt, Wt_, bt = dev(X, dt), dev(W, dt), None if b is None else dev(b)
    a = torch.full((n, H), float("nan"), device="cuda")
    capi.ggnn_banded_step_bits(dt, n, B, H, E, tb, Xt, Wt_, bt, a)
    np.testing.assert_array_equal(host(a), want)
    WT = dev(W.transpose(0, 2, 1), dt)
    z = torch.zeros((H, 3 * H), device="cuda", dtype=torch_dt(dt))
    ho, sv = torch.empty_like(Xt), torch.empty((n, 3 * H), device="cuda", dtype=torch_dt(dt))
    a.fill_(float("nan"))
    capi.ggnn_step_bits_gru(dt, n, B, H, E, tb, Xt, Wt_, WT, bt, z, z, torch.zeros(3 * H, device="cuda"), a, ho, sv)
    np.testing.assert_array_equal(host(a), want)
    np.testing.assert_array_equal(host(ho), X / 2)   # r = z = 1/2, n = 0
    da = rng.integers(-2, 3, (n, H)).astype(np.float64)
    dX = dev(rng.integers(-3, 4, (n, H)).astype(np.float64))
    dX0 = host(dX)
    dM = torch.full((E, n + 3, H), float("nan"), device="cuda", dtype=torch_dt(dt))
    capi.ggnn_banded_step_bits_bwd(dt, n, B, H, E, tbt, dev(da.T, dt), Wt_, dX, dX, dM, n + 3)
    wM = O.aggregate_transpose(n, s, d, e, da, E)
    np.testing.assert_array_equal(host(dM[:, :n]), wM)
    np.testing.assert_array_equal(host(dX), dX0 + np.einsum("eno,eho->nh", wM, W))


# fp32: up to 256 row tiles of 32 nodes a workgroup holds one of them and eight type groups (four at B = 32 with up to
# four types), up to 512 two and four (one and four at B = 32), above that more rows and two groups; fewer types than
# groups, more, one type (16 rows per wave at H = 256).
@pytest.mark.parametrize("B,H,E,nb,bias", [
    (32, 32, 3, 520, True), (64, 64, 2, 260, False), (128, 64, 5, 130, True), (256, 32, 1, 65, False),
    (512, 64, 3, 33, True), (128, 128, 9, 2, True), (256, 256, 2, 1, False), (512, 128, 1, 2, True),
    (32, 256, 10, 3, True), (64, 256, 2, 5, True), (32, 64, 4, 300, False), (32, 32, 5, 7, True), (32, 32, 9, 300, True),
    (64, 32, 10, 140, False), (128, 64, 3, 70, True), (32, 256, 1, 2, True), (32, 256, 1, 257, False),
    (64, 256, 1, 3, True), (64, 256, 1, 130, False), (64, 256, 1, 257, True), (128, 256, 1, 2, True),
    (128, 256, 1, 65, False), (256, 256, 1, 33, True), (128, 256, 1, 129, True), (512, 256, 1, 1, False)])
def test_f32_step_forms_integer_exact(B, H, E, nb, bias):
    say(f"f32 step form B={B} H={H} E={E} nb={nb} bias={bias}")
    _step_case("f32", B, H, E, nb, B + H + E, bias)


# bf16: the direct-weight kernel's workgroup forms (up to 256 row tiles of 32 nodes, up to 512, more), both
# sides of the sizes where another kernel takes over (H = 64: 128 tiles at B <= 128; in the forward with its GRU
# from 5 types on at B = 128, from 7 at B = 64 and at H = 32, B = 256).
@pytest.mark.parametrize("B,H,E,nb,bias", [
    (64, 64, 7, 2, True), (64, 64, 6, 64, False), (128, 64, 5, 1, True), (128, 64, 4, 32, True), (256, 32, 7, 16, True),
    (256, 32, 6, 3, False), (256, 32, 8, 17, False), (64, 64, 9, 64, True), (64, 64, 3, 65, True), (128, 64, 10, 32, False), (128, 64, 3, 33, False),
    (256, 64, 5, 3, True), (256, 64, 2, 20, False), (256, 64, 2, 65, True), (512, 32, 3, 2, True), (512, 32, 1, 33, False),
    (256, 32, 2, 16, True), (32, 128, 3, 4, True), (32, 128, 2, 520, False), (64, 128, 1, 260, True),
    (128, 128, 9, 2, False), (128, 128, 2, 40, True), (128, 128, 2, 130, True), (256, 128, 2, 17, False),
    (512, 128, 1, 33, True), (32, 256, 3, 5, True), (64, 256, 2, 70, False), (128, 256, 1, 40, True),
    (256, 256, 2, 1, True), (512, 256, 1, 2, True),
    (64, 128, 3, 140, True), (128, 128, 9, 70, False), (32, 128, 7, 300, True), (32, 256, 2, 300, True),
    (64, 256, 10, 130, False), (128, 256, 3, 70, True), (256, 64, 9, 33, True),
    # one type without W^T: the narrow kernel's streamed blocks
    (64, 128, 1, 130, True), (64, 128, 1, 128, False), (512, 64, 1, 65, True), (512, 64, 1, 64, False),
    (64, 256, 1, 1, True), (512, 256, 1, 1, False),
    # above the direct-weight kernel's sizes at H >= 128 with W^T and in reverse: the wide kernel
    (32, 128, 2, 1025, True), (64, 128, 1, 513, True), (128, 128, 3, 257, True), (256, 128, 1, 129, True),
    (512, 128, 2, 65, False), (32, 256, 2, 513, True), (64, 256, 1, 257, True), (128, 256, 3, 129, True),
    (256, 256, 1, 65, True), (256, 256, 2, 65, False), (512, 256, 2, 65, True), (512, 256, 1, 65, True)])
def test_bf16_step_forms_integer_exact(B, H, E, nb, bias):
    say(f"bf16 step form B={B} H={H} E={E} nb={nb} bias={bias}")
    _step_case("bf16", B, H, E, nb, B + H + E, bias)


@pytest.mark.parametrize("B", [32, 128, 512])
def test_f32_step_keeps_every_bit(B):
    """One message per node through W = I: the aggregate is the sender's state, bit for bit, over the whole
    range of float32 (the states are staged as three bf16 parts; the smallest part of 2^-90 is above the
    subnormal range)."""
    n, H = 2 * B, 32
    rng = np.random.default_rng(B)
    m = rng.integers(1 << 23, 1 << 24, (n, H)).astype(np.float64) * rng.choice([-1.0, 1.0], (n, H))
    X = m * np.exp2(rng.integers(-90, 127, (n, H)) - 23.0)
    src, dst = np.arange(n), (np.arange(n) + 1) % n
    keep = np.abs(src // B - dst // B) <= 1
    src, dst = src[keep], dst[keep]
    bits, bits_t, _, _, _ = capi.ggnn_banded_pack_bits(n, 1, B, src, dst, np.zeros(len(src), int))
    I = dev(np.eye(H)[None])
    a = torch.full((n, H), float("nan"), device="cuda")
    capi.ggnn_banded_step_bits("f32", n, B, H, 1, torch.from_numpy(bits).cuda(), dev(X), I, None, a)
    want = np.zeros((n, H))
    want[dst] = X[src]
    np.testing.assert_array_equal(host(a), want)
    dM, dX = torch.empty((1, n, H), device="cuda"), torch.empty((n, H), device="cuda")
    capi.ggnn_banded_step_bits_bwd("f32", n, B, H, 1, torch.from_numpy(bits_t).cuda(), dev(X.T), I, None, dX, dM, n)
    want = np.zeros((n, H))
    want[src] = X[dst]
    np.testing.assert_array_equal(host(dM[0]), want)
    np.testing.assert_array_equal(host(dX), want)


# bf16 node update: one, two or four tiles of 16 nodes per wave (up to 256 workgroups of the first, of the second,
# else), by two groups of waves at H = 64 and four at H = 32; the last workgroup partly or mostly past the end.
@pytest.mark.parametrize("H,n", [(32, 32), (32, 288), (32, 16416), (32, 32800), (64, 160), (64, 4128), (64, 8224),
                                 (64, 16416), (128, 32), (128, 4096), (128, 4128), (128, 8224), (256, 96), (256, 4096),
                                 (256, 4160), (256, 8224)])
def test_gru_update_forms(H, n):
    say(f"gru_update form H={H} n={n}")
    rng = np.random.default_rng(H + n)
    k = 1 / np.sqrt(H)
    a = round_to("f32", 3 * rng.standard_normal((n, H)))
    h = round_to("bf16", rng.standard_normal((n, H)))
    Wi, U = (round_to("bf16", rng.uniform(-k, k, (H, 3 * H))) for _ in range(2))
    b = round_to("f32", rng.uniform(-k, k, 3 * H))
    out = torch.full((n, H), float("nan"), device="cuda", dtype=torch.bfloat16)
    sv = torch.full((n, 3 * H), float("nan"), device="cuda", dtype=torch.bfloat16)
    args = ("bf16", n, H, dev(a), dev(h, "bf16"), dev(Wi, "bf16"), dev(U, "bf16"), dev(b))
    capi.ggnn_gru_update(*args, out, sv)
    y, r, z, nn = O.gru_forward(a, h, Wi, U, b)
    # Stored in bf16: half a unit in the last of 8 bits, at most 2^-8 of the value.  Before that r*h (|r*h| < 5) is
    # rounded to bf16, an error of at most 2^-8 |r h| in each of H terms times |U| <= H^-1/2: independent, about
    # 2^-8 rms(r h) / 3 in the candidate, six times which bounds the largest of 10^6 (the other operands are exact
    # or split to 16 bits, 2^-17).
    slack = 6 * 2.0 ** -8 * np.sqrt(np.mean((r * h) ** 2)) / 3
    for got, want in ((out, y), (sv, np.concatenate([r, z, nn], 1))):
        assert np.max(np.abs(host(got) - want) - 2.0 ** -8 * np.abs(want)) <= slack
    ns = torch.full((n, H), float("nan"), device="cuda", dtype=torch.bfloat16)
    capi.ggnn_gru_update(*args, ns, None)
    assert torch.equal(ns, out)


# Sparse step on grids around the sizes where all types' weights go to LDS, where they fit (E <= 14 at H = 64 in
# bf16); uneven shares of the groups, a receiver with more senders than the LDS copy of its group holds, odd E.
@pytest.mark.parametrize("dt,H,E,n", [("bf16", 64, 14, 16384), ("bf16", 64, 15, 16384), ("bf16", 64, 1, 16352),
                                      ("bf16", 32, 7, 20000), ("f32", 32, 11, 16416), ("f32", 64, 3, 16416)])
def test_sparse_step_forms_integer_exact(dt, H, E, n):
    say(f"sparse_step form dt={dt} H={H} E={E} n={n}")
    rng = np.random.default_rng(H + E + n)
    m = 4 * n
    src, dst, et = rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(0, E, m)
    dst[:600], et[:600] = n - 5, E - 1          # 600 senders of one receiver
    dst[600:700], et[600:700] = 17, 0
    X = rng.integers(-2, 3, (n, H)).astype(np.float64)
    W = rng.integers(-1, 2, (E, H, H)).astype(np.float64)
    bias = rng.integers(-2, 3, (E, H)).astype(np.float64) if E % 2 else None
    row_ptr, col, _ = capi.ggnn_sparse_csr(n, E, src, dst, et)
    a = torch.full((n, H), float("nan"), device="cuda")
    capi.ggnn_sparse_step(dt, n, H, E, torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), len(col),
                          dev(X, dt), dev(W.transpose(0, 2, 1), dt), None if bias is None else dev(bias), a)
    s, d, e, _ = O.dedupe_edges(src, dst, et)
    np.testing.assert_array_equal(host(a), O.aggregate(n, s, d, e, O.msg_transform(X, W, bias)))


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_parameters_keep_their_addresses(dt):
    """The parameters a captured pass reads are the ones a training step updates, also when training is set up
    after the capture; the flat buffers' gaps stay zero."""
    from ggnn_synth import backbone_graph, draw_candidates, draw_params, draw_readout
    from paper_1906_11786_amd.driver import BandedGGNN, compile_graphs
    E, H, n = 3, 32, 200
    comp = compile_graphs([backbone_graph(5, 0, n, E, span_mean=4.0, max_span=30)], 32, E, reorder=False)
    m = BandedGGNN(comp, H, 2, dt, draw_params(5, n, comp.n_pad, H, E, dt, with_bias=True))
    m.capture()
    before = [t.data_ptr() for t in (m.W, m.bias, m.Wi, m.U, m.b)]
    cands = draw_candidates(5, comp.offsets)
    m.setup_training(cands, *draw_readout(5, H), lr=0.1, momentum=0.9, weight_decay=0.01)
    m.train_step()
    assert before == [t.data_ptr() for t in (m.W, m.bias, m.Wi, m.U, m.b)]
    m.step()
    eager = {k: v.copy() for k, v in m.results().items()}
    for _ in range(3):
        m.X[1:].zero_()
        m.replay()
        torch.cuda.synchronize()
        for k, v in m.results().items():
            np.testing.assert_array_equal(v, eager[k])
    used = torch.zeros_like(m.master, dtype=torch.bool)
    for v in m._views(used):
        v.fill_(True)
    assert not m.master[~used].any() and not m.velocity[~used].any()


# bf16 node reverse at H >= 128: 32 nodes per workgroup up to 8,192 nodes, else 64, the last workgroup partly past the
# end; two buffers (test_step_bits_gru_bwd_in_place has dh in the upstream gradient's).
@pytest.mark.parametrize("H,n", [(128, 32), (128, 96), (128, 8192), (128, 8224), (256, 32), (256, 8224)])
def test_gru_update_bwd_forms(H, n):
    say(f"gru_update_bwd form H={H} n={n}")
    rng = np.random.default_rng(H + n)
    k = 1 / np.sqrt(H)
    a = round_to("f32", rng.standard_normal((n, H)))
    h = round_to("bf16", rng.standard_normal((n, H)))
    Wi, U = (round_to("bf16", rng.uniform(-k, k, (H, 3 * H))) for _ in range(2))
    b = round_to("f32", rng.uniform(-k, k, 3 * H))
    g = round_to("f32", rng.standard_normal((n, H)))
    gates = [round_to("bf16", x) for x in O.gru_forward(a, h, Wi, U, b)[1:]]
    want = O.gru_backward(g, a, h, *gates, Wi, U)
    ws_n = capi.ggnn_gru_update_bwd_workspace_bytes("bf16", n, H)
    ws = torch.empty(ws_n, dtype=torch.uint8, device="cuda")
    da = torch.full((H, n), float("nan"), device="cuda", dtype=torch.bfloat16)
    dh = torch.full((n, H), float("nan"), device="cuda")
    dWi, dU, db = torch.zeros((H, 3 * H), device="cuda"), torch.zeros((H, 3 * H), device="cuda"), torch.zeros(3 * H, device="cuda")
    capi.ggnn_gru_update_bwd("bf16", n, H, dev(g), dev(a), dev(h, "bf16"), dev(np.concatenate(gates, 1), "bf16"),
                             dev(Wi, "bf16"), dev(U, "bf16"), da, dh, dWi, dU, db, ws, ws_n)
    got = (host(da).T, host(dh), host(dWi), host(dU), host(db))
    for w, x in zip(want, got):
        assert relerr(x, w) <= TOL["bf16"]


# The reverse step whose GRU reverse is a launch of its own works in place (dh_prev takes the summed gradient, then
# dh): the same bits as with two buffers.  fp32 and small bf16 grids (gru_bwd_kernel), 32 and 64 nodes per workgroup
# at H >= 128 with the last one partly past the end.
@pytest.mark.parametrize("dt,B,H,n", [("f32", 32, 32, 96), ("f32", 64, 128, 8256), ("bf16", 64, 64, 4096),
                                      ("bf16", 32, 128, 8224), ("bf16", 32, 256, 96), ("bf16", 32, 256, 8224)])
def test_step_bits_gru_bwd_in_place(dt, B, H, n):
    say(f"step_bits_gru_bwd in place dt={dt} B={B} H={H} n={n}")
    E = 5
    rng = np.random.default_rng(B + H + n)
    k = 1 / np.sqrt(H)
    _, bits_t, _, _, _ = capi.ggnn_banded_pack_bits(n, E, B, *_edges(rng, n, 3 * n, E, 20))
    bits_t = torch.from_numpy(bits_t).cuda()
    da, h = (dev(round_to(dt, rng.standard_normal(s)), dt) for s in ((H, n), (n, H)))
    W = dev(round_to(dt, k * rng.standard_normal((E, H, H))), dt)
    Wi, U = (dev(round_to(dt, rng.uniform(-k, k, (H, 3 * H))), dt) for _ in range(2))
    gates = dev(round_to(dt, rng.uniform(0, 1, (n, 3 * H))), dt)
    dX_in = dev(rng.standard_normal((n, H)))
    dM = torch.empty((E, n, H), device="cuda", dtype=torch_dt(dt))
    dap, dhp = torch.empty_like(da), torch.full((n, H), float("nan"), device="cuda")
    gh = torch.empty_like(gates)
    capi.ggnn_step_bits_gru_bwd(dt, n, B, H, E, bits_t, da, W, dX_in, dM, n, Wi, U, h, gates, dap, dhp, gh)
    g, da2, dh2 = torch.empty_like(dX_in), torch.empty_like(da), torch.empty_like(dX_in)
    capi.ggnn_banded_step_bits_bwd(dt, n, B, H, E, bits_t, da, W, dX_in, g, dM, n)
    ws_n = capi.ggnn_gru_update_bwd_workspace_bytes(dt, n, H)
    ws = torch.empty(ws_n, dtype=torch.uint8, device="cuda")
    sums = [torch.zeros(s, device="cuda") for s in ((H, 3 * H), (H, 3 * H), (3 * H,))]
    capi.ggnn_gru_update_bwd(dt, n, H, g, g, h, gates, Wi, U, da2, dh2, *sums, ws, ws_n)
    assert torch.equal(dap, da2) and torch.equal(dhp, dh2)


# Sparse step with all weights in LDS, on both sides of the grids where it starts (1,024 or 1,250 groups at H = 64, by
# the types; 1,024, 1,250 or 2,049 at H = 32) and with long lists: up to four receivers of a group with more than 48
# senders of one type have them shared by the wave, five and more walk theirs one by one.
@pytest.mark.parametrize("dt,H,E,n", [("bf16", 64, 4, 16384), ("bf16", 64, 4, 16352), ("bf16", 64, 10, 20000),
                                      ("bf16", 64, 14, 20032), ("bf16", 64, 10, 19968), ("bf16", 32, 2, 16384),
                                      ("bf16", 32, 4, 20000), ("bf16", 32, 9, 32800), ("bf16", 32, 9, 32768),
                                      ("f32", 32, 8, 32800), ("f32", 64, 3, 20000), ("f32", 64, 7, 33056)])
def test_sparse_step_long_lists_integer_exact(dt, H, E, n):
    say(f"sparse_step long lists dt={dt} H={H} E={E} n={n}")
    rng = np.random.default_rng(H + E + n)
    src, dst, et = [rng.integers(0, n, n)], [rng.integers(0, n, n)], [rng.integers(0, E, n)]

    def senders(node, typ, count):
        src.append(rng.choice(n, count, replace=False))
        dst.append(np.full(count, node))
        et.append(np.full(count, typ))
    for q, count in enumerate((48, 49, 50, 63, 64, 65, 81)):     # receivers 32 .. 38: six long lists of one type
        senders(32 + q, 0, count)
    for q, count in zip((0, 7, 8, 15), (49, 64, 65, 300)):       # four of one type in the last group
        senders(n - 16 + q, E - 1, count)
    for typ in range(E):                                         # one receiver with long lists of every type
        senders(n // 2 + 5, typ, 60 + 97 * typ)
    senders(n // 2 + 16, 0, 3000)
    src, dst, et = (np.concatenate(x) for x in (src, dst, et))
    X = rng.integers(-2, 3, (n, H)).astype(np.float64)
    W = rng.integers(-1, 2, (E, H, H)).astype(np.float64)
    bias = rng.integers(-2, 3, (E, H)).astype(np.float64) if E % 2 else None
    row_ptr, col, _ = capi.ggnn_sparse_csr(n, E, src, dst, et)
    a = torch.full((n, H), float("nan"), device="cuda")
    capi.ggnn_sparse_step(dt, n, H, E, torch.from_numpy(row_ptr).cuda(), torch.from_numpy(col).cuda(), len(col),
                          dev(X, dt), dev(W.transpose(0, 2, 1), dt), None if bias is None else dev(bias), a)
    s, d, e, _ = O.dedupe_edges(src, dst, et)
    np.testing.assert_array_equal(host(a), O.aggregate(n, s, d, e, O.msg_transform(X, W, bias)))
