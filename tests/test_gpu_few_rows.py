"""The kernels that few-row and mid-row passes are made of, at the sizes where their tiles,
fragments and dispatch rules have edges, through the public entry points.

Velocities (not actions, which a step moves by v / H only) against the float64 oracle.
Bars as elsewhere (TOL_F32, TOL_BF16): at most two layers of about ten bf16-rounded tensors
each, 2^-9 apiece and independent, give sqrt(20) 2^-9 = 0.9 % in the 2-norm, and the largest
element over the largest value is about twice that.
"""

import numpy as np
import pytest

import synth
from tests.harness import TOL_BF16, TOL_F32, GpuRoll, have_gpu, rel_err, velocity_parity
from tests.test_gpu_full import _transformer_case

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

W = synth.workloads

BASE = dict(layers=2, width=256, n_q_heads=4, n_kv_heads=2, head_dim=64, mlp_dim=512, horizon=20, action_dim=7,
            prefix_len=40, n_fop=4, fop_obs_dim=16, dtype=W.BF16)


def _shape(**kw):
    return synth.RavelShape(name="few_rows", **{**BASE, **kw})


def _step_velocities(s, batch):
    # three steps: launched directly, recorded, replayed
    wts = synth.draw_weights(s, seed=4, stress=True)
    velocity_parity(s, wts, batch, list(range(batch)), [0, 1, 2], tol=TOL_F32 if s.dtype == W.F32 else TOL_BF16,
                    init_tobs=-2, persistent=None if s.dtype == W.F32 else False, sens_report=())


@pytest.mark.parametrize("kw,batch", [
    (dict(n_fop=1), 1),                                            # one token
    (dict(n_fop=16, horizon=16), 4),                               # a whole fragment, as many slots as tokens, most envs
    (dict(n_fop=17), 2),                                           # two fragments, 68 of 96 columns
    (dict(n_fop=32, horizon=33), 1),                               # 128 columns
    (dict(n_fop=33, horizon=40), 1),                               # 132 columns: separate projections
    (dict(n_fop=16, horizon=15), 1),                               # fewer slots than tokens: separate projections
    (dict(n_fop=5), 5),                                            # five envs: separate projections
    (dict(width=128, n_q_heads=2, n_kv_heads=1, head_dim=32), 3),  # smallest width and head
    (dict(width=1024, n_q_heads=8, n_kv_heads=1, head_dim=256, n_fop=16, horizon=17), 1),  # largest
    (dict(width=192), 1),                                          # not a multiple of 128
])
def test_adapter_fold_edges(kw, batch):
    _step_velocities(_shape(**kw), batch)


@pytest.mark.parametrize("batch", [1, 4, 5])  # folded, folded, separate projections
def test_adapter_of_tokens_whose_values_cancel(batch):
    """Two tokens of equal keys and values A + d, -A + d (d = A / 128, all exact in bf16): the
    attention row is d, while each token's own contribution is 128 times larger.  Rounding
    those contributions to bf16 (2^-9) would leave errors of 2^-9 128 / sqrt(2 . 3) = 10 % of
    the adapter's output; with their remainders kept the bar is that of every bf16 case."""
    from oracle.expert import Expert
    from oracle.training import expert_velocity, training_loss
    from tests.test_gpu_train import gpu_train
    s = _shape(n_fop=2)
    wts = synth.draw_weights(s, seed=4, stress=True)
    rng = np.random.default_rng(1)
    qd, kvd, w = 256, 128, s.width
    kv = np.zeros((2 * kvd, w), np.float32)
    kv[kvd:, 0], kv[kvd:, 1] = rng.choice([-1.0, 1.0], kvd), rng.choice([-1.0, 1.0], kvd)
    wts["layers.1.fop.kv.w"] = kv
    wts["layers.1.fop.o.w"] = W.bf16_round((64 * rng.standard_normal((w, qd))).astype(np.float32))
    wts["layers.1.fop.alpha"] = np.full(1, 5.0, np.float32)
    z = np.zeros((batch, 2, w), np.float32)
    z[:, 0, 0], z[:, 1, 0], z[:, :, 1] = 1.0, -1.0, 2.0**-7
    g = GpuRoll(s, wts, batch, 0)
    g.buf.set_option(g.rv.OPT_PERSISTENT, 0) if batch * s.horizon <= 64 else None
    ctx = [synth.draw_context(s, 0, e, 0) for e in range(batch)]
    for e in range(batch):
        g.set_context(e, *ctx[e], 0)
    target, noise = (rng.standard_normal((batch, s.horizon, s.action_dim)).astype(np.float32) for _ in range(2))
    ages = list(range(batch))
    _, v = gpu_train(g, target, noise, ages, z)
    ex = Expert(s, wts, np.float64)
    for e in range(batch):
        _, ref = training_loss(expert_velocity(ex, *ctx[e], ages[e], z[e]), target[e].astype(np.float64),
                               noise[e].astype(np.float64))
        err = rel_err(v[e], ref)
        print(f"env {e} of {batch}: velocity error {err:.3e}")
        assert err <= TOL_BF16


def test_a_model_without_folding_buffers_holds_its_weights_once():
    """The transposed query projections come with the first buffer that folds its adapters
    and are shared by the next."""
    import torch

    from paper_2609_34170_amd import ravel
    s = _shape(layers=8, width=1024, n_q_heads=16, n_kv_heads=1, head_dim=256, mlp_dim=64, prefix_len=0, n_fop=4)
    wts = synth.draw_weights(s, seed=4)
    copy = len(s.adapter_layers()) * 16 * 256 * 1024 * 2  # 34 MB; free memory is counted in pages of 2 MB

    def used(make):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        made = make()
        return made, before - torch.cuda.mem_get_info()[0]

    first = ravel.Model(s, wts)  # (loads the library's kernels)
    first.close()
    model, _ = used(lambda: ravel.Model(s, wts))
    sizes = [used(lambda: ravel.Buffer(model, b, 0)) for b in (5, 1, 1)]
    assert sizes[1][1] - sizes[2][1] > copy // 2, [n for _, n in sizes]


@pytest.mark.parametrize("kw,batch", [
    (dict(action_dim=1, horizon=1), 1),
    (dict(action_dim=16, horizon=16), 1),
    (dict(action_dim=17, horizon=17), 2),
    (dict(action_dim=33, horizon=48), 1),
    (dict(action_dim=64, horizon=128), 1),
    (dict(action_dim=65, horizon=20), 1),    # separate head and update
    (dict(width=2048, n_q_heads=8, n_kv_heads=2, head_dim=128, mlp_dim=256, layers=1, n_fop=0), 1),  # two K batches
])
def test_output_head_and_update_edges(kw, batch):
    _step_velocities(_shape(**{"n_fop": 0, **kw}), batch)


@pytest.mark.parametrize("kw,batch", [
    (dict(horizon=1), 1),
    (dict(horizon=32), 1), (dict(horizon=33), 1),      # 32-row tiles end
    (dict(horizon=64), 1), (dict(horizon=65), 1),      # the few-row kernels end
    (dict(horizon=43), 3), (dict(horizon=52), 5),      # 129 rows (K ranges 8 -> 4), 260 rows (4 -> 2)
    (dict(mlp_dim=80), 2), (dict(mlp_dim=1360), 1),    # hidden rows padded to whole K tiles
    (dict(mlp_dim=2112), 1), (dict(mlp_dim=6928), 1),  # 33 and 109 K tiles: the last range is shorter
    (dict(width=1040, n_q_heads=4, head_dim=64), 1),   # a last column tile that is nearly empty
])
def test_tiled_gemm_edges(kw, batch):
    _step_velocities(_shape(**kw), batch)


@pytest.mark.parametrize("horizon,batch", [(35, 2), (43, 3), (20, 1)])  # 70 and 129 rows; the few-row kernels
def test_widths_without_the_fused_residual_kernel(horizon, batch):
    _step_velocities(_shape(layers=1, width=4160, mlp_dim=128, n_fop=0, horizon=horizon), batch)


@pytest.mark.parametrize("horizon,mlp", [(16, 1536), (16, 1552), (17, 1536)])  # the last of the few-row kernels
def test_few_rows_of_a_long_k(horizon, mlp):
    _step_velocities(_shape(layers=2, width=2048, mlp_dim=mlp, horizon=horizon, fop_stride=2), 1)


@pytest.mark.parametrize("layers,horizon,batch,period", [
    (8, 25, 6, 3),   # modulation of 25600 columns: tiles of 64 columns
    (9, 25, 6, 3),   # of 28672: the first of tiles of 128 columns; 50 to 75 live rows of 150
    (9, 64, 5, 5),   # 128 to 320 live rows: whole row tiles and remainders
])
def test_modulation_of_distinct_conditionings(layers, horizon, batch, period):
    s = _shape(layers=layers, width=512, horizon=horizon, mlp_dim=128, n_fop=0, n_kv_heads=4)
    wts = synth.draw_weights(s, seed=4, stress=True)
    # the file's bar is for two layers; the errors of more add up as their square root
    velocity_parity(s, wts, batch, [0, batch - 1], [0, 2, 4], tol=TOL_BF16 * (layers / 2) ** 0.5, period=period,
                    stagger=True, sens_report=())


@pytest.mark.parametrize("hd,prefix,horizon,batch", [
    (64, 0, 9, 1), (64, 447, 20, 1), (64, 448, 20, 1),     # below and at eight key tiles
    (128, 1000, 64, 1), (256, 255, 16, 2), (256, 530, 50, 1), (32, 2000, 3, 1),
    (32, 70, 100, 40), (64, 200, 100, 40),                 # chunks of 128 rows, the last of 72
])
def test_attention_key_ranges(hd, prefix, horizon, batch):
    _step_velocities(_shape(head_dim=hd, prefix_len=prefix, horizon=horizon, layers=1, n_fop=0), batch)


@pytest.mark.parametrize("kw,batch,dead", [
    (dict(prefix_len=200), 1, (0, 64)),                 # the first key tile
    (dict(prefix_len=1000), 1, (448, 640)),             # whole tiles at the start of a key range
    (dict(prefix_len=200, head_dim=256, n_kv_heads=1), 6, (0, 32)),
    (dict(prefix_len=130, horizon=100, n_kv_heads=1), 40, (0, 64)),   # 128-row chunks
    (dict(prefix_len=90, dtype=W.F32, width=128), 1, (16, 32)),  # a wave's first keys
])
def test_keys_whose_scores_overflow(kw, batch, dead):
    """Queries of positive entries and a run of prefix keys near the largest negative bf16: their
    scores are -infinity in 32 bits, their weights 0 (exp of -1e40 in the oracle), and the
    other keys' softmax is what it is without them."""
    from oracle.expert import Expert
    from oracle.training import expert_velocity, training_loss
    from tests.test_gpu_train import gpu_train
    s = _shape(layers=1, n_fop=0, **kw)
    wts = synth.draw_weights(s, seed=4, stress=True)
    w = s.width
    wts["layers.0.mod.w"][:2 * w] = 0.0  # attention norm: scale -1, shift 1
    wts["layers.0.mod.b"][:2 * w] = np.repeat(np.float32([-1.0, 1.0]), w)
    qd = s.n_q_heads * s.head_dim
    wts["layers.0.qkv.w"][:qd] = np.abs(wts["layers.0.qkv.w"][:qd])
    g = GpuRoll(s, wts, batch, 0)
    if s.dtype == W.BF16 and batch * s.horizon <= 64:
        g.buf.set_option(g.rv.OPT_PERSISTENT, 0)
    ctx = []
    for e in range(batch):
        k, v = synth.draw_context(s, 0, e, 0)
        k[:, dead[0]:dead[1]] = -3e38
        ctx.append((k, v))
        g.set_context(e, k, v, 0)
    rng = np.random.default_rng(1)
    target, noise = (rng.standard_normal((batch, s.horizon, s.action_dim)).astype(np.float32) for _ in range(2))
    _, got = gpu_train(g, target, noise, [1] * batch)
    ex = Expert(s, wts, np.float64)
    for e in {0, batch - 1}:
        _, ref = training_loss(expert_velocity(ex, *ctx[e], 1, None), target[e].astype(np.float64),
                               noise[e].astype(np.float64))
        assert rel_err(got[e], ref) <= (TOL_F32 if s.dtype == W.F32 else TOL_BF16), e


@pytest.mark.parametrize("kw,batch", [
    (dict(horizon=1, action_dim=1, prefix_len=0), 1),
    (dict(horizon=17, mlp_dim=80, n_fop=3), 1),
    (dict(horizon=65, n_q_heads=2, n_kv_heads=1, head_dim=128, n_fop=1), 1),
    (dict(horizon=16, prefix_len=300, head_dim=32, n_kv_heads=4), 5),
])
def test_32_bit_models(kw, batch):
    _step_velocities(_shape(dtype=W.F32, width=128, **kw), batch)


@pytest.mark.parametrize("dtype,horizon,batch,S,width", [
    (W.BF16, 3, 1, 8, 256),      # more Euler steps than buffer rows: the modulation comes in parts
    (W.BF16, 20, 4, 5, 256), (W.BF16, 13, 6, 3, 256),
    (W.BF16, 70, 1, 72, 256),    # 70 rows at a time (tiles), then 2
    (W.BF16, 20, 4, 5, 192), (W.BF16, 20, 4, 5, 1152),  # widths whose modulation always takes tiles
    (W.BF16, 3, 1, 8, 1152), (W.BF16, 70, 1, 72, 192),
    (W.F32, 2, 1, 5, 256), (W.F32, 20, 4, 3, 256),
])
@pytest.mark.parametrize("offset", [W.OFFSET_MLP, W.OFFSET_CONCAT, W.OFFSET_ADAPTER])
def test_chunk_modulation_rows(dtype, horizon, batch, S, width, offset):
    kw = {**BASE, "dtype": dtype, "horizon": horizon, "offset_mode": offset, "width": width}
    _transformer_case("small_bf16", batch, S, np.float64, persistent=None if dtype == W.F32 else False, **kw)


def test_velocities_into_memory_of_any_alignment():
    import torch
    s = _shape(n_fop=0, action_dim=5)
    g = GpuRoll(s, synth.draw_weights(s, seed=4, stress=True), 2, 0)
    for e in range(2):
        g.set_context(e, *synth.draw_context(s, 0, e, 0), 0)
    gen = torch.Generator().manual_seed(0)
    y, n = (torch.randn((2, s.horizon, 5), generator=gen).to(g.dev) for _ in range(2))
    ages = torch.tensor([1, 3], dtype=torch.int64, device=g.dev)
    out = []
    for off in (0, 1):
        loss, v = torch.empty(2, device=g.dev), torch.empty(2 * s.horizon * 5 + 1, device=g.dev)
        v = v[off:off + 2 * s.horizon * 5].view(2, s.horizon, 5)
        g.buf.train_loss(y, n, ages, None, loss, v)
        torch.cuda.synchronize()
        out.append((loss.cpu().numpy(), v.cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("shape_kw", [dict(n_fop=0), dict(n_fop=0, dtype=W.F32, width=128)])
@pytest.mark.parametrize("where", ["target", "noise", "between"])
def test_velocities_in_place_of_an_input(shape_kw, where):
    """v_out over target, over noise, and over the end of one and the start of the other:
    the loss and the velocities are those of a call with memory of its own."""
    import torch
    s = _shape(**shape_kw)
    g = GpuRoll(s, synth.draw_weights(s, seed=4, stress=True), 2, 0)
    g.buf.set_option(g.rv.OPT_PERSISTENT, 0)
    for e in range(2):
        g.set_context(e, *synth.draw_context(s, 0, e, 0), 0)
    gen = torch.Generator().manual_seed(0)
    n, shp = 2 * s.horizon * s.action_dim, (2, s.horizon, s.action_dim)
    data = torch.randn(2 * n, generator=gen).to(g.dev)  # target, then noise
    ages = torch.tensor([1, 3], dtype=torch.int64, device=g.dev)
    out = []
    for own in (True, False):
        mem = data.clone()
        at = {"target": 0, "noise": n, "between": n // 2 // 4 * 4}[where]
        v = torch.empty(shp, device=g.dev) if own else mem[at:at + n].view(shp)
        loss = torch.empty(2, device=g.dev)
        g.buf.train_loss(mem[:n].view(shp), mem[n:].view(shp), ages, None, loss, v)
        torch.cuda.synchronize()
        out.append((loss.cpu().numpy(), v.cpu().numpy()))
    assert np.array_equal(out[0][1], out[1][1])
    assert np.array_equal(out[0][0], out[1][0])


@pytest.mark.parametrize("sets,rounds,graphs", [(1, 12, 1), (2, 6, 2), (12, 1, 0), (9, 2, 9), (12, 3, 12)])
def test_a_pointer_set_is_recorded_on_its_second_step(sets, rounds, graphs):
    import torch

    from paper_2609_34170_amd import ravel
    s = _shape()
    wts = synth.draw_weights(s, seed=4, stress=True)
    a, b = GpuRoll(s, wts, 1, 3), GpuRoll(s, wts, 1, 3, use_graph=False)
    for g in (a, b):
        g.buf.set_option(ravel.OPT_PERSISTENT, 0)
        g.set_context(0, *synth.draw_context(s, 0, 0, 0), 0)
    outs = [torch.empty((1, s.action_dim), device=a.dev) for _ in range(sets)]
    for st in range(sets * rounds):
        z = synth.draw_fop_tokens(s, 0, st, batch=1)
        a.fop.copy_(a.to_dev(z))
        a.buf.step(a.fop, outs[st % sets])
        torch.cuda.synchronize()
        assert np.array_equal(outs[st % sets].cpu().numpy(), b.step(z)), st
    assert a.buf.query(ravel.Q_GRAPHS) == graphs


@pytest.mark.parametrize("obs,batch,offset", [
    (8, 1, 0), (136, 3, 0), (128, 16, 0), (512, 17, 0), (520, 2, 0),
    (64, 64, 0), (64, 65, 0),      # the last in one launch, the first of the tiled product
    (64, 2, 1),                    # observations off a 16-byte boundary: converted first
])
def test_encoder_edges(obs, batch, offset):
    import torch
    s = _shape(fop_obs_dim=obs)
    wts = synth.draw_weights(s, seed=4, stress=True)
    g = GpuRoll(s, wts, batch, 0)
    x = np.random.default_rng(obs).standard_normal((batch, obs)).astype(np.float32)
    mem = torch.empty(batch * obs + 1, device=g.dev)[offset:offset + batch * obs].view(batch, obs)
    mem.copy_(torch.from_numpy(x))
    out = torch.empty((batch, s.n_fop, s.width), dtype=torch.bfloat16, device=g.dev)
    g.buf.fop_encode(mem, out)
    torch.cuda.synchronize()
    w = {k: np.asarray(v, np.float64) for k, v in wts.items() if k.startswith("fop.")}
    xb = torch.from_numpy(x).bfloat16().double().numpy()
    h = xb @ w["fop.w1"].T + w["fop.b1"]
    h = 0.5 * h * (1 + np.tanh(np.sqrt(2 / np.pi) * (h + 0.044715 * h**3)))
    ref = (h @ w["fop.w2"].T + w["fop.b2"]).reshape(out.shape)
    # two rounded tensors: the hidden rows (2^-9 each, independent) and the tokens
    assert rel_err(out.float().cpu().numpy(), ref) < 2.0**-7
