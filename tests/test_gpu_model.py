"""GPU parity of the model runtime (dare_model_*) against the model oracle.

The model keeps its caches inside, so the oracle keeps its own and both advance step by
step.  Each layer is checked on the residual stream the GPU itself fed it (the `trace`
output): the oracle runs the layer's attention block and feed-forward on that input and
its own caches, and the results are compared under the rules of parity_util.  Thresholds
sit in the wide gap between the drift of unchanged tokens (0 up to rounding) and of
changed ones, so the decisions are the same on both sides; refreshed counts are compared
exactly."""
import numpy as np
import pytest
import torch

from oracle import dare_oracle as orc
from oracle import dllm_oracle as dl
from paper_2605_08134_amd import synth
import parity_util as pu
from parity_util import dev, host, store

pytestmark = pytest.mark.gpu

EPS, ROPE = 1e-5, 10000.0


def _rng_normal(n):
    return np.random.default_rng(n).standard_normal(n)


def _build(Bm, params, cfg, dtype):
    dt = Bm.DARE_BF16 if dtype == "bf16" else Bm.DARE_F32
    m = Bm.DareModel(cfg["L"], cfg["d"], cfg["H"], cfg["ffn"], cfg["V"], cfg["B"], cfg["T"], dt, EPS, ROPE)
    for l, lp in enumerate(params["layers"]):
        m.set_layer(l, *[dev(lp[k], dtype) for k in ("attn_gain", "wq", "wk", "wv", "wo", "ffn_gain", "w_gate",
                                                      "w_up", "w_down")])
    m.set_io(dev(params["embed"], dtype), dev(params["final_gain"], dtype),
             dev(params["head"], dtype) if "head" in params else None)
    return m


def _zero_caches(cfg):
    z = np.zeros((cfg["B"], cfg["T"], cfg["d"]))
    return [dict(q_prev=np.zeros((cfg["B"], cfg["T"], cfg["d"] // cfg["H"])), k_cache=z, v_cache=z, o_cache=z)
            for _ in range(cfg["L"])]


def _gpu_step(m, cfg, dtype, modes, taus, ids):
    td = pu.tdtype(dtype)
    n = cfg["B"] * cfg["T"] * cfg["d"]
    hidden = torch.full((cfg["B"], cfg["T"], cfg["d"]), float("nan"), dtype=td, device="cuda")
    refreshed = torch.full((cfg["L"], cfg["B"]), -1, dtype=torch.int32, device="cuda")
    trace = torch.full((2 * cfg["L"] + 1, n), float("nan"), dtype=td, device="cuda")
    m.step(modes, taus, dev(ids), hidden, refreshed, trace)
    torch.cuda.synchronize()
    tr = host(trace).reshape(2 * cfg["L"] + 1, cfg["B"], cfg["T"], cfg["d"])
    return host(hidden), host(refreshed), tr


def _check_step(cfg, dtype, params, caches, modes, taus, ids, hidden, refreshed, tr, prefix=0, quantile=False,
                per_layer=None):
    """Layer by layer on the GPU's own residual stream; returns the oracle's new caches.
    per_layer: optional list that receives the oracle's result dict of every layer."""
    storage = "bf16" if dtype == "bf16" else None
    tol = pu.TOL[dtype]
    active = np.ones((cfg["B"], cfg["T"]), dtype=bool)
    active[:, :prefix] = False
    new_caches = []
    for l, lp in enumerate(params["layers"]):
        c = caches[l]
        x_in, x_mid, x_out = tr[2 * l], tr[2 * l + 1], tr[2 * l + 2]
        r = orc.block_step(modes[l], taus[l], x_in, "rms", lp["attn_gain"], None, EPS, lp["wq"], lp["wk"], lp["wv"],
                           lp["wo"], c["q_prev"], c["k_cache"], c["v_cache"], c["o_cache"], cfg["H"], storage=storage,
                           rope_base=ROPE, residual=True, quantile=quantile, prefix=prefix)
        assert np.array_equal(refreshed[l], r["sel_count"]), "layer %d refreshed %s, oracle %s" % (
            l, refreshed[l], r["sel_count"])
        if per_layer is not None:
            per_layer.append(r)
        rms_o = float(np.sqrt(np.mean(r["exact"]["out"] ** 2)))
        want_mid = r["exact"]["block_out"]
        if dtype == "f32":
            assert np.max(np.abs(x_mid - want_mid)) <= 1e-4 * rms_o, "layer %d attention block" % l
        else:
            ex = np.abs(x_mid - want_mid) - pu.half_ulp_bf16(want_mid) - pu.half_ulp_bf16(r["exact"]["out"])
            assert np.max(ex) <= tol * rms_o, "layer %d attention block: %g" % (l, np.max(ex) / rms_o)
        got_ffn, exact_ffn = dl.ffn_block(x_mid, lp["ffn_gain"], EPS, lp["w_gate"], lp["w_up"], lp["w_down"], storage,
                                          rows=active if prefix else None)
        f = exact_ffn - x_mid
        rms_f = float(np.sqrt(np.mean(f[active] ** 2)))
        if dtype == "f32":
            assert np.max(np.abs(x_out - exact_ffn)) <= 1e-4 * rms_f, "layer %d feed-forward" % l
        else:
            ex = np.abs(x_out - exact_ffn) - pu.half_ulp_bf16(exact_ffn) - pu.half_ulp_bf16(f)
            assert np.max(ex) <= tol * rms_f, "layer %d feed-forward: %g" % (l, np.max(ex) / rms_f)
        if prefix:
            assert np.array_equal(x_out[:, :prefix], x_mid[:, :prefix])
        new_caches.append({k: r[k] for k in ("q_prev", "k_cache", "v_cache", "o_cache")})
    y = orc.rms_norm(tr[-1], params["final_gain"], EPS)
    if dtype == "f32":
        assert pu.rel_err(hidden, y) <= 1e-5
    else:
        assert np.all(np.abs(hidden - y) <= pu.half_ulp_bf16(y) + 1e-5 * np.maximum(np.abs(y), 1.0))
    return new_caches


@pytest.fixture(scope="module")
def Bm():
    from paper_2605_08134_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("T,d,prefix,ffn", [
    (2048, 1024, 0, 6144), (1793, 1024, 0, 6144),    # 64 tiles of 256 x 128: not cut, 64 x 128 is faster
    (2048, 2048, 0, 6144), (1900, 2048, 107, 6144),  # 128 tiles; 1793 rows left by the prefix: one in the last row tile
    (2305, 2048, 0, 6144),                           # 160 tiles: more than the workspace holds
    (2305, 1024, 0, 9216),                           # 80 tiles, 144 k-steps; one row in the last row tile
])
def test_down_projection_cut_along_k(Bm, T, d, prefix, ffn):
    """The down projection (96 k-steps and more) with two workgroups on the halves of a tile's k.  Three
    steps in a row on the same ids: the sum does not depend on which workgroup comes first."""
    cfg = dict(L=1, d=d, H=d // 128, ffn=ffn, V=128, B=1, T=T)
    params = synth.make_model_params(T, 1, d, cfg["ffn"], cfg["V"], "bf16", with_head=False)
    m = _build(Bm, params, cfg, "bf16")
    ids = synth.make_ids(T, 1, T, cfg["V"], T // 2, cfg["V"] - 1)
    step = lambda: _gpu_step(m, cfg, "bf16", [orc.MODE_DENSE], [0.0], ids)
    hidden, refreshed, tr = step()
    caches = _check_step(cfg, "bf16", params, _zero_caches(cfg), [orc.MODE_DENSE], [0.0], ids, hidden, refreshed, tr)
    if prefix:
        m.set_prefix(prefix)
        hidden, refreshed, tr = step()
        _check_step(cfg, "bf16", params, caches, [orc.MODE_DENSE], [0.0], ids, hidden, refreshed, tr, prefix=prefix)
    for _ in range(2):
        again, _, trace = step()
        assert np.array_equal(again, hidden) and np.array_equal(trace, tr)
    m.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,T,d,prefix", [(1, 5, 64, 0), (1, 33, 2048, 32), (2, 40, 128, 7), (2, 19, 1088, 1)])
def test_hidden_state_with_and_without_trace(Bm, dtype, L, T, d, prefix):
    """The last sum and the final norm are one pass, which stores the sum only for a trace: the hidden state is that of
    the traced stream, frozen rows (the norm alone) included; a step that asks for neither runs too."""
    cfg = dict(L=L, d=d, H=d // 64, ffn=2 * d, V=64, B=3, T=T)
    params = synth.make_model_params(T, L, d, cfg["ffn"], cfg["V"], dtype, with_head=False)
    m = _build(Bm, params, cfg, dtype)
    ids = synth.make_ids(T, 3, T, cfg["V"], T // 3, cfg["V"] - 1)
    step = lambda: _gpu_step(m, cfg, dtype, [orc.MODE_DENSE] * L, [0.0] * L, ids)
    hidden, refreshed, tr = step()
    caches = _check_step(cfg, dtype, params, _zero_caches(cfg), [orc.MODE_DENSE] * L, [0.0] * L, ids, hidden, refreshed, tr)
    if prefix:
        m.set_prefix(prefix)
        hidden, refreshed, tr = step()
        _check_step(cfg, dtype, params, caches, [orc.MODE_DENSE] * L, [0.0] * L, ids, hidden, refreshed, tr, prefix=prefix)
    plain = torch.full((3, T, d), float("nan"), dtype=pu.tdtype(dtype), device="cuda")
    m.step([orc.MODE_DENSE] * L, [0.0] * L, dev(ids), plain)
    m.step([orc.MODE_DENSE] * L, [0.0] * L, dev(ids))
    again = step()[0]
    assert np.array_equal(host(plain), hidden) and np.array_equal(again, hidden)
    m.destroy()


# 40 rows: small tiles; 8192 x 4096: two rounds of 256 x 256
@pytest.mark.parametrize("B,T,ffn", [(1, 40, 256), (4, 2048, 2048)])
def test_gate_over_its_whole_range(Bm, B, T, ffn):
    """silu(g) * u for single gates g = v, -v and u = 1, -1 (one weight and one input each, so both are exact), from gates whose
    divisor 1 + exp(-g) is near the largest float to infinite ones."""
    d, n_gates = 256, 250
    cfg = dict(L=1, d=d, H=2, ffn=ffn, V=64, B=B, T=T)
    v = np.concatenate([np.arange(-88.5, -80.0, 0.5), [-64.5, -64.0, -63.5, 0.0, 1e-30, 1e-36, 1e30, 127.0],
                        20 * _rng_normal(n_gates)])[:n_gates]
    v = store(v.astype(np.float32), "bf16").astype(np.float64)
    at = np.arange(n_gates) * (ffn // 256) + np.arange(n_gates) % (ffn // 256)     # a gate's column
    z = np.zeros
    lp = dict(attn_gain=np.ones(d), ffn_gain=np.ones(d), wq=z((d, d)), wk=z((d, d)), wv=z((d, d)), wo=z((d, d)),
              w_gate=z((d, ffn)), w_up=z((d, ffn)), w_down=z((ffn, d)))
    lp["w_gate"][0, at], lp["w_up"][0, at], lp["w_down"][at, 2 + np.arange(n_gates)] = v / 16, 1 / 16, 1.0
    lp["w_gate"][1, at[5]], lp["w_up"][1, at[5]] = 3e38, 1 / 16
    embed = z((64, d))
    embed[:4, :2] = [[16, 0], [-16, 0], [0, 16], [0, -16]]      # normalised: the same, rounded to bf16
    m = _build(Bm, dict(layers=[lp], embed=embed, final_gain=np.ones(d)), cfg, "bf16")
    ids = np.arange(B * T, dtype=np.int32).reshape(B, T) % 4
    x = _gpu_step(m, cfg, "bf16", [orc.MODE_DENSE], [0.0], ids)[2][2]
    m.destroy()
    for sign, got in ((1, x[ids == 0]), (-1, x[ids == 1])):
        g = sign * v
        want = np.where(g < -88.7, 0.0, g / (1 + np.exp(-np.maximum(g, -88.7)))) * sign       # (exp(-g) past the largest float: 0)
        # a rounding to bf16 (2^-9) and exp of 32 bits (|g| 2^-24 and its own last bit)
        assert np.all(np.abs(got[:, 2:2 + n_gates] - want) <= 2.0 ** -8 * np.abs(want) + 1e-38)
    up, down = x[ids == 2], x[ids == 3]      # gates of +inf and -inf: inf and -inf / inf; 0 times them in the other columns
    assert np.all(up[:, 7] == np.inf) and np.all(np.isnan(np.delete(up, 7, axis=1))) and np.all(np.isnan(down))


# sequences, tokens, hidden, feed-forward: silu(gate) * up of more than 128 MB, stored past the L2, with 8 rows in the last row tile and half a
# column tile
GATE_PAST_THE_L2 = (4, 2050, 256, 8384), "256 x 256 four waves"


def test_gate_past_the_l2_has_the_bits_of_a_smaller_launch(Bm):
    """A sequence's rows of the last residual stream in a batch and alone; without attention, whose sums depend on the batch."""
    (B, T, d, ffn), _ = GATE_PAST_THE_L2
    assert B * T * ffn * 2 > 128 << 20 > T * ffn * 2
    cfg = dict(L=1, d=d, H=2, ffn=ffn, V=192, B=B, T=T)
    params = synth.make_model_params(17, 1, d, ffn, 192, "bf16", with_head=False)
    params["layers"][0]["wo"] = np.zeros((d, d))
    ids = np.random.default_rng(3).integers(0, 192, (B, T)).astype(np.int32)
    m = _build(Bm, params, cfg, "bf16")
    whole = _gpu_step(m, cfg, "bf16", [orc.MODE_DENSE], [0.0], ids)[2]
    for b in range(B):
        alone = _gpu_step(m, dict(cfg, B=1), "bf16", [orc.MODE_DENSE], [0.0], ids[b:b + 1])[2]
        assert np.all(np.isfinite(alone)) and np.any(alone[2] != alone[1])
        assert np.array_equal(whole[1][b], alone[1][0])
        assert np.array_equal(whole[2][b], alone[2][0])
    m.destroy()


def test_layers_share_the_workspace_of_attention_with_cut_keys(Bm):
    """The workspace that steps of 1921 tokens and more use (8.7 MB) is the model's: a layer takes
    no more memory at 2048 than at 1920 tokens than its own rows do (1/16 of about 14 MB)."""
    def per_layer(T):
        free = []
        for L in (1, 9):
            cfg = dict(L=L, d=128, H=1, ffn=128, V=128, B=1, T=T)
            params = synth.make_model_params(1, L, 128, 128, 128, "bf16", with_head=False)
            m = _build(Bm, params, cfg, "bf16")
            torch.cuda.synchronize()
            free.append(torch.cuda.mem_get_info()[0])
            m.destroy()
        return (free[0] - free[1]) / 8

    per_layer(1920)                              # (once, for what the allocator keeps)
    assert per_layer(2048) - per_layer(1920) < 4 * 2 ** 20


@pytest.mark.parametrize("T,prefix", [(2048, 0), (4100, 1000)])
def test_few_rows_of_long_sequences_in_two_layers(Bm, T, prefix):
    """Both layers cut the keys of their few refreshed rows over workgroups, in one workspace."""
    cfg = dict(L=2, d=256, H=2, ffn=256, V=256, B=1, T=T)
    params = synth.make_model_params(T, 2, 256, 256, 256, "bf16", with_head=False)
    m = _build(Bm, params, cfg, "bf16")
    ids = synth.make_ids(T, 1, T, 256, T // 2, 255)
    modes, taus = [orc.MODE_DENSE] * 2, [0.0] * 2
    caches = _check_step(cfg, "bf16", params, _zero_caches(cfg), modes, taus, ids, *_gpu_step(m, cfg, "bf16", modes, taus, ids))
    m.set_prefix(prefix)
    for t in range(3):
        ids[0, T - 2 - t] = 7 + t
        modes, taus = [orc.MODE_KVO] * 2, [1e-3] * 2
        caches = _check_step(cfg, "bf16", params, caches, modes, taus, ids, *_gpu_step(m, cfg, "bf16", modes, taus, ids),
                             prefix=prefix)
    m.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_small_model_blockwise_steps(Bm, dtype):
    cfg = dict(L=3, d=256, H=4, ffn=512, V=320, B=2, T=48)
    params = synth.make_model_params(5, cfg["L"], cfg["d"], cfg["ffn"], cfg["V"], dtype)
    m = _build(Bm, params, cfg, dtype)
    mask_id = cfg["V"] - 1
    ids = synth.make_ids(5, cfg["B"], cfg["T"], cfg["V"], 16, mask_id)
    rng = np.random.Generator(np.random.PCG64(17))
    steps = dl.blockwise_schedule(16, 32, 16, 1, rng)
    caches = _zero_caches(cfg)
    L = cfg["L"]
    plan = [([orc.MODE_DENSE] * L, [0.0] * L)]
    for mode in (orc.MODE_KVO, orc.MODE_KV, orc.MODE_O, [orc.MODE_DENSE, orc.MODE_KVO, orc.MODE_O]):
        plan.append(([mode] * L if isinstance(mode, int) else mode, [1e-3] * L))
    for t, (modes, taus) in enumerate(plan):
        if t > 0:
            for b in range(cfg["B"]):
                ids[b, steps[t - 1]] = rng.integers(0, mask_id)
        hidden, refreshed, tr = _gpu_step(m, cfg, dtype, modes, taus, ids)
        assert np.array_equal(tr[0], dl.embed(ids, params["embed"]).astype(np.float32))
        caches = _check_step(cfg, dtype, params, caches, modes, taus, ids, hidden, refreshed, tr)
        if t > 0 and modes[0] != orc.MODE_DENSE:
            assert (refreshed[0] == 1).all()          # layer 0: only the token whose id changed
    # the same ids again: nothing drifts, everything is reused, the output does not move
    h2, r2, _ = _gpu_step(m, cfg, dtype, [orc.MODE_KVO] * L, [0.0] * L, ids)
    assert (r2 == 0).all() and np.array_equal(h2, hidden)
    # logits of a few rows
    rows = np.array([0, 17, 95], dtype=np.int32)
    lg = host(m.logits(dev(hidden, dtype), dev(rows)))
    want = dl.logits(hidden.reshape(-1, cfg["d"])[rows], params["head"])
    pu.assert_close(lg, want, dtype)
    m.destroy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_small_model_prefix_and_quantile_rule(Bm, dtype):
    cfg = dict(L=2, d=128, H=2, ffn=256, V=192, B=2, T=40)
    params = synth.make_model_params(6, cfg["L"], cfg["d"], cfg["ffn"], cfg["V"], dtype, with_head=False)
    m = _build(Bm, params, cfg, dtype)
    ids = synth.make_ids(6, cfg["B"], cfg["T"], cfg["V"], 12, cfg["V"] - 1)
    L = cfg["L"]
    caches = _zero_caches(cfg)
    hidden, refreshed, tr = _gpu_step(m, cfg, dtype, [orc.MODE_DENSE] * L, [0.0] * L, ids)
    caches = _check_step(cfg, dtype, params, caches, [orc.MODE_DENSE] * L, [0.0] * L, ids, hidden, refreshed, tr)
    m.set_prefix(12)                                   # the prompt is frozen from here on
    ids[:, 20] = 3
    ids[:, 31] = 5
    modes, taus = [orc.MODE_KVO, orc.MODE_KV], [1e-3, 1e-3]
    hidden, refreshed, tr = _gpu_step(m, cfg, dtype, modes, taus, ids)
    caches = _check_step(cfg, dtype, params, caches, modes, taus, ids, hidden, refreshed, tr, prefix=12)
    assert (refreshed[0] == 2).all()
    # Quantile rule (Sec. 3.1 "Reuse rate allocation") against the oracle: per layer and sequence
    # the threshold is the k-th smallest drift score of the 28 tokens that are not frozen.  Layer 0
    # in KV mode recomputes every attention row, so in layer 1 every token has drifted a little and
    # the k-th smallest score is a real order statistic, not the zero of unchanged tokens.  The
    # rates are chosen layer by layer from the oracle's own run so that the k-th and the (k+1)-th
    # smallest score of both sequences are further apart than the two sides' scores can differ.
    m.set_rule(Bm.RULE_QUANTILE)
    ids[:, 25] = 7
    storage = "bf16" if dtype == "bf16" else None
    band = 3e-5 if dtype == "bf16" else 1e-6      # a rounding flip in the normalised bf16 state moves a score by up to 3e-5
    n_act = cfg["T"] - 12
    modes, phis = [orc.MODE_KV, orc.MODE_KVO], [0.5] * L
    for l in range(L):
        plan = dl.model_step(modes, phis, ids, params, caches, cfg["H"], EPS, ROPE, storage=storage, quantile=True,
                             prefix=12)
        srt = np.sort(plan["layers"][l]["scores"][:, 12:], axis=1)
        ok = [k for k in range(1, n_act) if np.all(srt[:, k] - srt[:, k - 1] > 10 * band) or
              (np.all(srt[:, k - 1] == 0.0) and np.all((srt[:, k] == 0.0) | (srt[:, k] > 10 * band)))]
        assert ok, "no rank with a clear gap in layer %d" % l
        k = min(ok, key=lambda k: abs(k - n_act // 2))
        phis[l] = (k - 0.5) / n_act                   # ceil(phi * n_act) = k
    hidden, refreshed, tr = _gpu_step(m, cfg, dtype, modes, phis, ids)
    res = []
    _check_step(cfg, dtype, params, caches, modes, phis, ids, hidden, refreshed, tr, prefix=12, quantile=True,
                per_layer=res)
    for l in range(L):
        tau_gpu = host(m.layer(l).thresholds(cfg["B"]))
        assert np.all(np.abs(tau_gpu - res[l]["tau"]) <= band), (l, tau_gpu, res[l]["tau"])
        assert np.array_equal(refreshed[l], (res[l]["reuse_mask"] == 0).sum(axis=1))
    assert (refreshed[0] >= 1).all() and (refreshed <= n_act).all()
    print("quantile rule, %s: rates %s, refreshed per layer and sequence %s" % (dtype, phis, refreshed.tolist()))
    with pytest.raises(Bm.DareError):
        m.step([orc.MODE_KVO] * L, [1.5] * L, dev(ids))
    m.destroy()


def test_model_argument_errors(Bm):
    with pytest.raises(Bm.DareError):
        Bm.DareModel(1, 100, 2, 128, 64, 1, 8, Bm.DARE_F32)          # hidden not a multiple of 64
    m = Bm.DareModel(2, 128, 2, 128, 64, 1, 8, Bm.DARE_F32)
    ids = torch.zeros((1, 8), dtype=torch.int32, device="cuda")
    with pytest.raises(Bm.DareError):
        m.step(0, 0.0, ids)                                           # no weights yet
    with pytest.raises(IndexError):
        m.layer(0)
    m.destroy()


def test_out_of_range_ids_embed_as_zero(Bm):
    cfg = dict(L=1, d=128, H=2, ffn=128, V=64, B=1, T=8)
    params = synth.make_model_params(7, 1, 128, 128, 64, "f32", with_head=False)
    m = _build(Bm, params, cfg, "f32")
    ids = np.array([[0, 63, 64, -1, 5, 1000, 2, 3]], dtype=np.int32)
    _, _, tr = _gpu_step(m, cfg, "f32", [0], [0.0], ids)
    want = np.where(((ids >= 0) & (ids < 64))[:, :, None], params["embed"][np.clip(ids, 0, 63)], 0.0)
    assert np.array_equal(tr[0], want.astype(np.float32))
    m.destroy()


def test_two_layers_at_llada_width(Bm):
    """Full layer width (hidden 4096, 32 x 128, feed-forward 12288), bf16, 2 layers, 256 tokens."""
    dtype = "bf16"
    cfg = dict(L=2, d=4096, H=32, ffn=12288, V=512, B=1, T=256)
    params = synth.make_model_params(8, cfg["L"], cfg["d"], cfg["ffn"], cfg["V"], dtype, with_head=False)
    m = _build(Bm, params, cfg, dtype)
    ids = synth.make_ids(8, 1, 256, 512, 128, 511)
    caches = _zero_caches(cfg)
    hidden, refreshed, tr = _gpu_step(m, cfg, dtype, [0, 0], [0.0, 0.0], ids)
    caches = _check_step(cfg, dtype, params, caches, [0, 0], [0.0, 0.0], ids, hidden, refreshed, tr)
    ids[0, [130, 141, 150, 200]] = [1, 2, 3, 4]
    modes, taus = [orc.MODE_KVO, orc.MODE_KVO], [1e-3, 1e-3]
    hidden, refreshed, tr = _gpu_step(m, cfg, dtype, modes, taus, ids)
    _check_step(cfg, dtype, params, caches, modes, taus, ids, hidden, refreshed, tr)
    assert refreshed[0].tolist() == [4]
    m.destroy()
