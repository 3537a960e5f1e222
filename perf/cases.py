"""Timed cases of the framework: one denoising step of a layer, of an attention block and of a
whole model, through the public Python entry points (``DareLayer.layer_step``,
``DareLayer.block_step``, ``DareModel.step`` / ``DareModel.logits``).

A case is a dict of plain values:

  kind       "layer" (layer_step), "block" (block_step: RMS norm, rotary embedding, residual sum)
             or "model" (DareModel.step and the logits of the current block)
  dtype      "bf16" or "f32"
  batch, seq, hidden, heads          the layer's shape (head_dim = hidden / heads)
  mode       "dense", "kv", "o" or "kvo"
  lo, hi     share of the tokens of a sequence whose hidden state (model: token id) changed since the
             last step, at least one token; each sequence draws its own share in [lo, hi].  These
             are the tokens that are refreshed
  rate_rule  thresholds by reuse rate (quantile) instead of by score
  prefix     frozen tokens at the start of every sequence
  layers, ffn, vocab, skip, block    model only: its size, the number of leading layers that stay dense,
             and the tokens per sequence whose logits are computed

Inputs follow the recipe of ``paper_2605_08134_amd/synth.py``: weights ~ N(0, 0.02^2), hidden states
~ N(0, 1), changed tokens move by 0.5 N(0, 1), the others by 0.01 N(0, 1), so that the drift has
two well separated modes and a threshold between them refreshes exactly the changed tokens.
Consecutive passes alternate between the two hidden states (or id lists): every pass sees the
same refreshed set while the caches really change, as ``bench.py`` does.
"""
import math

import torch

from paper_2605_08134_amd import binding, synth

MODES = {"dense": binding.MODE_DENSE, "kv": binding.MODE_KV, "o": binding.MODE_O, "kvo": binding.MODE_KVO}
EPS, ROPE_BASE = 1e-5, 10000.0
# between the drift of a token whose id changed (0.6 and more) and of the others (up to 0.1 in the
# deeper layers of short sequences) in a network of a few random layers
MODEL_TAU = 0.3


def _case(name, kind, batch, seq, hidden, heads, mode, lo=0.2, hi=None, dtype="bf16", rate_rule=False, prefix=0,
          layers=0, ffn=0, vocab=0, skip=0, block=0):
    c = dict(kind=kind, dtype=dtype, batch=batch, seq=seq, hidden=hidden, heads=heads, mode=mode, lo=lo,
             hi=lo if hi is None else hi, rate_rule=rate_rule, prefix=prefix, layers=layers, ffn=ffn, vocab=vocab,
             skip=skip, block=block)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the small fp32 configuration: the path that results are checked on; launches and host time
        _case("layer_kvo_tiny_f32", "layer", 1, 128, 256, 4, "kvo", dtype="f32"),
        # two short sequences of odd length in a narrow layer: a step bound by its launches
        _case("layer_kvo_small", "layer", 2, 201, 512, 4, "kvo"),
        # one or a few tokens unmasked per step and nearly everything reused: the usual step of
        # decoding one sequence, a stream over the weights
        _case("layer_kvo_few", "layer", 1, 1024, 4096, 32, "kvo", lo=0.004),
        # the headline of bench.py: 80 % reuse of K/V and outputs
        _case("layer_kvo_1024", "layer", 1, 1024, 4096, 32, "kvo"),
        # K/V reuse only, at the low end of the reuse range
        _case("layer_kv_half", "layer", 1, 1024, 4096, 32, "kv", lo=0.5),
        # the dense step: it fills the caches, and it is every refresh-interval step
        _case("layer_dense_1024", "layer", 1, 1024, 4096, 32, "dense"),
        # output reuse in the block of a model, thresholds set by reuse rate, odd lengths
        _case("block_o_ragged", "block", 3, 777, 4096, 32, "o", lo=0.25, rate_rule=True),
        # the batched workload: 8 sequences, each with its own share of refreshed tokens
        _case("layer_kvo_8x2048", "layer", 8, 2048, 4096, 32, "kvo", lo=0.05, hi=0.30),
        # its dense step, as the block of a model calls it
        _case("block_dense_8x2048", "block", 8, 2048, 4096, 32, "dense"),
        # decoding one sequence with a whole model (four of its layers): one token unmasked per step,
        # and the logits of the current block of 32
        _case("model_kvo_1024", "model", 1, 1024, 4096, 32, "kvo", lo=0.0, layers=4, ffn=12288, vocab=126464, block=32),
        # a batch of short sequences: the first layer stays dense, a moderate share is refreshed
        _case("model_kvo_16x256", "model", 16, 256, 4096, 32, "kvo", lo=0.10, hi=0.15, layers=3, ffn=12288,
              vocab=126464, skip=1, block=32),
        # long sequences with a frozen prompt (prefix caching), four tokens unmasked per step
        _case("model_prefix_4x4096", "model", 4, 4096, 4096, 32, "kvo", lo=0.001, layers=2, ffn=12288, vocab=126464,
              prefix=2048, block=32),
    ]


def draw(rng):
    """One more case of the ranges above; it costs no more than the largest listed one."""
    top = max(_cost(c) for c in listed())
    logu = lambda a, b: math.exp(rng.uniform(math.log(a), math.log(b)))
    while True:
        kind = rng.choice(["layer", "layer", "layer", "block", "block", "model"])
        if kind == "layer" and rng.random() < 0.15:
            # fp32, the path for checks: small sizes only
            hidden, dh = rng.choice([256, 512, 1024]), 64
            batch, seq = rng.randint(1, 2), int(logu(32, 257))
            dtype = "f32"
        else:
            hidden = rng.choice([512, 1024, 2048, 3072, 4096, 4096, 4096])
            dh = 64 if hidden <= 1024 and rng.random() < 0.5 else 128
            batch = rng.choice([1, 1, 1, 2, 3, 4, 6, 8, 16])
            seq = int(logu(64, 4100))
            dtype = "bf16"
        mode = rng.choice(["dense", "kv", "o", "kvo", "kvo", "kvo"])
        lo = logu(0.002, 0.6)
        rate_rule = kind != "model" and rng.random() < 0.25
        hi = lo if rate_rule else min(0.6, lo * rng.uniform(1.0, 3.0))
        prefix = rng.randint(1, seq // 2) if kind != "layer" and rng.random() < 0.4 else 0
        kw = {}
        if kind == "model":
            layers = rng.randint(1, 4)
            hi, lo = min(hi, 0.15), min(lo, 0.15)
            kw = dict(layers=layers, ffn=hidden * 3, vocab=rng.choice([32000, 126464]), block=rng.choice([8, 32, 64]),
                      skip=rng.choice([0, 0, 1]))
        c = _case(None, kind, batch, seq, hidden, hidden // dh, mode, lo, hi, dtype, rate_rule, prefix, **kw)
        if _cost(c) <= top and batch * seq <= 16384:
            return c


def _counts(c):
    """Changed (= refreshed) tokens of each sequence: spread evenly over [lo, hi]."""
    b, act = c["batch"], c["seq"] - c["prefix"]
    share = [c["lo"] + (c["hi"] - c["lo"]) * (i + 0.5) / b for i in range(b)]
    return [min(act, max(1, round(s * act))) for s in share]


def _changed(c, gen):
    """Bool [batch, seq] on the CPU: the changed tokens, none of them frozen."""
    m = torch.zeros(c["batch"], c["seq"], dtype=torch.bool)
    for b, n in enumerate(_counts(c)):
        m[b, c["prefix"] + torch.randperm(c["seq"] - c["prefix"], generator=gen)[:n]] = True
    return m


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    gen, cpu = torch.Generator(device=dev), torch.Generator()
    gen.manual_seed(seed)
    cpu.manual_seed(seed)
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    d, b, t = case["hidden"], case["batch"], case["seq"]
    rn = lambda *shape: torch.randn(shape, device=dev, dtype=td, generator=gen)
    weight = lambda *shape: rn(*shape).mul_(synth.WEIGHT_STD)
    gain = lambda: rn(d).mul_(0.1).add_(1.0)
    changed = _changed(case, cpu)
    st = {"case": case, "turn": 0}
    if case["kind"] == "model":
        n, f, v = case["layers"], case["ffn"], case["vocab"]
        m = binding.DareModel(n, d, case["heads"], f, v, b, t, binding.DARE_BF16, EPS, ROPE_BASE)
        for l in range(n):
            m.set_layer(l, gain(), weight(d, d), weight(d, d), weight(d, d), weight(d, d), gain(), weight(d, f),
                        weight(d, f), weight(f, d))
        m.set_io(rn(v, d), gain(), weight(d, v))
        # a prompt and, behind it, mask ids (the last id); the changed tokens differ between the
        # two id lists
        ids = torch.randint(0, v - 1, (b, t), generator=cpu, dtype=torch.int32)
        ids[:, max(case["prefix"], t // 2):] = v - 1
        other = torch.where(changed, torch.randint(0, v - 1, (b, t), generator=cpu, dtype=torch.int32), ids)
        rows = torch.cat([torch.arange(t - min(t, case["block"]), t, dtype=torch.int32) + i * t for i in range(b)])
        mode = MODES[case["mode"]]
        st.update(model=m, inputs=[other.to(dev), ids.to(dev)], rows=rows.to(dev),
                  modes=[binding.dare_policy_mode(mode, l, 1, case["skip"], 0) for l in range(n)],
                  hidden=torch.empty((b, t, d), dtype=td, device=dev),
                  refreshed=torch.zeros((n, b), dtype=torch.int32, device=dev))
        m.step(binding.MODE_DENSE, 0.0, st["inputs"][1])  # fills the caches of every layer
        m.set_prefix(case["prefix"])
        return st
    layer = binding.DareLayer(*(weight(d, d) for _ in range(4)), n_heads=case["heads"], max_batch=b, max_seq=t)
    sigma = torch.where(changed, synth.SIGMA_PERTURBED, synth.SIGMA_STABLE).to(dev)
    prev = torch.randn((b, t, d), device=dev, generator=gen)
    cur = prev + sigma[:, :, None] * torch.randn((b, t, d), device=dev, generator=gen)
    caches = layer.new_state(b, t)
    st.update(layer=layer, caches=caches, inputs=[cur.to(td), prev.to(td)],
              mask=torch.zeros((b, t), dtype=torch.uint8, device=dev),
              # the counts are a reuse mode's: the dense step has no use for them
              count=None if case["mode"] == "dense" else torch.zeros((b,), dtype=torch.int32, device=dev),
              out=caches["o_cache"])
    if case["kind"] == "block":
        layer.block_attach("rms", gain(), None, EPS, ROPE_BASE, True)
        st["out"] = torch.empty((b, t, d), dtype=td, device=dev)
    _layer_call(st, binding.MODE_DENSE, 0.0, st["inputs"][1])  # fills the caches
    st["tau"] = synth.TAU_SEPARATING
    layer.set_prefix(case["prefix"])
    if case["rate_rule"]:
        act = t - case["prefix"]
        layer.set_threshold_rule(binding.RULE_QUANTILE)
        st["tau"] = (act - _counts(case)[0] - 0.5) / act if act > _counts(case)[0] else 0.0
    return st


def _layer_call(st, mode, tau, x):
    call = st["layer"].block_step if st["case"]["kind"] == "block" else st["layer"].layer_step
    k = st["caches"]
    call(mode, tau, x, k["q_prev"], k["k_cache"], k["v_cache"], k["o_cache"], st["out"], st["mask"], None, st["count"],
         None)


def run(state):
    x = state["inputs"][state["turn"] & 1]
    state["turn"] += 1
    if "model" in state:
        m = state["model"]
        m.step(state["modes"], MODEL_TAU, x, state["hidden"], state["refreshed"])
        return {"hidden": state["hidden"], "logits": m.logits(state["hidden"], state["rows"]),
                "refreshed": state["refreshed"]}
    _layer_call(state, MODES[state["case"]["mode"]], state["tau"], x)
    return {"out": state["out"], "mask": state["mask"], "count": state["count"], **state["caches"]}


def _layer_work(c, mode):
    """(flops, bytes) of one layer step: weights, hidden states and caches each touched once."""
    b, t, d = c["batch"], c["seq"], c["hidden"]
    es = 2 if c["dtype"] == "bf16" else 4
    dh = d // c["heads"]
    act, ref = b * (t - c["prefix"]), sum(_counts(c))
    kv = ref if mode in ("kv", "kvo") else act       # rows whose K and V are projected
    o = ref if mode in ("o", "kvo") else act         # rows with queries, attention and output
    flops = 2 * d * (2 * kv * d + 2 * o * d + (act - o) * dh) + 4 * o * t * d
    # weights; hidden states in; K and V rows written, the others read; output rows; score cache
    bytes_ = es * (4 * d * d + act * d + 2 * b * t * d + o * d) + 8 * act * dh + b * t
    return flops, bytes_


def work(case):
    d, es = case["hidden"], 2 if case["dtype"] == "bf16" else 4
    tok = case["batch"] * case["seq"]
    act = case["batch"] * (case["seq"] - case["prefix"])
    if case["kind"] != "model":
        flops, bytes_ = _layer_work(case, case["mode"])
        if case["kind"] == "block":  # the residual sum of every row: the cached output in, the sum out
            bytes_ += 2 * tok * d * es
        return {"flops": flops, "bytes": bytes_}
    f, v = case["ffn"], case["vocab"]
    rows = case["batch"] * min(case["seq"], case["block"])
    flops, bytes_ = 2 * rows * d * v, es * (d * v + rows * v + 2 * tok * d)
    for l in range(case["layers"]):
        a, m = _layer_work(case, "dense" if l < case["skip"] else case["mode"])
        flops += a + 6 * act * d * f
        bytes_ += m + es * 3 * d * f
    return {"flops": flops, "bytes": bytes_}


def _cost(case):
    w = work(case)
    return max(w["flops"] / 2.5e15, w["bytes"] / 8e12)


def tolerance(case):
    """About four times the difference between the results and the same step in float64 with the
    stored tensors rounded to the case's type: fp32 3e-7 at hidden 256 (6e-7 expected at 1024), one
    bf16 layer 3.2e-3 (largest element 0.017), four model layers 9.8e-3 (0.061)."""
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4, "differ": 0.0}
    if case["kind"] == "model":
        return {"rel": 0.03, "max": 0.25, "differ": 0.0}
    return {"rel": 1.2e-2, "max": 0.07, "differ": 0.0}
