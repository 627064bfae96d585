"""Performance cases of the library: what a user has it do, through its public entry points.

Four kinds of work, at the shapes of the workloads in ``workloads/``:

* ``decode``: one decode step (one new token per sequence over a paged KV cache), with the output layer and the argmax
  where the workload carries a vocabulary;
* ``unit``: one finetune unit, a layer's LoRA forward and backward over one micro-batch;
* ``train``: one training step of a stack of layers: forward, output layer with cross entropy, backward, AdamW on every
  adapter;
* ``colocated``: a finetune unit beside decode steps, each task on its own stream and both in one pool.

``listed()`` are the cases looked at one by one, ``draw()`` gives more of the same ranges.  Weights, caches and inputs are
random with the distributions of ``workloads/synth.py``, made on the device.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import workloads as wl
from paper_2511_11729_amd import binding as hb

DEV = "cuda:0"
PAGE = 16                   # tokens per KV page
BLOCK = 2 << 20             # bytes per block of the pool
IN_FLIGHT = 3               # finetune units a caller keeps enqueued before it waits for the oldest
DECODE_PER_UNIT = 8         # decode steps issued beside one finetune unit in the colocated case
WEIGHT = dict(q="wq", k="wk", v="wv", o="wo", gate="wg", up="wu", down="wd")
TARGETS = {"qv": ("q", "v"), "qkvo": ("q", "k", "v", "o"), "all": wl.LORA_TARGETS}


# --------------------------------------------------------------------------------------------- the cases
def listed():
    return [
        # a toy layer in fp32: what a first test of an installation runs, all launches and latency
        {"name": "decode_tiny_f32", "kind": "decode", "config": 0, "layers": 1, "batch": 4, "dist": "uniform", "length": 96},
        # a chat with one user: the whole 7B model, one sequence, weights read once per token
        {"name": "decode_7b_b1", "kind": "decode", "config": 2, "layers": 32, "batch": 1, "dist": "const", "length": 1024},
        # the benchmark's decode step: one 7B layer, 8 sequences of uneven length
        {"name": "decode_7b_layer_b8", "kind": "decode", "config": 1, "layers": 1, "batch": 8, "dist": "uniform", "length": 1152},
        # an odd batch on a model with q, k, v biases, groups of 7 query heads and a large vocabulary
        {"name": "decode_qwen_b21", "kind": "decode", "config": 5, "layers": 4, "batch": 21, "dist": "lognormal", "length": 800},
        # the largest batch before the tiled path, multi-head attention over long uneven caches
        {"name": "decode_13b_b32", "kind": "decode", "config": 3, "layers": 4, "batch": 32, "dist": "lognormal", "length": 1200},
        # a loaded server: the largest batch, grouped-query attention, uneven caches
        {"name": "decode_8b_b256", "kind": "decode", "config": 4, "layers": 4, "batch": 256, "dist": "lognormal", "length": 800},
        # the smallest finetune unit: launches and latency
        {"name": "unit_tiny_f32", "kind": "unit", "config": 0, "micro": 2, "seq": 128, "rank": 8, "targets": "qv"},
        # the benchmark's finetune unit
        {"name": "unit_7b", "kind": "unit", "config": 1, "micro": 4, "seq": 512, "rank": 16, "targets": "qkvo"},
        # a ragged micro-batch: neither the rows nor the sequence length fill tiles; biases, groups of 7
        {"name": "unit_qwen_3x344", "kind": "unit", "config": 5, "micro": 3, "seq": 344, "rank": 16, "targets": "qkvo"},
        # the largest unit: every projection adapted at the largest rank, 1024-token sequences
        {"name": "unit_13b", "kind": "unit", "config": 3, "micro": 4, "seq": 1024, "rank": 64, "targets": "all"},
        # a training step at the 8B grouped-query shape with its 128k-class output layer, two layers deep
        {"name": "train_8b", "kind": "train", "config": 4, "layers": 2, "micro": 8, "seq": 512, "rank": 32, "targets": "qkvo"},
        # the benchmark itself: the finetune unit beside decode steps issued back to back
        {"name": "colocated_7b", "kind": "colocated", "config": 1, "batch": 8, "dist": "uniform", "length": 1152, "micro": 4,
         "seq": 512, "rank": 16, "targets": "qkvo"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["decode"] * 5 + ["unit"] * 3 + ["train", "colocated"])
    if kind in ("decode", "colocated"):
        config = rng.choice([0, 1, 2, 3, 4, 5]) if kind == "decode" else 1
        c = {"kind": kind, "config": config, "dist": rng.choice(["const", "uniform", "lognormal"])}
        if config == 0:
            c.update(layers=rng.randint(1, 2), batch=_log_int(rng, 1, 16), length=_log_int(rng, 16, 384))
        elif kind == "decode":
            c.update(layers=1 if config == 1 else rng.randint(1, 6), batch=_log_int(rng, 1, 256), length=_log_int(rng, 32, 4096))
        else:
            c.update(batch=_log_int(rng, 1, 24), length=_log_int(rng, 64, 1400))
    else:
        config = rng.choice([0, 1, 3, 4, 5]) if kind == "unit" else rng.choice([2, 4, 5])
        c = {"kind": kind, "config": config}
        if kind == "train":
            c["layers"] = rng.randint(1, 2)
    if kind != "decode":
        c.update(micro=rng.randint(1, 8), seq=8 * _log_int(rng, 2, 128), rank=rng.choice([8, 16, 32, 64]),
                 targets=rng.choice(["qv", "qkvo", "all"]))
    return c


def draw(rng):
    """One more case; none with more rows, work or cached tokens than the largest listed ones."""
    cases = listed()
    most = {k: max(work(x)[k] for x in cases) for k in ("bytes", "flops")}
    kv_most = max(_kv_bytes(x) for x in cases if "length" in x)
    while True:
        c = _draw_once(rng)
        if c["kind"] != "decode" and c["micro"] * c["seq"] > (2048 if c["kind"] == "colocated" else 4096):
            continue
        if all(work(c)[k] <= most[k] for k in most) and ("length" not in c or _kv_bytes(c) <= kv_most):
            return c


# --------------------------------------------------------------------------------------------- shapes and floors
def _model(c):
    return dataclasses.replace(wl.workload(c["config"]).model, n_layers=c.get("layers", 1))


def _lengths(c):
    """Cached tokens per sequence: part of the case, the same for every seed."""
    n, w = c["length"], wl.workload(c["config"])
    dist = {"const": ("const", n), "uniform": ("uniform", max(1, n // 4), 2 * n - n // 4),
            "lognormal": ("lognormal", n, 0.6, 8192)}[c["dist"]]
    return np.maximum(1, wl.draw_lengths(w, c["batch"], dist)).astype(np.int32)


def _kv_bytes(c):
    m = _model(c)
    return m.n_layers * int((_lengths(c).astype(np.int64) + 1).sum()) * 2 * m.kv_row_bytes


def _decode_work(c):
    m, n = _model(c), _lengths(c)
    B, L, eb, QD = c["batch"], m.n_layers, m.elem_bytes, m.n_q * m.head_dim
    head = m.vocab * m.hidden
    tokens = int((n.astype(np.int64) + 1).sum())
    nbytes = eb * (L * m.layer_params + head) + _kv_bytes(c) + B * m.hidden * 8 + B * m.vocab * 4
    return nbytes, 2.0 * B * (L * m.layer_params + head) + 4.0 * L * tokens * QD


def _unit_work(c, L=1):
    m, T = _model(c), c["micro"] * c["seq"]
    QD = m.n_q * m.head_dim
    ad = sum(sum(m.proj_shape(p)) for p in TARGETS[c["targets"]]) * c["rank"]
    # frozen weights forward and for dX; causal attention 2 + 5 products; adapters forward 2, dX 2, dA and dB 2 each way
    flops = 4.0 * T * m.layer_params + 7.0 * c["micro"] * c["seq"] ** 2 * QD + 6.0 * T * ad
    return L * (m.elem_bytes * (m.layer_params + ad) + 8 * ad) + 16 * T * m.hidden, L * flops


def work(c):
    if c["kind"] == "decode":
        b, f = _decode_work(c)
    elif c["kind"] == "unit":
        b, f = _unit_work(c)
    elif c["kind"] == "train":
        m, T = _model(c), c["micro"] * c["seq"]
        b, f = _unit_work(c, m.n_layers)
        ad = sum(sum(m.proj_shape(p)) for p in TARGETS[c["targets"]]) * c["rank"] * m.n_layers
        b += m.elem_bytes * m.vocab * m.hidden + 28 * ad     # output layer; AdamW: master, m, v, gradient, 16-bit copy
        f += 4.0 * T * m.vocab * m.hidden
    else:
        b, f = _unit_work(c)
        db, df = _decode_work(c)
        b, f = b + DECODE_PER_UNIT * db, f + DECODE_PER_UNIT * df
    return {"bytes": float(b), "flops": float(f)}


def tolerance(c):
    """About four times the error against the same path in float64 (torch, on the device), measured at the listed cases."""
    L = c.get("layers", 1)
    if c["config"] == 0 and c["kind"] == "decode":
        return {"rel": 1e-5, "max": 1e-4}                    # fp32 throughout
    if c["kind"] in ("decode", "colocated"):                 # bf16 operands: 2.6e-3 at one layer, 5.8e-3 at 4, 1.55e-2 at 32
        return {"rel": min(0.03, 0.0105 * math.sqrt(L)), "max": 0.06 * math.sqrt(L)}
    if c["kind"] == "unit":                                  # half operands: 0.8e-3 to 2.3e-3, largest single error 3e-2
        return {"rel": 8e-3, "max": 0.12}
    return {"rel": 1.6e-2, "max": 0.3}                       # a stack of units; the second moments carry the error twice


# --------------------------------------------------------------------------------------------- set-up
class _Rand:
    """Seeded device tensors."""

    def __init__(self, seed):
        self.g = torch.Generator(DEV)
        self.g.manual_seed(seed)

    def __call__(self, shape, std, dtype=torch.float32, mean=0.0):
        t = torch.randn(shape, generator=self.g, device=DEV, dtype=dtype)
        if std != 1.0:
            t.mul_(std)
        return t.add_(mean) if mean else t


def _layers(m, rnd, dt):
    out = []
    for _ in range(m.n_layers):
        lw = {WEIGHT[p]: rnd(m.proj_shape(p), 0.02, dt) for p in wl.LORA_TARGETS}
        lw["g1"], lw["g2"] = rnd((m.hidden,), 0.02, mean=1.0), rnd((m.hidden,), 0.02, mean=1.0)
        if m.qkv_bias:
            for p in "qkv":
                lw["b" + p] = rnd((m.proj_shape(p)[0],), 0.5)
        out.append(lw)
    return out


def _extras(m, rnd, dt):
    if m.vocab < 1:
        return {}
    return dict(vocab=m.vocab, emb=rnd((m.vocab, m.hidden), 1.0, dt), g_final=rnd((m.hidden,), 0.02, mean=1.0),
                w_lm=rnd((m.vocab, m.hidden), 0.02, dt))


def _shape_args(m):
    return dict(n_layers=m.n_layers, hidden=m.hidden, n_q_heads=m.n_q, n_kv_heads=m.n_kv, head_dim=m.head_dim, ffn=m.ffn,
                rms_eps=m.rms_eps, rope_base=m.rope_base, dtype=hb.HARLI_BF16 if m.dtype == "bf16" else hb.HARLI_F32)


def _unit_chunks(m, T, units, chunk):
    """Pool chunks for the saved activations of `units` finetune calls (a unit's tensors take whole adjacent chunks)."""
    act = T * m.hidden * 12 + T * m.n_q * m.head_dim * 4 + T * m.n_kv * m.head_dim * 4 + T * m.ffn * 6
    return units * (act // chunk + 3)


def _setup(c, seed, *, decode, ft_units):
    """Pool, context and the decode inputs of a case.  `ft_units`: finetune calls whose activations the pool holds."""
    torch.cuda.set_device(0)
    m, rnd = _model(c), _Rand(seed)
    dt = torch.bfloat16 if m.dtype == "bf16" else torch.float32
    s = {"kind": c["kind"], "m": m, "stream": torch.cuda.current_stream()}
    chunk = m.n_layers * 2 * BLOCK
    n = _lengths(c) if decode else np.array([1], np.int32)
    pages = (n + 1 + PAGE - 1) // PAGE
    n_chunks = -(-int(pages.sum()) // (BLOCK // (PAGE * m.kv_row_bytes))) + 1
    small = 0
    T = c["micro"] * c["seq"] if ft_units else 0
    if ft_units:
        n_chunks += _unit_chunks(m, T, ft_units, chunk)
        small = 64 << 20
    nbytes = small + n_chunks * chunk
    s["cache"] = rnd((nbytes // m.elem_bytes,), 1.0, dt) if decode else torch.zeros(nbytes // m.elem_bytes, dtype=dt, device=DEV)
    s["slab"] = s["cache"].view(torch.uint8)
    s["pool"] = hb.Pool(s["slab"], nbytes, block_bytes=BLOCK, n_layers=m.n_layers, page_tokens=PAGE, kv_row_bytes=m.kv_row_bytes,
                        small_pool_bytes=small)
    extras = _extras(m, rnd, dt) if c["kind"] in ("decode", "train") else {}
    s["ctx"] = hb.Context(s["pool"], layers=_layers(m, rnd, dt), max_batch=len(n), max_seq_len=int(n.max()) + 8,
                          max_ft_tokens=T, **_shape_args(m), **extras)
    if decode:
        ids = np.array(s["pool"].alloc_pages(int(pages.sum())), np.int32)
        ids = ids[np.random.default_rng(seed).permutation(len(ids))]     # logical pages scattered over physical ones
        table = np.full((len(n), int(pages.max()) + 1), -1, np.int32)
        at = 0
        for b, k in enumerate(pages):
            table[b, :k] = ids[at:at + k]
            at += k
        s["step"] = dict(batch=len(n), kv_len=torch.from_numpy(n).to(DEV), page_table=torch.from_numpy(table).to(DEV),
                         max_pages=table.shape[1], max_kv_len=int(n.max()) + 1,
                         x_out=torch.empty(len(n), m.hidden, device=DEV))
        if m.vocab:
            s["step"].update(token_ids=torch.randint(0, m.vocab, (len(n),), generator=rnd.g, device=DEV, dtype=torch.int32),
                             logits=torch.empty(len(n), m.vocab, device=DEV),
                             next_token=torch.empty(len(n), dtype=torch.int32, device=DEV))
        else:
            s["step"]["x_in"] = rnd((len(n), m.hidden), 1.0)
    if ft_units:
        _setup_adapters(s, c, rnd, dt)
    return s


def _setup_adapters(s, c, rnd, dt):
    """Adapters of every layer and their gradients, each kind in one flat buffer with a view per tensor."""
    m, names, r = s["m"], TARGETS[c["targets"]], c["rank"]
    shapes = [(l, p, i, sh) for l in range(m.n_layers) for p in names
              for i, sh in ((0, (m.proj_shape(p)[1], r)), (1, (r, m.proj_shape(p)[0])))]
    total = sum(a * b for _, _, _, (a, b) in shapes)

    def flat(dtype):
        buf, views, at = torch.zeros(total, dtype=dtype, device=DEV), [], 0
        for _, _, _, (a, b) in shapes:
            views.append(buf[at:at + a * b].view(a, b))
            at += a * b
        return buf, views

    s["param"], pv = flat(dt)
    s["grad"], gv = flat(torch.float32)
    for (_, _, i, sh), v in zip(shapes, pv):
        v.copy_(rnd(sh, 0.01 if i else 0.125, dt))
    per = [[{}, {}, {}, {}] for _ in range(m.n_layers)]        # A, B, dA, dB by target
    for (l, p, i, _), v, g in zip(shapes, pv, gv):
        per[l][i][p], per[l][2 + i][p] = v, g
    s["A"], s["B"], s["dA"], s["dB"] = ([per[l][k] for l in range(m.n_layers)] for k in range(4))
    s["ctx"].lora_attach(r, 2.0 * r, names, s["A"], s["B"])
    T = c["micro"] * c["seq"]
    s["shape"] = (c["micro"], c["seq"])
    s["done"] = []
    if c["kind"] == "train":
        s["t"] = 0
        s["master"], mv = flat(torch.float32)
        s["m1"], m1 = flat(torch.float32)
        s["m2"], m2 = flat(torch.float32)
        s["master"].copy_(s["param"])
        s["update"] = list(zip(mv, m1, m2, gv, pv))
        s["emb"] = rnd((m.vocab, m.hidden), 1.0)
        s["tok"] = torch.randint(0, m.vocab, s["shape"], generator=rnd.g, device=DEV)
        tg = torch.full(s["shape"], -1, dtype=torch.int32, device=DEV)
        tg[:, :-1] = s["tok"][:, 1:]
        s["tok"], s["tg"] = s["tok"].reshape(-1), tg.reshape(-1)
        s["acts"] = [torch.empty(T, m.hidden, device=DEV) for _ in range(m.n_layers + 1)]
        s["d"] = [torch.empty(T, m.hidden, device=DEV) for _ in range(2)]
        s["loss"] = torch.zeros(1, device=DEV)
    else:
        s["X"] = rnd((T, m.hidden), 1.0)
        s["dY"] = rnd((T, m.hidden), 1.0 / (T * m.hidden))
        s["Y"], s["dX"] = torch.empty(T, m.hidden, device=DEV), torch.empty(T, m.hidden, device=DEV)


def prepare(c, seed):
    if c["kind"] == "decode":
        return _setup(c, seed, decode=True, ft_units=0)
    if c["kind"] == "train":
        return _setup(c, seed, decode=False, ft_units=c["layers"] * (IN_FLIGHT + 1))
    s = _setup(c, seed, decode=c["kind"] == "colocated", ft_units=IN_FLIGHT + 1)
    if c["kind"] == "colocated":
        s["streams"] = (torch.cuda.Stream(), torch.cuda.Stream())
    return s


# --------------------------------------------------------------------------------------------- one pass
def _wait_for_room(s):
    """The activations of a unit return to the pool when the GPU has passed it: a caller keeps a few units enqueued."""
    if len(s["done"]) >= IN_FLIGHT:
        s["done"].pop(0).synchronize()


def _mark_done(s, stream):
    ev = torch.cuda.Event()
    ev.record(stream)
    s["done"].append(ev)


def _unit(s, stream):
    _wait_for_room(s)
    saved = s["ctx"].lora_fwd(0, s["X"], s["Y"], *s["shape"], stream=stream)
    s["ctx"].lora_bwd(0, s["dY"], s["dX"], saved, s["dA"][0], s["dB"][0], stream=stream)
    _mark_done(s, stream)
    return {"Y": s["Y"], "dX": s["dX"], "grads": s["grad"]}


def _train(s, stream):
    ctx, acts, L = s["ctx"], s["acts"], s["m"].n_layers
    _wait_for_room(s)
    s["t"] += 1
    torch.index_select(s["emb"], 0, s["tok"], out=acts[0])
    saved = [ctx.lora_fwd(l, acts[l], acts[l + 1], *s["shape"], stream=stream) for l in range(L)]
    d, dn = s["d"]
    ctx.head_fwd_bwd(acts[L], s["tg"], s["loss"], d, stream=stream)
    for l in range(L - 1, -1, -1):
        ctx.lora_bwd(l, d, dn, saved[l], s["dA"][l], s["dB"][l], stream=stream)
        d, dn = dn, d
    for master, m1, m2, grad, param in s["update"]:
        hb.adamw_step(master, m1, m2, grad, param, step=s["t"], lr=1e-4, zero_grad=True, stream=stream)
    _mark_done(s, stream)
    return {"loss": s["loss"], "hidden": acts[L], "dX": d, "master": s["master"], "m1": s["m1"], "m2": s["m2"], "param": s["param"]}


def run(s):
    if s["kind"] == "unit":
        return _unit(s, s["stream"])
    if s["kind"] == "train":
        return _train(s, s["stream"])
    if s["kind"] == "decode":
        s["ctx"].decode_step(stream=s["stream"], **s["step"])
        # the chosen tokens are left out: where two logits lie within their rounding either is right
        return {"x_out": s["step"]["x_out"], "cache": s["cache"], "logits": s["step"].get("logits")}
    dec, ft = s["streams"]
    for st in s["streams"]:
        st.wait_stream(s["stream"])
    out = _unit(s, ft)
    for _ in range(DECODE_PER_UNIT):
        s["ctx"].decode_step(stream=dec, **s["step"])
    for st in s["streams"]:
        s["stream"].wait_stream(st)
    return {"x_out": s["step"]["x_out"], **out}
