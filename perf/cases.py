"""What the performance of this library is measured on.

A node of the ring does three things: it takes a sample's first visit (the whole prompt, in one call or in pieces),
it takes later visits (the newest position of one sample, or of all the samples whose messages wait in its queue),
and, on the starter, it turns returning hidden states into tokens.  The cases are calls of these entry points on
the model shapes and partitions of `synth.py` (the benchmark workloads and the paper's own models), from one message
of a small fp32 node to a long first visit, in both storage types.

Weights follow `synth.make_weights` (N(0, 0.02^2) matrices) with gains and biases off their neutral values, hidden
states that cross a node's boundary are N(0, 1), token ids are uniform; everything is made on the GPU from the seed.

A decode case keeps generating: every pass extends the caches by one position, and when they are full the samples
are dropped and the next requests, with the same prompts, take their places.
"""
import torch

from paper_2505_18164_amd import mdi, synth as S

# shape name -> (preset, layers of the largest partition, the node is the starter: embedding in, output layers on)
SHAPES = {
    "gpt2": (S.gpt2_small, 4, True),          # 12 layers cut in three
    "nanollama": (S.nanollama, 7, True),      # the paper's 304M model, cuts 5/7 and 2/5/5
    "tinyllama": (S.tinyllama, 12, True),     # the paper's 1.1B model, cuts 10/12 and 6/8/8; 11 of 22 in the benchmark
    "llama2_7b": (S.llama2_7b, 8, False),     # layers 8 - 15: a secondary node
    "llama3_8b": (S.llama3_8b, 8, False),     # 32 layers cut in four
}
PROMPTS_AT_ONCE = 2048                        # a longer context is filled in pieces of this many positions
STEP_INPUTS = 8                               # different inputs a decode case goes round


def listed():
    return [
        # The smallest call: the starter of a 4-layer fp32 GPT-2 node turns one returning state into a token and
        # forwards it.  All latency: 110 MB of weights, 20 exchanges between workgroups.
        {"name": "gpt2 fp32 one token", "kind": "starter", "shape": "gpt2", "dtype": "fp32", "layers": 4, "n": 1, "ctx": 16, "shared": False},
        # One node of GPT-2 cut in three, three samples in flight (as many as nodes), their queue drained in one call.
        {"name": "gpt2 queue of 3", "kind": "queue", "shape": "gpt2", "dtype": "bf16", "layers": 4, "n": 3, "ctx": 128, "shared": True},
        # The starter of a TinyLlama ring: four samples come back, get their tokens and go on through 11 layers.
        {"name": "tinyllama starter, 4 samples", "kind": "starter", "shape": "tinyllama", "dtype": "bf16", "layers": 11, "n": 4, "ctx": 512, "shared": True},
        # The paper's own rule on a large partition: one message per call.
        {"name": "llama2-7b one message", "kind": "queue", "shape": "llama2_7b", "dtype": "bf16", "layers": 8, "n": 1, "ctx": 1024, "shared": False},
        # The headline of the benchmark: eight samples in flight share a pass over the weights.
        {"name": "llama2-7b queue of 8", "kind": "queue", "shape": "llama2_7b", "dtype": "bf16", "layers": 8, "n": 8, "ctx": 1024, "shared": True},
        # A full pass late in long generations: sixteen samples, grouped kv heads, caches of 6144 positions.
        {"name": "llama3-8b queue of 16, long", "kind": "queue", "shape": "llama3_8b", "dtype": "bf16", "layers": 8, "n": 16, "ctx": 6144, "shared": True},
        # First visit of a short, odd prompt to the paper's fp32 model (the larger part of the 5/7 cut).
        {"name": "nanollama fp32 prompt of 100", "kind": "visit", "shape": "nanollama", "dtype": "fp32", "layers": 7, "T": 100, "pieces": 1},
        # First visit of an ordinary, ragged prompt to the starter of a TinyLlama ring.
        {"name": "tinyllama prompt of 333", "kind": "visit", "shape": "tinyllama", "dtype": "bf16", "layers": 11, "T": 333, "pieces": 1},
        # The benchmark's first visit, in one call ...
        {"name": "llama2-7b prompt of 1024", "kind": "visit", "shape": "llama2_7b", "dtype": "bf16", "layers": 8, "T": 1024, "pieces": 1},
        # ... and in pieces, as a node takes it that must not stall the other samples for the whole visit.
        {"name": "llama2-7b prompt in 4 pieces", "kind": "visit", "shape": "llama2_7b", "dtype": "bf16", "layers": 8, "T": 1024, "pieces": 4},
        # The largest: a long document's first visit to a quarter of the 8B model.
        {"name": "llama3-8b prompt of 6000", "kind": "visit", "shape": "llama3_8b", "dtype": "bf16", "layers": 8, "T": 6000, "pieces": 1},
        # The starter draws tokens for sixteen returning samples over the large vocabulary.
        {"name": "llama3-8b tokens for 16", "kind": "head", "shape": "llama3_8b", "dtype": "bf16", "n": 16, "top_k": 50},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over the logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    shape = rng.choice(list(SHAPES))
    make, most, _ = SHAPES[shape]
    # the small models are run in fp32 as well (the paper's boards have no 16-bit arithmetic), the large ones in bf16
    dtype = rng.choice(["fp32", "bf16"]) if shape in ("gpt2", "nanollama") else "bf16"
    max_ctx = make()["max_ctx"]
    kind = rng.choice(["queue", "queue", "visit", "visit", "starter", "head"])
    layers = rng.randint(1, most)
    if kind == "visit":
        T = _log(rng, 1, min(max_ctx, 6000 if dtype == "bf16" else 1024))
        return {"kind": "visit", "shape": shape, "dtype": dtype, "layers": layers, "T": T,
                "pieces": rng.choice([1, 1, rng.randint(2, 6)]) if T >= 64 else 1}
    if kind == "head":
        return {"kind": "head", "shape": shape, "dtype": dtype, "n": rng.randint(1, 16), "top_k": rng.choice([1, rng.randint(2, 64)])}
    if kind == "starter" and not SHAPES[shape][2]:
        kind = "queue"
    return {"kind": kind, "shape": shape, "dtype": dtype, "layers": layers, "n": rng.choice([1, rng.randint(2, 16), rng.randint(2, 16)]),
            "ctx": _log(rng, 16, max_ctx * 3 // 4), "shared": rng.random() < 0.75}


# ----------------------------------------------------------------------------
def _cfg(case):
    cfg = SHAPES[case["shape"]][0](dtype=S.DT_F32 if case["dtype"] == "fp32" else S.DT_BF16)
    cfg["n_layer"] = max(cfg["n_layer"], case.get("layers", 0))
    return cfg


def _layer_range(case, cfg):
    n = case.get("layers", 0)
    lo = 0 if SHAPES[case["shape"]][2] else min(8, cfg["n_layer"] - n)
    return lo, lo + n


def _weights(cfg, lo, hi, embed, head, gen):
    """Random-init weights on the GPU: matrices N(0, 0.02^2) in the storage type, gains around 1 and biases around 0."""
    dt = mdi.torch_dtype(cfg["dtype"])

    def mat(*shape):
        t = torch.randn(shape, generator=gen, device="cuda", dtype=dt)
        return t.mul_(S.WEIGHT_STD)

    def vec(n, centre):
        return torch.randn((n,), generator=gen, device="cuda").mul_(0.1).add_(centre)

    ln = cfg["norm_kind"] == S.NORM_LAYERNORM
    w = {"layers": {}}
    for layer in range(lo, hi):
        shapes = S.layer_tensor_shapes(cfg)
        lw = {name: mat(*shape) for name, shape in shapes.items()}
        for k in ("1", "2"):
            lw["ln%s_g" % k] = vec(cfg["d_model"], 1.0)
            if ln:
                lw["ln%s_b" % k] = vec(cfg["d_model"], 0.0)
        if cfg["has_bias"]:
            for b, m in (("bq", "wq"), ("bk", "wk"), ("bv", "wv"), ("bo", "wo"), ("b1", "w1"), ("b2", "w2")):
                if m in shapes:
                    lw[b] = vec(shapes[m][0], 0.0)
        w["layers"][layer] = lw
    if embed or (head and cfg["tie_embed"]):
        w["wte"] = mat(cfg["vocab"], cfg["d_model"])
    if embed and cfg["pos_kind"] == S.POS_LEARNED:
        w["wpe"] = mat(cfg["max_ctx"], cfg["d_model"])
    if head:
        w["lnf_g"] = vec(cfg["d_model"], 1.0)
        if ln:
            w["lnf_b"] = vec(cfg["d_model"], 0.0)
        if not cfg["tie_embed"]:
            w["lm_head"] = mat(cfg["vocab"], cfg["d_model"])
    return w


def _inputs(cfg, embed, T, gen):
    """T positions that enter a node: token ids at the starter, else the previous node's hidden states."""
    if embed:
        return torch.randint(0, cfg["vocab"], (T,), generator=gen, device="cuda", dtype=torch.int32)
    return torch.randn((T, cfg["d_model"]), generator=gen, device="cuda", dtype=mdi.torch_dtype(cfg["dtype"]))


def _hidden(cfg, shape, gen):
    return torch.randn((*shape, cfg["d_model"]), generator=gen, device="cuda", dtype=mdi.torch_dtype(cfg["dtype"]))


def _cuts(T, pieces):
    """T positions in `pieces` pieces of about equal length."""
    return [T * (i + 1) // pieces - T * i // pieces for i in range(pieces)]


def _first_visits(st):
    """(Re)fills every sample's cache from its prompt, long ones in pieces."""
    part, cut = st["part"], st["cuts"]
    for s, prompt in enumerate(st["prompts"]):
        part.seq_reset(s)
        at = 0
        for t in cut:
            part.prefill_chunk(s, prompt[at:at + t], st["prompt_out"][:t])
            at += t
    st["len"] = sum(cut)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    cfg = _cfg(case)
    lo, hi = _layer_range(case, cfg)
    kind, n, dt = case["kind"], case.get("n", 1), mdi.torch_dtype(cfg["dtype"])
    embed = hi > lo and SHAPES[case["shape"]][2]
    head = kind in ("starter", "head")
    st = {"case": dict(case), "V": cfg["vocab"]}
    page = 64 if cfg["d_model"] >= 2048 else 16
    if kind == "visit":
        T, cuts = case["T"], _cuts(case["T"], case["pieces"])
        st["part"] = mdi.Partition(cfg, _weights(cfg, lo, hi, embed, head, gen), lo, hi, has_embed=embed, max_seqs=2,
                                   kv_page_tokens=page, max_prefill=max(cuts))
        st["in"] = list(torch.split(_inputs(cfg, embed, T, gen), cuts))
        st["out"] = [torch.empty((t, cfg["d_model"]), dtype=dt, device="cuda") for t in cuts]
        return st
    if head:
        st["states"] = _hidden(cfg, (STEP_INPUTS, n), gen)
        st["tokens"] = torch.empty((n,), dtype=torch.int32, device="cuda")
        st["logits"] = torch.empty((n, cfg["vocab"]), dtype=torch.float32, device="cuda")
        st["step"] = 0
    if kind == "head":
        st["part"] = mdi.Partition(cfg, _weights(cfg, lo, lo, False, True, gen), lo, lo, has_head=True, max_seqs=n)
        return st
    ctx = case["ctx"]
    cuts = _cuts(ctx, -(-ctx // PROMPTS_AT_ONCE))
    st["part"] = mdi.Partition(cfg, _weights(cfg, lo, hi, embed, head, gen), lo, hi, has_embed=embed, has_head=head,
                               max_seqs=n, kv_page_tokens=page, max_prefill=max(cuts))
    st["prompts"] = [_inputs(cfg, embed, ctx, gen) for _ in range(n)]
    st["prompt_out"] = torch.empty((max(cuts), cfg["d_model"]), dtype=dt, device="cuda")
    st["cuts"], st["max_ctx"] = cuts, cfg["max_ctx"]
    if kind == "queue":
        st["inputs"] = [[_inputs(cfg, embed, 1, gen)[0:1].reshape(-1) for _ in range(n)] for _ in range(STEP_INPUTS)]
    st["out"] = [torch.empty((cfg["d_model"],), dtype=dt, device="cuda") for _ in range(n)]
    st["step"] = 0
    _first_visits(st)
    return st


def _tokens(st, states, top_k):
    """Output layers of the samples whose hidden states came back: tokens and logits."""
    part, n, k = st["part"], len(states), st["step"]
    if n == 1:
        if top_k == 1:
            part.sample_greedy(0, states[0], st["tokens"], st["logits"])
        else:
            part.sample_topk(0, states[0], 0.8, top_k, 1234, k, st["tokens"], st["logits"])
    else:
        part.sample_batch(list(range(n)), states, 0.8, top_k, 1234, [k] * n, st["tokens"], st["logits"])


def run(st):
    case, part = st["case"], st["part"]
    kind = case["kind"]
    if kind == "visit":
        part.seq_reset(0)
        for x, y in zip(st["in"], st["out"]):
            part.prefill_chunk(0, x, y)
        return st["out"]
    k = st["step"] % STEP_INPUTS
    if kind == "head":
        _tokens(st, list(st["states"][k]), case["top_k"])
        st["step"] += 1
        return st["tokens"], st["logits"]
    n = case["n"]
    if st["len"] + 1 > st["max_ctx"]:
        _first_visits(st)
    if kind == "starter":
        _tokens(st, list(st["states"][k]), 1)
        ins = [st["tokens"][s:s + 1] for s in range(n)]
    else:
        ins = st["inputs"][k]
    if n == 1:
        part.decode_step(0, ins[0], st["out"][0])
    elif case["shared"]:
        part.decode_batch(list(range(n)), ins, st["out"])
    else:
        part.decode_steps(list(range(n)), ins, st["out"])
    st["step"] += 1
    st["len"] += 1
    return (st["tokens"], st["logits"], st["out"]) if kind == "starter" else st["out"]


# ----------------------------------------------------------------------------
def work(case):
    """Bytes: every matrix once per pass (once per call for the pieces of a first visit, which are calls of their own),
    every sample's cached keys and values once, what is appended to the caches, inputs and outputs.  Operations: the
    products, and attention over the positions that are visible."""
    cfg = _cfg(case)
    esz = 4 if case["dtype"] == "fp32" else 2
    d, H, K, h, F, V = (cfg[k] for k in ("d_model", "n_head", "n_kv_head", "head_dim", "d_ff", "vocab"))
    layers, kind, n = case.get("layers", 0), case["kind"], case.get("n", 1)
    mats = layers * ((H + 2 * K) * h * d + d * H * h + (3 if cfg["mlp_kind"] == S.MLP_SWIGLU else 2) * d * F)
    kv = layers * 2 * K * h * esz                    # bytes of one position's keys and values
    nbytes = flops = 0.0
    if kind == "visit":
        T, at = case["T"], 0
        for t in _cuts(T, case["pieces"]):
            nbytes += mats * esz + kv * (at + t) + 2 * t * d * esz
            flops += 2.0 * t * mats + 4.0 * layers * H * h * (t * at + t * (t + 1) / 2)
            at += t
        return {"bytes": nbytes, "flops": flops}
    if kind in ("starter", "head"):
        nbytes += V * d * esz + n * (d * esz + V * 4 + 4)
        flops += 2.0 * n * V * d
    if kind != "head":
        # a queue that is not shared makes a pass over the weights for every message: that is what the call promises
        passes = 1 if case["shared"] or n == 1 else n
        nbytes += passes * mats * esz + n * (kv * (case["ctx"] + 1) + 2 * d * esz)
        flops += n * (2.0 * mats + 4.0 * layers * H * h * (case["ctx"] + 1))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the paths differ by from the same arithmetic in 64 bits, in which nothing between the
    storage types is rounded (relative, and largest single difference):
    fp32 (sums of up to 5120 products): 3.0e-6 and 1.3e-5 behind seven layers, 1e-7 and 4e-7 for logits;
    bf16, logits: 1.7e-3 and 8e-3;
    bf16, hidden states behind 4 / 8 / 11 layers: 3.4e-3 / 8.5e-3 / 1.34e-2, and up to 6e-2 (caches, hand-offs and
    the vectors between the products are bf16; another order of sums moves them to the neighbouring value)."""
    if case["dtype"] == "fp32":
        return {"rel": 1.2e-5, "max": 6e-5}
    return {"rel": 7e-3, "max": 3e-2} if case["kind"] == "head" else {"rel": 2e-2, "max": 0.2}
