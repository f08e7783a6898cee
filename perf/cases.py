"""The work that programs have this library do, as cases whose speed is measured.

A case is one iteration of the denoising step (or the part of it that a path has of its own) through the public calls of
the package, on the model shapes of this repository's configurations:

  decode   psd_decode for one iteration of Alg. 1 on whole sequences: stage-1 call, commit, drafts, verification call over
           the K drafts, acceptance -- what a generation spends its time on
  steps    the same iteration as separate calls, for programs that keep the loop in their own hands
  cached   one iteration of a context-causal block model against its KV caches, as separate calls
  prefill  the prompt's keys and values of such a model into its KV caches
  approx   one iteration of a bidirectional model under the approximate KV cache: the refreshing call on the whole
           sequences, then the verification on the block rows
  decide   the decision kernels alone on given tables, for programs that run a model of their own

Weights are random.  They are drawn once per process and model, from a seed of their own: a program loads its model once
and then takes prompt after prompt.  The token embeddings carry most of the residual stream, as in trained models, which
keeps rounding differences from growing layer by layer; the mask token's row is smaller, so that what a masked position
predicts comes from its context.  Confidences stay flat and below the threshold, as with every random model here, so an
iteration always makes both of its model calls.
"""
from collections import OrderedDict
from dataclasses import dataclass

import numpy as np
import torch

import paper_2605_15609_amd as psd
from paper_2605_15609_amd.binding import pack_qkv

DEVICE = "cuda:0"


@dataclass(frozen=True)
class Shape:
    name: str
    dtype: str
    n_layers: int
    d_model: int
    n_heads: int
    n_kv_heads: int
    d_head: int
    d_ffn: int
    vocab: int
    rms_eps: float
    rope_theta: float
    qkv_bias: bool
    logit_scale: float = 1.0
    attention: str = "bidirectional"

    @property
    def mask_id(self):
        return self.vocab - 1


SHAPES = {
    "tiny": Shape("tiny-fp32", "fp32", 2, 64, 4, 4, 16, 256, 256, 1e-5, 1e4, False),
    "small": Shape("small-bf16", "bf16", 8, 512, 8, 8, 64, 1408, 32000, 1e-5, 1e4, False),
    "llada": Shape("llada8b-shaped", "bf16", 32, 4096, 32, 32, 128, 12288, 126464, 1e-5, 5e5, False),
    "dream": Shape("dream7b-shaped", "bf16", 28, 3584, 28, 4, 128, 18944, 152064, 1e-6, 1e6, True),
}
# rows of the rotary tables (a library handle takes sequences up to this length)
MAX_SEQ = 2048


def _case(name, path, model, B, prompt, gen, L, K, layers=0, graph="chain"):
    c = {"path": path, "model": model, "layers": layers or SHAPES[model].n_layers, "B": B, "prompt": prompt, "gen": gen, "L": L,
         "K": K, "graph": graph}
    return dict(c, name=name) if name else c


def listed():
    return [
        # decisions for a batch of a program's own model: the smallest calls, launches are all there is
        _case("decide", "decide", "small", 16, 256, 1024, 64, 8),
        # the fp32 path at the size of its configuration: a debugging session steps through a generation
        _case("tiny fp32 iteration", "decode", "tiny", 1, 16, 32, 32, 2),
        # a small model, one user
        _case("small iteration", "decode", "small", 1, 128, 256, 32, 4),
        # a small model, several users, prompts of no round length, blocks of 24, a multi-parent draft graph
        _case("small ragged batch", "decode", "small", 5, 77, 120, 24, 4, graph="lattice"),
        # one user of an 8B model (the repository's third configuration)
        _case("8B iteration", "decode", "llada", 1, 256, 256, 32, 4),
        # three users of an 8B model, prompts of no round length, loop in the program's own hands
        _case("8B ragged steps", "steps", "llada", 3, 301, 256, 32, 4),
        # one user of a 7B model with grouped KV heads and biases, longer sequence, deeper drafts (fourth configuration)
        _case("7B grouped iteration", "decode", "dream", 1, 512, 512, 32, 6),
        # a full batch: 16 sequences of 1280 tokens, 128 drafts verified in one call (fifth configuration, 8 of 32 layers)
        _case("batch of 16, 128 drafts", "decode", "llada", 16, 256, 1024, 64, 8, layers=8),
        # block-causal serving: one user ...
        _case("8B cached iteration", "cached", "llada", 1, 256, 256, 32, 4),
        # ... several users on a model with grouped KV heads ...
        _case("7B grouped cached batch", "cached", "dream", 4, 512, 512, 32, 6),
        # ... and the prompt that comes before it
        _case("8B prefill", "prefill", "llada", 1, 512, 256, 32, 1),
        # a bidirectional model under the approximate cache
        _case("8B approximate cache", "approx", "llada", 1, 256, 256, 32, 4),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def spread(lo, hi):      # whole numbers, evenly over their logarithm
        return int(round(lo * (hi / lo) ** rng.random()))

    most = max(_cost(c) for c in listed())
    while True:
        path = rng.choice(["decode", "decode", "decode", "steps", "cached", "cached", "prefill", "approx", "decide"])
        model = "small" if path == "decide" else rng.choice(["small", "llada", "dream"] + (["tiny"] if path in ("decode", "steps") else []))
        cached = path in ("cached", "prefill", "approx")
        L = rng.choice([16, 32, 48, 64]) if cached else rng.choice([16, 20, 24, 32, 32, 40, 64])
        prompt, gen = spread(16, 1024), L * spread(2, 16)
        if path in ("cached", "prefill"):
            prompt = max(1, prompt // L) * L      # prompts of whole blocks
        if path == "approx" and rng.random() < 0.5:
            prompt = prompt // 8 * 8
        graph, K = ("lattice", rng.choice([2, 4, 8])) if rng.random() < 0.25 else ("chain", rng.randint(2, 8))
        layers = {"tiny": 2, "small": 8, "llada": rng.choice([8, 32]), "dream": rng.choice([7, 28])}[model]
        case = _case("", path, model, spread(1, 16), prompt, gen, L, K, layers, graph)
        # a case as large as the largest listed one at most, and sequences that the handle takes; sequences of no round
        # length come in small batches, and a generation of a few tokens comes with others (or its one commit more or less
        # would be a large share of it)
        N, calls = prompt + gen, case["B"] * (1 + K)
        few = path == "decode" or path == "steps" or path == "approx"
        if N > MAX_SEQ - 64 or _cost(case) > most or (few and N % 8 and calls * N * N > 15 * 600 * 600):
            continue
        if model != "tiny" and case["B"] * N < 400:
            continue
        return case


def _shape(case):
    s = SHAPES[case["model"]]
    causal = case["path"] in ("cached", "prefill")
    return Shape(**dict(s.__dict__, n_layers=case["layers"], attention="block_causal" if causal else "bidirectional"))


# -------------------------------------------------------------------------------------------------------------- weights
_weights, _models = {}, OrderedDict()


def _draw_weights(name):
    s = SHAPES[name]
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000 + sorted(SHAPES).index(name))
    dtype = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    d, hq, hkv, f, v = s.d_model, s.n_heads * s.d_head, s.n_kv_heads * s.d_head, s.d_ffn, s.vocab

    def normal(std, *dims, dtype=dtype):
        return torch.empty(dims, dtype=dtype, device=DEVICE).normal_(0.0, std, generator=g)

    def ones(n):
        return torch.ones(n, dtype=torch.float32, device=DEVICE)

    std = 1.28 / d ** 0.5         # 0.02 at d_model 4096
    emb = normal(1.0, v, d)
    emb[s.mask_id] *= 0.3
    tensors = {"tok_emb": emb, "lm_head": normal(0.5 * std, v, d), "final_norm": ones(d)}
    half = s.d_head // 2
    freq = s.rope_theta ** (-torch.arange(half, dtype=torch.float64) * 2.0 / s.d_head)
    angle = torch.arange(MAX_SEQ, dtype=torch.float64)[:, None] * freq[None, :]
    tensors["rope_cos"], tensors["rope_sin"] = angle.cos().float().to(DEVICE), angle.sin().float().to(DEVICE)
    out = std / (2.0 * s.n_layers) ** 0.5
    layers = []
    for _ in range(s.n_layers):
        lt = {"attn_norm": ones(d), "wq": normal(std, hq, d), "wk": normal(std, hkv, d), "wv": normal(std, hkv, d),
              "wo": normal(out, d, hq), "ffn_norm": ones(d), "w_gate": normal(std, f, d), "w_up": normal(std, f, d),
              "w_down": normal(out, d, f), "bq": None, "bk": None, "bv": None}
        if s.qkv_bias:
            for b, n in (("bq", hq), ("bk", hkv), ("bv", hkv)):
                lt[b] = normal(0.02, n, dtype=torch.float32)
        pack_qkv(lt)
        layers.append(lt)
    return tensors, layers


def _model(case):
    """The program's model, loaded once: its handle for this path (a cut of `layers` layers shares the tensors)."""
    s = _shape(case)
    if s not in _models:
        if case["model"] not in _weights:
            _weights[case["model"]] = _draw_weights(case["model"])
        tensors, layers = _weights[case["model"]]
        while len(_models) >= 4:
            _models.popitem(last=False)[1].close()
        _models[s] = psd.Model(s, MAX_SEQ, tensors, layers[: s.n_layers], DEVICE)
    _models.move_to_end(s)
    return _models[s]


# --------------------------------------------------------------------------------------------------------------- inputs
_zipf = {}


def _text(rng, vocab, dims):
    """Token ids with the frequencies of text: rank r of the truncated Zipf law p(r) ~ r^-1.1; never the mask token."""
    if vocab not in _zipf:
        c = np.cumsum(np.arange(1, vocab, dtype=np.float64) ** -1.1)
        _zipf[vocab] = c / c[-1]
    return np.minimum(np.searchsorted(_zipf[vocab], rng.random(dims)), vocab - 2).astype(np.int32)


def _graph(case):
    if case["graph"] == "lattice":
        return psd.lattice_graph(case["K"].bit_length() - 1)
    return psd.chain_graph(case["K"])


def prepare(case, seed):
    model = _model(case)
    rng = np.random.default_rng([seed, 7])
    v, mask = model.shape.vocab, model.shape.mask_id
    B, P, G, L, K = case["B"], case["prompt"], case["gen"], case["L"], case["K"]
    N = P + G
    path = case["path"]
    # the prompt, blocks that are finished, and masks from the active block on; sequences of a batch are on blocks of their
    # own where the call lets them (psd_decode), on a common one elsewhere
    blocks = rng.integers(0, G // L, size=B)
    if path != "decode":
        blocks[:] = blocks[0]
    starts = [int(P + b * L) for b in blocks]
    tokens = _text(rng, v, (B, N))
    for b, start in enumerate(starts):
        tokens[b, start:] = mask
    state = {"path": path, "model": model, "L": L, "K": K, "N": N, "prompt": P, "starts": starts, "start": starts[0], "policy": psd.Policy(0.9, 1),
             "graph": _graph(case)}
    if path == "decide":
        # a block of which 70 % is masked and the tables of a model of the program's own: confidences on both sides of the
        # threshold, verifier predictions that repeat the first ones with probability 0.7
        start = starts[0]
        tokens[:, start:start + L] = np.where(rng.random((B, L)) < 0.7, mask, _text(rng, v, (B, L)))
        open_ = tokens[:, start:start + L] == mask
        top1 = np.where(open_, _text(rng, v, (B, L)), tokens[:, start:start + L])
        conf = np.where(open_, rng.random((B, L)), -1.0)
        v_top1 = np.where(rng.random((B, K, L)) < 0.7, top1[:, None, :], _text(rng, v, (B, K, L)))
        for name, a, dtype in (("top1", top1, torch.int32), ("conf", conf, torch.float32), ("v_top1", v_top1, torch.int32),
                               ("v_conf", rng.random((B, K, L)), torch.float32)):
            state[name] = torch.from_numpy(np.ascontiguousarray(a)).to(DEVICE, dtype)
    state["given"] = torch.from_numpy(tokens).to(DEVICE)
    state["tokens"] = state["given"].clone()
    if path == "cached":
        state["cache"] = psd.KvCache(model, B, N)
        psd.psd_kv_prefill(model, state["tokens"], state["start"], L, state["cache"])
    elif path == "prefill":
        state["cache"] = psd.KvCache(model, B, P)
        nbytes = 2 * model.shape.n_layers * model.shape.n_kv_heads * model.shape.d_head * (P + (P + 63) // 64 * 64) * B
        state["kv"] = state["cache"].mem[:nbytes].view(torch.bfloat16)
    elif path == "approx":
        state["cache"] = psd.KvCache(model, B, N - L)
    return state


# ------------------------------------------------------------------------------------------------------------- one pass
def run(state):
    path, model, L = state["path"], state["model"], state["L"]
    tokens, start, policy, graph = state["tokens"], state["start"], state["policy"], state["graph"]
    if path == "prefill":
        psd.psd_kv_prefill(model, tokens, state["prompt"], L, state["cache"])
        return {"kv": state["kv"]}
    tokens.copy_(state["given"])      # every pass starts from the same generation
    if path == "decode":
        psd.psd_decode(model, tokens, state["starts"], L, policy, graph, max_iterations=1)
        return {"tokens": tokens}
    if path == "decide":
        mask, n = psd.psd_select_unmask(model, tokens, start, L, state["top1"], state["conf"], policy)
        sigma, m, drafts = psd.psd_build_drafts(model, tokens, start, L, state["top1"], state["conf"], graph)
        k_star, accepted = psd.psd_accept(model, tokens, drafts, start, L, sigma, m, graph, policy, state["v_top1"], state["v_conf"])
        return {"tokens": tokens, "mask": mask, "n": n, "sigma": sigma, "m": m, "drafts": drafts, "k_star": k_star, "accepted": accepted}
    # one iteration of Alg. 1 by separate calls
    B, N, K = tokens.shape[0], state["N"], graph.K
    if path == "steps":
        top1, conf = psd.psd_forward_confidence(model, tokens, start, L)
    elif path == "cached":
        top1, conf = psd.psd_forward_confidence_cached(model, tokens, start, L, state["cache"])
    else:
        top1, conf = psd.psd_forward_confidence_approx(model, tokens, start, L, state["cache"], refresh=True)
    psd.psd_select_unmask(model, tokens, start, L, top1, conf, policy)
    sigma, m, drafts = psd.psd_build_drafts(model, tokens, start, L, top1, conf, graph)
    if path == "steps":
        psd.psd_verify_accept(model, tokens, drafts, start, L, sigma, m, graph, policy)
    else:
        rows = drafts.view(B * K, N)
        if path == "cached":
            v_top1, v_conf = psd.psd_forward_confidence_cached(model, rows, start, L, state["cache"], seqs_per_cache=K)
        else:
            v_top1, v_conf = psd.psd_forward_confidence_approx(model, rows, start, L, state["cache"], refresh=False, seqs_per_cache=K)
        psd.psd_accept(model, tokens, drafts, start, L, sigma, m, graph, policy, v_top1.view(B, K, L), v_conf.view(B, K, L))
    return {"conf": conf, "tokens": tokens, "drafts": drafts}


# ------------------------------------------------------------------------------------------------- what a pass cannot avoid
def _call(s, S, N, L, keys, head=True, last=True):
    """(bytes, flops) of one model call over S sequences of N rows, each of which sees `keys` keys on average: every weight
    once, every row through every layer; in the last layer all rows give keys and values and only the L block rows of a
    sequence (last=False: none) go further; head: the LM-head pass on those rows."""
    size = 2 if s.dtype == "bf16" else 4
    d, hq, hkv, f = s.d_model, s.n_heads * s.d_head, s.n_kv_heads * s.d_head, s.d_ffn
    kv, rest = 2 * d * hkv, 2 * d * hq + 3 * d * f
    full, tail = S * N * (s.n_layers - 1), S * L if last else 0
    flops = 2.0 * ((full + S * N) * kv + (full + tail) * rest) + 4.0 * hq * keys * (full + tail)
    nbytes = size * (s.n_layers * kv + (s.n_layers - (0 if last else 1)) * rest) + S * N * d * size
    if head:
        flops += 2.0 * S * L * s.vocab * d
        nbytes += s.vocab * d * size + S * L * 8
    return float(nbytes), flops


def work(case):
    s, path = _shape(case), case["path"]
    B, P, L, K = case["B"], case["prompt"], case["L"], case["K"]
    N = P + case["gen"]
    row = 2 * s.n_kv_heads * s.d_head * s.n_layers * 2        # bytes of a position's keys and values
    if path == "decide":
        return {"bytes": float(B * (4 * N * (K + 2) + 8 * L * (K + 1) + 5 * L + 12 + K)), "flops": float(B * K * L * (L + K))}
    if path == "prefill":
        nbytes, flops = _call(s, B, P, L, (P + L) / 2, head=False, last=False)
        return {"bytes": nbytes + B * P * row, "flops": flops}
    if path == "cached":
        held = P + case["gen"] / 2                            # the active block is anywhere in the generated part
        one, two = _call(s, B, L, L, held + L), _call(s, B * K, L, L, held + L)
        return {"bytes": one[0] + two[0] + 2 * B * held * row, "flops": one[1] + two[1]}
    one = _call(s, B, N, L, N)
    two = _call(s, B * K, L, L, N) if path == "approx" else _call(s, B * K, N, L, N)
    more = 2 * B * (N - L) * row if path == "approx" else 0
    return {"bytes": one[0] + two[0] + more, "flops": one[1] + two[1]}


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / 1e15


def tolerance(case):
    # decisions on given tables are whole numbers and the same everywhere
    if case["path"] == "decide":
        return "exact"
    # fp32 sums in another order: 1e-6 in the confidences
    if case["model"] == "tiny":
        return {"rel": 1e-5, "differ": 0.0}
    # bf16 operands: with other kernels of the same precision (the library's plain ones) keys and values move by 0.54 %,
    # confidences by 0.5 - 1.2 %; a near tie in the order of the confidences then swaps two positions of a sequence here and
    # there (0.4 % of the tokens of a batch at most)
    return {"rel": 0.02 if case["path"] == "prefill" else 0.03, "differ": 0.01}
