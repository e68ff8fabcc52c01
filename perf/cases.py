"""The work that the framework is timed on: pruned prefill layers from 512 to 131072 tokens, a whole prefill with the
Preserve/Slim schedule, one decoded token's layer, and the scoring / selection / compaction calls on their own.

Shapes are the repository's workloads (paper_2508_06447_amd/inputs.py): the LLaMA-3.1-8B-shaped and Qwen2.5-7B-shaped
layers in bf16 and the small fp32 layer.  Weights are N(0, 0.02^2) and hidden states N(0, 1) with 1 % of the tokens four
times as large.  As in a trained model, some blocks of the prompt are about what the local window is about: their rows
and the window's share a direction, and the Query and Key projections of a head group are correlated, so these blocks
score higher and the retained set does not hang on the last bit of a score.
"""
from __future__ import annotations

import ctypes
import math

import torch

import paper_2508_06447_amd as slim
from paper_2508_06447_amd import inputs

# family -> the workload that has its shapes (hidden, heads, ffn, rope, biases)
FAMILY = {"llama": inputs.WORKLOADS["cfg3"], "qwen": inputs.WORKLOADS["cfg6"], "small": inputs.WORKLOADS["cfg1"]}
RESPONSE_ROOM = 64                     # rows a decoding program keeps free behind the response tokens it has


def listed():
    return [
        # the small fp32 layer: what someone runs to check numbers, and the smallest call of the library
        dict(name="small_fp32_layer", kind="layer", family="small", tokens=512, block=16, window=32, keep=0.5, gains=True),
        # a layer behind the last pruning layer of a 32k prefill: 8 blocks left, nothing dropped
        dict(name="layer_512", kind="layer", family="llama", tokens=512, block=64, window=64, keep=1.0, gains=False),
        # an ordinary prompt whose length is no multiple of anything, with the model's own RMSNorm gains
        dict(name="layer_2983_gains", kind="layer", family="llama", tokens=2983, block=64, window=64, keep=0.5, gains=True),
        # the 8k, 32k and 128k pruning layers of the benchmark (gains folded into the weights, as a server keeps them)
        dict(name="layer_8192", kind="layer", family="llama", tokens=8192, block=64, window=64, keep=0.5, gains=False),
        dict(name="layer_32768", kind="layer", family="llama", tokens=32768, block=64, window=64, keep=0.3, gains=False),
        dict(name="layer_131072", kind="layer", family="llama", tokens=131072, block=128, window=128, keep=0.2, gains=False),
        # the second model family: 7 query heads per kv head, biases, feature counts that are no multiple of 256
        dict(name="qwen_layer_32768", kind="layer", family="qwen", tokens=32768, block=64, window=64, keep=0.375, gains=False),
        # a whole prefill of a 4k prompt: 16 layers, pruning at layers 4, 8 and 12 down to two blocks
        dict(name="prefill_4096_16_layers", kind="model", family="llama", tokens=4096, layers=16, window=64),
        # one decoded token's layer: 8k active prompt tokens; and the whole of a 32k prompt behind a longer answer
        dict(name="decode_128_blocks", kind="decode", family="llama", slots=128, response=16),
        dict(name="decode_512_blocks", kind="decode", family="llama", slots=512, response=301),
        # a decoding step's choice of blocks from the stored unit keys (window = the last 4 tokens, the paper's)
        dict(name="decode_choice_32768", kind="choice", family="llama", tokens=32768, window=4, keep=0.25),
        # scoring, selection and compaction for a program that has Query and Key states of its own
        dict(name="prune_32768", kind="prune", family="llama", tokens=32768, window=64, keep=0.3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "model", "decode", "decode", "choice", "prune", "small"])
    family = rng.choice(["llama", "llama", "qwen"])
    if kind == "small":
        return dict(kind="layer", family="small", tokens=_log(rng, 128, 1024), block=16, window=32, keep=round(rng.uniform(0.2, 1.0), 3),
                    gains=True)
    if kind == "layer":
        c = dict(kind="layer", family=family, tokens=_log(rng, 200, 98304), block=rng.choice([64, 64, 128]),
                 window=rng.choice([4, 64, 64, 128]), keep=rng.choice([1.0, round(rng.uniform(0.125, 0.75), 3)]),
                 gains=rng.choice([False, False, True]))
        most = work(listed()[5])["flops"]
        while work(c)["flops"] > 0.9 * most:
            c["tokens"] = c["tokens"] * 2 // 3
        return c
    if kind == "model":
        return dict(kind="model", family=family, tokens=_log(rng, 1024, 6144), layers=rng.choice([8, 12]), window=rng.choice([4, 64]))
    if kind == "decode":
        return dict(kind="decode", family="llama", slots=_log(rng, 8, 512), response=_log(rng, 1, 1500))
    return dict(kind=kind, family=family, tokens=_log(rng, 2048, 131072), window=rng.choice([4, 16, 64]), keep=round(rng.uniform(0.1, 0.6), 3))


def _schedule(case):
    """Pruning at a quarter, half and three quarters of the layers, to 50 %, 25 % and 12.5 % of the incoming blocks."""
    L = case["layers"]
    return slim.schedule_keep_counts(case["tokens"], 64, L, {L // 4: 0.5, L // 2: 0.25, 3 * L // 4: 0.125})


class _Draw:
    """Seeded tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.host = torch.Generator()
        self.host.manual_seed(seed)

    def normal(self, *shape, std=1.0, dtype=torch.bfloat16):
        t = torch.empty(*shape, dtype=dtype, device="cuda")
        return t.normal_(0.0, std, generator=self.g)

    def some(self, n, k):
        """k of n indices."""
        return torch.randperm(n, generator=self.host)[:k]


def _weights(d, wl, dtype, gains):
    qd, kvd, Hd, F = wl.n_q_heads * wl.head_dim, wl.n_kv_heads * wl.head_dim, wl.hidden, wl.ffn
    w = dict(wk=d.normal(kvd, Hd, std=0.02, dtype=dtype), wv=d.normal(kvd, Hd, std=0.02, dtype=dtype),
             wo=d.normal(Hd, qd, std=0.02, dtype=dtype), w_gate=d.normal(F, Hd, std=0.02, dtype=dtype),
             w_up=d.normal(F, Hd, std=0.02, dtype=dtype), w_down=d.normal(Hd, F, std=0.02, dtype=dtype))
    group = wl.n_q_heads // wl.n_kv_heads
    of_key = w["wk"].view(wl.n_kv_heads, 1, wl.head_dim, Hd).expand(-1, group, -1, -1).reshape(qd, Hd)
    w["wq"] = (0.8 * of_key + d.normal(qd, Hd, std=0.6 * 0.02, dtype=dtype)).to(dtype)
    if wl.qkv_bias:
        w.update(bq=d.normal(qd, std=0.5, dtype=dtype), bk=d.normal(kvd, std=0.5, dtype=dtype), bv=d.normal(kvd, std=0.5, dtype=dtype))
    if gains:
        w.update(g_attn=1 + d.normal(Hd, std=0.1, dtype=dtype), g_ffn=1 + d.normal(Hd, std=0.1, dtype=dtype))
    return w


def _relevance(d, n_tokens, block, window, keeps):
    """Per token: how much of the window's direction its row has.  keeps: block counts of the successive prunings, largest
    first; the first and the last block and those under the window are in every set."""
    nb = slim.n_blocks(n_tokens, block)
    always = {0} | set(range(max(0, (n_tokens - window) // block), nb))
    order = sorted(always) + [int(b) for b in d.some(nb, nb) if int(b) not in always]
    level = torch.zeros(nb)
    for k in keeps:
        level[order[:max(k, len(always))]] += 1.0
    rows = level.repeat_interleave(block)[:n_tokens].clone()
    rows[max(0, n_tokens - window):] = max(1.0, float(level.max()))
    return rows.cuda()


def _hidden(d, n_tokens, hidden, rows, dtype):
    x = d.normal(n_tokens, hidden, dtype=dtype)
    direction = d.normal(hidden, dtype=dtype)
    x.addcmul_(rows.to(dtype)[:, None], direction[None, :])
    x[d.some(n_tokens, max(1, n_tokens // 100)).cuda()] *= 4.0
    return x


def _shape(wl, block, window, dtype):
    return slim.make_shape(wl.hidden, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.ffn, block, wl.unit, window, dtype, wl.rope_theta,
                           wl.rms_eps)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    d, wl, lib = _Draw(seed), FAMILY[case["family"]], slim.load_library()
    dtype = torch.float32 if wl.dtype == "fp32" else torch.bfloat16
    Hq, Hkv, hd = wl.n_q_heads, wl.n_kv_heads, wl.head_dim
    N = case.get("tokens")
    if case["kind"] == "layer":
        nb = slim.n_blocks(N, case["block"])
        keep = inputs.keep_count(case["keep"], nb)
        rows = _relevance(d, N, case["block"], min(case["window"], N), [keep] if keep < nb else [])
        shape = _shape(wl, case["block"], case["window"], dtype)
        return dict(kind="layer", shape=shape, weights=_weights(d, wl, dtype, case["gains"]), keep=keep,
                    x=_hidden(d, N, wl.hidden, rows, dtype), pos=torch.arange(N, dtype=torch.int32, device="cuda"),
                    workspace=_bytes(slim.pruned_layer_workspace_bytes(shape, N, keep)))
    if case["kind"] == "model":
        keeps = _schedule(case)
        rows = _relevance(d, N, 64, min(case["window"], N), [k for k in keeps if k])
        shape = _shape(wl, 64, case["window"], dtype)
        need = lib.slim_prefill_model_workspace_bytes(ctypes.byref(shape), len(keeps), (ctypes.c_int * len(keeps))(*keeps), N)
        return dict(kind="model", shape=shape, keeps=keeps, x=_hidden(d, N, wl.hidden, rows, dtype),
                    weights=[_weights(d, wl, dtype, False) for _ in range(case["layers"])],
                    pos=torch.arange(N, dtype=torch.int32, device="cuda"), workspace=_bytes(need))
    if case["kind"] == "decode":
        slots, resp, block = case["slots"], case["response"], 64
        nb = 4 * slots                                    # a quarter of the prompt's blocks is active
        prompt = nb * block - 27                          # the last one is short
        held = torch.cat([torch.tensor([nb - 1]), d.some(nb - 1, slots - 1)])[torch.randperm(slots, generator=d.host)]
        room = RESPONSE_ROOM + resp
        shape = _shape(wl, block, 64, dtype)
        return dict(kind="decode", shape=shape, weights=_weights(d, wl, dtype, False), x=d.normal(wl.hidden, dtype=dtype),
                    pool=d.normal(slots, 2, block, Hkv, hd, dtype=dtype), held=held.to(torch.int32).cuda(), prompt=prompt,
                    k=d.normal(room, Hkv, hd, dtype=dtype), v=d.normal(room, Hkv, hd, dtype=dtype), response=resp,
                    workspace=_bytes(lib.slim_decode_layer_workspace_bytes(ctypes.byref(shape), slots, resp)))
    # Query and Key states of a program's own: the keys of the relevant blocks lean towards the window's queries
    nb = slim.n_blocks(N, 64)
    keep = inputs.keep_count(case["keep"], nb)
    about = d.normal(Hkv, 1, hd)
    q = (d.normal(case["window"], Hkv, Hq // Hkv, hd) + about).reshape(case["window"], Hq, hd)
    k = d.normal(N, Hkv, hd)
    k.addcmul_(0.5 * _relevance(d, N, 64, 1, [keep]).to(dtype)[:, None, None], about.view(1, Hkv, hd))
    state = dict(kind=case["kind"], q=q, keep=keep, n=N, Hkv=Hkv, kept=torch.empty(keep, dtype=torch.int32, device="cuda"),
                 scores=torch.empty(nb, dtype=torch.float32, device="cuda"), workspace=_bytes(lib.slim_score_blocks_workspace_bytes(Hkv, hd)))
    if case["kind"] == "choice":
        return dict(state, units=slim.slim_unit_keys(k, 64, wl.unit))
    return dict(state, k=k, x=d.normal(N, wl.hidden), unit=wl.unit)


def run(s):
    if s["kind"] == "layer":
        return slim.slim_pruned_layer(s["shape"], s["weights"], s["x"], s["pos"], s["keep"], workspace=s["workspace"])
    if s["kind"] == "model":
        return slim.slim_prefill_model(s["shape"], s["weights"], s["x"], s["pos"], s["keeps"], workspace=s["workspace"])
    if s["kind"] == "decode":
        x, q = slim.slim_decode_layer(s["shape"], s["weights"], s["x"], s["prompt"] + s["response"], s["pool"], s["held"], s["prompt"], s["k"],
                                      s["v"], s["response"], workspace=s["workspace"])
        return x, q, s["k"], s["v"]
    if s["kind"] == "choice":
        scores = slim.slim_score_blocks_from_unit_keys(s["q"], s["units"], s["n"], s["Hkv"], 64, 8, scores=s["scores"], workspace=s["workspace"])
        return scores, slim.slim_select_topk_blocks(scores, s["keep"], kept=s["kept"])
    scores = slim.slim_score_blocks(s["q"], s["k"], 64, s["unit"], scores=s["scores"], workspace=s["workspace"])
    kept = slim.slim_select_topk_blocks(scores, s["keep"], kept=s["kept"])
    x, pos = slim.slim_compact_tokens(s["x"], kept, 64)
    keys, _ = slim.slim_compact_tokens(s["k"], kept, 64, want_pos=False)
    return scores, kept, x, pos, keys


def _layer_work(wl, N, n, window, es):
    """(flops, weight bytes) of one layer: keys of all N tokens, everything else of the n that continue."""
    qd, kvd, Hd, F = wl.n_q_heads * wl.head_dim, wl.n_kv_heads * wl.head_dim, wl.hidden, wl.ffn
    flops = 2 * N * Hd * kvd + 2 * n * Hd * (qd + kvd) + 2 * n * n * qd + 2 * n * qd * Hd + 6 * n * Hd * F
    if n < N:
        flops += 2 * min(window, N) * Hd * qd + 2 * N * kvd
    return flops, es * (2 * qd * Hd + 2 * kvd * Hd + 3 * Hd * F)


def work(case):
    wl = FAMILY[case["family"]]
    es = 4 if wl.dtype == "fp32" else 2
    qd, kvd, Hd, F = wl.n_q_heads * wl.head_dim, wl.n_kv_heads * wl.head_dim, wl.hidden, wl.ffn
    if case["kind"] == "layer":
        N, block = case["tokens"], case["block"]
        n = inputs.kept_tokens(N, block, inputs.keep_count(case["keep"], slim.n_blocks(N, block)))
        flops, weights = _layer_work(wl, N, n, case["window"], es)
        return {"bytes": weights + (N + n) * (Hd * es + 4), "flops": flops}
    if case["kind"] == "model":
        n, flops, weights = case["tokens"], 0, 0
        for k in _schedule(case):
            m = inputs.kept_tokens(n, 64, k) if k else n
            f, w = _layer_work(wl, n, m, case["window"], es)
            flops, weights, n = flops + f, weights + w, m
        return {"bytes": weights + (case["tokens"] + n) * (Hd * es + 4), "flops": flops}
    if case["kind"] == "decode":
        keys = case["slots"] * 64 - 27 + case["response"] + 1
        weights = 2 * qd * Hd + 2 * kvd * Hd + 3 * Hd * F
        return {"bytes": es * (weights + 2 * keys * kvd + 2 * Hd + qd), "flops": 2 * weights + 4 * keys * qd}
    N = case["tokens"]
    keep = inputs.keep_count(case["keep"], slim.n_blocks(N, 64))
    n = inputs.kept_tokens(N, 64, keep)
    if case["kind"] == "choice":
        return {"bytes": 4 * slim.n_blocks(N, 64) * (64 // wl.unit) * kvd + es * case["window"] * qd, "flops": 2 * N // wl.unit * kvd}
    return {"bytes": es * (N * kvd + case["window"] * qd + 2 * n * (Hd + kvd)) + 4 * n, "flops": 2 * N * kvd}


def tolerance(case):
    """What two correct implementations may differ by.  Measured against the same path in float32 from the same inputs: bf16
    layers rel 3.6e-3 to 4.3e-3, max 0.02; 16 layers rel 1.3e-2, max 0.07; the scores on given keys and the fp32 layer 2e-7."""
    if case["kind"] in ("choice", "prune") or FAMILY[case["family"]].dtype == "fp32":
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] == "model":
        return {"rel": 0.03, "max": 0.3}
    return {"rel": 1.5e-2, "max": 0.1}
