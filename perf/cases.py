"""The calls of this library whose speed is followed, through the public binding only.

Three kinds of call, as a serving program makes them:

  first_token  a new sequence: open, prompt pass, first step, its logits, close (time to first token)
  decode       open, prompted sequences that go on: `steps` steps in one call, the last step's logits
  response     a whole short response: open, prompt, all its steps (drawn by the sampler), close

Models are the repository's workloads.  `depth` = 4 takes a quarter of the layers and of the
vocabulary at full width: every launch keeps its size and its share of the step, and inputs are made
four times as fast; `depth` = 1 is the whole model.  Tokens are teacher-forced, so that two
implementations see the same inputs at every step whatever the last bits of their logits are.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import workloads as wl
from paper_2603_09215_amd import Spark

ROOM = 4096   # tokens a decoding sequence may grow before its program starts a new one


def listed():
    return [
        # the smallest model, fp32, a whole sampled response: launches and latency, no bandwidth
        dict(name="tiny_fp32_response", kind="response", model="tiny", depth=1, batch=1, lo=16, hi=16, steps=64, aligned=False),
        # the headline: one speaker, whole model, 512-token prompt, greedy
        dict(name="step_b1_decode", kind="decode", model="step_audio_2_mini", depth=1, batch=1, lo=512, hi=512, steps=12, aligned=False),
        # one speaker on the other backbone, one whole 13 : 26 cycle (flushes of four rows)
        dict(name="glm_b1_decode", kind="decode", model="glm_4_voice", depth=4, batch=1, lo=1024, hi=1024, steps=39, aligned=False),
        # a few speakers: three rows below the exit layer, up to nine above
        dict(name="step_b3_decode", kind="decode", model="step_audio_2_mini", depth=4, batch=3, lo=256, hi=2048, steps=12, aligned=False),
        # a small batch
        dict(name="step_b8_decode", kind="decode", model="step_audio_2_mini", depth=4, batch=8, lo=256, hi=2048, steps=12, aligned=False),
        # the batched workload: 32 speakers, mixed schedules, every step has full-depth rows
        dict(name="step_b32_decode", kind="decode", model="step_audio_2_mini", depth=4, batch=32, lo=256, hi=2048, steps=12, aligned=False),
        # a larger one whose schedules are aligned: 48 rows below, flushes of up to 144 above
        dict(name="step_b48_aligned", kind="decode", model="step_audio_2_mini", depth=4, batch=48, lo=256, hi=2048, steps=12, aligned=True),
        # long contexts
        dict(name="glm_b8_long_decode", kind="decode", model="glm_4_voice", depth=4, batch=8, lo=8192, hi=8192, steps=12, aligned=False),
        # a short utterance, ragged
        dict(name="step_first_token_37", kind="first_token", model="step_audio_2_mini", depth=4, batch=1, lo=37, hi=37, steps=1, aligned=False),
        # the benchmark prompts of the two backbones, the first on the whole model
        dict(name="step_first_token_512", kind="first_token", model="step_audio_2_mini", depth=1, batch=1, lo=512, hi=512, steps=1, aligned=False),
        dict(name="glm_first_token_1024", kind="first_token", model="glm_4_voice", depth=4, batch=1, lo=1024, hi=1024, steps=1, aligned=False),
        # a long recording
        dict(name="glm_first_token_8192", kind="first_token", model="glm_4_voice", depth=4, batch=1, lo=8192, hi=8192, steps=1, aligned=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "first_token", "first_token", "response"])
    if kind == "response":
        return dict(kind=kind, model="tiny", depth=1, batch=_log_int(rng, 1, 8), lo=_log_int(rng, 1, 64), hi=64,
                    steps=rng.randint(16, 64), aligned=bool(rng.getrandbits(1)))
    model = rng.choice(["step_audio_2_mini", "glm_4_voice"])
    if kind == "first_token":
        n = _log_int(rng, 2, 8192)
        return dict(kind=kind, model=model, depth=4, batch=1, lo=n, hi=n, steps=1, aligned=False)
    batch = _log_int(rng, 1, 48)
    # prompts: a quarter of the longest to the longest, 64 k prompt tokens in all at most
    hi = _log_int(rng, 64, min(8192, 65536 // batch))
    return dict(kind=kind, model=model, depth=4, batch=batch, lo=max(1, hi // 4), hi=hi, steps=rng.randint(6, 18),
                aligned=bool(rng.getrandbits(1)))


# ---------------------------------------------------------------------------------- model and inputs

def _model(case):
    w = wl.WORKLOADS[case["model"]]
    s, q = w.shape, int(case["depth"])
    if q == 1:
        return w, s, w.schedule
    shape = s.replace(n_layers=s.n_layers // q, vocab_text=s.vocab_text // q, vocab_speech=s.vocab_speech // q)
    return w, shape, w.schedule.replace(exit_layer=w.schedule.exit_layer // q)


_weights = {}   # the one model that is loaded: a program has one, and opens its contexts on it


def _load(case):
    _, shape, _ = _model(case)
    if shape not in _weights:
        _weights.clear()
        torch.cuda.empty_cache()
        if shape.dtype == wl.DTYPE_BF16:
            _weights[shape] = wl.make_weights_on_device(shape, seed=0)
        else:
            _weights[shape] = wl.make_weights(shape, seed=0)
        gain = torch.Generator().manual_seed(5)
        for name in wl.GAIN_TENSORS:   # gains as a trained model has them, away from 1
            t = 1.0 + 0.1 * torch.randn(wl.tensor_shapes(shape)[name], generator=gain, dtype=torch.float32)
            _weights[shape][name] = t.cuda() if shape.dtype == wl.DTYPE_BF16 else t.numpy()
    return _weights[shape]


def _inputs(case, seed):
    """prompts, cycle offsets, and the ids forced at the `steps` positions of one call"""
    w, shape, sched = _model(case)
    n, steps = case["batch"], case["steps"]
    lens = [int(x) for x in wl.make_prompt_lengths(n, case["lo"], case["hi"], seed=3)]
    prompts = [wl.make_prompt(shape, m, seed=1000 * seed + i, ids=w.prompt_ids) for i, m in enumerate(lens)]
    cyc = sched.n_text + sched.n_speech
    offsets = [0 if case["aligned"] else i % cyc for i in range(n)]
    forced = np.stack([wl.make_forced_stream(shape, steps, sched.n_text, sched.n_speech, off, seed=1000 * seed + 500 + i)
                       for i, off in enumerate(offsets)], axis=1)
    words = np.random.Generator(np.random.Philox(seed)).integers(0, 2 ** 64, size=(steps, n), dtype=np.uint64)
    return prompts, offsets, forced, words


def _open(state):
    state["ids"] = [state["spark"].seq_open(off) for off in state["offsets"]]
    for sid, p in zip(state["ids"], state["prompts"]):
        state["spark"].prefill(sid, p)
    state["left"] = state["room"]


def _close(state):
    for sid in state["ids"]:
        state["spark"].seq_close(sid)


def prepare(case, seed):
    _, shape, sched = _model(case)
    prompts, offsets, forced, words = _inputs(case, seed)
    room = ROOM if case["kind"] == "decode" else case["steps"]
    longest = (max(len(p) for p in prompts) + room + 63) // 64 * 64
    spark = Spark(shape, sched, _load(case), max_batch=case["batch"], max_seq_len=longest, kv_page_tokens=64)
    state = dict(spark=spark, kind=case["kind"], steps=case["steps"], prompts=prompts, offsets=offsets, forced=forced,
                 words=words, room=room)
    if case["kind"] == "response":
        spark.set_sampling(0.7, 0.9)
    if case["kind"] == "decode":
        _open(state)
    return state


def run(state):
    spark, steps = state["spark"], state["steps"]
    if state["kind"] == "decode":
        if state["left"] < steps:   # the responses have reached their longest: the next ones begin
            _close(state)
            _open(state)
        _, depth = spark.decode(steps, state["ids"], state["forced"])
        state["left"] -= steps
        return {"logits": [spark.get_logits(s)[0] for s in state["ids"]], "depth": depth}
    _open(state)
    if state["kind"] == "response":
        token, depth = spark.decode_sampled(steps, state["ids"], state["words"], state["forced"])
    else:
        token, depth = spark.step(state["ids"], state["forced"][0])
    out = {"logits": [spark.get_logits(s)[0] for s in state["ids"]], "depth": depth}
    if state["kind"] == "response":
        out["token"] = token   # fp32: a draw does not hang on the last bits of a 16-bit cache entry
    _close(state)
    return out


# ---------------------------------------------------------------------------------- what a pass needs

def _full_depth(sched, n_layers, g, offset, j):
    """(is text, runs full depth) of generated token g after j speech tokens"""
    slot = (g + offset) % (sched.n_text + sched.n_speech)
    if slot < sched.n_text:
        return True, True
    index = j if sched.scope == wl.SCOPE_STREAM else slot - sched.n_text
    return False, sched.exit_layer == n_layers or sched.period_k <= 1 or index % sched.period_k == sched.phase


def work(case):
    _, s, sched = _model(case)
    esz = 2 if s.dtype == wl.DTYPE_BF16 else 4
    d, F, V, L, e = s.d_model, s.d_ffn, s.vocab, s.n_layers, sched.exit_layer
    q, kv = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    layer = (q + 2 * kv) * d + d * q + 3 * F * d       # weight elements
    lens = [int(x) for x in wl.make_prompt_lengths(case["batch"], case["lo"], case["hi"], seed=3)]
    nbytes = flops = 0.0

    def rows(layers, pos_count, ctx_sum):   # projections and attention of rows through some layers
        return layers * (2.0 * layer * pos_count + 4.0 * q * ctx_sum)

    if case["kind"] != "decode":            # the prompt: every weight once, every K/V entry written once
        for n in lens:
            if n > 1:
                nbytes += L * layer * esz + (n - 1) * (d * esz + L * 2 * kv * esz)
                flops += rows(L, n - 1, (n - 1) * n / 2)
    offsets = [0 if case["aligned"] else i % (sched.n_text + sched.n_speech) for i in range(len(lens))]
    j, pend, ctx = [0] * len(lens), [0] * len(lens), [n - 1 for n in lens]
    for g in range(case["steps"]):
        any_full = any_ee = False
        up_kv = 0
        for i in range(len(lens)):
            text, full = _full_depth(sched, L, g, offsets[i], j[i])
            j[i] += not text
            ctx[i] += 1
            flops += rows(e, 1, ctx[i]) + 2.0 * V * d
            if full:
                any_full = True
                flops += rows(L - e, pend[i] + 1, (pend[i] + 1) * ctx[i])
                up_kv += ctx[i]
                pend[i] = 0
            else:
                any_ee = True
                flops += 2.0 * d * d
                pend[i] += 1
        nbytes += e * (layer * esz + sum(ctx) * 2 * kv * esz)
        if any_full:
            nbytes += (L - e) * (layer * esz + up_kv * 2 * kv * esz) + V * d * esz
        if any_ee:
            nbytes += (V + d) * d * esz
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured against exact(): 2.3e-7 .. 2.5e-7 (fp32 throughout: sums of up to 1024 terms in some
    # order, through four layers).  Two correct implementations are 1.4 times that apart; four times
    # that, with some room for another draw.
    if wl.WORKLOADS[case["model"]].shape.dtype == wl.DTYPE_FP32:
        return {"rel": 2e-6, "max": 3e-5, "differ": 0.0}
    # bf16 cache: another order of the fp32 sums makes some entries round to the neighbouring bf16
    # value, and the layers above carry that on.  Measured against exact(): 1.4e-4 .. 6.7e-4 at a
    # quarter of the depth, 6.7e-4 .. 9.7e-4 at the whole of it.
    return {"rel": 5e-3, "max": 0.04, "differ": 0.0}


# ---------------------------------------------------------------------------------- the same in 64 bits

EXACT_TOKENS = 17000   # prompt tokens that exact() runs: the first sequences of a large batch


def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, angle):   # x [T][heads][hd], pairs (i, i + hd/2)
    h = x.shape[-1] // 2
    c, s = torch.cos(angle)[:, None, :], torch.sin(angle)[:, None, :]
    return torch.cat([x[..., :h] * c - x[..., h:] * s, x[..., h:] * c + x[..., :h] * s], -1)


def _forward(shape, sched, W, ids, depth):
    """logits of the last of `ids`, run to `depth` layers: a plain causal transformer in 64 bits.  Early
    exits change nothing else: the cache that a step sees is complete in every layer it runs.  What the
    library defines as its formats is kept: cache entries rounded to the model's type, rotary angles
    formed in 32 bits."""
    dev = "cuda:0"
    get = lambda name, l=None: torch.as_tensor(W[name] if l is None else W[name][l]).to(dev)   # noqa: E731
    T, hd, nq, nkv, d = len(ids), shape.head_dim, shape.n_q_heads, shape.n_kv_heads, shape.d_model
    grp = nq // nkv
    store = (lambda t: t.bfloat16().double()) if shape.dtype == wl.DTYPE_BF16 else (lambda t: t.float().double())
    inv = torch.tensor([shape.rope_base ** (-2.0 * i / hd) for i in range(hd // 2)], dtype=torch.float64, device=dev).float()
    angle = (torch.arange(T, device=dev).float()[:, None] * inv[None, :]).double()
    x = torch.as_tensor(W["embed"][ids] if isinstance(W["embed"], np.ndarray)
                        else W["embed"][torch.as_tensor(ids, device=dev).long()]).to(dev).double()
    at = torch.arange(T, device=dev)
    for l in range(depth):
        n = _norm(x, get("attn_norm", l), shape.rms_eps)
        qh = _rope((n @ get("wq", l).double().T).view(T, nq, hd), angle)
        kh = store(_rope((n @ get("wk", l).double().T).view(T, nkv, hd), angle))
        vh = store((n @ get("wv", l).double().T).view(T, nkv, hd))
        out = torch.empty(T, nq, hd, dtype=torch.float64, device=dev)
        for r0 in range(0, T, 1024):
            r1 = min(T, r0 + 1024)
            for h in range(nq):
                sc = (qh[r0:r1, h] @ kh[:r1, h // grp].T) / math.sqrt(hd)
                sc.masked_fill_(at[None, :r1] > at[r0:r1, None], -math.inf)
                out[r0:r1, h] = torch.softmax(sc, -1) @ vh[:r1, h // grp]
        x = x + out.view(T, nq * hd) @ get("wo", l).double().T
        n = _norm(x, get("mlp_norm", l), shape.rms_eps)
        for r0 in range(0, T, 2048):
            m = n[r0:r0 + 2048]
            a = torch.nn.functional.silu(m @ get("wg", l).double().T) * (m @ get("wu", l).double().T)
            x[r0:r0 + 2048] += a @ get("wd", l).double().T
    h = x[-1]
    if depth == shape.n_layers:
        return (get("lm_head").double() @ _norm(h, get("final_norm"), shape.rms_eps)).cpu().numpy()
    u = h + get("lens_a").double() @ h + get("lens_b").double()
    return (get("lens_head").double() @ _norm(u, get("lens_norm"), shape.rms_eps)).cpu().numpy()


def exact(case, seed):
    _, shape, sched = _model(case)
    W = _load(case)
    prompts, offsets, forced, _ = _inputs(case, seed)
    logits, depth, spent = [], np.zeros((case["steps"], case["batch"]), dtype=np.int32), 0
    for i, (p, off) in enumerate(zip(prompts, offsets)):
        j = 0
        for g in range(case["steps"]):
            text, full = _full_depth(sched, shape.n_layers, g, off, j)
            j += not text
            depth[g, i] = shape.n_layers if full else sched.exit_layer
        spent += len(p)
        if i and spent > EXACT_TOKENS:
            logits.append(None)
            continue
        ids = np.concatenate([p, forced[:-1, i]]).astype(np.int64)
        logits.append(_forward(shape, sched, W, ids, int(depth[-1, i])))
    out = {"logits": logits, "depth": depth if case["kind"] != "first_token" else depth[0]}
    if case["kind"] == "response":
        out["token"] = None
    return out
