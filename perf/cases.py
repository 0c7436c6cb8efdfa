"""The work that this serving engine is timed on: closed sets of requests, prefill iterations, decode iterations and mixed
iterations, each through blink_submit / blink_run / blink_wait / blink_poll_outputs as a serving program calls them.

Models. The layers have the shapes of the repository's configurations: llama3_8b (bf16, grouped-query attention), churn (bf16,
multi-head attention), moe_30b_a3b (mixture of experts), tiny and sched_stress (fp32). The two large ones are cut to a few
layers and to a vocabulary in about that proportion, so that making an engine takes about a second; a layer's work and the share
that the layers have of a pass are those of the whole model. Matrices are N(0, 1/fan_in), so that activations keep
the size they have in a trained model. The head is tied to the embeddings, shifted by one token id: the next token is then
decided by a wide margin, as a trained model decides most of its tokens, and two correct engines that round differently
emit the same tokens, so that what they compute can be compared number by number. The checkpoint is the same for every seed;
the requests are drawn from it.

Kinds of pass:
  set      a closed set of requests from submission to the last token
  prefill  prompts submitted, one prefill iteration, first tokens
  decode   the next `iters` decode iterations of a batch that is already running
  mixed    chunked prefill: a prompt arrives while a batch decodes; iterations until its first token, each with all decodes

Outputs: every token of the pass, and the logits of its last iteration.
"""
import functools
import math

import numpy as np
import torch

import paper_2604_07609_amd as blink

MODELS = {
    "tiny": dict(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, d_ffn=1024, vocab=4096, dtype=0,
                 rms_eps=1e-5, rope_theta=10000.0),
    "sched_stress": dict(n_layers=1, d_model=128, n_q_heads=2, n_kv_heads=2, head_dim=64, d_ffn=512, vocab=8192, dtype=0,
                         rms_eps=1e-5, rope_theta=10000.0),
    "churn": dict(n_layers=8, d_model=1024, n_q_heads=16, n_kv_heads=16, head_dim=64, d_ffn=4096, vocab=32000, dtype=1,
                  rms_eps=1e-5, rope_theta=10000.0),
    # four of the 32 layers of the 8B shape
    "llama3_8b": dict(n_layers=4, d_model=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ffn=14336, vocab=8192, dtype=1,
                      rms_eps=1e-5, rope_theta=500000.0),
    # two of the 48 layers of the 30B mixture of experts
    "moe_30b_a3b": dict(n_layers=2, d_model=2048, n_q_heads=32, n_kv_heads=4, head_dim=128, d_ffn=768, n_experts=128, n_active=8,
                        vocab=6144, dtype=1, rms_eps=1e-6, rope_theta=1000000.0),
}
# the sampling parameters of the workloads: temperature, top-k, top-p
GREEDY = (0.0, 0, 1.0)
SAMPLED = (0.8, 50, 0.9)
SAMPLING = {"tiny": GREEDY, "sched_stress": GREEDY, "churn": GREEDY, "llama3_8b": SAMPLED, "moe_30b_a3b": SAMPLED}
BUDGET = 8192          # prompt tokens of a prefill iteration, as in every configuration
DECODE_BUDGET = 2048   # output tokens a decoding request may still emit: far more than a measurement asks for


def listed():
    return [
        # the smallest engine: eight short chat turns on the fp32 model, latency and launches only
        dict(name="tiny_set", kind="set", model="tiny", n=8, lo=16, hi=64, out=32),
        # the scheduler's workload: 512 short sequences on a one-layer model, the scheduler step and the sampler dominate
        dict(name="stress_decode", kind="decode", model="sched_stress", n=512, lo=4, hi=32, iters=8),
        # a small bf16 model serving a set to completion: multi-head attention, prefill and decode
        dict(name="churn_set", kind="set", model="churn", n=16, lo=64, hi=700, out=64),
        # time to first token of one ordinary prompt
        dict(name="prefill_509", kind="prefill", model="llama3_8b", n=1, lo=509, hi=509),
        # the prefill iteration of a saturated engine: two or three ragged prompts, about 1700 tokens
        dict(name="prefill_1700", kind="prefill", model="llama3_8b", n=3, lo=350, hi=790),
        # the largest prefill iteration: two prompts that fill the token budget
        dict(name="prefill_8k", kind="prefill", model="llama3_8b", n=2, lo=3900, hi=4096),
        # decode of a lightly loaded, a half loaded (odd batch) and a full engine at the contexts of the chat workload
        dict(name="decode_16", kind="decode", model="llama3_8b", n=16, lo=300, hi=1500, iters=16),
        dict(name="decode_61", kind="decode", model="llama3_8b", n=61, lo=300, hi=1500, iters=8),
        dict(name="decode_256", kind="decode", model="llama3_8b", n=256, lo=300, hi=1500, iters=8),
        # chunked prefill with 2048 tokens per iteration: a long prompt beside a decoding batch
        dict(name="mixed_192", kind="mixed", model="llama3_8b", n=192, lo=300, hi=1500, prompt=3500, budget=2048),
        # the mixture of experts: decode and prefill
        dict(name="moe_decode_96", kind="decode", model="moe_30b_a3b", n=96, lo=200, hi=1000, iters=8),
        dict(name="moe_prefill_2k", kind="prefill", model="moe_30b_a3b", n=4, lo=400, hi=650),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["set", "prefill", "prefill", "prefill", "decode", "decode", "decode", "mixed"])
    if kind == "set":
        model = rng.choice(["tiny", "churn"])
        lo = rng.randint(5, 100)
        hi = min(lo + rng.randint(0, 600), 128 - 33 if model == "tiny" else 900)
        return dict(kind=kind, model=model, n=_log_int(rng, 1, 8 if model == "tiny" else 20), lo=min(lo, hi), hi=hi, out=rng.randint(4, 32 if model == "tiny" else 64))
    if kind == "prefill":
        model = rng.choice(["llama3_8b", "llama3_8b", "moe_30b_a3b", "churn"])
        total = _log_int(rng, 20, 8192 if model == "llama3_8b" else 4000 if model == "moe_30b_a3b" else 2048)
        n = rng.randint(max(1, -(-total // 4096)), max(2, min(8, total // 16)))
        mean = total // n
        lo = max(1, int(mean * rng.uniform(0.5, 1.0)))
        return dict(kind=kind, model=model, n=n, lo=lo, hi=max(lo, min(2 * mean - lo, 4096, 8192 // n)))
    if kind == "mixed":
        budget = rng.choice([512, 1024, 2048])
        n = _log_int(rng, 4, min(200, budget // 2))
        lo = rng.randint(30, 500)
        return dict(kind=kind, model="llama3_8b", n=n, lo=lo, hi=lo + rng.randint(0, 1000), prompt=_log_int(rng, 100, 3500), budget=budget)
    model = rng.choice(["llama3_8b", "llama3_8b", "llama3_8b", "moe_30b_a3b", "churn", "sched_stress"])
    n = _log_int(rng, 1, {"llama3_8b": 256, "moe_30b_a3b": 128, "churn": 64, "sched_stress": 512}[model])
    lo = 4 if model == "sched_stress" else rng.randint(8, 400)
    hi = 32 if model == "sched_stress" else lo + rng.randint(0, 1100)
    return dict(kind=kind, model=model, n=n, lo=lo, hi=hi, iters=rng.randint(4, 8))


# ---- the checkpoint ------------------------------------------------------------------------------------------------
def _tensors(m):
    """(name, tensor on the GPU) in blob order; bf16 models' matrices in bf16, gains in fp32."""
    d, hd, nq, nkv, F, V, E, L = (m["d_model"], m["head_dim"], m["n_q_heads"], m["n_kv_heads"], m["d_ffn"], m["vocab"],
                                  m.get("n_experts", 0), m["n_layers"])
    g = torch.Generator(device="cuda").manual_seed(20260)
    wt = torch.bfloat16 if m["dtype"] == 1 else torch.float32

    def normal(*shape, std):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std

    def matrix(*shape):
        return normal(*shape, std=shape[-1] ** -0.5).to(wt)

    def gain():
        return 1.0 + normal(d, std=0.1)

    embed = normal(V, d, std=math.sqrt(L)).to(wt)
    yield "embed", embed
    for l in range(L):
        yield f"{l}.g1", gain()
        yield f"{l}.wq", matrix(nq * hd, d)
        yield f"{l}.wk", matrix(nkv * hd, d)
        yield f"{l}.wv", matrix(nkv * hd, d)
        yield f"{l}.wo", matrix(d, nq * hd)
        yield f"{l}.g2", gain()
        if E:
            yield f"{l}.wr", matrix(E, d)
        yield f"{l}.wg", matrix(*((E, F, d) if E else (F, d)))
        yield f"{l}.wu", matrix(*((E, F, d) if E else (F, d)))
        yield f"{l}.wd", matrix(*((E, d, F) if E else (d, F)))
    yield "gf", gain()
    e = embed.float()
    head = normal(V, d, std=d ** -0.5) + 16.0 * d ** -0.5 * (e / e.norm(dim=1, keepdim=True)).roll(1, 0)
    yield "lm", head.to(wt)


@functools.lru_cache(maxsize=1)
def _blob(model):
    """The checkpoint as one host array, as a loader would have it."""
    parts = []
    for _, t in _tensors(MODELS[model]):
        parts.append(t.reshape(-1).view(torch.uint8).cpu().numpy())
    return np.concatenate(parts)


# ---- requests and engine --------------------------------------------------------------------------------------------
def _lengths(case, seed):
    return np.random.default_rng(seed).integers(case["lo"], case["hi"] + 1, case["n"])


def _prompts(case, seed):
    rng = np.random.default_rng([seed, 1])
    V = MODELS[case["model"]]["vocab"]
    return [rng.integers(0, V, int(n)).astype(np.int32) for n in _lengths(case, seed)]


def _new_prompt(case, seed):
    return np.random.default_rng([seed, 2]).integers(0, MODELS[case["model"]]["vocab"], case["prompt"]).astype(np.int32)


class _State:
    def __init__(self, case, seed):
        self.case, self.prompts, self.seed = case, _prompts(case, seed), seed
        self.model = MODELS[case["model"]]
        self.sampling = SAMPLING[case["model"]]
        kind, n = case["kind"], case["n"]
        out = {"set": case.get("out", 0), "prefill": 1}.get(kind, DECODE_BUDGET)
        longest = max(len(p) for p in self.prompts) + out
        blocks = sum((len(p) + out + 15) // 16 for p in self.prompts)
        budget, slots = BUDGET, n
        if kind == "mixed":
            self.prompt = _new_prompt(case, seed)
            longest = max(longest, len(self.prompt) + 1)
            blocks += len(self.prompt) // 16 + 1
            budget, slots = case["budget"], n + 1
        engine = dict(kv_block_size=16, kv_num_blocks=int(blocks), max_batch=slots, max_seq_len=(longest + 15) // 16 * 16,
                      max_prefill_tokens=budget, ring_slots=1 << max(4, (2 * slots - 1).bit_length()), eos_token_id=-1,
                      chunked_prefill=kind == "mixed")
        self.out = out
        self.eng = blink.Engine(self.model, engine, _blob(case["model"]), flags=blink.FLAG_KEEP_LOGITS)
        self.used = 0
        if kind in ("decode", "mixed"):
            self.start_batch()

    def submit(self, prompt, out, seed):
        t, k, p = self.sampling
        return self.eng.submit(prompt, out, t, k, p, seed)

    def start_batch(self):
        """The batch that the pass finds running: every request prefilled, its first token out."""
        ids = [self.submit(p, self.out, self.seed * 1000 + i) for i, p in enumerate(self.prompts)]
        got = 0
        while got < len(ids):
            self.eng.run(1)
            self.eng.wait()
            ev = self.eng.drain()
            got += int(np.count_nonzero(ev["flags"] & blink.EVENT_FIRST))
        self.used = 1

    def iterations(self):
        if self.case["kind"] == "mixed":
            return -(-self.case["prompt"] // (self.case["budget"] - self.case["n"]))
        if self.case["kind"] == "decode":
            return self.case["iters"]
        prefills, room = 0, 0      # prompts are admitted in order while they fit the iteration
        for p in self.prompts:
            if len(p) > room:
                prefills, room = prefills + 1, BUDGET
            room -= len(p)
        return prefills + self.out - 1

    def room(self, iters):
        """Starts the batch again once its requests are nearly used up (the first of a chunked start is up to 300 tokens ahead)."""
        if self.used + iters + 300 >= self.out:
            while self.eng.stats()["n_running"]:
                self.eng.run(16)
                self.eng.wait()
                self.eng.drain()
            self.start_batch()
        self.used += iters

    def result(self, ev, rows):
        ev = ev[np.lexsort((ev["index"], ev["request_id"]))]
        v = self.model["vocab"]
        logits = self.eng.debug_read(blink.DBG.LOGITS, np.float32, max_bytes=4 * rows * v).reshape(rows, v)
        return {"tokens": ev["token"].astype(np.int64), "logits": logits}

    def __del__(self):
        eng = getattr(self, "eng", None)
        if eng is not None:
            eng.shutdown()


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    case, eng = state.case, state.eng
    kind, n = case["kind"], case["n"]
    rows, iters = n, state.iterations()
    if kind in ("set", "prefill"):
        for i, p in enumerate(state.prompts):
            state.submit(p, state.out, state.seed * 1000 + i)
    else:
        state.room(iters)
        if kind == "mixed":
            state.submit(state.prompt, 1, state.seed * 1000 + 999)
            rows = n + 1
    eng.run(iters)
    eng.wait()
    return state.result(eng.drain(1 << 14), rows)


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def work(case):
    m = MODELS[case["model"]]
    d, hd, nq, nkv, F, V, E, L = (m["d_model"], m["head_dim"], m["n_q_heads"], m["n_kv_heads"], m["d_ffn"], m["vocab"],
                                  m.get("n_experts", 0), m["n_layers"])
    es = 2 if m["dtype"] == 1 else 4
    n, mean = case["n"], (case["lo"] + case["hi"]) / 2
    attn_w = d * (nq + 2 * nkv) * hd + d * nq * hd

    def layer(tokens):
        """(weights read, multiply-adds per token) of a layer's matrices for an iteration of that many tokens."""
        if not E:
            return attn_w + 3 * d * F, attn_w + 3 * d * F
        k = m["n_active"]
        distinct = E * (1 - (1 - k / E) ** tokens)
        return attn_w + d * E + distinct * 3 * d * F, attn_w + d * E + k * 3 * d * F

    def iteration(tokens, rows, kv_tokens, pairs):
        """tokens through the layers, rows through the head, kv_tokens read from the cache, (query, key) pairs per head."""
        w, mac = layer(tokens)
        nbytes = L * (w * es + (kv_tokens + tokens) * 2 * nkv * hd * es) + V * d * es + tokens * d * es + rows * V * 4
        flops = 2.0 * (L * (tokens * mac + pairs * nq * 2 * hd) + rows * V * d)
        return np.array([nbytes, flops])

    var = (case["hi"] - case["lo"]) ** 2 / 12.0
    prompt_pairs = n * (mean * mean + var + mean) / 2
    if case["kind"] == "prefill":
        got = iteration(n * mean, n, 0, prompt_pairs)
    elif case["kind"] == "decode":
        got = sum(iteration(n, n, n * (mean + i), n * (mean + i + 1)) for i in range(case["iters"]))
    elif case["kind"] == "set":
        got = iteration(n * mean, n, 0, prompt_pairs) + sum(iteration(n, n, n * (mean + i), n * (mean + i + 1)) for i in range(case["out"] - 1))
    else:
        room, left, at, got, i = case["budget"] - n, case["prompt"], 0, 0, 0
        while left:
            c = min(room, left)
            got = got + iteration(n + c, n + (c == left), n * (mean + i) + at, n * (mean + i + 1) + c * at + c * (c + 1) / 2)
            at, left, i = at + c, left - c, i + 1
    return {"bytes": float(got[0]), "flops": float(got[1])}


def tolerance(case):
    # about four times the distance from the 64-bit result: fp32 sums 4e-7 to 6e-7; bf16 weights with half-precision activations
    # 2.4e-4 to 5e-4 (a rounding that falls the other way in one layer travels through the rest)
    return {"rel": 2.5e-6} if MODELS[case["model"]]["dtype"] == 0 else {"rel": 2e-3}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------
def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * theta ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _norm(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g


def _ffn(h, W, l, m):
    silu = torch.nn.functional.silu
    if not m.get("n_experts"):
        return (silu(h @ W[f"{l}.wg"].T) * (h @ W[f"{l}.wu"].T)) @ W[f"{l}.wd"].T
    top, idx = (h @ W[f"{l}.wr"].T).topk(m["n_active"], dim=-1)
    p, out = torch.softmax(top, -1), torch.zeros_like(h)
    for e in range(m["n_experts"]):
        t, k = (idx == e).nonzero(as_tuple=True)
        if len(t):
            x = h[t]
            y = (silu(x @ W[f"{l}.wg"][e].double().T) * (x @ W[f"{l}.wu"][e].double().T)) @ W[f"{l}.wd"][e].double().T
            out.index_add_(0, t, y * p[t, k][:, None])
    return out


def _last_logits(m, seqs):
    """Logits behind the last token of every sequence."""
    nq, nkv, hd, L, eps = m["n_q_heads"], m["n_kv_heads"], m["head_dim"], m["n_layers"], m["rms_eps"]
    G = nq // nkv
    cu = np.cumsum([0] + [len(s) for s in seqs])
    last = torch.tensor(cu[1:] - 1, device="cuda")
    ids = torch.from_numpy(np.concatenate(seqs).astype(np.int64)).cuda()
    pos = torch.from_numpy(np.concatenate([np.arange(len(s)) for s in seqs])).cuda()
    W, tensors, x = {}, _tensors(m), None
    for name, t in tensors:
        if name == "embed":
            x = t[ids].double()
            continue
        W[name] = t if t.dim() == 3 else t.double()     # the experts' stacks are widened one expert at a time
        l, what = name.split(".") if "." in name else (None, name)
        if what == "wd":                                # the layer is complete
            l = int(l)
            final = l + 1 == L
            q = torch.empty(len(ids), nq * hd, device="cuda", dtype=torch.float64)
            k, v = (torch.empty(len(ids), nkv * hd, device="cuda", dtype=torch.float64) for _ in range(2))
            for s in range(0, len(ids), 8192):
                h = _norm(x[s:s + 8192], W[f"{l}.g1"], eps)
                q[s:s + 8192], k[s:s + 8192], v[s:s + 8192] = h @ W[f"{l}.wq"].T, h @ W[f"{l}.wk"].T, h @ W[f"{l}.wv"].T
            att = torch.empty(len(seqs) if final else len(ids), nq * hd, device="cuda", dtype=torch.float64)
            for i in range(len(seqs)):
                a, b = int(cu[i]), int(cu[i + 1])
                kk = _rope(k[a:b].view(-1, nkv, hd), pos[a:b], m["rope_theta"]).transpose(0, 1)            # [nkv][n][hd]
                vv = v[a:b].view(-1, nkv, hd).transpose(0, 1).contiguous()
                for q0 in range(b - 1 if final else a, b, 1024):
                    q1 = min(q0 + 1024, b)
                    qq = _rope(q[q0:q1].view(-1, nq, hd), pos[q0:q1], m["rope_theta"]).view(q1 - q0, nkv, G, hd)
                    mask = pos[a:b][None, :] > pos[q0:q1][:, None]
                    for j in range(nkv):
                        s = (qq[:, j].reshape(-1, hd) @ kk[j].T.contiguous() / math.sqrt(hd)).view(q1 - q0, G, -1)
                        o = torch.softmax(s.masked_fill(mask[:, None], -math.inf), -1).view((q1 - q0) * G, -1) @ vv[j]
                        at = slice(i, i + 1) if final else slice(q0, q1)
                        att[at, j * G * hd:(j + 1) * G * hd] = o.view(q1 - q0, G * hd)
            del q, k, v
            if final:
                x = x[last]
            for s in range(0, len(x), 8192):
                y = x[s:s + 8192] + att[s:s + 8192] @ W[f"{l}.wo"].T
                x[s:s + 8192] = y + _ffn(_norm(y, W[f"{l}.g2"], eps), W, l, m)
            W = {}
    return _norm(x, W["gf"], eps) @ W["lm"].T


def _emitted(case, seed):
    """Output tokens that every request of the batch has when the pass begins. With chunked prefill the batch is started in mixed
    iterations: the requests whose prompts are done decode while the rest of the budget goes to the others, in order."""
    lens = [int(x) for x in _lengths(case, seed)]
    if case["kind"] != "mixed":
        return np.full(len(lens), 1 if case["kind"] == "decode" else 0)
    left, out = list(lens), np.zeros(len(lens), dtype=np.int64)
    while out.min() == 0:
        room = case["budget"] - int((out > 0).sum())
        out[out > 0] += 1
        for i in range(len(lens)):
            c = min(room, left[i])
            if left[i] and c:
                left[i], room = left[i] - c, room - c
                out[i] = left[i] == 0
    return out


def exact(case, seed):
    m = MODELS[case["model"]]
    steps = {"set": case.get("out"), "prefill": 1, "decode": case.get("iters"),
             "mixed": -(-case.get("prompt", 0) // (case.get("budget", 1 << 30) - case["n"]))}[case["kind"]]
    seqs, toks = [], []
    for p, had in zip(_prompts(case, seed), _emitted(case, seed)):
        out = (p[-1] + 1 + np.arange(had + steps)) % m["vocab"]    # every next token is the current one plus one: the wide margin of the head
        seqs.append(np.concatenate([p, out[:-1]]))
        toks.append(out[had:])
    if case["kind"] == "mixed":
        seqs.append(_new_prompt(case, seed))
        toks.append((seqs[-1][-1:] + 1) % m["vocab"])
    return {"tokens": np.concatenate(toks).astype(np.int64), "logits": _last_logits(m, seqs)}
