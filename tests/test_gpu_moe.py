"""GPU parity of the mixture-of-experts FFN: router, selection, grouped expert GEMMs and the weighted sum, every
iteration against the oracle. The oracle is fed the engine's routing (a half-precision router logit may order two nearly
equal experts differently from an exact one) and reports its own: the two must agree wherever the oracle's margin is
clear of the engine's arithmetic, and the logits must then agree to the stated tolerance."""
import numpy as np
import pytest

import synth
from tests import parity
from tests.test_gpu_parity import setup, sampled, _fixed_prompts

pytestmark = pytest.mark.gpu


def free_run_tokens(lib, cfg, eng, blob, reqs):
    ev, trace, st = parity.run_engine(lib, cfg, eng, blob, reqs)
    assert st["free_blocks"] == eng["kv_num_blocks"] and st["committed_blocks"] == 0 and st["n_running"] == 0
    out = {}
    for rid, idx, tok in sorted((int(x["request_id"]), int(x["index"]), int(x["token"])) for x in ev):
        out.setdefault(rid, []).append(tok)
    return out


def test_moe_stepwise(lib):
    """Eight experts, two active: prefill and decode iterations of the mini mix, every other request sampling."""
    cfg, eng, raw, blob = setup("mini_moe", 141)
    reqs = sampled(synth.make_workload("mini", cfg["vocab"], 241, n_requests=9), 141)
    toks = {}
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, reqs, rtol=2e-2, tokens_out=toks)
    print("mini_moe: worst relative logit error", worst)
    # the free-running loop (one window, HIP graph) produces the same tokens as the iteration-by-iteration run
    assert free_run_tokens(lib, cfg, eng, blob, reqs) == toks


@pytest.mark.parametrize("prompts,max_new", [([530, 260, 7, 90], 4), ([33] * 40 + [17] * 8, 5), ([100, 60, 30], 4)])
def test_moe16_stepwise(lib, prompts, max_new):
    """Sixteen experts, four active. Long prompts: an expert gets well over 64 tokens of a prefill iteration (the tiled
    GEMM schedules, groups that start at every multiple of 16). 48 short requests: decode iterations of 48 tokens,
    12 per expert on average (independent waves with one to four token blocks per expert, some experts empty). Three
    prompts of 190 tokens in all: the router GEMM on its 65..256-token schedule."""
    cfg, eng, raw, blob = setup("mini_moe16", 142)
    reqs = _fixed_prompts(cfg, prompts, max_new, 242)
    toks = {}
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, reqs, rtol=2e-2, tokens_out=toks)
    print("mini_moe16", len(prompts), "requests: worst relative logit error", worst)
    assert free_run_tokens(lib, cfg, eng, blob, reqs) == toks


def test_moe_on_the_chain_without_merge_kernels(lib):
    """Bit 7 of the tuning word: the launcher always runs the kernel chain without the decode attention's merge kernels,
    whose scheduler step hands out whole contexts (it does so by itself only once many sequences run). Contexts of up to
    540 tokens, two rounds of KV blocks per item."""
    cfg, eng, raw, blob = setup("mini_moe16", 143)
    reqs = _fixed_prompts(cfg, [530, 260, 7, 90], 4, 243)
    toks = {}
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, reqs, rtol=2e-2, tokens_out=toks, tune=0x80)
    print("mini_moe16 on the short chain: worst relative logit error", worst)


@pytest.mark.parametrize("mode", ["chunked_prefill", "preemption", "prefix_cache"])
def test_moe_with_the_scheduler_extensions(lib, mode):
    """The routed FFN under the scheduler's optional modes (mixed prefill + decode iterations with a budget of 48 tokens; on-demand
    KV growth with preemptions in a pool of 14 blocks; prefix caching on prompts with common heads): the modes change
    which tokens an iteration carries, not what the model computes for them."""
    cfg, eng, raw, blob = setup("mini_moe", 145)
    reqs = synth.make_workload("mini", cfg["vocab"], 245, n_requests=10)
    if mode == "chunked_prefill":
        eng = dict(eng, chunked_prefill=True, max_prefill_tokens=48)
    elif mode == "preemption":
        eng = dict(eng, preemption=True, kv_num_blocks=14, max_batch=4)
        for r in reqs:
            r["prompt"] = r["prompt"][:40]
    else:
        eng = dict(eng, prefix_cache=True, kv_num_blocks=40)
        reqs = synth.with_shared_prefixes(reqs, cfg["vocab"], 345, n_prefixes=2, prefix_len=(16, 50), share=0.8)
        reqs = [dict(r, prompt=r["prompt"][: eng["max_seq_len"] - r["max_new_tokens"] - 1]) for r in reqs]
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, reqs, rtol=2e-2)
    print("mini_moe with", mode, ": worst relative logit error", worst)


def test_moe_one_expert_equals_dense(lib):
    """One expert, one active: the routed path must reproduce the dense FFN of the same matrices (its weight is 1)."""
    cfg, eng, raw, blob = setup("mini_moe", 143)
    cfg1 = dict(cfg, n_experts=1, n_active=1)
    raw1 = synth.make_weights(cfg1, 143, gain_jitter=0.1)
    dense = {k: v for k, v in cfg1.items() if k not in ("n_experts", "n_active")}
    rawd = {k: (v[0] if k.endswith((".wg", ".wu", ".wd")) else v) for k, v in raw1.items() if not k.endswith(".wr")}
    reqs = synth.make_workload("mini", cfg["vocab"], 243, n_requests=6)
    a = free_run_tokens(lib, cfg1, eng, synth.pack_blob(cfg1, raw1), reqs)
    b = free_run_tokens(lib, dense, eng, synth.pack_blob(dense, rawd), reqs)
    same = sum(x == y for r in a for x, y in zip(a[r], b[r]))
    total = sum(len(v) for v in a.values())
    print("one expert vs dense: equal tokens", same, "of", total)
    assert a.keys() == b.keys() and same >= 0.9 * total   # different GEMM schedules round differently: greedy near-ties may flip


def test_moe_rejects_bad_configs(lib):
    cfg, eng, raw, blob = setup("mini_moe", 144)
    for bad in (dict(n_active=0), dict(n_active=9), dict(n_experts=300)):
        with pytest.raises(lib.BlinkError):
            lib.Engine(dict(cfg, **bad), eng, blob)
    with pytest.raises(lib.BlinkError):
        lib.Engine(dict(cfg, dtype=0), eng, blob)


def test_few_expert_items_are_spread_over_the_chip(lib):
    """Gate/up and down of one token at the widths of moe_30b_a3b: 192 and 256 wave items of eight experts. 24 and 15 us a
    launch with the items spread over the compute units; 50 and 25 with eight neighbouring items in every workgroup (39 and 26 with four)."""
    cfg = dict(synth.model_config("moe_30b_a3b"), n_layers=1, vocab=1024)
    eng = dict(synth.engine_config("moe_30b_a3b"), kv_num_blocks=64, max_batch=2, max_seq_len=256, max_prefill_tokens=256, ring_slots=4)
    d, hd, E = cfg["d_model"], cfg["head_dim"], cfg["n_experts"]
    layer = 2 * 4 * d + 2 * ((cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * hd * d + d * cfg["n_q_heads"] * hd + E * d + E * 3 * d * cfg["d_ffn"])
    e = lib.Engine(cfg, eng, np.zeros(2 * 2 * cfg["vocab"] * d + layer + 4 * d, dtype=np.uint8))
    us = {}
    try:
        e.submit(np.zeros(4, np.int32), 200)
        e.run(1)
        e.wait()
        for phase in (18, 19):
            e.time_phase(phase)
            e.run(20)
            e.wait()
            us[phase] = float(np.min(e.phase_times_ms()[:20])) * 1e3
    finally:
        e.shutdown()
    print("one token: gate/up %.1f us, down %.1f us" % (us[18], us[19]))
    assert us[18] < 34 and us[19] < 22
