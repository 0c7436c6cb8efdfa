"""GPU parity of the kernels that share operand tiles through LDS, at the sizes where a tile can go wrong: prompt attention
(shared KV tiles), the bf16 tile GEMMs in every tile shape, and the fp32 GEMMs in both of their schedules. Every iteration
against the oracle."""
import numpy as np
import pytest

import synth
from tests import parity
from tests.test_gpu_parity import setup, _fixed_prompts

pytestmark = pytest.mark.gpu

# A bf16 model's activations are rounded to half precision (2^-11) at about four places per layer; over two or three layers
# that is sqrt(12) * 2^-11 = 1.7e-3 of a logit's own scale, and at most twice that at the worst of the few thousand
# logits of a run. One key, one k-step or one row too many or too few moves a logit by several per cent.
RTOL = 4e-3


@pytest.mark.parametrize("chunked", [False, True])
@pytest.mark.parametrize("name", ["mini_churn", "mini_kv8", "mini_gqa", "mini_gqa128", "mini_g6", "mini_g8"])
def test_prompt_attention_with_shared_kv_tiles(lib, name, chunked):
    """1, 2, 3, 4, 6 and 8 q heads per kv head (so 128, 64 or 32 queries per work item), head dimensions 64 and 128. Prompts one
    below, at and above the item, the 64-key step and the 16-token block, one shorter than a query tile; with chunked
    prefill, chunks that begin in the middle of a block and items beside decoding sequences."""
    cfg, eng, raw, blob = setup(name, 61)
    prompts = [33, 5, 127, 130, 64, 321, 509]
    eng = dict(eng, max_batch=7, max_seq_len=540, kv_num_blocks=110, max_prefill_tokens=2048, ring_slots=16)
    if chunked:
        eng.update(chunked_prefill=True, max_prefill_tokens=203)
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 3, 261), rtol=RTOL)
    print(name, "chunked" if chunked else "whole prompts", "worst relative logit error", worst)


def ragged(dtype, **more):
    cfg = dict(synth.model_config("mini_gqa"), d_model=160, n_q_heads=3, n_kv_heads=1, d_ffn=352, vocab=1003, dtype=dtype, **more)
    raw = synth.make_weights(cfg, 62, gain_jitter=0.1)
    return cfg, raw, synth.pack_blob(cfg, raw)


@pytest.mark.parametrize("model", ["dense", "moe"])
@pytest.mark.parametrize("shape", [0, 1, 2, 3, 4, 6, 7])
def test_tile_gemms_in_every_shape(lib, shape, model):
    """Bits 12-14 of the tuning word force the tile shape: 64x64, 128x64, 128x128, 256x128, 256x192, 256x256 (0: the
    automatic choice). K of 5 and 11 steps of 32 (the last pair is half padding), rows that end inside every tile, 65 to
    330 tokens in an iteration, expert groups from none to several tiles."""
    if model == "moe":
        cfg, eng, raw, blob = setup("mini_moe16", 62)
    else:
        eng = synth.engine_config("mini_gqa")
        cfg, raw, blob = ragged(1)
    eng = dict(eng, max_batch=6, max_seq_len=400, kv_num_blocks=96, max_prefill_tokens=512, ring_slots=16)
    for prompts in ([65], [257, 73]):
        worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 2, 262), rtol=RTOL, tune=shape << 12)
        print(model, "shape", shape, "prompts", prompts, "worst relative logit error", worst)


@pytest.mark.parametrize("prompts", [[1], [17], [33, 15], [509, 16], [511, 500, 490]])
def test_fp32_gemms_in_both_schedules(lib, prompts):
    """A workgroup's waves share a tile's K (few tiles) or take a tile each (QKV and gate/up at 525 tokens, every GEMM
    over the prompt at 1501): one token, one more than a tile of them, ragged last tiles of tokens and of rows. Tolerance: the
    rounding of sums of up to 352 products (sqrt(352) * 2^-24) in each of some ten GEMMs in a row."""
    cfg, raw, blob = ragged(0)
    eng = dict(synth.engine_config("mini_gqa"), max_batch=6, max_seq_len=540, kv_num_blocks=110, max_prefill_tokens=2048, ring_slots=16)
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 2, 263), rtol=1e-5)
    print("fp32", prompts, "worst relative logit error", worst)
