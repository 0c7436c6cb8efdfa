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


# bits 16-19 of the tuning word: 15 forces prompt attention with shared KV tiles, 3 the kernel with a query tile per wave; 0: the scheduler's choice
SHARED_TILES, WAVE_PER_TILE = 15 << 16, 3 << 16


@pytest.mark.parametrize("kernel", [SHARED_TILES, WAVE_PER_TILE])
@pytest.mark.parametrize("chunked", [False, True])
@pytest.mark.parametrize("name", ["mini_churn", "mini_kv8", "mini_gqa", "mini_gqa128", "mini_g6", "mini_g8"])
def test_prompt_attention_with_shared_kv_tiles(lib, name, chunked, kernel):
    """1, 2, 3, 4, 6 and 8 q heads per kv head (so 128, 64 or 32 queries per work item), head dimensions 64 and 128. Prompts one
    below, at and above the item, the 64-key step and the 16-token block, one shorter than a query tile; with chunked
    prefill, chunks that begin in the middle of a block and items beside decoding sequences. The kernel with a query tile per
    wave on the same prompts."""
    cfg, eng, raw, blob = setup(name, 61)
    prompts = [33, 5, 127, 130, 64, 321, 509]
    eng = dict(eng, max_batch=7, max_seq_len=540, kv_num_blocks=110, max_prefill_tokens=2048, ring_slots=16)
    if chunked:
        eng.update(chunked_prefill=True, max_prefill_tokens=203)
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 3, 261), rtol=RTOL, tune=kernel)
    print(name, "chunked" if chunked else "whole prompts", "worst relative logit error", worst)


@pytest.mark.parametrize("kernel", [0, SHARED_TILES, WAVE_PER_TILE])
def test_prompt_tails_behind_a_cached_head(lib, kernel):
    """32 q / 8 kv heads of 128: tails of 1 to 130 tokens behind a cached head of 1040 in one iteration, on every kernel and on the
    scheduler's choice."""
    cfg, eng, raw, blob = setup("mini_heads32", 64)
    tails = [1, 16, 17, 31, 32, 33, 64, 65, 130]
    eng = dict(eng, prefix_cache=True, max_batch=len(tails) + 1, max_seq_len=1200, kv_num_blocks=200, max_prefill_tokens=1060, ring_slots=16)
    rng = np.random.default_rng(64)
    head = rng.integers(0, cfg["vocab"], 1040).astype(np.int32)
    reqs = [dict(arrival_s=0.0, prompt=np.concatenate([head, rng.integers(0, cfg["vocab"], n).astype(np.int32)]), max_new_tokens=3,
                 temperature=0.0, top_k=0, top_p=1.0, seed=i) for i, n in enumerate([3] + tails)]
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, reqs, rtol=RTOL, tune=kernel)
    print("tails, tuning word", hex(kernel), "worst relative logit error", worst)


@pytest.mark.parametrize("heads", [(32, 8, 128), (16, 16, 64)])
def test_prompt_attention_takes_the_faster_kernel(lib, heads):
    """Launch times of both kernels and of the scheduler's choice: few queries behind a long context, where the keys of a query
    tile have to be split between waves (62 us against 147 for 64 queries behind 4096 tokens), and prompts from
    position 0, where the shared tiles win (85 against 137 at 2048 tokens). The choice may cost a quarter and 4 us more than the better one."""
    nq, nkv, hd = heads
    cfg = dict(synth.model_config("mini_heads32"), n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, n_layers=1)
    eng = dict(synth.engine_config("mini_heads32"), prefix_cache=True, max_batch=16, max_seq_len=4400, kv_num_blocks=4000, max_prefill_tokens=8192, ring_slots=32)
    blob = synth.pack_blob(cfg, synth.make_weights(cfg, 65))
    rng = np.random.default_rng(65)

    def prompt(n):
        return rng.integers(0, cfg["vocab"], n).astype(np.int32)

    heads_cached = [prompt(4100) for _ in range(4)]
    us = {}
    for kernel in (0, SHARED_TILES, WAVE_PER_TILE):
        e = lib.Engine(cfg, eng, blob, tune=kernel)
        try:
            for h in heads_cached:
                e.submit(h, 1)
                e.run(1)
                e.wait()
                e.drain()
            e.time_phase(4)
            for n, cached, tokens in ((1, 4096, 64), (4, 4096, 32), (1, 1024, 128), (1, 0, 2048), (3, 0, 700)):
                best = np.inf
                for rep in range(4):
                    for i in range(n):
                        e.submit(np.concatenate([heads_cached[i % 4][:cached], prompt(tokens)]), 1)
                    e.run(1)
                    e.wait()
                    e.drain()
                    best = min(best, float(e.phase_times_ms()[0]) * 1e3)
                us.setdefault((n, cached, tokens), []).append(best)
        finally:
            e.shutdown()
    for case, t in us.items():
        print(heads, "prompts, cached, tokens", case, "us: choice %.1f, shared %.1f, wave per tile %.1f" % tuple(t))
    assert all(t[0] < 1.25 * min(t[1:]) + 4.0 for t in us.values()), us


def ragged(dtype, d_model=160, **more):
    cfg = dict(synth.model_config("mini_gqa"), d_model=d_model, n_q_heads=3, n_kv_heads=1, d_ffn=352, vocab=1003, dtype=dtype, **more)
    raw = synth.make_weights(cfg, 62, gain_jitter=0.1)
    return cfg, raw, synth.pack_blob(cfg, raw)


def wide_engine(lib, tune=0):
    """Two layers of the llama3_8b widths, weights all zero: for launch times."""
    cfg = dict(synth.model_config("llama3_8b"), n_layers=2, vocab=1024)
    eng = dict(synth.engine_config("llama3_8b"), kv_num_blocks=600, max_batch=4, max_seq_len=8192, max_prefill_tokens=8192, ring_slots=8)
    d, hd = cfg["d_model"], cfg["head_dim"]
    layer = 2 * 4 * d + 2 * ((cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * hd * d + d * cfg["n_q_heads"] * hd + 3 * d * cfg["d_ffn"])
    return lib.Engine(cfg, eng, np.zeros(2 * 2 * cfg["vocab"] * d + cfg["n_layers"] * layer + 4 * d, dtype=np.uint8), tune=tune)


def test_the_tile_shape_chosen_is_about_the_fastest(lib):
    """QKV (6144 x 4096), the attention output projection (4096 x 4096) and down (4096 x 14336) at 100 to 8000 tokens with every shape forced and with the
    automatic choice, which may cost an eighth more than the best of them (with one set of constants for all epilogues
    it took 51 us against 39 for QKV at 100 tokens, 561 against 464 at 8000)."""
    us = {}
    for shape in (0, 1, 2, 3, 4, 6, 7):
        e = wide_engine(lib, tune=shape << 12)
        try:
            for phase in (2, 5, 8):
                e.time_phase(phase)
                for tokens in (100, 300, 1000, 2048, 4000, 8000):
                    best = np.inf
                    for rep in range(4):
                        e.submit(np.zeros(tokens, np.int32), 1)
                        e.run(1)
                        e.wait()
                        e.drain()
                        best = min(best, float(e.phase_times_ms()[0]) * 1e3 / 2)
                    us.setdefault((phase, tokens), []).append(best)
        finally:
            e.shutdown()
    for case, t in us.items():
        print("phase, tokens", case, "us: choice %.1f, shapes" % t[0], ["%.1f" % x for x in t[1:]])
    assert all(t[0] < 1.125 * min(t[1:]) for t in us.values()), us


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


@pytest.mark.parametrize("shape", [2, 3, 4, 6, 7])
def test_the_tile_shape_does_not_move_a_bit(lib, shape):
    """A mixture of experts chooses by the largest router logits, so the residual stream behind a prompt iteration has the same bits in every tile
    shape as with 64 x 64 tiles, which have another epilogue: 1900 tokens of four ragged prompts (a sum of squares that was
    contracted in another order moved some in a hundred tokens)."""
    cfg, eng, raw, blob = setup("mini_moe16", 62)
    eng = dict(eng, max_batch=6, max_seq_len=600, kv_num_blocks=160, max_prefill_tokens=2048, ring_slots=16)
    out = []
    for tune in (1 << 12, shape << 12):
        e = lib.Engine(cfg, eng, blob, tune=tune)
        try:
            for r in _fixed_prompts(cfg, [530, 477, 590, 303], 1, 268):
                e.submit(r["prompt"], 1)
            e.run(1)
            e.wait()
            out.append(e.debug_read(11, np.uint32).reshape(1900, cfg["d_model"]))
        finally:
            e.shutdown()
    assert (out[0] == out[1]).all(), "%d tokens differ" % (out[0] != out[1]).any(axis=1).sum()


@pytest.mark.parametrize("slices", [2, 3])
@pytest.mark.parametrize("shape", [1, 2, 3, 4])
def test_tile_gemms_with_k_in_slices(lib, shape, slices):
    """Bits 24-27 of the tuning word cut K of every tile of the QKV, attention output and down projections into slices, which the workgroup that
    comes last adds up: K of 3 and 6 pairs of k-steps (slices of one to three pairs, one of them half padding), 17 to 330 tokens and
    decode iterations, twice over (the counters are zeros again after every launch)."""
    cfg, raw, blob = ragged(1)
    eng = dict(synth.engine_config("mini_gqa"), max_batch=24, max_seq_len=400, kv_num_blocks=96, max_prefill_tokens=512, ring_slots=64)
    for prompts in ([65], [257, 73], [61], [3] * 19):
        worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 3, 264), rtol=RTOL, tune=shape << 12 | slices << 24)
        print("shape", shape, "slices", slices, "prompts", prompts, "worst relative logit error", worst)


@pytest.mark.parametrize("prompts", [[1], [17], [33, 15], [509, 16], [511, 500, 490], [3] * 270])
def test_fp32_gemms_in_both_schedules(lib, prompts):
    """A workgroup's waves share a tile's K (few tiles) or, from 1025 tiles of 16 x 16 on, take 32 x 32 each with the whole of K: gate/up (44 row
    tiles) at 525 tokens, every GEMM of a layer (20, 14, 44 and 14 row tiles) at 1501, the LM head (63, the last row pair half
    and the last tile partly empty) over 270 sequences. One token, one more than a tile of them, ragged last tiles of tokens and
    of rows. Tolerance: the rounding of sums of up to 352 products (sqrt(352) * 2^-24) in each of some ten GEMMs in a row."""
    cfg, raw, blob = ragged(0, d_model=224)
    n = len(prompts)
    eng = dict(synth.engine_config("mini_gqa"), max_batch=max(6, n), max_seq_len=540, kv_num_blocks=max(110, 2 * n), max_prefill_tokens=2048,
               ring_slots=16 if n < 16 else 512)
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 2, 263), rtol=1e-5)
    print("fp32", prompts if n < 16 else n, "worst relative logit error", worst)


@pytest.mark.parametrize("heads", [(2, 2, 64), (4, 2, 64), (3, 1, 64), (8, 1, 64), (6, 1, 64), (2, 2, 128), (3, 1, 128), (8, 2, 128)])
def test_fp32_attention(lib, heads):
    """1, 2, 3, 4, 6 and 8 q heads per kv head of 64 and 128 dimensions (whole and partly filled groups of heads): contexts of one
    key, around a block of 16, around the four blocks of the four waves (64), around a step of every wave (256 and 128 keys) and behind it; prompts, then
    decode iterations that cross those edges. Tolerance: the rounding of sums of up to 600 products (sqrt(600) * 2^-24) in each of some ten steps."""
    nq, nkv, hd = heads
    cfg = dict(synth.model_config("mini_gqa"), d_model=96, n_q_heads=nq, n_kv_heads=nkv, head_dim=hd, d_ffn=192, vocab=1003, dtype=0)
    raw = synth.make_weights(cfg, 66, gain_jitter=0.1)
    prompts = [1, 15, 16, 62, 65, 126, 254, 257, 530]
    eng = dict(synth.engine_config("mini_gqa"), max_batch=len(prompts), max_seq_len=560, kv_num_blocks=140, max_prefill_tokens=2048, ring_slots=16)
    worst = parity.stepwise_check(lib, cfg, eng, raw, synth.pack_blob(cfg, raw), _fixed_prompts(cfg, prompts, 5, 266), rtol=1.5e-5)
    print("fp32 attention", heads, "worst relative logit error", worst)


@pytest.mark.parametrize("name,prompts", [("mini_gqa128", [1030, 2070, 7, 511, 1023]), ("mini_gqa", [6300, 512, 40]), ("mini_kv8", [1030] * 24)])
def test_decode_attention_merges_chunks_itself(lib, name, prompts):
    """Bit 3 of the tuning word: always the chain without the merge kernel whose attention kernel merges a context's chunks. One chunk, two
    to thirteen, contexts that grow by a chunk on the way, and more items than workgroups (24 sequences x 8 kv heads x 3 chunks)."""
    cfg, eng, raw, blob = setup(name, 67)
    blocks = sum((n + 20) // 16 + 1 for n in prompts)
    eng = dict(eng, max_batch=len(prompts), max_seq_len=max(prompts) + 16, kv_num_blocks=blocks, max_prefill_tokens=8192, ring_slots=32)
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 5, 267), rtol=RTOL, tune=0x8)
    print(name, "chunks merged in the attention kernel, worst relative logit error", worst)


@pytest.mark.parametrize("name,prompts", [("mini_gqa128", [1030, 2070, 4090, 6300, 7]), ("mini_gqa", [1030, 2070, 4090, 6300, 7]), ("mini_kv8", [2600] * 12)])
def test_where_chunks_are_merged_does_not_move_a_bit(lib, name, prompts):
    """The launcher chooses from a hint of the host, which is some iterations old, whether the attention kernel merges a context's chunks (bit 3
    of the tuning word: always) or a kernel behind it does (bit 5: always), so the two give the same bits: contexts of one to thirteen
    chunks, up to four of them in one batch of loads, more in several; logits of five decode iterations."""
    cfg, eng, raw, blob = setup(name, 67)
    blocks = sum((n + 20) // 16 + 1 for n in prompts)
    eng = dict(eng, max_batch=len(prompts), max_seq_len=max(prompts) + 16, kv_num_blocks=blocks, max_prefill_tokens=1 << 15, ring_slots=32)
    logits = []
    for tune in (0x20, 0x8, 0):
        e = lib.Engine(cfg, eng, blob, tune=tune, flags=lib.FLAG_KEEP_LOGITS)
        try:
            for r in _fixed_prompts(cfg, prompts, 6, 267):
                e.submit(r["prompt"], 6)
            rows = []
            for _ in range(6):
                e.run(1)
                e.wait()
                rows.append(e.debug_read(lib.DBG.LOGITS, np.uint32).reshape(len(prompts), cfg["vocab"]))
            logits.append(np.stack(rows))
        finally:
            e.shutdown()
    assert (logits[0][0] == logits[1][0]).all()
    for other in logits[1:]:
        assert (logits[0] == other).all(), "%d of %d rows differ" % ((logits[0] != other).any(axis=2).sum(), 6 * len(prompts))


def one_product_per_sum(cfg, seed):
    """Weights with which every sum over K has one term that is not zero, so that no order of summation shows: what an output projection
    adds to the residual stream is zero, and every row of gate, up, down and the LM head has a single element."""
    raw = synth.make_weights(cfg, seed, gain_jitter=0.1)
    rng = np.random.default_rng(seed)
    for name, w in raw.items():
        what = name.split(".")[-1]
        if what == "wo":
            w[:] = 0
        elif what in ("wg", "wu", "wd", "lm"):
            row = np.arange(w.shape[0])
            w[:] = 0
            w[row, rng.integers(0, w.shape[1], w.shape[0])] = synth.f32_to_bf16_bits(rng.uniform(0.5, 1.5, w.shape[0]).astype(np.float32))
    return raw


@pytest.mark.parametrize("tune", [0, 2, 0x40, 0x1000, 0x1040, 0x2000, 0x3000, 0x4000, 0x6000, 0x7000, 0x1000 | 2 << 24, 0x1040 | 2 << 24, 0x4000 | 2 << 24])
def test_every_residual_epilogue_sums_the_squares_in_one_order(lib, tune):
    """Without an order of summation over K to tell them apart the streaming schedule (one to four blocks of tokens), its and the tiles' epilogues
    tile by tile (bit 6), the tiles of every shape and K in slices give a token the same norm scales: the logits behind 64 last
    tokens, which the last of these scales multiplies, have the same bits in iterations of 1 to 704 tokens. (A sum of squares that was contracted
    in another order in some tile shapes moved two rows of the 64.)"""
    cfg = dict(synth.model_config("mini_gqa128"))
    blob = synth.pack_blob(cfg, one_product_per_sum(cfg, 69))
    eng = dict(synth.engine_config("mini_gqa128"), max_batch=64, max_seq_len=32, kv_num_blocks=128, max_prefill_tokens=1024, ring_slots=256)
    rng = np.random.default_rng(69)
    last = rng.integers(0, cfg["vocab"], 64)

    def logits(tune, shapes):
        """Of every (sequences, tokens of each), an iteration after the other."""
        e = lib.Engine(cfg, eng, blob, tune=tune, flags=lib.FLAG_KEEP_LOGITS)
        try:
            for first, n, each in shapes:
                for tok in last[first:first + n]:
                    e.submit(np.concatenate([rng.integers(0, cfg["vocab"], each - 1), [tok]]), 1)
                e.run(1)
                e.wait()
                assert len(e.drain()) == n
                yield e.debug_read(lib.DBG.LOGITS, np.uint32).reshape(n, cfg["vocab"])
        finally:
            e.shutdown()

    alone = np.concatenate(list(logits(0, [(i, 1, 1) for i in range(64)])))
    shapes = [(0, 1, 1), (0, 16, 1), (16, 33, 1), (3, 61, 1), (0, 64, 1), (0, 64, 2), (0, 64, 5), (0, 64, 11)]
    for (first, n, each), got in zip(shapes, logits(tune, shapes)):
        assert (got == alone[first:first + n]).all(), "%d x %d tokens: %d rows differ" % (n, each, (got != alone[first:first + n]).any(axis=1).sum())


@pytest.mark.parametrize("prompts", [[1], [40], [130], [530, 477]])
def test_epilogues_tile_by_tile_do_not_move_a_bit(lib, prompts):
    """Bit 6 of the tuning word: epilogues that load their operands tile by tile. The residual stream of a mixture of experts behind prompts that take the
    streaming schedule, its grid of 64 x 64 items and (forced) 64 x 64 tiles has the same bits with and without it: the rotary
    embedding and the sums of squares are one computation in both."""
    cfg, eng, raw, blob = setup("mini_moe16", 62)
    eng = dict(eng, max_batch=6, max_seq_len=600, kv_num_blocks=160, max_prefill_tokens=2048, ring_slots=16)
    out = []
    for tune in (1 << 12, 1 << 12 | 0x40):
        e = lib.Engine(cfg, eng, blob, tune=tune if sum(prompts) > 256 else tune & 0x40)
        try:
            for r in _fixed_prompts(cfg, prompts, 1, 270):
                e.submit(r["prompt"], 1)
            e.run(1)
            e.wait()
            out.append(e.debug_read(lib.DBG.HIDDEN, np.uint32))
        finally:
            e.shutdown()
    assert out[0].size == sum(prompts) * cfg["d_model"] and (out[0] == out[1]).all(), "%d values differ" % (out[0] != out[1]).sum()


def test_fp32_down_projection_with_few_tokens_has_the_chip_to_itself(lib):
    """Down 1024 x 4096 at 509 tokens is 512 items of 32 x 32, at 2036 tokens 2048, one for every wave of the chip: the quarter of the work may take
    two thirds of the time (117 us against 250; with eight neighbouring items per workgroup it was 64 busy compute units and 246)."""
    cfg = dict(synth.model_config("mini_gqa"), n_layers=2, d_model=1024, n_q_heads=8, n_kv_heads=8, head_dim=128, d_ffn=4096, vocab=512, dtype=0)
    eng = dict(synth.engine_config("mini_gqa"), max_batch=2, max_seq_len=2048, kv_num_blocks=256, max_prefill_tokens=2048, ring_slots=16)
    e = lib.Engine(cfg, eng, synth.pack_blob(cfg, synth.make_weights(cfg, 71)))
    us = {}
    try:
        e.time_phase(8)
        for tokens in (509, 2036):
            for rep in range(5):
                e.submit(np.zeros(tokens, np.int32), 1)
                e.run(1)
                e.wait()
                e.drain()
                us[tokens] = min(us.get(tokens, np.inf), float(e.phase_times_ms()[0]) * 1e3 / 2)
    finally:
        e.shutdown()
    print(us)
    assert us[509] < us[2036] * 2 / 3, us


@pytest.mark.parametrize("slices", [5, 8])
@pytest.mark.parametrize("shape", [1, 2, 3])
def test_tile_gemms_with_k_in_many_slices(lib, shape, slices):
    """The workgroup that comes last adds four slices of 128 x 64 tiles at a time, eight of 64 x 64 and one of 128 x 128: five and eight slices,
    so that there are second and partly filled batches; K of 9 and 11 pairs of k-steps (slices of one to three pairs)."""
    cfg = dict(synth.model_config("mini_gqa"), n_layers=1, d_model=576, n_q_heads=9, n_kv_heads=3, head_dim=64, d_ffn=704, vocab=1003)
    raw = synth.make_weights(cfg, 72, gain_jitter=0.1)
    eng = dict(synth.engine_config("mini_gqa"), max_batch=24, max_seq_len=400, kv_num_blocks=96, max_prefill_tokens=512, ring_slots=64)
    for prompts in ([65], [61], [128], [3] * 19):
        worst = parity.stepwise_check(lib, cfg, eng, raw, synth.pack_blob(cfg, raw), _fixed_prompts(cfg, prompts, 3, 272), rtol=RTOL, tune=shape << 12 | slices << 24)
        print("shape", shape, "slices", slices, "prompts", prompts, "worst relative logit error", worst)


@pytest.mark.parametrize("prompts", [[17], [61], [65], [257, 73], [400, 109]])
def test_eight_slices_by_the_planner_s_own_choice(lib, prompts):
    """Down 256 x 6400 (100 pairs of k-steps) is in eight slices from 17 tokens on without being asked to."""
    cfg, eng, raw, blob = setup("mini_wide2", 73)
    eng = dict(eng, max_batch=4, max_seq_len=420, kv_num_blocks=96)
    worst = parity.stepwise_check(lib, cfg, eng, raw, blob, _fixed_prompts(cfg, prompts, 2, 273), rtol=RTOL)
    print("prompts", prompts, "worst relative logit error", worst)


def test_iterations_beyond_16384_tokens(lib):
    """Down 160 x 9216 has K in slices up to 16384 tokens, exactly one item per compute unit, and whole beyond: 42 prompts of 400 tokens in one
    iteration of 16800 give the logits that they give in iterations of 4000."""
    cfg = dict(synth.model_config("mini_gqa"), n_layers=2, d_model=160, n_q_heads=4, n_kv_heads=4, head_dim=64, d_ffn=9216, vocab=1003)
    blob = synth.pack_blob(cfg, synth.make_weights(cfg, 74, gain_jitter=0.1))
    rows = []
    for budget in (4000, 20000):
        eng = dict(synth.engine_config("mini_gqa"), max_batch=42, max_seq_len=416, kv_num_blocks=42 * 26, max_prefill_tokens=budget, ring_slots=64)
        e = lib.Engine(cfg, eng, blob, flags=lib.FLAG_KEEP_LOGITS)
        try:
            for r in _fixed_prompts(cfg, [400] * 42, 1, 274):
                e.submit(r["prompt"], 1)
            got = []
            while sum(len(g) for g in got) < 42:
                e.run(1)
                e.wait()
                e.drain()
                got.append(e.debug_read(lib.DBG.LOGITS, np.float32).reshape(-1, cfg["vocab"]))
            rows.append(np.concatenate(got))
        finally:
            e.shutdown()
    assert len(got) == 1
    error = np.abs(rows[0] - rows[1]).max(axis=1) / np.abs(rows[0]).max(axis=1)
    print("worst relative difference", error.max())
    assert error.max() < RTOL
