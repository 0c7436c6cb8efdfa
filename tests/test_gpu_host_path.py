"""The host side of the ABI on the GPU: what a call does when a phase has no kernels, when another library's HIP call has failed
on the same thread, and while long kernels run."""
import ctypes
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def tiny_engine(lib, **kw):
    cfg, eng = synth.model_config("tiny"), synth.engine_config("tiny")
    return lib.Engine(cfg, eng, synth.pack_blob(cfg, synth.make_weights(cfg, 1000)), **kw)


@pytest.mark.parametrize("phase", [1, 2, 3, 6, 9, 13])
def test_timing_a_phase_with_or_without_kernels_leaves_the_loop_running(lib, phase):
    """An fp32 model has no kernels of its own for the norms (1, 6, 9), the rotary step (3) and phase 13: their time is 0 in every
    iteration of every window, and the windows serve their requests."""
    e = tiny_engine(lib, pump_depth=2)
    try:
        e.time_phase(phase)
        for window in range(3):
            e.submit(np.arange(20), 6)
            e.run(6)
            e.wait()
            assert len(e.drain()) == 6
            times = e.phase_times_ms()
            assert len(times) >= 6 and ((times[:6] > 0).all() if phase == 2 else not times.any())
    finally:
        e.shutdown()


def failed_hip_call():
    """A HIP call of this thread that fails without touching the GPU, as a program's own handling of an error may leave it."""
    name = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    assert ctypes.CDLL(name).hipSetDevice(9999) != 0


def test_an_error_of_an_earlier_hip_call_is_not_taken_for_the_engine_s_own(lib):
    """Making an engine, submit, run, poll, the clock probe and the stand-alone sampler look at their own launches only. (A submit
    that reported such an error had already marked its ring slot as taken, so that the ring refused every later one.)"""
    failed_hip_call()
    e = tiny_engine(lib)
    try:
        for round_ in range(2):
            failed_hip_call()
            assert e.submit(np.arange(20), 4) == round_
            failed_hip_call()
            e.run(4)
            e.wait()
            failed_hip_call()
            assert len(e.drain()) == 4
            failed_hip_call()
            e.clock_sync()
            failed_hip_call()
            row = np.arange(100, dtype=np.float32)[None]
            assert lib.sample_rows(row, [dict(temperature=0.0, top_k=0, top_p=1.0, seed=0)], [0])[0] == 99
    finally:
        e.shutdown()


def test_submit_and_poll_beside_long_kernels(lib):
    """Submit and poll need a place on the chip for a moment and must not wait for the GEMM launch that occupies it to end.
    Prefill iterations of 8192 tokens at the widths of the llama3_8b shape: launches of 0.4 to 1.5 ms one behind the other, so
    that a call which waited for the end of one would take about half a millisecond at the median; 25 to 35 us without the wait."""
    cfg = dict(synth.model_config("llama3_8b"), n_layers=2, vocab=1024)
    eng = dict(synth.engine_config("llama3_8b"), kv_num_blocks=60 * 260, max_batch=64, max_seq_len=4112, max_prefill_tokens=8192, ring_slots=256)
    d, hd = cfg["d_model"], cfg["head_dim"]
    layer = 2 * 4 * d + 2 * ((cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * hd * d + d * cfg["n_q_heads"] * hd + 3 * d * cfg["d_ffn"])
    blob = np.zeros(2 * 2 * cfg["vocab"] * d + cfg["n_layers"] * layer + 4 * d, dtype=np.uint8)
    e = lib.Engine(cfg, eng, blob)
    rng = np.random.default_rng(1)
    took = {"submit": [], "poll": []}
    try:
        for _ in range(60):
            e.submit(np.zeros(4096, np.int32), 1)
        e.run(0)
        end = time.perf_counter() + 0.1
        while time.perf_counter() < end:
            t0 = time.perf_counter()
            e.poll()
            t1 = time.perf_counter()
            time.sleep(rng.uniform(0, 1e-3))
            t2 = time.perf_counter()
            e.submit(np.zeros(16, np.int32), 1)
            took["poll"].append(t1 - t0)
            took["submit"].append(time.perf_counter() - t2)
            time.sleep(rng.uniform(0, 1e-3))
        e.stop()
        st = e.stats()
    finally:
        e.shutdown()
    for name, v in took.items():
        print(name, "median %.0f us of %d calls" % (np.median(v) * 1e6, len(v)), "prefill iterations", st["prefill_iterations"])
    assert st["prefill_iterations"] >= 5 and st["next_ticket"] < 60 + len(took["submit"])      # prefills ran all along
    assert np.median(took["submit"]) < 150e-6 and np.median(took["poll"]) < 150e-6


def test_the_last_iteration_of_a_window_is_enqueued_ahead(lib):
    """Device time from the end of an iteration to the scheduler step of the next: no longer before the second and last
    iteration of a window of two than inside a window of six (15 us each; 21 when the launcher waited for the first of two to end)."""
    cfg, eng = synth.model_config("mini_churn"), dict(synth.engine_config("mini_churn"), max_batch=4, max_seq_len=1000, kv_num_blocks=256)
    e = lib.Engine(cfg, eng, synth.pack_blob(cfg, synth.make_weights(cfg, 49)), flags=lib.FLAG_TRACE)
    gaps = {2: [], 6: []}
    try:
        e.submit(np.arange(50), 900)
        e.run(1)
        e.wait()
        for i in range(50):
            for n, g in gaps.items():
                e.run(n)
                e.wait()
                t = e.trace(n)
                g.append((t["t_sched_begin_ns"][-1].astype(np.int64) - t["t_publish_end_ns"][-2].astype(np.int64)) / 1e3)
    finally:
        e.shutdown()
    short, long = (np.median(gaps[n][5:]) for n in (2, 6))
    print("gap before the last iteration of 2: %.1f us, of 6: %.1f us" % (short, long))
    assert short < long + 3.0


@pytest.mark.parametrize("n,cap", [(1, 2), (8, 5), (9, 4096), (256, 7), (257, 300)])
def test_poll_in_pieces_and_the_logits_behind_it(lib, n, cap):
    """Polls of `cap` records (a slot's records in several polls, one strip of 256 slots and one more) bring every token of every request
    once and in order, completed slots are free again, and the logits of the last iteration (8192 floats a row: within the first
    256 KB, that and one more row, several pieces of 512 KB) have their maximum at the token that each request got."""
    cfg = synth.model_config("sched_stress")
    eng = dict(synth.engine_config("sched_stress"), max_batch=n, ring_slots=512)
    e = lib.Engine(cfg, eng, synth.pack_blob(cfg, synth.make_weights(cfg, 1000)), flags=lib.FLAG_KEEP_LOGITS)
    try:
        for window in range(2):
            rng = np.random.default_rng(window)
            ids = [e.submit(rng.integers(0, cfg["vocab"], 5 + i % 4), 3) for i in range(n)]
            e.run(3)
            e.wait()
            got = {i: [] for i in ids}
            while True:
                ev = e.poll(cap)
                if ev.size == 0:
                    break
                assert ev.size <= cap
                for r in ev:
                    assert r["index"] == len(got[r["request_id"]])
                    got[r["request_id"]].append(int(r["token"]))
            assert all(len(t) == 3 for t in got.values())
            logits = e.debug_read(lib.DBG.LOGITS, np.float32).reshape(n, cfg["vocab"])
            assert [int(x) for x in logits.argmax(1)] == [got[i][2] for i in ids]
    finally:
        e.shutdown()


@pytest.mark.parametrize("n,out,cap", [(300, 9, 1 << 16), (300, 9, 2500), (40, 60, 1 << 16), (512, 40, 1 << 16), (3, 1500, 1 << 16), (2, 1100, 2100)])
def test_polls_of_many_records(lib, n, out, cap):
    """More than 2048 new records of 256 slots come with a second launch, a workgroup per 1024 of a slot: strips of slots on either side of
    that, polls that end inside a slot, slots with more records than one workgroup takes. Every token once and in order, and the
    slots can be taken again afterwards."""
    cfg = synth.model_config("sched_stress")
    eng = dict(synth.engine_config("sched_stress"), max_batch=n, max_seq_len=out + 8, kv_num_blocks=n * (out // 16 + 2), ring_slots=512)
    e = lib.Engine(cfg, eng, synth.pack_blob(cfg, synth.make_weights(cfg, 1000)))
    rng = np.random.default_rng(n)
    try:
        for window in range(2):
            ids = [e.submit(rng.integers(0, cfg["vocab"], 3 + i % 3), out) for i in range(n)]
            e.run(out)
            e.wait()
            got, polls = [], 0
            while True:
                ev = e.poll(cap)
                if ev.size == 0:
                    break
                assert ev.size <= cap
                got.append(ev)
                polls += 1
            assert polls == -(-n * out // cap)
            ev = np.concatenate(got)
            order = np.lexsort((np.arange(len(ev)), ev["request_id"]))
            assert (ev["request_id"][order].reshape(n, out) == np.array(ids)[:, None]).all()
            ev = ev[order].reshape(n, out)
            assert (ev["index"] == np.arange(out)).all() and (np.diff(ev["iteration"].astype(np.int64), axis=1) == 1).all()
            assert (ev["flags"] == np.where(np.arange(out) == 0, lib.EVENT_FIRST, 0) + np.where(np.arange(out) == out - 1, lib.EVENT_LAST, 0)).all()
            if window == 0:
                first = ev["token"]
                rng = np.random.default_rng(n)
            else:
                assert (ev["token"] == first).all()
            e.set_exit_when_idle(True)
            e.run(0)
            e.wait()
            e.set_exit_when_idle(False)
    finally:
        e.shutdown()


def test_a_poll_of_many_records_takes_no_longer_than_two_launches(lib):
    """512 slots with 120 records each: 61440 records are 1 MB over the bus and 2 MB of events, 140 us a poll (one workgroup for all of
    them took 290)."""
    cfg = synth.model_config("sched_stress")
    eng = dict(synth.engine_config("sched_stress"), max_seq_len=128, kv_num_blocks=512 * 8, ring_slots=512)
    e = lib.Engine(cfg, eng, synth.pack_blob(cfg, synth.make_weights(cfg, 1000)))
    took = []
    try:
        for _ in range(5):
            for i in range(512):
                e.submit(np.full(4, i), 120)
            e.run(120)
            e.wait()
            t0 = time.perf_counter()
            ev = e.poll(1 << 16)
            took.append((time.perf_counter() - t0) * 1e6)
            assert len(ev) == 512 * 120
            e.set_exit_when_idle(True)
            e.run(0)
            e.wait()
            e.set_exit_when_idle(False)
    finally:
        e.shutdown()
    print("61440 records: %.0f us a poll" % min(took))
    assert min(took) < 230


def test_decode_iterations_behind_a_prefill_run_their_own_batch_s_chain(lib):
    """40 sequences x 8 kv heads of 64 x 3 chunks are more than three attention items per compute unit, where a kernel behind the
    attention merges the chunks: it is there (phase 12) from the first decode iteration behind the prefill iterations, although those
    had no decode attention themselves, and is not there for 4 sequences."""
    cfg = synth.model_config("mini_kv8")
    eng = dict(synth.engine_config("mini_kv8"), max_prefill_tokens=16384)
    e = lib.Engine(cfg, eng, synth.pack_blob(cfg, synth.make_weights(cfg, 50)))
    rng = np.random.default_rng(50)
    try:
        for n in (40, 4):
            for _ in range(n):
                e.submit(rng.integers(0, cfg["vocab"], 1100), 12)
            first = 0
            while first < n:
                e.run(1)
                e.wait()
                first += len(e.drain())
            e.time_phase(12)
            e.run(4)
            e.wait()
            t = e.phase_times_ms()[:4]
            print(n, "sequences, merge kernel in the first four decode iterations, us:", t * 1e3)
            assert (t > 0).all() if n == 40 else not t.any(), (n, t)
            e.time_phase(-1)
            e.set_exit_when_idle(True)
            e.run(0)
            e.wait()
            e.drain()
            e.set_exit_when_idle(False)
    finally:
        e.shutdown()
