"""The host side of the ABI on the GPU: what a call does when a phase has no kernels, when another library's HIP call has failed
on the same thread, and while long kernels run."""
import ctypes

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
