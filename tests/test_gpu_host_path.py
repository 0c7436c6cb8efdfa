"""The host side of the ABI on the GPU: what a call does when a phase has no kernels, when another library's HIP call has failed
on the same thread, and while long kernels run."""
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
