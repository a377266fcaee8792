"""The points that the phase trace names are the ones the kernel stamps: each
``SI_TRACE_MARK`` / ``SI_TRACE_WAVE`` number of ``owned.hip`` has a name in
``phase_trace.py`` and every name a stamp, within the kernel's trace slots."""

import os
import re

from paper_2411_12692_amd import build, phase_trace


def _stamps(macro):
    with open(os.path.join(build.CSRC, "owned.hip")) as f:
        return {int(n) for n in re.findall(macro + r"\((\d+)\)", f.read())}


def _limit(name):
    with open(os.path.join(build.CSRC, "si_device.h")) as f:
        return int(re.search(r"constexpr int %s = (\d+);" % name, f.read()).group(1))


def test_every_named_point_is_stamped():
    assert _stamps("SI_TRACE_MARK") == set(phase_trace.BLOCK_MARKS)
    assert _stamps("SI_TRACE_WAVE") == set(phase_trace.WAVE_MARKS)


def test_stamps_fit_the_trace():
    assert max(phase_trace.BLOCK_MARKS) < _limit("kTraceBlockMarks") <= phase_trace.SLOTS == _limit("kTraceSlots")
    assert max(phase_trace.WAVE_MARKS) < phase_trace.WAVE_SLOTS == _limit("kTraceWaveMarks")
