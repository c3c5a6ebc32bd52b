"""Which kernels a context launches, on which streams, and how these are joined: against a HIP
runtime that only writes down what it is asked (no GPU)."""
import pytest

import hip_record as hr
from paper_1306_1821_amd import binding

GROUPS = [64, 16, 128, 64, 32]   # four size groups: three side streams


def failing(call, nth):
    """A trajectory of divided chains whose nth `call` is refused, then one without a refusal."""
    c = hr.Context(GROUPS)
    c.group()
    hr.runtime.record_fail(call.encode(), nth)
    first, again = c.log(1), c.log(2)
    return first, again, hr.lib.hmc_last_error(c.ctx).decode()


# a trajectory records the fork and three ends, and waits three times for each of them
@pytest.mark.parametrize("call,nth", [("hipEventRecord", k) for k in (1, 2, 3, 4)] +
                         [("hipStreamWaitEvent", k) for k in (1, 2, 3, 4, 5, 6)] + [("hipGetLastError", 1)])
def test_parts_are_joined_when_a_call_fails(call, nth):
    """The failure is reported, and no stream is left running past the call's place in the
    caller's stream; the next call works."""
    (log, st), (after, st2), why = hr.call(failing, call, nth)
    assert binding.STATUS.get(st) == "EDEVICE"
    assert "refused" in why
    assert hr.unjoined(log) == []
    assert st2 == binding.HMC_OK and len(hr.streams(after)) == 4 and hr.unjoined(after) == []
