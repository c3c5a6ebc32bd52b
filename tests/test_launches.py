"""Which kernels a context launches, on which streams, and how these are joined: against a HIP
runtime that only writes down what it is asked (no GPU)."""
import ctypes
import re

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


def learned_forms(launch):
    c = hr.Context(GROUPS)
    for cls in range(3):
        c.check(hr.lib.hmc_set_launch(c.ctx, cls, launch[cls]))
    c.learned()
    out = [c.log()]
    c.timing(True)
    out.append(c.log())
    c.graph(True)
    out.append(c.log())
    kinds = re.compile(r"yzpass_n.*ELi[123]EE")   # the learned mass's, not the plain data force (0)
    return [sorted(k for k in hr.kernels(log) if kinds.search(k)) for log, _ in out]


@pytest.mark.parametrize("launch,planes", [((-1, -1, -1), True), ((0, -1, -1), True), ((0, 0, 0), False), ((-1, 0, -1), False)])
def test_learned_mass_batch_has_one_form(launch, planes):
    """The passes a learned mass takes in a batch of several sizes follow from its launches
    alone: the same plane passes with pass timing on, off, and captured."""
    direct, timed, captured = hr.call(learned_forms, launch)
    assert bool(direct) == planes
    assert direct == timed == captured


def tuned(sizes, group):
    c = hr.Context(sizes)
    if group:
        c.group()
    before = hr.streams(c.log()[0])
    c.autotune()
    return len(before), [len(hr.streams(c.log(sweep=sweep)[0])) for sweep in (False, True)]


@pytest.mark.parametrize("sizes,parts", [([192] * 2, 2), ([128] * 6, 2), ([256] * 3, 2), ([64, 128, 64, 192], 3),
                                         ([8, 16], 2), ([128] * 5, 1), ([64] * 48, 1), ([256], 1)])
def test_autotuner_keeps_the_parts(sizes, parts):
    """Contexts on either side of the sizes from which chains advance in parts, with every
    launch timed faster than the one before it: the autotuner's last candidate, a grid of its
    own, would put all chains on one stream."""
    before, after = hr.call(tuned, sizes, len(set(sizes)) > 1)
    assert before == parts and after == [parts, parts]


def weight_gradient_blocks(units):
    hr.runtime.record_compute_units(units)
    params = (ctypes.c_float * hr.lib.cnn_param_count())()
    net, field = ctypes.c_void_p(), ctypes.c_void_p(1 << 50)
    assert hr.lib.cnn_create(params, ctypes.c_void_p(hr.STREAM), ctypes.byref(net)) == binding.HMC_OK
    out = []
    for n in (16, 128):
        hr.runtime.record_clear()
        assert hr.lib.cnn_gradient(net, n, field, field, None, None) == binding.HMC_OK
        out.append([w[2] for w in hr.words() if w[0] == "launch" and "k_wgrad" in w[3]])
    return out


def test_weight_gradient_sums_are_split_alike_on_every_device():
    """The partial sums of a weight gradient, and so its rounding, follow from the grid size alone."""
    whole = hr.call(weight_gradient_blocks, 256)
    assert whole == hr.call(weight_gradient_blocks, 32) and len(whole[0]) == len(whole[1]) == 4


def copies(sizes):
    c = hr.Context(sizes)
    out = []
    for change in (lambda: hr.lib.hmc_set_step(c.ctx, 0, ctypes.c_double(0.1)),
                   lambda: hr.lib.hmc_set_mass(c.ctx, len(sizes) - 1, ctypes.c_void_p(1 << 50))):
        hr.runtime.record_clear()
        c.check(change())
        out.append(sum(w[0] == "copy" for w in hr.words()))
    return out


@pytest.mark.parametrize("sizes", [[64], GROUPS, [192] * 2, [8] * 3])
def test_a_changed_chain_is_one_copy(sizes):
    """Step size and mass live in the chains' descriptors: however many arrays of them a
    context has (all chains, size groups, parts), a change goes to the device at once."""
    assert hr.call(copies, sizes) == [1, 1]


def small_forms(sizes, group):
    c = hr.Context(sizes, rj=True)
    if group:
        c.group()
    out = []
    for timing, graph in ((False, False), (False, True), (True, False)):
        c.timing(timing)
        c.graph(graph)
        log, _ = c.log(sweep=True)
        out.append([sum(name in k for k in hr.kernels(log)) for name in ("k_small_trajectory", "k_small_joint")])
    return out


@pytest.mark.parametrize("sizes,group,launches", [([8] * 2, False, 1), ([16], False, 1), ([8, 16, 32], True, 2),
                                                  ([8, 16, 32], False, 0), ([32] * 2, False, 0)])
def test_small_grids_run_in_one_workgroup(sizes, group, launches):
    """The one-workgroup trajectory and joint move, direct and captured; the passes while timed."""
    direct, captured, timed = hr.call(small_forms, sizes, group)
    assert direct == captured == [launches, launches] and timed == [0, 0]


def convolution_blocks(sizes):
    params = (ctypes.c_float * hr.lib.cnn_param_count())()
    net, field = ctypes.c_void_p(), ctypes.c_void_p(1 << 50)
    assert hr.lib.cnn_create(params, ctypes.c_void_p(hr.STREAM), ctypes.byref(net)) == binding.HMC_OK
    out = []
    for n in sizes:
        hr.runtime.record_clear()
        assert hr.lib.cnn_forward(net, n, field, field, field) == binding.HMC_OK
        assert hr.lib.cnn_gradient(net, n, field, field, None, None) == binding.HMC_OK
        out.append([int(w[2]) for w in hr.words() if w[0] == "launch" and "k_conv" in w[3]])
    return out


def test_small_convolutions_spread_over_the_compute_units():
    """Four layers forward, four in training and three backward: at least a workgroup for every
    four x planes, two y rows and sixteen z voxels, or for every compute unit."""
    sizes = range(4, 133, 4)
    for n, blocks in zip(sizes, hr.call(convolution_blocks, list(sizes))):
        assert len(blocks) == 11 and min(blocks) >= min(256, n // 4 * (n // 2) * -(-n // 16)), (n, blocks)
