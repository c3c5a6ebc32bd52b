"""Host-side tests without a GPU: the library against a HIP runtime (hip_record.c) that runs
nothing and writes down the launches, event records and waits it is asked for.

`call(function, *args)` runs the function in a process of its own in which libhmc.so is bound to
that runtime; the function uses Context and returns plain values.
"""
import ctypes
import multiprocessing
import os
import subprocess
import sys
import tempfile
import types

from paper_1306_1821_amd import binding, build

HERE = os.path.dirname(os.path.abspath(__file__))
STREAM = 7   # the caller's stream


def _bind(path):
    global runtime, lib
    runtime = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)   # ahead of libhmc.so's own dependency
    runtime.record_text.restype = ctypes.c_char_p
    sys.modules["torch"] = types.ModuleType("torch")       # its HIP runtime stays out
    lib = binding.lib()


def call(function, *args):
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    with tempfile.TemporaryDirectory() as tmp:
        path = os.path.join(tmp, "hip_record.so")
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", path, os.path.join(HERE, "hip_record.c")], check=True)
        with multiprocessing.get_context("spawn").Pool(1, _bind, (path,)) as pool:
            return pool.apply_async(function, args).get(timeout=100)


def words():
    """The record since it was cleared, as lists of words."""
    return [line.split() for line in runtime.record_text().decode().splitlines()]


class Context:
    """A sampler of chains of the given grid sizes, on buffers that no kernel touches."""

    def __init__(self, sizes, steps=3, rj=False):
        k = len(sizes)
        cfgs, bufs = (binding.HmcConfig * k)(), (binding.HmcBuffers * k)()
        for i, n in enumerate(sizes):
            c, b = cfgs[i], bufs[i]
            c.n, c.box, c.n_sub, c.n_bins = n, 500.0, 2, 3
            c.alpha_prior, c.seed, c.chain_id, c.n_leapfrog, c.eps = 1.0, 1, i, steps, 0.05
            c.rj_move = int(rj)
            for j, name in enumerate(("R", "counts", "delta_k", "mom_k", "grad_k", "delta_r", "alpha", "beta", "work")):
                setattr(b, name, (16 * i + j + 1) << 40)
            b.work_bytes = lib.hmc_workspace_bytes(ctypes.byref(c))
        ones = (ctypes.c_double * (3 * k))(*[1.0] * (3 * k))
        self.ctx = ctypes.c_void_p()
        st = lib.hmc_init_batch(cfgs, bufs, k, ones, ones, ones, ctypes.c_void_p(STREAM), ctypes.byref(self.ctx))
        assert st == binding.HMC_OK, lib.hmc_last_error(None)
        self.chains = k

    def check(self, st):
        assert st == binding.HMC_OK, lib.hmc_last_error(self.ctx)

    def group(self):
        """One launch per size group for every pass class."""
        for cls in range(3):
            self.check(lib.hmc_set_launch(self.ctx, cls, -1))

    def learned(self):
        for i in range(self.chains):
            self.check(lib.hmc_set_mass(self.ctx, i, ctypes.c_void_p(1 << 50)))

    def timing(self, on):
        self.check(lib.hmc_timing(self.ctx, int(on), None, None))

    def graph(self, on):
        self.check(lib.hmc_use_graph(self.ctx, int(on)))

    def autotune(self):
        self.check(lib.hmc_autotune(self.ctx, 2, None))

    def log(self, index=1, sweep=False):
        """The record of one queued trajectory (or sweep), and its status."""
        runtime.record_clear()
        out = ctypes.c_void_p(1 << 51)
        if sweep:
            st = lib.gibbs_sweep_async(self.ctx, index, out)
        else:
            st = lib.leapfrog_trajectory_async(self.ctx, index, out, out)
        return words(), st

    def close(self):
        lib.hmc_destroy(self.ctx)


def kernels(log):
    """Names of the launched kernels, in order."""
    return [w[3] for w in log if w[0] == "launch"]


def streams(log):
    """Streams that kernels were launched to."""
    return sorted({int(w[1]) for w in log if w[0] == "launch"})


def unjoined(log, stream=STREAM):
    """Streams with launches that neither `stream` nor the host waits for after their last one."""
    open_, at = set(), {}
    for w in log:
        if w[0] == "launch" and int(w[1]) != stream:
            open_.add(int(w[1]))
        elif w[0] == "sync":
            open_.discard(int(w[1]))
        elif w[0] == "record":
            at[w[2]] = int(w[1]) if int(w[1]) in open_ else None
        elif w[0] == "wait" and int(w[1]) == stream:
            open_.discard(at.get(w[2]))
    return sorted(open_)
