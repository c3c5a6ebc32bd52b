"""Contexts whose chains advance in parts on streams of their own: a chain's results are those of
the undivided context (which runs while pass timing is on) and, alone, its own."""
import numpy as np
import pytest

from gpu_common import chain_spec, plain_mock, start_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1306_1821_amd.binding import Sampler  # noqa: E402

MIXED = [(8, 3), (64, 20), (16, 7), (64, 20), (32, 12)]


def records(specs, mks, mode, grouped, passes=2):
    s = Sampler(specs)
    for i, mk in enumerate(mks):
        s.set_state(i, np.roll(start_state(mk)[0], i, axis=0))
    if grouped:
        for cls in range(3):
            s.set_launch(cls, -1)
    if mode == "whole":
        s.timing(1)
    s.use_graph(mode == "graph")
    out = [[] for _ in specs]
    for i in range(passes):
        dH, acc = s.trajectory(100 + i)
        sw = s.sweep(i)
        _ = s.state(0)["delta_k"].sum()                  # eager work between replays
        for c in range(len(specs)):
            st = s.state(c)
            out[c] += [dH[c], acc[c]] + [np.asarray(sw[c][k]) for k in sorted(sw[c])] + [st[k] for k in sorted(st)]
    s.close()
    return out


def same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_size_groups_on_their_own_streams():
    mks = [plain_mock(n, 500.0, nb, nsub=2) for n, nb in MIXED]
    specs = [chain_spec(mk, nsteps=5, eps=0.05, seed=7, chain_id=c, rj=True) for c, mk in enumerate(mks)]
    whole = records(specs, mks, "whole", True)
    for mode in ("parts", "graph"):
        for a, b in zip(whole, records(specs, mks, mode, True)):
            same(a, b)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,chains", [(192, 3), (128, 6)])   # uneven halves; the smallest that splits
def test_halves_of_one_size(n, chains):
    mk = plain_mock(n, 500.0, 16, nsub=1)
    specs = [chain_spec(mk, nsteps=3, eps=0.03, seed=7, chain_id=c, rj=True) for c in range(chains)]
    parts = records(specs, [mk] * chains, "parts", False, passes=1)
    for a, b in zip(parts, records(specs, [mk] * chains, "whole", False, passes=1)):
        same(a, b)
    for a, b in zip(parts, records(specs, [mk] * chains, "graph", False, passes=1)):
        same(a, b)
    same(parts[0], records(specs[:1], [mk], "parts", False, passes=1)[0])
