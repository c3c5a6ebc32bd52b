"""A learned mass in a batch of several sizes whose size groups advance on streams of their own."""
import numpy as np
import pytest

from gpu_common import chain_spec, dh_tol, plain_mock, rel_l2, start_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1306_1821_amd.binding import Sampler  # noqa: E402

SIZES = (64, 32, 128, 64)
KINDS = ("learned", "diagonal", "diagonal", "learned")
FIELDS = ("delta_k", "mom_k", "grad_k", "delta_r")


def sampler(chains):
    s = Sampler([chain_spec(plain_mock(SIZES[c], 500.0, 8, nsub=1), nsteps=4, eps=0.03, seed=29, chain_id=c, rj=True)
                 for c in chains])
    for i, c in enumerate(chains):
        n = SIZES[c]
        s.set_state(i, np.roll(start_state(plain_mock(n, 500.0, 8, nsub=1))[0], 3 * c, axis=2))
        lv = 0.5 * np.random.default_rng(c).standard_normal((n, n, n)) - 2.0
        s.set_mass(i, lv.astype(np.float32), kind=KINDS[c])
    return s


def batch(launch, timing=False, graph=False):
    """dH, decisions and states after one trajectory, then after a sweep and another trajectory."""
    s = sampler(range(len(SIZES)))
    for cls in range(3):
        s.set_launch(cls, launch[cls])
    s.timing(1 if timing else 0)
    s.use_graph(graph)
    out = []
    for i in range(2):
        dH, acc = s.trajectory(10 + i)
        out.append((dH, acc, [s.state(c) for c in range(len(SIZES))]))
        s.sweep(i)
        _ = s.state(0)["delta_k"].sum()   # eager work between replays
    s.close()
    return out


@pytest.mark.timeout(300)
def test_learned_mass_in_a_divided_batch():
    """Divided, timed (undivided), replayed, and with the x passes in one launch: the same bits.
    One trajectory against the same chains with one launch over all of them (no plane passes)
    and against each chain alone: the bounds of the plane passes' own comparison (2e-6 per
    trajectory, dH within twice its float32 bound)."""
    parts = batch((-1, -1, -1))
    for other in (batch((-1, -1, -1), timing=True), batch((-1, -1, -1), graph=True), batch((0, -1, -1))):
        for (da, aa, sa), (db, ab, sb) in zip(parts, other):
            assert np.array_equal(da, db) and np.array_equal(aa, ab)
            for a, b in zip(sa, sb):
                for k in FIELDS:
                    assert np.array_equal(a[k], b[k]), k
    alone = []
    for c in range(len(SIZES)):
        s = sampler([c])
        dH, acc = s.trajectory(10)
        alone.append((dH[0], acc[0], s.state(0)))
        s.close()
    dH, acc, states = parts[0]
    for db, ab, sb in (batch((0, 0, 0))[0], [list(x) for x in zip(*alone)]):
        for c, n in enumerate(SIZES):
            assert abs(dH[c] - db[c]) < 2 * dh_tol(n) and acc[c] == ab[c], (c, dH[c], db[c])
            for k in FIELDS:
                assert rel_l2(states[c][k], sb[c][k]) < 2e-6, (c, k)
