"""Learned-mass trajectories: the plane passes against the separate passes."""
import numpy as np
import pytest

from gpu_common import chain_spec, dh_tol, plain_mock, rel_l2, start_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1306_1821_amd.binding import Sampler  # noqa: E402


@pytest.mark.parametrize("n,chains,kind,nsteps", [(32, 3, "learned", 5), (64, 2, "learned", 1),
                                                  (64, 2, "diagonal", 4), (128, 2, "learned", 4),
                                                  (192, 1, "learned", 3), (256, 1, "diagonal", 2)])
def test_plane_passes_match_separate_passes(n, chains, kind, nsteps):
    """Every state array of each chain to float32 rounding (the bound of the plain mass's
    comparison, 2e-6, per trajectory), dH within twice its float32 bound."""
    mk = plain_mock(n, 500.0, 16, nsub=1)
    d = start_state(mk)[0]
    lv = (0.5 * np.random.default_rng(n).standard_normal((n, n, n)) - 2.0).astype(np.float32)
    got = []
    for planes in (True, False):
        s = Sampler([chain_spec(mk, nsteps=nsteps, eps=0.03, seed=29, chain_id=c) for c in range(chains)])
        s.set_plane_pass(planes)
        for c in range(chains):
            s.set_state(c, np.roll(d, 3 * c, axis=2))
            s.set_mass(c, np.roll(lv, c, axis=0), kind=kind)
        dH, acc = s.trajectory(0)
        got.append((dH, acc, [s.state(c) for c in range(chains)]))
        s.close()
    (da, aa, sa), (db, ab, sb) = got
    assert np.all(np.abs(da - db) < 2 * dh_tol(n)) and np.array_equal(aa, ab)
    for a, b in zip(sa, sb):
        for k in ("delta_k", "mom_k", "grad_k", "delta_r"):
            assert rel_l2(a[k], b[k]) < 2e-6, (k, rel_l2(a[k], b[k]))
