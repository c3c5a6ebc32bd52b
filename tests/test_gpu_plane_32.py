"""The y-z plane pass at 32^3 (two planes per workgroup): against the separate passes and the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import test_gpu_hmc as hmc_tests  # noqa: E402
from gpu_common import chain_spec, dh_tol, mock, rel_l2, start_state  # noqa: E402
from paper_1306_1821_amd.binding import Sampler  # noqa: E402


def test_plane_pass_32_matches_separate_passes_and_oracle():
    hmc_tests.test_plane_pass_matches_separate_passes_and_oracle("cfg1", 0.05, 10)


def test_chains_of_one_context_use_their_own_planes():
    """Three chains with other starts: trajectories with the plane pass and with the separate
    passes end within the bounds of the test above."""
    mk = mock("cfg1")
    d = start_state(mk)[0]
    got = []
    for fused in (True, False):
        s = Sampler([chain_spec(mk, nsteps=6, seed=23, chain_id=c) for c in range(3)])
        s.set_plane_pass(fused)
        for c in range(3):
            s.set_state(c, np.roll(d, 5 * c, axis=c))
        dH, acc = s.trajectory(0)
        got.append((dH, acc, [s.state(c) for c in range(3)]))
        s.close()
    (da, aa, sa), (db, ab, sb) = got
    assert np.all(np.abs(da - db) < 2 * dh_tol(32)) and np.array_equal(aa, ab)
    for a, b in zip(sa, sb):
        for k in ("delta_k", "mom_k", "grad_k", "delta_r"):
            assert rel_l2(a[k], b[k]) < 2e-6, k
