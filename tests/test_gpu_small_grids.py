"""8^3 and 16^3 contexts: the one-workgroup trajectory and joint move against the separate
passes, which run while pass timing is on."""
import numpy as np
import pytest

from gpu_common import chain_spec, plain_mock, start_state

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1306_1821_amd.binding import Sampler  # noqa: E402


# steps 1: the start and end passes alone; eps 0.6: rejected trajectories and joint moves too
@pytest.mark.parametrize("n,nb,nsub,chains,nsteps,eps,kw", [
    (8, 4, 2, 1, 1, 0.05, {}), (8, 3, 1, 3, 7, 0.6, {}), (8, 4, 5, 2, 6, 0.1, dict(tau_mode=True)),
    (16, 8, 2, 1, 1, 0.05, {}), (16, 1, 1, 2, 2, 0.05, {}), (16, 7, 3, 3, 9, 0.6, {}),
    (16, 8, 2, 2, 5, 0.1, dict(alpha_prior=0.0, rj_log_bound=0.02))])
def test_one_workgroup_equals_separate_passes(n, nb, nsub, chains, nsteps, eps, kw):
    """Bit for bit: every state array, energy error, decision and draw, direct and replayed."""
    mk = plain_mock(n, 500.0, nb, nsub)
    runs = []
    for mode in ("passes", "fused", "graph"):
        s = Sampler([chain_spec(mk, nsteps=nsteps, eps=eps, seed=91, chain_id=c, rj=True, **kw)
                     for c in range(chains)])
        for c in range(chains):
            s.set_state(c, start_state(mk)[0])
        if mode == "passes":
            s.timing(1)
        s.use_graph(mode == "graph")
        out = []
        for i in range(4):
            out += list(s.trajectory(100 + i))
            for st in s.sweep(i):
                out += [np.asarray(st[k]) for k in sorted(st)]
            for c in range(chains):
                st = s.state(c)
                out += [st[k] for k in sorted(st)]
        if mode == "passes":
            assert s.timing(0)[1].sum() > 0
        s.close()
        runs.append(out)
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert np.array_equal(a, b), (np.shape(a), a, b)
