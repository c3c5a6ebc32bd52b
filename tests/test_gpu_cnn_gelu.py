"""The network's bf16 GELU and GELU' against their erfcf forms, at every float32 z."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1306_1821_amd.binding import CNN, HmcError  # noqa: E402


def test_short_gelu_rounds_as_the_erfcf_form():
    """Every float32 bit pattern as z (both tails, subnormals, infinities, NaN), v = 1 and three
    draws of v per z: no bf16 value differs, and every deviation is below the bound that
    decides where the short form may stand."""
    net = CNN(np.zeros(16034, np.float32))
    for seed in range(4):
        differ, worst = net.gelu_check(seed=seed)
        print(f"seed {seed}: differ {differ}, deviation over bound {worst}", flush=True)
        assert differ == (0, 0)
        assert 0 < worst[0] < 1 and 0 < worst[1] < 1
    with pytest.raises(HmcError):
        net.gelu_check(first=4, count=1 << 32)
    net.close()
