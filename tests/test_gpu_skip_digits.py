"""XS256 skips by distances of one, two and three hexadecimal digits, on both sides of
the state counts at which products per state give way to a table of the whole map,
against the serial CPU oracle.  Whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [8191, 8192, 65535, 65536, 300001])
@pytest.mark.parametrize("k", [1, 15, 1 << 60, 0x11, 0xF0000000000000F0, 0x9000000000000007, 0x111, 0x1000000000030002])
def test_skip_digits(oracle, S, k):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    st = torch.empty((8, S), dtype=torch.int32, device="cuda")
    R.rng_seed(R.RNG_XS256, 21, 0, S, st)
    R.rng_skip(R.RNG_XS256, st, S, k)
    torch.cuda.synchronize()
    ref = oracle.seed(oracle.XS256, 21, S)
    oracle.skip(oracle.XS256, ref, k)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), ref)
