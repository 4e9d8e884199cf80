"""The fused consumer on few streams (windows of blocks, lanes started from the
stream's state) and on many (one lane per stream): count and final states
against the serial CPU oracle.  Whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["MWC32", "XS256", "XS32", "KISS", "MWC1616"])
@pytest.mark.parametrize("S,n", [(1, 255), (1, 256), (1, 4097), (3, 8192), (63, 100003), (2, 1 << 20), (64, 10001), (1000, 20001),
                                 (5000, 513), (4097, 9000), (65, 1)])
def test_pi_windows(oracle, name, S, n):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o = R.GENERATORS[name], oracle.GENERATORS[name]
    st = torch.empty((R.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), 5, dtype=torch.int64, device="cuda")
    R.rng_seed(g, 8, 0, S, st)
    R.rng_fused_pi(g, st, S, n, cnt)
    torch.cuda.synchronize()
    ref_st = oracle.seed(o, 8, S)
    assert int(cnt.item()) == 5 + oracle.fused_pi(o, ref_st, n, threads=8)
    oracle.skip(o, end := oracle.seed(o, 8, S), n)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), end)
