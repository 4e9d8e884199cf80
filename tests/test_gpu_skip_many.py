"""rng_skip of many XS256 states (one table of M^k per workgroup) against the
serial CPU oracle, bit for bit: on both sides of the count from which on the
table is built, distances of one and of many digits.  Whole numbers: no
tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,k", [(8192, 1), (8191, 77), (65537, 16), (65600, 274877907944), (100001, (1 << 64) - 1), (131071, 0x123456789ABCDEF),
                                 (200000, 1 << 63), (300007, 255)])
def test_skip_many_xs256(oracle, S, k):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    o = oracle.GENERATORS["XS256"]
    st = torch.empty((8, S), dtype=torch.int32, device="cuda")
    R.rng_seed(R.RNG_XS256, 4, 0, S, st)
    special = torch.tensor([[0] * 8, [-1] * 8, [1] + [0] * 7, [0] * 7 + [-(1 << 31)]], dtype=torch.int32, device="cuda").T
    st[:, 40:44] = special  # all bits clear, all set, first and last alone
    ref = np.ascontiguousarray(st.cpu().numpy().view(np.uint32))
    R.rng_skip(R.RNG_XS256, st, S, k)
    torch.cuda.synchronize()
    oracle.skip(o, ref, k)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), ref)
