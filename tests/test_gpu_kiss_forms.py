"""Whole-tile KISS rows on both sides of the sizes at which the kernel takes the
other form of the step (f32 rows of 256 numbers from 3 2^25 to 2^28 numbers, u32
rows of 1024 to 4096 over 2^k streams from 2^28 on), against the serial CPU oracle,
bit for bit.  Whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,S,N", [("f32", (3 << 17) - 64, 256), ("f32", 3 << 17, 256), ("u32", 1 << 18, 1024),
                                    ("u32", 1 << 16, 4096), ("u32", 1 << 17, 2048)])
def test_kiss_forms(oracle, dt, S, N):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o, t = R.RNG_KISS, oracle.KISS, R.DTYPES[dt]
    st = torch.empty((R.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    R.rng_seed(g, 77, 0, S, st)
    out = torch.empty((S, N), dtype=torch.int32, device="cuda")
    R.rng_generate(g, st, S, N, t, out)
    torch.cuda.synchronize()
    ref_st = oracle.seed(o, 77, S)
    ref = oracle.generate(o, ref_st, N, t, threads=16).view(np.uint32)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), ref_st)
