"""The tuner keeps the stored shape for calls that kernels with a launch shape of
their own take (windows, chunks, rows off whole tiles): it would be timing noise.
Whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,S,N", [("KISS", 1, 100000), ("XS256", 1000, 1000), ("XS32", 300, 777), ("MWC32", 4096, 1024),
                                      ("MWC1616", 70001, 333), ("MWC32", 10, 100)])
def test_autotune_leaves_the_shape(oracle, name, S, N):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o, t = R.GENERATORS[name], oracle.GENERATORS[name], R.RNG_U32
    st = torch.empty((R.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    out = torch.empty(S * N, dtype=torch.int32, device="cuda")
    main, runs, mine = R.rng_get_shape(g, t), R.rng_row_shape(g, t, 1 << 20, 1024), R.rng_row_shape(g, t, S, N)
    R.rng_seed(g, 3, 0, S, st)
    wg, un, us = R.rng_autotune(g, t, S, N, st, out, 3)
    assert (wg, un) == mine and us > 0
    assert R.rng_get_shape(g, t) == main and R.rng_row_shape(g, t, 1 << 20, 1024) == runs
    torch.cuda.synchronize()
    # one warm-up call and three timed ones
    ref_st = oracle.seed(o, 3, S)
    oracle.skip(o, ref_st, 3 * N)
    ref = oracle.generate(o, ref_st, N, t, threads=8).view(np.uint32).reshape(-1)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), ref)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), ref_st)
