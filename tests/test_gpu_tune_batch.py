"""The batch tuner does not choose between row limits that plan the same rows."""
import pytest

pytestmark = pytest.mark.gpu


def test_batch_autotune_keeps_the_longest_rows():
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, n, L = R.RNG_XS32, 16, 5000  # rows far below every limit
    st = torch.empty((1, n), dtype=torch.int32, device="cuda")
    R.rng_seed(g, 3, 0, n, st)
    out = torch.empty(n * 5024, dtype=torch.int32, device="cuda")
    reqs = R.make_requests([(g, 0, st.data_ptr() + 4 * i, n, 0, L, out.data_ptr() + 4 * 5024 * i) for i in range(n)])
    h = R.rng_batch_create(n, n * L)
    try:
        R.rng_batch_set(h, reqs)
        wg, un, chunk, us = R.rng_batch_autotune(h, reps=1)
        assert chunk == 4096 and R.rng_batch_get_shape(h) == (wg, un, 4096)
    finally:
        torch.cuda.synchronize()
        R.rng_batch_destroy(h)
