"""Rows and chunks of any length whatever launch shape is set for whole-tile rows,
and XS256 rows of an odd number of 4 KiB that the four-chunk schedule does not take
(stream counts off 64, outputs off 16 bytes), against the serial CPU oracle, bit for
bit.  Whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GENS = ["MWC32", "XS256", "XS32", "KISS", "MWC1616"]


def run(oracle, name, dt, S, N, off):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o, t = R.GENERATORS[name], oracle.GENERATORS[name], R.DTYPES[dt]
    st = torch.empty((R.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    R.rng_seed(g, 31, 0, S, st)
    buf = torch.full((S * N + off + 32,), -7, dtype=torch.int32, device="cuda")
    ref_st = oracle.seed(o, 31, S)
    for _ in range(2):  # the second call continues from the states that the first wrote
        R.rng_generate(g, st, S, N, t, buf[off:off + S * N])
        torch.cuda.synchronize()
        ref = oracle.generate(o, ref_st, N, t, threads=8).view(np.uint32)
        h = buf.cpu().numpy()
        assert (h[:off] == -7).all() and (h[off + S * N:] == -7).all()
        assert np.array_equal(h[off:off + S * N].view(np.uint32).reshape(S, N), ref)
        assert np.array_equal(st.cpu().numpy().view(np.uint32), ref_st)


@pytest.mark.parametrize("S", [64, 1088, 4097, 4160])
@pytest.mark.parametrize("N", [1024, 3072, 5120])
@pytest.mark.parametrize("off", [0, 1, 4])
def test_xs256_odd_4k_rows(oracle, S, N, off):
    run(oracle, "XS256", "u32", S, N, off)


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("wg", [64, 512, 1024])
@pytest.mark.parametrize("S,N,off", [(5, 777, 0), (70, 300, 1), (4096, 1024, 0), (4097, 1001, 2), (66000, 129, 4)])
def test_rows_at_any_tuned_shape(oracle, name, wg, S, N, off):
    import paper_1101_1846_amd as R
    g = R.GENERATORS[name]
    old = [(t, R.rng_get_shape(g, t), R.rng_row_shape(g, t, 4096, 1024)) for t in (R.RNG_U32, R.RNG_F32)]
    try:
        for t, _, _ in old:
            R.rng_set_shape(g, t, wg, 4)
            R.rng_set_row_shape(g, t, 4096, 1024, wg, 4)
        run(oracle, name, "f32", S, N, off)
    finally:
        for t, main, runs in old:
            R.rng_set_shape(g, t, *main)
            R.rng_set_row_shape(g, t, 4096, 1024, *runs)
