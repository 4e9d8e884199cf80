"""Batch requests whose slice crosses position 2^64 of its stream: offset + length
above 2^64, in one tile, at the carry between two tiles and over many, against the
serial CPU oracle started by a skip of `offset`.  Whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["MWC32", "XS256", "XS32", "KISS", "MWC1616"])
@pytest.mark.parametrize("chunk", [0, 64, 4096])
@pytest.mark.parametrize("graph", [0, 1])
def test_slice_crosses_2_64(oracle, name, chunk, graph):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o = R.GENERATORS[name], oracle.GENERATORS[name]
    top = 1 << 64
    # (offset, length): the end below, at and above 2^64; 2^64 inside the first tile, at a tile's start, in a later one
    reqs = [(top - 1, 1), (top - 1, 2), (top - 1, 5000), (top - 4096, 4096), (top - 4096, 4097), (top - 100, 70001),
            (top - 65536, 65537), (top - 70000, 300000), (top - 5, 0), (top - 1, 0), (3, 100)]
    n = len(reqs)
    pool = torch.empty((R.rng_state_words(g), n), dtype=torch.int32, device="cuda")
    R.rng_seed(g, 23, 0, n, pool)
    at = np.concatenate([[0], np.cumsum([(length + 40) // 32 * 32 for _, length in reqs])])
    out = torch.full((int(at[-1]) + 64,), -7, dtype=torch.int32, device="cuda")
    table = [(g, i % 2, pool.data_ptr() + 4 * i, n, off, length, out.data_ptr() + 4 * int(at[i]))
             for i, (off, length) in enumerate(reqs)]
    h = R.rng_batch_create(n, sum(length for _, length in reqs))
    try:
        R.rng_batch_set_graph(h, graph)
        if chunk:
            R.rng_batch_set_shape(h, 0, 0, chunk)
        R.rng_batch_set(h, R.make_requests(table))
        R.rng_batch_launch(h)
        torch.cuda.synchronize()
    finally:
        R.rng_batch_destroy(h)
    got = out.cpu().numpy().view(np.uint32)
    for i, (off, length) in enumerate(reqs):
        st = np.ascontiguousarray(oracle.seed(o, 23, n)[:, i:i + 1])
        oracle.skip(o, st, off)
        if length:
            ref = oracle.generate(o, st, length, i % 2, threads=1).view(np.uint32).reshape(-1)
            assert np.array_equal(got[at[i]:at[i] + length], ref), reqs[i]
        assert np.array_equal(pool.cpu().numpy().view(np.uint32)[:, i], st[:, 0]), reqs[i]
        assert (got[at[i] + length:at[i + 1]] == 0xFFFFFFF9).all(), reqs[i]
