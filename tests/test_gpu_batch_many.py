"""Batches of thousands of short requests (more tiles than the grid has waves, pulled
from several counters; from 2048 requests on those that are short enough share tiles)
against the serial CPU oracle, bit for bit, launched twice from one plan, directly and
as a graph.  Whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GENS = ["MWC32", "XS256", "XS32", "KISS", "MWC1616"]


@pytest.mark.parametrize("n,longest,chunk,wg,graph", [(2049, 64, 0, 0, 0), (2300, 64, 0, 0, 0), (4500, 300, 0, 0, 0), (4500, 300, 64, 64, 0),
                                                       (3000, 2000, 0, 1024, 0), (5000, 130, 0, 0, 1), (2700, 250, 512, 512, 0),
                                                       (9000, 700, 0, 0, 0), (9000, 1000, 0, 256, 1)])
def test_many_short_requests(oracle, n, longest, chunk, wg, graph):
    rng = np.random.RandomState(n)
    length = rng.randint(0, longest + 1, n)
    length[:8] = [0, 1, longest, 32, 33, 63, 64, 65]
    offset = np.where(rng.randint(0, 4, n) == 0, rng.randint(1, 1 << 40, n), 0)
    run(oracle, rng, length, offset, chunk, wg, graph)


# above 4096 requests the root kernel takes several per wave, but not where most states
# move by an offset; requests of more than 64 tiles among them
@pytest.mark.parametrize("n,moved", [(4097, 9), (4097, 1), (8200, 40)])
def test_root_of_many(oracle, n, moved):
    rng = np.random.RandomState(n + moved)
    length = rng.randint(0, 40, n)
    length[[5, n // 2, n - 1]] = 300000, 262144, 270001
    offset = np.where(np.arange(n) % moved == 0, rng.randint(1, 1 << 10, n), 0)
    run(oracle, rng, length, offset, 64, 0, 0)


def run(oracle, rng, length, offset, chunk, wg, graph):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    n = len(length)
    gen, dtype, pad = rng.randint(0, 5, n), rng.randint(0, 2, n), rng.randint(0, 5, n)
    pools = []
    for g in GENS:
        st = torch.empty((R.rng_state_words(R.GENERATORS[g]), n), dtype=torch.int32, device="cuda")
        R.rng_seed(R.GENERATORS[g], 19, 0, n, st)
        pools.append(st)
    at = np.cumsum(np.concatenate([[8], length + pad + 3]))
    out = torch.full((int(at[-1]) + 64,), -7, dtype=torch.int32, device="cuda")
    table = [(R.GENERATORS[GENS[gen[i]]], int(dtype[i]), pools[gen[i]].data_ptr() + 4 * i, n, int(offset[i]), int(length[i]),
              out.data_ptr() + 4 * int(at[i])) for i in range(n)]
    h = R.rng_batch_create(n, int(length.sum()))
    ref_pools = [oracle.seed(oracle.GENERATORS[g], 19, n) for g in GENS]
    try:
        R.rng_batch_set_graph(h, graph)
        if chunk or wg:
            R.rng_batch_set_shape(h, wg, 0, chunk)
        R.rng_batch_set(h, R.make_requests(table))
        for _ in range(2):  # the second launch continues from the states that the first wrote
            R.rng_batch_launch(h)
            torch.cuda.synchronize()
            got = out.cpu().numpy().view(np.uint32)
            used = np.zeros(len(got), dtype=bool)
            for i in range(n):
                o = oracle.GENERATORS[GENS[gen[i]]]
                st = np.ascontiguousarray(ref_pools[gen[i]][:, i:i + 1])
                if offset[i]:
                    oracle.skip(o, st, int(offset[i]))
                if length[i]:
                    ref = oracle.generate(o, st, int(length[i]), int(dtype[i]), threads=1).view(np.uint32).reshape(-1)
                    assert np.array_equal(got[at[i]:at[i] + length[i]], ref), (i, table[i])
                ref_pools[gen[i]][:, i] = st[:, 0]
                used[at[i]:at[i] + length[i]] = True
            assert (got[~used] == 0xFFFFFFF9).all()
            for p, q in zip(pools, ref_pools):
                assert np.array_equal(p.cpu().numpy().view(np.uint32), q)
    finally:
        R.rng_batch_destroy(h)
