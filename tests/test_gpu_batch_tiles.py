"""Batch tiles (64 rows of 32 to 4096 samples, a wave's lanes started from the
request's state) against the serial CPU oracle, bit for bit: lengths around row
and tile ends, offsets whose jump has low, high and many bits, outputs at any
4-byte alignment, empty requests, and the longest rows.  Whole numbers: no
tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GENS = ["MWC32", "XS256", "XS32", "KISS", "MWC1616"]


@pytest.fixture(scope="module")
def rng():
    import paper_1101_1846_amd as R
    R.rng_init()
    return R


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available()
    return T


def _check(rng, torch, oracle, reqs, chunk):
    """reqs: (generator name, dtype name, offset, length, words before the output)."""
    n = len(reqs)
    pools = {g: torch.empty((rng.rng_state_words(rng.GENERATORS[g]), n), dtype=torch.int32, device="cuda") for g in GENS}
    for g, st in pools.items():
        rng.rng_seed(rng.GENERATORS[g], 17, 0, n, st)
    pos, at = 16, []
    for _, _, _, length, pad in reqs:
        at.append(pos + pad)
        pos = (pos + pad + length + 64) // 32 * 32
    out = torch.full((pos + 64,), -7, dtype=torch.int32, device="cuda")
    table = [(rng.GENERATORS[g], rng.DTYPES[t], pools[g].data_ptr() + 4 * i, n, off, length, out.data_ptr() + 4 * at[i])
             for i, (g, t, off, length, _) in enumerate(reqs)]
    h = rng.rng_batch_create(n, max(1, sum(r[3] for r in reqs)))
    try:
        if chunk:
            rng.rng_batch_set_shape(h, 0, 0, chunk)
        rng.rng_batch_set(h, rng.make_requests(table))
        rng.rng_batch_launch(h)
        torch.cuda.synchronize()
    finally:
        rng.rng_batch_destroy(h)
    got = out.cpu().numpy().view(np.uint32)
    used = np.zeros(len(got), dtype=bool)
    for i, (g, t, off, length, _) in enumerate(reqs):
        o = oracle.GENERATORS[g]
        st = np.ascontiguousarray(oracle.seed(o, 17, n)[:, i:i + 1])
        if off:
            oracle.skip(o, st, off)
        if length:
            ref = oracle.generate(o, st, length, rng.DTYPES[t], threads=1).view(np.uint32).reshape(-1)
            assert np.array_equal(got[at[i]:at[i] + length], ref), reqs[i]
        used[at[i]:at[i] + length] = True
        assert np.array_equal(pools[g].cpu().numpy().view(np.uint32)[:, i], st[:, 0]), reqs[i]
    assert (got[~used] == 0xFFFFFFF9).all()


@pytest.mark.parametrize("g", GENS)
@pytest.mark.parametrize("chunk", [0, 64, 4096])
def test_tile_edges(rng, torch, oracle, g, chunk):
    lengths = [1, 31, 32, 33, 2047, 2048, 2049, 4096, 4097, 65535, 65536, 65537 + 64]
    offsets = [0, 1, (1 << 40) - 1, 0, 4096, (1 << 63) + 5]
    reqs = [(g, ("u32", "f32")[i % 2], offsets[i % 6], n, (0, 1, 2, 3, 4, 5, 7)[i % 7]) for i, n in enumerate(lengths)]
    _check(rng, torch, oracle, reqs + [(g, "u32", 12345, 0, 0), (g, "u32", 0, 0, 0)], chunk)


def test_longest_rows_and_mixed_generators(rng, torch, oracle):
    reqs = [(g, t, 3 * k, n, k % 3) for k, (g, t, n) in enumerate(
        (g, t, n) for g in GENS for t in ("u32", "f32") for n in (5, 64 * 4096 + 1, 3 * 64 * 4096 - 7))]
    _check(rng, torch, oracle, reqs, 4096)
