"""Rows of any length, count and alignment (rng_generate with one row per lane)
against the serial CPU oracle, bit for bit: lengths around whole lines (32
numbers) and tiles (128), partial last groups, every residue of the output
within a line, and more groups than one pass of the waves takes.  Whole
numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GENS = ["MWC32", "XS256", "XS32", "KISS", "MWC1616"]
GUARD = 0xFFFFFFF9


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


def _check(rng, torch, oracle, name, dt, S, N, off):
    g, o, t = rng.GENERATORS[name], oracle.GENERATORS[name], rng.DTYPES[dt]
    st = torch.empty((rng.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    rng.rng_seed(g, 5, 0, S, st)
    buf = torch.full((S * N + off + 64,), -7, dtype=torch.int32, device="cuda")
    rng.rng_generate(g, st, S, N, t, buf[off:off + S * N])
    torch.cuda.synchronize()
    ref_st = oracle.seed(o, 5, S)
    ref = oracle.generate(o, ref_st, N, t, threads=8).view(np.uint32)
    h = buf.cpu().numpy().view(np.uint32)
    assert (h[:off] == GUARD).all() and (h[off + S * N:] == GUARD).all()
    assert np.array_equal(h[off:off + S * N].reshape(S, N), ref)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), ref_st)


@pytest.mark.parametrize("N", [32, 33, 63, 64, 95, 100, 127, 129, 159, 160, 161, 191, 255, 257, 288, 1000, 1001, 4111])
@pytest.mark.parametrize("S,off", [(64, 0), (1, 3), (65, 8), (191, 29), (1030, 0)])
def test_rows_xs256(rng, torch, oracle, S, N, off):
    _check(rng, torch, oracle, "XS256", "u32", S, N, off)


@pytest.mark.parametrize("off", range(32))
def test_rows_every_residue(rng, torch, oracle, off):
    _check(rng, torch, oracle, "XS256", "f32", 130, 387, off)


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("dt,S,N,off", [("u32", 65536 + 64, 100, 0), ("f32", 65536 + 7, 125, 4), ("u32", 98304 - 1, 296, 1),
                                        ("f32", 131072, 127, 0), ("u32", 65599, 288, 0), ("f32", 70001, 161, 19)])
def test_rows_generators(rng, torch, oracle, name, dt, S, N, off):
    _check(rng, torch, oracle, name, dt, S, N, off)


@pytest.mark.parametrize("name", ["MWC32", "XS256"])
def test_rows_more_groups_than_one_pass(rng, torch, oracle, name):
    _check(rng, torch, oracle, name, "u32", (1 << 20) + 65, 33, 5)
