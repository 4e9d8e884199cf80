"""Streams cut into chunks, all of a stream in one wave (rng_generate with fewer
streams than the device has lanes), against the serial CPU oracle, bit for bit:
chunk counts from 2 to 64, row lengths that leave a longer last chunk, every
generator, partial last groups and misaligned outputs.  Whole numbers: no
tolerance."""
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


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("dt,S,N,off", [
    ("u32", 1025, 128, 0), ("f32", 1033, 129, 3), ("u32", 2000, 255, 0), ("f32", 4096, 1024, 0), ("u32", 4099, 1000, 17),
    ("f32", 1500, 4097, 1), ("u32", 1100, 16383, 0), ("f32", 20001, 193, 31), ("u32", 40000, 256, 0), ("f32", 65000, 130, 2),
    ("u32", 1030, 70016, 0), ("f32", 7, 200, 5), ("u32", 64, 2047, 0), ("u32", 1, 128, 0), ("f32", 3, 1999, 30)])
def test_row_chunks(rng, torch, oracle, name, dt, S, N, off):
    g, o, t = rng.GENERATORS[name], oracle.GENERATORS[name], rng.DTYPES[dt]
    st = torch.empty((rng.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    rng.rng_seed(g, 23, 0, S, st)
    buf = torch.full((S * N + off + 64,), -7, dtype=torch.int32, device="cuda")
    ref_st = oracle.seed(o, 23, S)
    for _ in range(2):  # the second call continues from the states that the first wrote
        rng.rng_generate(g, st, S, N, t, buf[off:off + S * N])
        torch.cuda.synchronize()
        ref = oracle.generate(o, ref_st, N, t, threads=8).view(np.uint32)
        h = buf.cpu().numpy().view(np.uint32)
        assert (h[:off] == GUARD).all() and (h[off + S * N:] == GUARD).all()
        assert np.array_equal(h[off:off + S * N].reshape(S, N), ref)
        assert np.array_equal(st.cpu().numpy().view(np.uint32), ref_st)
