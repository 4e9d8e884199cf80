"""One long sequence over the device (split, leapfrog and few-stream bulk
generation) against the serial CPU oracle, bit for bit, at the edges of its
windows (64 blocks of 32, 64 or 128 numbers), of 128-byte lines and of the
thread count.  Whole numbers: no tolerance."""
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


def _host(t):
    import torch as T
    T.cuda.synchronize()
    return t.cpu().numpy().view(np.uint32)


def _one(torch, rng, op, name, dt, total, threads, off, alias):
    """The call's numbers and final state, with 64 guard words on each side of the output."""
    g = rng.GENERATORS[name]
    st = torch.empty((rng.rng_state_words(g), 1), dtype=torch.int32, device="cuda")
    rng.rng_seed(g, 91, 0, 1, st)
    fin = st if alias else torch.zeros_like(st)
    buf = torch.full((total + off + 128,), -7, dtype=torch.int32, device="cuda")
    out = buf[64 + off:64 + off + total]
    size = rng.rng_split_workspace_bytes if op == "split" else rng.rng_leapfrog_workspace_bytes
    call = rng.rng_generate_split if op == "split" else rng.rng_generate_leapfrog
    nb = size(g, threads)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    call(g, st, total, threads, rng.DTYPES[dt], out, fin, ws, nb)
    h = _host(buf)
    assert (h[:64 + off] == np.uint32(0xFFFFFFF9)).all() and (h[64 + off + total:] == np.uint32(0xFFFFFFF9)).all()
    return h[64 + off:64 + off + total], _host(fin).reshape(-1)


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("op", ["split", "leapfrog"])
@pytest.mark.parametrize("dt,total,threads,off", [
    ("u32", 1, 1, 0), ("f32", 31, 7, 1), ("u32", 33, 64, 31), ("f32", 2047, 2, 0), ("u32", 2048, 2048, 3),
    ("u32", 2049 + 29, 100, 3), ("f32", 100003, 1000, 30), ("u32", (1 << 21) - 1, 1 << 14, 0),
    ("f32", (1 << 21) + 4097, 4099, 17), ("u32", (1 << 23) + 8192, 1 << 16, 0), ("u32", (1 << 23) + 8191 + 5, 99991, 27),
    ("f32", 20 * (1 << 20) + 1, 3, 2)])
def test_sequence_edges(rng, torch, oracle, name, op, dt, total, threads, off):
    o = oracle.GENERATORS[name]
    ref_st = oracle.seed(o, 91, 1)
    ref = oracle.generate(o, ref_st, total, rng.DTYPES[dt], threads=1).view(np.uint32).reshape(-1)
    for alias in (False, True):
        out, fin = _one(torch, rng, op, name, dt, total, threads, off, alias)
        assert np.array_equal(out, ref)
        assert np.array_equal(fin, ref_st.reshape(-1))


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("dt,S,N,off", [("u32", 1, 2048, 1), ("f32", 3, 2079, 5), ("u32", 63, 4099, 0),
                                        ("f32", 40, 70001, 31), ("u32", 7, (1 << 20) + 13, 2), ("f32", 33, 1 << 18, 0)])
def test_few_streams(rng, torch, oracle, name, dt, S, N, off):
    g, o, t = rng.GENERATORS[name], oracle.GENERATORS[name], rng.DTYPES[dt]
    st = torch.empty((rng.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    rng.rng_seed(g, 12, 0, S, st)
    buf = torch.full((S * N + off + 64,), -7, dtype=torch.int32, device="cuda")
    rng.rng_generate(g, st, S, N, t, buf[off:off + S * N])
    ref_st = oracle.seed(o, 12, S)
    ref = oracle.generate(o, ref_st, N, t, threads=8).view(np.uint32)
    h = _host(buf)
    assert (h[:off] == np.uint32(0xFFFFFFF9)).all() and (h[off + S * N:] == np.uint32(0xFFFFFFF9)).all()
    assert np.array_equal(h[off:off + S * N].reshape(S, N), ref)
    assert np.array_equal(_host(st), ref_st)
