"""Which kernel takes a call's rows (line by line, chunks of a wave, windows of a
sequence, or the general one), on both sides of each limit, against the serial
CPU oracle, bit for bit, and the fused consumer around the limit of its windows.
Whole numbers: no tolerance."""
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
    R.rng_seed(g, 29, 0, S, st)
    buf = torch.full((S * N + off + 32,), -7, dtype=torch.int32, device="cuda")
    ref_st = oracle.seed(o, 29, S)
    for _ in range(2):  # the second call continues from the states that the first wrote
        R.rng_generate(g, st, S, N, t, buf[off:off + S * N])
        torch.cuda.synchronize()
        ref = oracle.generate(o, ref_st, N, t, threads=8).view(np.uint32)
        h = buf.cpu().numpy()
        assert (h[:off] == -7).all() and (h[off + S * N:] == -7).all()
        assert np.array_equal(h[off:off + S * N].view(np.uint32).reshape(S, N), ref)
        assert np.array_equal(st.cpu().numpy().view(np.uint32), ref_st)


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("dt,S,N,off", [
    ("u32", 63, 168, 0), ("u32", 64, 168, 0), ("f32", 100, 188, 4), ("u32", 100, 192, 4), ("f32", 500, 396, 0),
    ("u32", 8193, 400, 0), ("f32", 1024, 1532, 0), ("u32", 1025, 1532, 8), ("f32", 1025, 1536, 8), ("u32", 16385, 300, 0),
    ("f32", 70, 127, 1), ("u32", 70, 129, 1), ("f32", 33000, 96, 0), ("u32", 32768, 96, 0), ("f32", 65537, 100, 0),
    ("u32", 8191, 512, 0), ("f32", 8192, 512, 0), ("f32", 511, 8188, 0), ("u32", 513, 8192, 0), ("f32", 600, 16384, 0),
    ("u32", 513, 16380, 0), ("u32", 8192, 3072, 0), ("f32", 12289, 4096, 0), ("u32", 8200, 3104, 0)])
def test_row_rules(oracle, name, dt, S, N, off):
    run(oracle, name, dt, S, N, off)


@pytest.mark.parametrize("S,n", [(64, 262145), (200, 530637), (8192, 255), (8192, 3000), (8193, 3000)])
def test_pi_limits(oracle, S, n):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o = R.GENERATORS["XS256"], oracle.GENERATORS["XS256"]
    st = torch.empty((R.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    R.rng_seed(g, 8, 0, S, st)
    R.rng_fused_pi(g, st, S, n, cnt)
    torch.cuda.synchronize()
    assert int(cnt.item()) == oracle.fused_pi(o, oracle.seed(o, 8, S), n, threads=8)
    end = oracle.seed(o, 8, S)
    oracle.skip(o, end, n)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), end)
