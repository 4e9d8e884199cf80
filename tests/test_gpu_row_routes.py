"""The limits between the kernels that take a call's rows, on both sides, where
test_gpu_row_rules.py does not reach: fewer rows than lanes, whole tiles and short
rows of more than 65536 streams, 16 KiB runs at as many runs as CUs, XS256 windows
above 1024 streams, the four-chunk rows between them, and the fused consumer in
chunks.  Against the serial CPU oracle, bit for bit; whole numbers: no tolerance."""
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
    R.rng_seed(g, 37, 0, S, st)
    buf = torch.full((S * N + off + 32,), -7, dtype=torch.int32, device="cuda")
    ref_st = oracle.seed(o, 37, S)
    for _ in range(2):  # the second call continues from the states that the first wrote
        R.rng_generate(g, st, S, N, t, buf[off:off + S * N])
        torch.cuda.synchronize()
        ref = oracle.generate(o, ref_st, N, t, threads=16).view(np.uint32)
        h = buf.cpu().numpy()
        assert (h[:off] == -7).all() and (h[off + S * N:] == -7).all()
        assert np.array_equal(h[off:off + S * N].view(np.uint32).reshape(S, N), ref)
        assert np.array_equal(st.cpu().numpy().view(np.uint32), ref_st)


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("dt,S,N,off", [
    # fewer rows than lanes
    ("u32", 3, 127, 1), ("f32", 33, 128, 1), ("u32", 63, 128, 4), ("f32", 10, 96, 0), ("u32", 1, 339, 4), ("f32", 63, 340, 0),
    ("u32", 7, 512, 4), ("f32", 2, 2500, 0), ("u32", 33, 4095, 3), ("f32", 5, 4100, 0), ("u32", 20, 5999, 2), ("f32", 20, 6000, 4),
    # whole tiles and lines
    ("u32", 8192, 1024, 0), ("f32", 8256, 1024, 0), ("u32", 8255, 1024, 0), ("u32", 12288, 4096, 0), ("u32", 9000, 12288, 0),
    ("u32", 200, 96, 0), ("u32", 5000, 416, 0),
    # more than 65536 streams
    ("u32", 65536, 512, 4), ("f32", 65537, 512, 4), ("u32", 66001, 640, 8), ("u32", 66001, 516, 4), ("f32", 262144, 200, 4),
    ("u32", 262145, 200, 0), ("u32", 262200, 256, 4), ("u32", 66001, 60, 0), ("f32", 70000, 64, 4),
    # windows, chunks and rows of the cheap generators and of KISS
    ("u32", 256, 11999, 4), ("f32", 257, 12000, 4), ("u32", 512, 19999, 1), ("f32", 300, 20000, 0), ("u32", 8191, 1300, 4),
    ("f32", 8192, 1100, 0), ("u32", 8192, 1096, 4), ("f32", 9000, 1700, 4),
    # 16 KiB runs at 256 runs of 64 lanes and one more
    ("u32", 65536, 1024, 0), ("u32", 65792, 1024, 0), ("f32", 32896, 2048, 0)])
def test_routes(oracle, name, dt, S, N, off):
    run(oracle, name, dt, S, N, off)


@pytest.mark.parametrize("dt,S,N,off", [("u32", 4097, 16385, 0), ("f32", 4097, 16384, 3), ("u32", 1025, 16385, 1),
                                        ("f32", 1025, 20001, 2), ("u32", 4096, 3072, 4), ("f32", 4096, 3072, 1),
                                        ("u32", 1088, 5120, 4), ("u32", 66000, 1024, 0), ("u32", 130000, 1024, 0)])
def test_xs256_long_rows(oracle, dt, S, N, off):
    run(oracle, "XS256", dt, S, N, off)


# XS256 chunks of the fused consumer: above the windows' stream counts, and where
# the windows' starts and idle lanes would take 3 10^8 steps (8192 x 33000 and 70001;
# 8192 x 36900 stays below)
@pytest.mark.parametrize("S,n", [(8193, 8193), (8192, 33000), (8192, 36900), (8192, 70001), (8192, 8192)])
def test_xs256_pi_chunks(oracle, S, n):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o = R.GENERATORS["XS256"], oracle.GENERATORS["XS256"]
    st = torch.empty((R.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    R.rng_seed(g, 8, 0, S, st)
    R.rng_fused_pi(g, st, S, n, cnt)
    torch.cuda.synchronize()
    ref_st = oracle.seed(o, 8, S)
    assert int(cnt.item()) == oracle.fused_pi(o, ref_st, n, threads=16)
    oracle.skip(o, end := oracle.seed(o, 8, S), n)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), end)


# few numbers per stream: a lane each up to these lengths, a window with idle lanes above
@pytest.mark.parametrize("name,S,n", [("XS256", 1, 339), ("XS256", 1, 341), ("XS256", 300, 387), ("XS256", 300, 389),
                                      ("XS256", 8192, 1650), ("XS256", 8192, 1651), ("KISS", 63, 319), ("KISS", 63, 321),
                                      ("MWC32", 8, 255), ("XS32", 63, 257), ("MWC1616", 5, 513), ("KISS", 7, 512)])
def test_pi_short(oracle, name, S, n):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o = R.GENERATORS[name], oracle.GENERATORS[name]
    st = torch.empty((R.rng_state_words(g), S), dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), 9, dtype=torch.int64, device="cuda")
    R.rng_seed(g, 8, 0, S, st)
    R.rng_fused_pi(g, st, S, n, cnt)
    torch.cuda.synchronize()
    ref_st = oracle.seed(o, 8, S)
    assert int(cnt.item()) == 9 + oracle.fused_pi(o, ref_st, n, threads=8)
    oracle.skip(o, end := oracle.seed(o, 8, S), n)
    assert np.array_equal(st.cpu().numpy().view(np.uint32), end)
