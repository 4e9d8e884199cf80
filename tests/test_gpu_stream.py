"""A call without a stream runs on torch's current one, inside and outside a
stream context."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_default_stream_is_the_current_one(oracle):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    side = torch.cuda.Stream()
    assert R._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert R._stream(None) == side.cuda_stream
        st = torch.empty((2, 256), dtype=torch.int32, device="cuda")
        out = torch.empty((256, 512), dtype=torch.int32, device="cuda")
        R.rng_seed(R.RNG_MWC32, 3, 0, 256, st)
        R.rng_generate(R.RNG_MWC32, st, 256, 512, R.RNG_U32, out)
        side.synchronize()
        got = out.cpu().numpy().view(np.uint32)
    assert R._stream(None) == torch.cuda.current_stream().cuda_stream
    o = oracle.GENERATORS["MWC32"]
    assert np.array_equal(got, oracle.generate(o, oracle.seed(o, 3, 256), 512, R.RNG_U32, threads=2))
