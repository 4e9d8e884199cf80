"""Start and final states that lie inside the output of a split or leapfrogged
sequence, or inside its workspace: the numbers come from the state as it was before
the call, and the final state is written last, over the numbers.  Against the serial
CPU oracle; whole numbers: no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GENS = ["MWC32", "XS256", "XS32", "KISS", "MWC1616"]


@pytest.mark.parametrize("name", GENS)
@pytest.mark.parametrize("total,threads", [(40, 1), (5000, 64), (300007, 1000)])
# where the states lie: words into the output, "ws" words into the workspace, None: a buffer of its own
@pytest.mark.parametrize("op,start,final", [
    (op, start, final) for op in ("split", "noalloc", "leapfrog")
    for start, final in (("first", None), ("last", None), (None, "first"), (None, "last"), ("mid", "mid"), ("first", "last"),
                         ("mid", "half"), ("first", "ws"), ("ws", "ws"), ("ws", "first"), (None, "ws"))
    if op != "noalloc" or "ws" not in (start, final)])
def test_states_inside_the_output(oracle, name, op, total, threads, start, final):
    import torch
    import paper_1101_1846_amd as R
    R.rng_init()
    g, o = R.GENERATORS[name], oracle.GENERATORS[name]
    w = R.rng_state_words(g)
    nb = max(R.rng_split_workspace_bytes(g, threads), R.rng_leapfrog_workspace_bytes(g, threads))
    buf = torch.full((total + 16,), -7, dtype=torch.int32, device="cuda")
    ws = torch.zeros(nb // 4, dtype=torch.int32, device="cuda")
    # "mid" straddles nothing; "half" overlaps "mid" by part of a state
    at = {"first": 0, "last": total - w, "mid": (total - w) // 2, "half": (total - w) // 2 + w // 2}

    def place(where):
        if where is None:
            return torch.zeros(w, dtype=torch.int32, device="cuda"), None
        if where == "ws":
            return ws[:w], None
        return buf[at[where]:at[where] + w], at[where]

    (st, _), (fin, f) = place(start), place(final)
    R.rng_seed(g, 44, 0, 1, st)
    out = buf[:total]
    if op == "noalloc":
        R.rng_generate_split_noalloc(g, st, total, threads, 0, out, fin)
    else:
        call = R.rng_generate_split if op == "split" else R.rng_generate_leapfrog
        call(g, st, total, threads, 0, out, fin, ws, nb)
    torch.cuda.synchronize()
    ref_st = oracle.seed(o, 44, 1)
    ref = oracle.generate(o, ref_st, total, 0, threads=1).view(np.uint32).reshape(-1).copy()
    ref_st = ref_st.reshape(-1)
    if f is not None:
        ref[f:f + w] = ref_st
    got = buf.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[:total], ref)
    assert (got[total:] == 0xFFFFFFF9).all()
    assert np.array_equal(fin.cpu().numpy().view(np.uint32), ref_st)
