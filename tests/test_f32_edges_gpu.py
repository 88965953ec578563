"""The fp32 path at the edges of its tiles: chunks of 1 to 64 rows (the 16-row
blocks of the triangular inverse and of the products that skip its zero
blocks), several chunks, packed sequences with empty ones, the forward that
keeps its intermediates in the rows of the output, the training pair and the
no-allocation entry point.  Against the fp64 oracle at the operator's bar for
fp32 inputs (1e-5 of the largest entry: about 64 sums of 64 products, each with
a rounding error of 2^-24)."""
import pytest

from comba_inputs import random_case
from gpu_helpers import check_bwd, check_fwd, to_device

pytestmark = pytest.mark.gpu

CASES = [dict(B=1, T=t, H=1) for t in (1, 15, 16, 17, 33, 63, 64, 65)] + \
    [dict(B=2, T=130, H=3), dict(B=3, T=257, H=5), dict(T=0, H=3, seqlens=[1, 0, 64, 65, 200, 0])]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: "-".join(str(v) for v in kw.values()))
@pytest.mark.parametrize("bt", [False, True], ids=["tied", "separate"])
def test_f32_tile_edges(kw, bt):
    import torch

    import paper_2506_02475_amd as comba

    print("case", kw, bt, flush=True)
    w = random_case(seed=53, dk=64, dv=64, in_dtype="f32", dht=True, beta_tilde=bt, **kw)
    check_fwd(w)
    check_bwd(w)
    # the pair that keeps its state and the stateless calls: the same arithmetic
    a = to_device(w)
    args = (a["q"], a["k"], a["v"], a["g"], a["beta"], a["d"], a["h0"])
    kws = dict(cu_seqlens=a["cu_seqlens"], beta_tilde=a["beta_tilde"])
    o, ht = comba.comba_chunk_fwd(*args, **kws)
    o_s, ht_s, ws = comba.comba_chunk_fwd_save(*args, **kws)
    o_n, ht_n = comba.comba_chunk_fwd_noalloc(*args, **kws)
    gr = comba.comba_chunk_bwd(*args, a["dO"], a["dht"], **kws)
    gr_s = comba.comba_chunk_bwd_saved(*args, a["dO"], a["dht"], workspace=ws, **kws)
    torch.cuda.synchronize()
    for x in (o_s, o_n):
        assert torch.equal(o, x)
    for x in (ht_s, ht_n):
        assert torch.equal(ht, x)
    for name in gr:
        assert torch.equal(gr[name], gr_s[name]), name
