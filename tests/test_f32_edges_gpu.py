"""The fp32 path at the edges of its tiles: chunks of 1 to 64 rows (the 16-row
blocks of the triangular inverse and of the products that skip its zero
blocks), several chunks, packed sequences with empty ones, the forward that
keeps its intermediates in the rows of the output, the training pair and the
no-allocation entry point.  Against the fp64 oracle at the operator's bar for
fp32 inputs (1e-5 of the largest entry: about 64 sums of 64 products, each with
a rounding error of 2^-24)."""
import numpy as np
import pytest

import oracle
from comba_inputs import random_case
from gpu_helpers import check_bwd, check_fwd, gpu_bwd, gpu_fwd, to_device

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


def test_one_empty_sequence():
    # one chunk slot, empty: dd has one partial and it is zero
    w = random_case(T=0, H=3, dk=64, dv=64, in_dtype="f32", seed=3, dht=True, seqlens=[0])
    gr = gpu_bwd(w)
    assert not gr["dd"].any() and np.array_equal(gr["dh0"], w.dht)


def test_more_chains_than_one_grid_dimension():
    """18,000 chains: the chains' grid has two dimensions (more than 65,536
    workgroups); bit for bit the two halves of the batch."""
    import torch

    import paper_2506_02475_amd as comba

    print("case 4500 rows, 4 heads", flush=True)
    w = random_case(B=4500, T=2, H=4, dk=64, dv=64, in_dtype="f32", seed=7, dht=True)
    a = to_device(w)
    names = ("q", "k", "v", "g", "beta")

    def call(i, j):
        args = tuple(a[n][i:j].contiguous() for n in names) + (a["d"], a["h0"][i:j].contiguous())
        o, ht = comba.comba_chunk_fwd(*args)
        gr = comba.comba_chunk_bwd(*args, a["dO"][i:j].contiguous(), a["dht"][i:j].contiguous())
        return dict({n: gr[n] for n in ("dq", "dk", "dv", "dg", "dbeta", "dh0")}, o=o, ht=ht)

    whole, lo, hi = call(0, 4500), call(0, 2250), call(2250, 4500)
    torch.cuda.synchronize()
    for n, x in whole.items():
        assert torch.equal(x, torch.cat([lo[n], hi[n]])), n


@pytest.mark.parametrize("gate,corr,bar", [(0.01, 0.9, 5.8e-7), (0.01, 0.99, 6.6e-7),
                                           (0.0, 0.99, 7.4e-7)])
def test_similar_keys_and_slow_gates(gate, corr, bar):
    """Where fp32 rounding adds up most: keys correlated with one another, states
    that hardly decay.  The bar on o (2-norm) lies between the error of the
    chunk form's products on Q and K themselves and that of products on a
    rounded Q - d K, which the sums over similar keys do not average out."""
    w = random_case(B=1, T=512, H=8, dk=64, dv=64, in_dtype="f32", seed=11, dht=True)
    w.g *= np.float32(gate)
    base = np.random.default_rng(12).standard_normal((1, 1, 8, 64)).astype(np.float32)
    base /= np.linalg.norm(base, axis=-1, keepdims=True)
    k = np.float32(np.sqrt(corr)) * base + np.float32(np.sqrt(1 - corr)) * w.k
    w.k[...] = (k / np.linalg.norm(k, axis=-1, keepdims=True)).astype(np.float32)
    o, ht = gpu_fwd(w)
    ro, _ = oracle.step_fwd(w.q, w.k, w.v, w.g, w.beta, w.d, w.h0)
    err = np.linalg.norm(o.astype(np.float64) - ro) / np.linalg.norm(ro)
    print("2-norm error of o: %.3g" % err, flush=True)
    check_fwd(w)
    check_bwd(w)
    assert err <= bar
