"""The scans' forms (LDS layout, operand loads, slice width) against each other.

Which form runs depends on the chains that are at work per CU, so the same row is
computed alone (few chains) and inside batches that pass each rule (320 to 1,024
chains of 32 columns on 256 CUs): its outputs, final state and gradients must be
bit for bit the same, since no form changes a row's arithmetic.  Ragged last
chunks and both sides' head sizes.  Packed batches, with empty sequences, are
computed with the host offsets (whole-row forward scan) and without them (the
lengths are not known: the direct one)."""
import copy
import os

import numpy as np
import pytest

from comba_inputs import random_case
from gpu_helpers import gpu_bwd, gpu_fwd, maxrel, to_device

pytestmark = pytest.mark.gpu

# enough full chunks and equal enough lengths for the whole-row form on 256 CUs
PACKED = [dict(H=16, dk=128, dv=128, seqlens=[448, 0, 511, 512, 575] * 6),
          dict(H=16, dk=128, dv=64, seqlens=[640, 1, 639, 705, 0] * 12),
          dict(H=16, dk=64, dv=64, seqlens=[513, 0, 640, 576, 64] * 13)]


# nearly full chunks: 64 rows take the whole-row form
FULL = [(128, 128, 127), (128, 64, 191), (128, 256, 127), (64, 64, 703), (64, 128, 639)]


@pytest.mark.parametrize("B", [20, 33, 64])
@pytest.mark.parametrize("dk,dv,T", [(128, 128, 130), (64, 64, 65), (64, 128, 63), (128, 64, 200),
                                     (128, 256, 70)] + FULL)
def test_a_row_does_not_depend_on_its_batch(B, dk, dv, T):
    import torch

    import paper_2506_02475_amd as comba

    H = 4 * 128 // dv  # 16 chains of 32 columns per row
    print("case B%d H%d dk%d dv%d T%d" % (B, H, dk, dv, T), flush=True)
    w = random_case(B=B, T=T, H=H, dk=dk, dv=dv, in_dtype="bf16", seed=83, dht=True)
    a = to_device(w)
    names = ("q", "k", "v", "g", "beta")

    def calls(x, h0, dO, dht):
        args = tuple(x[n] for n in names) + (a["d"], h0)
        o, ht = comba.comba_chunk_fwd(*args)
        o_s, ht_s, ws = comba.comba_chunk_fwd_save(*args)
        gr = comba.comba_chunk_bwd_saved(*args, dO, dht, workspace=ws)
        assert torch.equal(o, o_s) and torch.equal(ht, ht_s)
        return o, ht, gr

    o, ht, gr = calls(a, a["h0"], a["dO"], a["dht"])
    for b in (0, B - 1):
        one = {n: a[n][b:b + 1].contiguous() for n in names}
        o1, ht1, gr1 = calls(one, a["h0"][b:b + 1].contiguous(), a["dO"][b:b + 1].contiguous(),
                             a["dht"][b:b + 1].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(o1[0], o[b]) and torch.equal(ht1[0], ht[b])
        for n in ("dq", "dk", "dv", "dg", "dbeta", "dh0"):
            assert torch.equal(gr1[n][0], gr[n][b]), n


@pytest.mark.parametrize("kw", PACKED, ids=lambda kw: "%d-%d" % (kw["dk"], kw["dv"]))
def test_packed_forms_agree(kw):
    import torch

    import paper_2506_02475_amd as comba

    print("case", kw["H"], kw["dk"], kw["dv"], len(kw["seqlens"]), flush=True)
    w = random_case(T=0, in_dtype="bf16", seed=89, dht=True, **kw)
    a = to_device(w)
    args = tuple(a[n] for n in ("q", "k", "v", "g", "beta", "d", "h0"))
    host = np.concatenate([[0], np.cumsum(kw["seqlens"])]).astype(np.int32)
    res = []
    for h in (None, host):
        kws = dict(cu_seqlens=a["cu_seqlens"], cu_seqlens_host=h)
        o, ht = comba.comba_chunk_fwd(*args, **kws)
        o_s, ht_s, ws = comba.comba_chunk_fwd_save(*args, **kws)
        gr = comba.comba_chunk_bwd_saved(*args, a["dO"], a["dht"], workspace=ws, **kws)
        res.append(dict(gr, o=o, ht=ht, o_s=o_s, ht_s=ht_s))
    torch.cuda.synchronize()
    for n, x in res[0].items():
        assert torch.equal(x, res[1][n]), n
    assert torch.equal(res[0]["o"], res[0]["o_s"]) and torch.isfinite(res[0]["dq"]).all()


@pytest.mark.parametrize("dv,P", [(128, 8), (64, 16)])
def test_segmented_reverse_scans_in_the_unpadded_form(dv, P, monkeypatch):
    """448 / 480 chains in the reverse state pass, 512 in the reverse scan: both
    unpadded.  Against the unsegmented scans (64 / 32 chains: padded), as the two
    agree elsewhere (operands of about 16 bits in both: outputs 2e-4, gradients
    5e-4 of the largest entry)."""
    print("case dv%d P%d" % (dv, P), flush=True)
    w = random_case(B=1, T=8192, H=16, dk=128, dv=dv, in_dtype="bf16", seed=41, dht=True)
    w.g *= np.linspace(0.0, 1.0, 16, dtype=np.float32)  # heads with and without decay
    monkeypatch.setenv("COMBA_SCAN_SEGMENTS", "1")
    o, ht = gpu_fwd(w)
    gr = gpu_bwd(w)
    monkeypatch.setenv("COMBA_SCAN_SEGMENTS", str(P))
    o2, ht2 = gpu_fwd(w)
    gr2 = gpu_bwd(w)
    for h in range(16):
        assert maxrel(o2[:, :, h], o[:, :, h]) <= 2e-4 and maxrel(ht2[:, h], ht[:, h]) <= 2e-4, h
    for n in ("dq", "dk", "dv", "dg", "dbeta", "dh0"):
        assert maxrel(gr2[n], gr[n]) <= 5e-4, n


# few chains (16-column slices where nothing is stored, padded tiles), many
# (whole rows, unpadded tiles), and the fp32 kernels
NONFINITE = [("bf16", 128, 1), ("bf16", 128, 64), ("bf16", 64, 1), ("bf16", 256, 1), ("f32", 64, 2)]


@pytest.mark.parametrize("dtype,d,B", NONFINITE)
@pytest.mark.parametrize("where", ["k", "v", "q"])
def test_non_finite_values_in_every_form(dtype, d, B, where):
    """A NaN in chunk 1 of row 0, head 0, and an infinite upstream gradient in its
    chunk 2: what depends on them is not finite, everything else bit for bit the
    clean run's."""
    import torch

    import paper_2506_02475_amd as comba

    print("case", dtype, d, B, where, flush=True)
    clean = random_case(B=B, T=191, H=4, dk=d, dv=d, in_dtype=dtype, seed=61, dht=True)
    bad = copy.deepcopy(clean)
    getattr(bad, where)[0, 70, 0, 7] = np.nan
    bad.dO[0, 150, 0, 3] = np.inf

    def run(w):
        a = to_device(w)
        args = tuple(a[n] for n in ("q", "k", "v", "g", "beta", "d", "h0"))
        o, ht = comba.comba_chunk_fwd(*args)
        o_s, ht_s, ws = comba.comba_chunk_fwd_save(*args)
        gr = comba.comba_chunk_bwd_saved(*args, a["dO"], a["dht"], workspace=ws)
        gr_r = comba.comba_chunk_bwd(*args, a["dO"], a["dht"])
        out = dict(gr, o=o, ht=ht, o_s=o_s, ht_s=ht_s)
        out.update({n + "_r": x for n, x in gr_r.items()})
        torch.cuda.synchronize()
        return {n: x.cpu().numpy() for n, x in out.items()}

    rc, rb = run(clean), run(bad)
    for n, x in rc.items():
        y = rb[n]
        assert np.isfinite(x).all(), n
        if n.startswith("dd"):  # sums over the rows of a head
            assert np.array_equal(x[1:], y[1:]) and not np.isfinite(y[0]), n
            continue
        assert np.array_equal(x[1:], y[1:]), n                        # other rows
        heads = 1 if n.startswith(("ht", "dh0")) else 2               # [N, H, ..] or [B, T, H, ..]
        assert np.array_equal(np.take(x[0], [1, 2, 3], heads - 1), np.take(y[0], [1, 2, 3], heads - 1)), n
    for n in ("o", "o_s"):
        assert np.array_equal(rb[n][0, :64, 0], rc[n][0, :64, 0]), n  # before the chunk
        col = slice(None) if where == "k" else 7
        if where != "q":  # the state takes it up
            assert not np.isfinite(rb[n][0, 128:, 0, col]).any(), n
        else:
            assert not np.isfinite(rb[n][0, 70, 0]).all()
    for n in ("ht", "ht_s"):
        assert np.isfinite(rb[n][0, 0]).all() == (where == "q"), n
    for n in ("dq", "dk", "dv", "dg", "dbeta", "dh0"):
        for m in (n, n + "_r"):
            y = rb[m][0, 0] if n == "dh0" else rb[m][0, :, 0]
            assert not np.isfinite(y).all(), m
