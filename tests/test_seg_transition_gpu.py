"""The segments' transition products when they underflow (few long rows).

The product of a segment's transitions stops being formed once it is exactly
zero.  One call holds heads whose gates decay fast (zero after a few chunks),
slowly (never) and not at all, so that workgroups leave the loop at different
chunks; it must agree with the unsegmented scans as the two agree elsewhere
(outputs 2e-4, gradients 5e-4 of the largest entry: the operands carry about
16 bits in both).  A non-finite key in a skipped chunk must still reach every
later output of its head, and every earlier gradient that depends on it."""
import os

import numpy as np
import pytest

from comba_inputs import random_case
from gpu_helpers import gpu_bwd, gpu_fwd, maxrel, to_device

pytestmark = pytest.mark.gpu
ENV = "COMBA_SCAN_SEGMENTS"


@pytest.fixture(autouse=True)
def _env():
    old = os.environ.get(ENV)
    yield
    if old is None:
        os.environ.pop(ENV, None)
    else:
        os.environ[ENV] = old


def _mixed(d, T, P):
    print("mixed decay: d%d T%d P%d" % (d, T, P), flush=True)
    w = random_case(B=1, T=T, H=4, dk=d, dv=d, in_dtype="bf16", seed=97, dht=True)
    w.g *= np.array([1.0, 0.002, 0.0, 0.05], np.float32)
    return w


@pytest.mark.parametrize("d,T,P", [(64, 1024, 4), (128, 2048, 8), (256, 512, 2)])
def test_mixed_decay(d, T, P):
    w = _mixed(d, T, P)
    os.environ[ENV] = "1"
    o, ht = gpu_fwd(w)
    gr = gpu_bwd(w)
    os.environ[ENV] = str(P)
    o2, ht2 = gpu_fwd(w)
    gr2 = gpu_bwd(w)
    for h in range(4):
        assert maxrel(o2[:, :, h], o[:, :, h]) <= 2e-4, h
        assert maxrel(ht2[:, h], ht[:, h]) <= 2e-4, h
    for name in ("dq", "dk", "dv", "dg", "dbeta", "dh0"):
        assert maxrel(gr2[name], gr[name]) <= 5e-4, name


def _nan_in_a_skipped_chunk():
    """Four segments of 256 tokens; a NaN key of head 0 in the last chunk of segment 1
    (tokens 448-511).  The product of that head's transitions is exactly zero
    before it: every factor's norm is at most its decay (unit keys, beta < 1), and
    the decay over the chunks before it is below the smallest positive fp32."""
    w = _mixed(64, 1024, 4)
    assert w.g[0, 256:448, 0].sum() < np.log(2.0 ** -149) - 1
    w.k[0, 460, 0, 5] = np.nan
    return w


def test_a_nan_in_a_skipped_chunk_reaches_the_later_segments():
    w = _nan_in_a_skipped_chunk()
    os.environ[ENV] = "4"
    o, ht = gpu_fwd(w)
    assert np.isfinite(o[0, :448, 0]).all()
    assert np.isnan(o[0, 512:, 0]).all() and np.isnan(ht[0, 0]).all()
    assert np.isfinite(o[:, :, 1:]).all() and np.isfinite(ht[:, 1:]).all()


@pytest.mark.parametrize("saved", [False, True], ids=["stateless", "saved"])
def test_a_nan_in_a_skipped_chunk_reaches_the_earlier_gradients(saved):
    import torch

    import paper_2506_02475_amd as comba

    w = _nan_in_a_skipped_chunk()
    os.environ[ENV] = "4"
    a = to_device(w)
    args = tuple(a[n] for n in ("q", "k", "v", "g", "beta", "d", "h0"))
    if saved:
        _, _, ws = comba.comba_chunk_fwd_save(*args)
        gr = comba.comba_chunk_bwd_saved(*args, a["dO"], a["dht"], workspace=ws)
    else:
        gr = comba.comba_chunk_bwd(*args, a["dO"], a["dht"])
    torch.cuda.synchronize()
    gr = {n: x.cpu().numpy() for n, x in gr.items()}
    # through the state gradient that leaves segment 1, over zero transitions
    assert np.isnan(gr["dh0"][0, 0]).all()
    for n in ("dk", "dv"):
        assert np.isnan(gr[n][0, :448, 0]).all(), n
    # dq of tokens before the chunk depends on no later token
    assert np.isfinite(gr["dq"][0, :448, 0]).all() and np.isnan(gr["dq"][0, 512:, 0]).all()
    for n in ("dq", "dk", "dv", "dg", "dbeta"):
        assert np.isfinite(gr[n][:, :, 1:]).all(), n
    assert np.isfinite(gr["dh0"][0, 1:]).all()
