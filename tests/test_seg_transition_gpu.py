"""The segments' transition products when they underflow (few long rows).

The product of a segment's transitions stops being formed once it is exactly
zero.  One call holds heads whose gates decay fast (zero after a few chunks),
slowly (never) and not at all, so that workgroups leave the loop at different
chunks; it must agree with the unsegmented scans as the two agree elsewhere
(outputs 2e-4, gradients 5e-4 of the largest entry: the operands carry about
16 bits in both).  A non-finite key in a skipped chunk must still reach every
later output of its head."""
import os

import numpy as np
import pytest

from comba_inputs import random_case
from gpu_helpers import gpu_bwd, gpu_fwd, maxrel

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


def test_a_nan_in_a_skipped_chunk_reaches_the_later_segments():
    w = _mixed(64, 1024, 4)
    w.k[0, 300, 0, 5] = np.nan          # head 0 decays: segment 1's product is zero by its chunk 4
    os.environ[ENV] = "4"
    o, ht = gpu_fwd(w)
    assert np.isfinite(o[0, :256, 0]).all()
    assert np.isnan(o[0, 320:, 0]).all() and np.isnan(ht[0, 0]).all()
    assert np.isfinite(o[:, :, 1:]).all() and np.isfinite(ht[:, 1:]).all()
