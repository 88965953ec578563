"""The sequence and chunk tables of packed batches: one launch for up to 1,024
sequences (256 per pass, several workgroups filling chunk slots), two beyond.
The chunk-wise forward over many short, empty and chunk-long sequences against
the token-by-token entry point, which uses no tables (2e-3, the operator's bar
for bf16 inputs)."""
import numpy as np
import pytest

from comba_inputs import random_case
from gpu_helpers import maxrel, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 257, 1024, 1025])
def test_many_sequences(n):
    import torch

    import paper_2506_02475_amd as comba

    print("sequences:", n, flush=True)
    rng = np.random.default_rng(n)
    lens = [int(x) for x in rng.choice([0, 1, 2, 5, 64, 65], size=n)]
    w = random_case(T=0, H=1, dk=64, dv=64, in_dtype="bf16", seed=n, grad=False, seqlens=lens)
    a = to_device(w)
    args = (a["q"], a["k"], a["v"], a["g"], a["beta"], a["d"], a["h0"])
    o, ht = comba.comba_chunk_fwd(*args, cu_seqlens=a["cu_seqlens"])
    o2, ht2 = comba.comba_recurrent_fwd(*args, cu_seqlens=a["cu_seqlens"])
    torch.cuda.synchronize()
    if o.numel():
        assert maxrel(o.cpu().numpy(), o2.cpu().numpy()) <= 2e-3
    assert maxrel(ht.cpu().numpy(), ht2.cpu().numpy()) <= 2e-3
