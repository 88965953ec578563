"""The forward scan's 16-column slices (few chains) against its 32-column ones.

The stateless forward takes 16-column slices when they are at most one per CU,
the forward that saves its state always 32: outputs and final states must be
bit for bit the same, on both sides of the rule (128 chains of 32 columns on 256
CUs), for every head size, ragged chunks, packed sequences and no states."""
import pytest

from comba_inputs import random_case
from gpu_helpers import check_fwd, to_device

pytestmark = pytest.mark.gpu

CASES = [dict(B=1, T=65, H=1, dk=64, dv=64), dict(B=2, T=130, H=3, dk=128, dv=128),
         dict(B=1, T=200, H=2, dk=64, dv=128), dict(B=1, T=63, H=5, dk=128, dv=64),
         dict(B=1, T=129, H=3, dk=256, dv=256), dict(B=3, T=70, H=1, dk=128, dv=256),
         dict(B=1, T=90, H=2, dk=256, dv=128), dict(B=2, T=100, H=16, dk=128, dv=128),
         dict(B=2, T=100, H=17, dk=128, dv=128),
         dict(T=0, H=3, dk=128, dv=128, seqlens=[0, 1, 64, 65, 300])]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: "-".join(str(v) for v in kw.values()))
@pytest.mark.parametrize("states", [False, True], ids=["no_states", "states"])
def test_slice_widths_agree(kw, states):
    import torch

    import paper_2506_02475_amd as comba

    print("case", kw, states, flush=True)
    w = random_case(seed=71, in_dtype="bf16", h0=states, grad=False, beta_tilde=True, **kw)
    a = to_device(w)
    args = (a["q"], a["k"], a["v"], a["g"], a["beta"], a["d"], a["h0"])
    kws = dict(cu_seqlens=a["cu_seqlens"], beta_tilde=a["beta_tilde"], output_final_state=states)
    o, ht = comba.comba_chunk_fwd(*args, **kws)
    o2, ht2, _ = comba.comba_chunk_fwd_save(*args, **kws)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and (not states or torch.equal(ht, ht2))
    if states:
        check_fwd(w)
