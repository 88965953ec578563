"""comba_chunk_bwd_saved_in_dtype: the gradient kernels' bf16 stores.

The values are those of comba_chunk_bwd_saved rounded to nearest even, bit for
bit, at the edges of the kernels' tiles: chunks of 1 to 64 rows, every head
size (the persistent and the 128-column-pass kernel), odd head counts, tied and
separate feedback strength, packed sequences with empty ones; and with several
chunk-heads per workgroup of the persistent kernel (768 and more, one workgroup
per CU), which copies its next one's operands during the stores, some of those
in empty chunk slots."""
import numpy as np
import pytest

from comba_inputs import attach_beta_tilde, random_case

pytestmark = pytest.mark.gpu

CASES = [
    dict(B=1, T=1, H=1, dk=64, dv=64), dict(B=2, T=65, H=3, dk=128, dv=128),
    dict(B=1, T=127, H=5, dk=64, dv=128), dict(B=1, T=63, H=3, dk=128, dv=64),
    dict(B=1, T=70, H=3, dk=256, dv=256), dict(B=2, T=130, H=1, dk=128, dv=256),
    dict(B=1, T=33, H=2, dk=256, dv=128), dict(T=0, H=3, dk=128, dv=128, seqlens=[1, 0, 64, 79]),
    dict(B=8, T=1000, H=6, dk=128, dv=128), dict(B=6, T=700, H=9, dk=64, dv=128),
    dict(T=0, H=6, dk=128, dv=128, seqlens=[70, 0, 128, 1] * 40),
]


@pytest.mark.parametrize("kw", CASES, ids=lambda kw: "-".join(str(v)[:20] for v in kw.values()))
@pytest.mark.parametrize("separate", [False, True], ids=["tied", "separate"])
def test_bf16_gradients_are_the_rounded_fp32_ones(kw, separate):
    import torch

    import paper_2506_02475_amd as comba
    from gpu_helpers import to_device

    print("case", kw, separate, flush=True)
    w = random_case(seed=31, in_dtype="bf16", dht=True, **kw)
    if separate:
        attach_beta_tilde(w, "b_beta", seed=2)
    a = to_device(w)
    args = (a["q"], a["k"], a["v"], a["g"], a["beta"], a["d"], a["h0"])
    kws = dict(cu_seqlens=a["cu_seqlens"], beta_tilde=a.get("beta_tilde"))
    _, _, ws = comba.comba_chunk_fwd_save(*args, **kws)
    ref = comba.comba_chunk_bwd_saved(*args, a["dO"], a["dht"], workspace=ws, **kws)
    got = comba.comba_chunk_bwd_saved_in_dtype(*args, a["dO"], a["dht"], workspace=ws, **kws)
    torch.cuda.synchronize()
    assert set(got) == set(ref)
    for name, x in ref.items():
        lo = name in ("dq", "dk", "dv", "dbeta", "dbeta_tilde")
        assert got[name].dtype == (torch.bfloat16 if lo else torch.float32), name
        assert torch.equal(got[name], x.to(got[name].dtype)), name
    assert np.isfinite(ref["dq"].cpu().numpy()).all()
