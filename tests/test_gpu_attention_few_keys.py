"""GPU parity of the attention forward that has all keys in LDS (up to 128) at the edges of its blocks of 32 keys, query tiles of 128 and head
widths, plain and causal (more, as many and fewer queries than keys), with plain and with sharp logits."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import ops
from test_gpu_ops import TOL_BF16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gain,row_shift", [(1.0, 0.0), (8.0, 80.0)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dh", [40, 64, 72, 96])
def test_few_keys(dh, causal, gain, row_shift):
    import torch
    from paper_2405_01248_amd import binding as B
    from paper_2405_01248_amd.harness import _np_to_dev, _dev_to_np, rel_err
    from softmax_schedule import head_logits
    for Nk in (1, 31, 32, 33, 64, 65, 77, 96, 97, 128):
        for Nq in sorted({1, Nk, 33, 130}):
            Bt, H = 2, 5      # (ten heads: the map of workgroups to heads has a remainder)
            d = H * dh
            q, k, v, _ = si.make_attention_inputs(Bt, H, Nq, Nk, dh, seed=Nq * 131 + Nk, gain=gain, row_shift=row_shift)
            dq, dk, dv = (_np_to_dev(t, "bf16") for t in (q, k, v))
            o = torch.empty((Bt, Nq, d), dtype=torch.bfloat16, device="cuda:0")
            lse = torch.zeros((Bt, H, Nq), dtype=torch.float32, device="cuda:0")
            B.op_attention_fwd(B.DP_BF16, Bt, H, Nq, Nk, dh, causal, 1.0 / np.sqrt(dh), dq, d, dk, d, dv, d, o, d, lse)
            torch.cuda.synchronize()
            s = head_logits(q, k, H, causal)
            m = s.max(axis=-1)
            ref_lse = m + np.log(np.exp(s - m[..., None]).sum(axis=-1))
            e = rel_err(_dev_to_np(o), ops.attention_fwd(q, k, v, H, causal))
            e_lse = float(np.max(np.abs(_dev_to_np(lse) - ref_lse))) / max(1.0, float(np.max(np.abs(ref_lse))))
            assert e <= TOL_BF16 and e_lse <= 1e-3, (Nq, Nk, e, e_lse)
