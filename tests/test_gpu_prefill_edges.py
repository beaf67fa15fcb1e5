"""Multi-query attention whose logits all lie far below zero: the rows of a
partial key tile past a segment's end must take no part in a row's reference
maximum or sums (as zero rows with logit 0 they would outweigh every real
one).  Segments that end inside a tile first, in the middle and last, and one
of fewer rows than a tile, with the keys walked whole and split; per-segment
statistics.

Tolerance: the attention bar; lse 1e-3 absolute at magnitude 60 (fp32)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle as ref  # noqa: E402
import paper_2609_32831_amd as uc  # noqa: E402
import workloads as gen  # noqa: E402
from gpu_util import check_attention, dev, rand_rows, sm_scale  # noqa: E402


@pytest.mark.parametrize("rows", [(33,), (5, 64), (100, 70, 32), (40, 1100, 7), (5, 1100)], ids=str)
def test_logits_far_below_zero(rows):
    print(f"CASE low_logits {rows}", flush=True)
    B, Hq, Hkv, M, D = 1, 4, 1, 20, 128
    # a shared direction with opposite signs in keys and queries: logits of about -60
    u = 6.0 / np.sqrt(D) * np.ones(D)
    def shifted(seed, n, sign):
        x = ref.widen(rand_rows(seed, 1, n, D, "bf16"), "bf16") + sign * u * 1.8
        return gen.round_to(x.astype(np.float32), "bf16")
    k = [shifted(3 + i, n, -1.0) for i, n in enumerate(rows)]
    v = [rand_rows(40 + i, 1, n, D, "bf16") for i, n in enumerate(rows)]
    q = shifted(90, Hq * M, 5.0).reshape(B, Hq, M, D)
    segs = [uc.dense_segment(dev(a, "bf16").view(B, Hkv, -1, D), dev(b, "bf16").view(B, Hkv, -1, D))
            for a, b in zip(k, v)]
    K, V = (np.concatenate([ref.widen(x, "bf16") for x in t], axis=1).reshape(B, Hkv, -1, D) for t in (k, v))
    ids = np.repeat(np.arange(len(rows)), rows).astype(np.int32)
    sm = sm_scale(D)
    o_ref, lse_ref, sl_ref, _ = ref.attend(ref.widen(q, "bf16"), K, V, None, ids, len(rows), sm)
    assert lse_ref.max() < -25
    o = torch.empty(B, Hq, M, D, device="cuda")
    lse = torch.empty(B, Hq, M, device="cuda")
    sl = torch.empty(B, Hq, M, len(rows), device="cuda")
    uc.uc_attend_mixed(uc.make_shape(B, Hq, Hkv, D), segs, dev(q, "bf16"), M, sm, o, lse, sl)
    assert uc.uc_last_kernel() == "prefill_mfma"
    torch.cuda.synchronize()
    check_attention(o.cpu().numpy(), o_ref, str(rows))
    assert np.allclose(lse.cpu().numpy(), lse_ref, rtol=0, atol=1e-3)
    assert np.allclose(sl.cpu().numpy(), sl_ref, rtol=0, atol=1e-3)
