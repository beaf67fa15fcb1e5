"""Multi-query attention with the keys split among workgroups (calls whose
query blocks leave CUs idle): one tile short of and past the number of tiles
that gives two splits, splits that end inside a segment, a packed segment's
residual tail and partial tiles at a split's end, and per-segment statistics
of segments that only some splits see.  The allocation-free call, whose array
may hold fewer splits, agrees with the workspace call.

Tolerance: the attention bar; lse as in the other prefill tests."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle as ref  # noqa: E402
import paper_2609_32831_amd as uc  # noqa: E402
from gpu_util import check_attention, dev, mixed_case, rand_rows, sm_scale  # noqa: E402

# B, Hq, Hkv, M, sizes (text, vit_full, vit_keep, pack, tail, cap)
CASES = [
    (1, 7, 1, 3, (480, 10, 0, 0, 0, 1)),            # 15 tiles: unsplit
    (1, 7, 1, 3, (481, 10, 0, 0, 0, 1)),            # 16 tiles: two splits, the last tile partial
    (1, 7, 1, 37, (33, 400, 300, 640 + 17, 5, 8)),  # views that end inside a split
    (2, 8, 2, 40, (1000, 2000, 1777, 2048 + 63, 100, 128)),
    (1, 28, 4, 203, (100, 900, 1024, 4096, 3, 8)),  # the records exceed the static array
]


@pytest.mark.parametrize("case", CASES, ids=[f"s{i}" for i in range(len(CASES))])
def test_split(case):
    B, Hq, Hkv, M, sizes = case
    print(f"CASE split {case}", flush=True)
    D = 128
    segs, K, V, ids = mixed_case(B, Hq, Hkv, D, "bf16", sizes[:1] + (max(sizes[1], sizes[2]),) + sizes[2:], seed=M)
    q = rand_rows(31, B * Hq, M, D, "bf16").reshape(B, Hq, M, D)
    sm, shape, qd = sm_scale(D), uc.make_shape(B, Hq, Hkv, D), dev(q, "bf16")
    o_ref, lse_ref, sl_ref, _ = ref.attend(ref.widen(q, "bf16"), K, V, None, ids, 4, sm)
    fin = np.isfinite(sl_ref)
    for call in (uc.uc_attend_mixed, uc.uc_attend_mixed_noalloc):
        for stats in (True, False):
            o = torch.full((B, Hq, M, D), 9.0, device="cuda")
            lse = torch.empty(B, Hq, M, device="cuda")
            sl = torch.empty(B, Hq, M, 4, device="cuda") if stats else None
            call(shape, segs, qd, M, sm, o, lse, sl)
            assert uc.uc_last_kernel() == "prefill_mfma"
            torch.cuda.synchronize()
            check_attention(o.cpu().numpy(), o_ref, call.__name__)
            assert np.allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-4)
            if stats:
                got = sl.cpu().numpy()
                assert np.array_equal(np.isfinite(got), fin)
                assert np.allclose(got[fin], sl_ref[fin], rtol=1e-5, atol=1e-4)
