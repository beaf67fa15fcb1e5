"""Infinite elements stay where the formula puts them.  The library promises
no particular result for them, but work done for padding (query rows past the
last one, value rows past a tile's end) must not turn a finite or infinite
result into NaN: a key whose logits are all -inf has score 0 and leaves the
others alone, and an infinite value makes its own channel infinite.

Tolerance: scores 1e-5 relative (32-bit exponentials), attention the bar."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle as ref  # noqa: E402
import paper_2609_32831_amd as uc  # noqa: E402
from gpu_util import check_attention, dev, rand_rows, sm_scale  # noqa: E402


@pytest.mark.parametrize("dtype,D,Hq,W", [("bf16", 128, 16, 1), ("bf16", 128, 7, 3), ("f32", 64, 1, 3)])
def test_score_of_a_key_at_minus_infinity(dtype, D, Hq, W):
    print(f"CASE score_inf {dtype} Hq={Hq} W={W}", flush=True)
    n, bad = 300, 5
    k = torch.from_numpy(ref.widen(rand_rows(1, 1, n, D, dtype), dtype)).float()
    q = torch.from_numpy(ref.widen(rand_rows(2, Hq, W, D, dtype), dtype)).float()
    q[..., 9] = q[..., 9].abs().clamp_(min=0.5)  # exact in either type
    rest = [i for i in range(n) if i != bad]
    want, _ = ref.score64(q.double().numpy()[None], k[:, rest].double().numpy()[None], np.zeros(n - 1, np.int32), 1,
                          sm_scale(D))
    k[:, bad, 9] = -np.inf
    kd, qd = (x.to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()[None] for x in (k, q))
    out, mass = torch.empty(1, 1, n, device="cuda"), torch.empty(1, 1, 1, device="cuda")
    uc.uc_score_importance(uc.make_shape(1, Hq, 1, D), [uc.dense_segment(kd, kd)], qd, W, sm_scale(D), [out], mass)
    torch.cuda.synchronize()
    got = out.cpu().double().numpy().reshape(-1)
    assert got[bad] == 0.0
    assert np.linalg.norm(got[rest] - want.reshape(-1)) <= 1e-5 * np.linalg.norm(want)
    assert abs(float(mass) - Hq * W) <= 1e-5 * Hq * W


@pytest.mark.parametrize("dtype,D", [("f16", 128), ("f32", 64)])
def test_infinite_value_at_a_tile_end(dtype, D):
    """The last row of a partial 16-row tile."""
    print(f"CASE value_inf {dtype} D={D}", flush=True)
    n, Hq, M = 70, 4, 2
    k, v, q = (rand_rows(s, *x, D, dtype) for s, x in ((1, (1, n)), (2, (1, n)), (3, (Hq, M))))
    o_ref = ref.attend(ref.widen(q, dtype).reshape(1, Hq, M, D), ref.widen(k, dtype)[None], ref.widen(v, dtype)[None],
                       None, np.zeros(n, np.int32), 1, sm_scale(D))[0]
    v = v.copy()
    v[0, n - 1, 11] = np.inf
    o = torch.empty(1, Hq, M, D, device="cuda")
    uc.uc_attend_mixed(uc.make_shape(1, Hq, 1, D),
                       [uc.dense_segment(dev(k, dtype)[None], dev(v, dtype)[None])],
                       dev(q.reshape(1, Hq, M, D), dtype), M, sm_scale(D), o)
    assert uc.uc_last_kernel() == "attend_wide"
    torch.cuda.synchronize()
    got = o.cpu().numpy()
    assert np.all(got[..., 11] == np.inf)
    got[..., 11] = o_ref[..., 11]
    check_attention(got, o_ref, "other channels")
