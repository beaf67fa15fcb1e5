"""Multi-query attention with the keys split among workgroups (calls whose
query blocks leave CUs idle): one key tile short of the number from which
calls are split and exactly that many, splits that end inside a segment, a
packed segment's residual tail and partial tiles at a split's end, and
per-segment statistics of segments that only some splits see.  The
allocation-free call gives the workspace call's bits.  Whether a call was split
shows in its workspace: the splits' records lie behind what a plan, which
never splits, needs.

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

# B, Hq, Hkv, M, sizes (text, vit_full, vit_keep, pack, tail, cap), whether the keys are split
CASES = [
    (1, 7, 1, 3, (992, 10, 0, 0, 0, 1), False),            # 31 tiles
    (1, 7, 1, 3, (961, 10, 0, 0, 0, 1), False),            # 31 tiles, the last of one row
    (1, 7, 1, 3, (993, 10, 0, 0, 0, 1), True),             # 32 tiles, the last of one row
    (1, 7, 1, 3, (1024, 10, 0, 0, 0, 1), True),            # 32 whole tiles
    (1, 7, 1, 37, (33, 400, 300, 640 + 17, 5, 8), True),   # views that end inside a split
    (2, 8, 2, 40, (1000, 2000, 1777, 2048 + 63, 100, 128), True),
    (1, 28, 4, 203, (100, 900, 1024, 4096, 3, 8), True),   # records of 30 MB
    (1, 28, 4, 1180, (600, 500, 400, 0, 3, 8), False),     # 260 query blocks: the chip is full
]


@pytest.mark.parametrize("case", CASES, ids=[f"s{i}" for i in range(len(CASES))])
def test_split(case):
    B, Hq, Hkv, M, sizes, split = case
    print(f"CASE split {case}", flush=True)
    D = 128
    segs, K, V, ids = mixed_case(B, Hq, Hkv, D, "bf16", sizes[:1] + (max(sizes[1], sizes[2]),) + sizes[2:], seed=M)
    q = rand_rows(31, B * Hq, M, D, "bf16").reshape(B, Hq, M, D)
    sm, shape, qd = sm_scale(D), uc.make_shape(B, Hq, Hkv, D), dev(q, "bf16")
    o_ref, lse_ref, sl_ref, _ = ref.attend(ref.widen(q, "bf16"), K, V, None, ids, 4, sm)
    fin = np.isfinite(sl_ref)
    plan = uc.AttendPlan(shape, segs, None, torch.bfloat16, M, sm)
    unsplit = int(uc.lib.uc_plan_workspace_size(plan._h))
    plan.close()
    ws = torch.full((uc.uc_attend_workspace_size(shape, segs, uc.UC_BF16, M),), 171, dtype=torch.uint8, device="cuda")
    uc.uc_attend_mixed(shape, segs, qd, M, sm, torch.empty(B, Hq, M, D, device="cuda"), ws=ws)
    torch.cuda.synchronize()
    assert bool((ws[unsplit:] != 171).any()) == split
    seen = {}
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
            out = (o, lse) + ((sl,) if stats else ())
            assert all(map(torch.equal, out, seen.setdefault(stats, out)))
            if stats:
                got = sl.cpu().numpy()
                assert np.array_equal(np.isfinite(got), fin)
                assert np.allclose(got[fin], sl_ref[fin], rtol=1e-5, atol=1e-4)


def test_split_rounds_like_unsplit():
    """A call with its keys split gives what the unsplit kernel gives for the
    same rows, up to the order of the sums: three requests one at a time (21
    query rows of one KV head, split) against the same three in a batch whose
    query blocks fill the chip (unsplit).  No reference is raised after the
    first tile: that takes a logit 8 above its maximum in base 2, and these
    have a standard deviation of 1.4.

    Tolerance: both sum the same products in binary32, 47 tiles of 32 rows one
    after another or in up to 16 runs merged at the end; a sum of n terms taken
    in another order moves by about sqrt(n) 2^-24 of the terms' norm, 4e-7
    here, and the bound is ten times that (probabilities rounded to fp16
    against other references move the result by 2.7e-4)."""
    B, Hq, M, n, D = 260, 7, 3, 1500, 128
    print(f"CASE split_rounding B={B} M={M} n={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    k, v, q = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
               for s in ((B, 1, n, D), (B, 1, n, D), (B, Hq, M, D)))

    def attend(b):
        x = [t[b].contiguous() for t in (k, v, q)]
        rows = x[2].shape[0]
        o = torch.empty(rows, Hq, M, D, device="cuda")
        uc.uc_attend_mixed(uc.make_shape(rows, Hq, 1, D), [uc.dense_segment(x[0], x[1])], x[2], M, sm_scale(D), o)
        assert uc.uc_last_kernel() == "prefill_mfma"
        return o

    whole = attend(slice(0, B))
    for b in range(3):
        one = attend(slice(b, b + 1))
        rel = float((one - whole[b:b + 1]).norm() / whole[b].norm())
        assert rel <= 4e-6, (b, rel)


@pytest.mark.parametrize("dtype,D,heads,n,large,small", [
    ("bf16", 128, (28, 4), 8192, 4096, 40),  # unsplit at 4096 query rows, split at 40
    ("f32", 64, (1, 1), 49152, 17, 16),       # two query blocks, then one with more records per row
], ids=["prefill", "wide"])
def test_workspace_of_the_largest_query_block(dtype, D, heads, n, large, small):
    """A workspace sized for the largest query block serves a smaller one,
    whose own reported size is larger."""
    Hq, Hkv = heads
    print(f"CASE workspace_largest {dtype} {heads} {large} {small}", flush=True)
    k, v = (rand_rows(s, Hkv, n, D, dtype) for s in (1, 2))
    segs = [uc.dense_segment(dev(k, dtype).view(1, Hkv, n, D), dev(v, dtype).view(1, Hkv, n, D))]
    shape, sm = uc.make_shape(1, Hq, Hkv, D), sm_scale(D)
    have, want = (uc.uc_attend_workspace_size(shape, segs, uc.NAME_DT[dtype], m) for m in (large, small))
    assert have < want
    q = rand_rows(3, Hq, small, D, dtype).reshape(1, Hq, small, D)
    o_ref = ref.attend(ref.widen(q, dtype), ref.widen(k, dtype)[None], ref.widen(v, dtype)[None], None,
                       np.zeros(n, np.int32), 1, sm)[0]
    for size in (have, want):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        o = torch.empty(1, Hq, small, D, device="cuda")
        uc.uc_attend_mixed(shape, segs, dev(q, dtype), small, sm, o, ws=ws)
        torch.cuda.synchronize()
        check_attention(o.cpu().numpy(), o_ref, f"{size} bytes")
