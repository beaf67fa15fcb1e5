"""The binary32 matrix-core kernels (every input outside the bf16 kernels) at
the edges of their 16-row tiles, 64-row chunks and 16-query blocks: element
types mixed within a call, head dims 64 and 128, every code width, row groups
of 8 and 16, queries at an unaligned address, and more records per row than
one wave merges at a time.  The same calls under UC_PATH_VALU run the
vector-ALU kernels; both are held to the oracle.

Tolerance: with every product and sum in binary32 the result differs from
the oracle's by the rounding of the logits (|s| < 2^6 here, so an absolute
error below 64 * 2^-24 * sqrt(D) / 2 = 2.2e-5 in the exponent) and of the
sums; 1e-4 relative bounds both with a factor of four."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle as ref  # noqa: E402
import paper_2609_32831_amd as uc  # noqa: E402
from gpu_util import dev, packed_from_oracle, rand_rows, sm_scale  # noqa: E402

# D, query dtype, B, Hkv, G, M, segments: ("d", dtype, rows, spare) dense, ("p", dtype, rows, group, bits)
CASES = [
    (64, "f32", 1, 1, 1, 1, [("d", "f32", 1, 0)]),
    (64, "f32", 1, 2, 4, 4, [("d", "f16", 15, 3), ("d", "f32", 16, 0), ("p", "f32", 17, 8, 4)]),
    (64, "f16", 2, 1, 3, 6, [("d", "bf16", 65, 0), ("p", "f16", 63, 16, 2), ("p", "bf16", 40, 8, 8)]),
    (64, "bf16", 1, 4, 7, 1, [("p", "bf16", 129, 64, 4), ("d", "bf16", 64, 7)]),
    (128, "f16", 1, 2, 7, 1, [("d", "f16", 1537, 1), ("p", "f16", 1000, 32, 8), ("d", "f16", 1, 4)]),
    (128, "f32", 1, 1, 17, 1, [("d", "f32", 100, 0), ("p", "f32", 31, 16, 8), ("p", "f32", 9, 8, 2)]),
    (128, "bf16", 1, 1, 1, 33, [("p", "bf16", 47, 8, 4), ("d", "f32", 33, 2), ("d", "f16", 0, 5)]),
    # 4096 rows of one head: 64-row chunks, so four waves merge a row's records
    (64, "f32", 1, 1, 2, 1, [("d", "f32", 4096, 0)]),
]


def _build(case):
    D, _, B, Hkv, _, _, specs = case
    BH = B * Hkv
    segs, ks, vs, ids = [], [], [], []
    for i, s in enumerate(specs):
        kind, dt, n = s[:3]
        if kind == "d":
            cap = max(n + s[3], 1)
            k, v = rand_rows(11 * i + 1, BH, cap, D, dt, outliers=(3,)), rand_rows(11 * i + 2, BH, cap, D, dt)
            segs.append(uc.dense_segment(dev(k, dt).reshape(B, Hkv, cap, D), dev(v, dt).reshape(B, Hkv, cap, D),
                                         n_rows=n))
            k, v = ref.widen(k[:, :n], dt), ref.widen(v[:, :n], dt)
        else:
            g, bits = s[3:]
            pk = ref.quantize(rand_rows(11 * i + 1, BH, n, D, dt, 2.0, outliers=(3,)),
                              rand_rows(11 * i + 2, BH, n, D, dt), dt, g, [bits] * BH)
            segs.append(packed_from_oracle(B, Hkv, n, D, g, dt, pk))
            k, v = ref.dequant(pk, n, D, g, dt)
        ks.append(k)
        vs.append(v)
        ids += [i] * n
    K, V = (np.concatenate(x, axis=1).reshape(B, Hkv, -1, D) for x in (ks, vs))
    return segs, K, V, np.asarray(ids, np.int32)


def _close(got, want):
    got, want = np.asarray(got, np.float64), np.asarray(want, np.float64)
    assert np.linalg.norm(got - want) <= 1e-4 * max(np.linalg.norm(want), 1e-30)


@pytest.mark.parametrize("path", ["auto", "valu"])
@pytest.mark.parametrize("case", CASES, ids=[f"w{i}" for i in range(len(CASES))])
def test_wide(case, path):
    D, q_dt, B, Hkv, G, M, specs = case
    print(f"CASE wide {path} {case}", flush=True)
    segs, K, V, ids = _build(case)
    Hq, n = Hkv * G, len(segs)
    q = rand_rows(99, B * Hq, M, D, q_dt).reshape(B, Hq, M, D)
    shape, sm = uc.make_shape(B, Hq, Hkv, D), sm_scale(D)
    qd = dev(q, q_dt)
    # the same values one element past an aligned address
    buf = torch.empty(qd.numel() + 1, dtype=qd.dtype, device="cuda")
    buf[1:] = qd.reshape(-1)
    qu = buf[1:].view(qd.shape)
    o_ref, lse_ref, sl_ref, _ = ref.attend(ref.widen(q, q_dt), K, V, None, ids, n, sm)
    sc_ref, ms_ref = ref.score64(ref.widen(q, q_dt), K, ids, n, sm)
    prev = uc.uc_set_path(uc.UC_PATH_VALU if path == "valu" else uc.UC_PATH_AUTO)
    try:
        for x in (qd, qu):
            for stats in (True, False):
                o = torch.empty(B, Hq, M, D, device="cuda")
                lse = torch.empty(B, Hq, M, device="cuda")
                sl = torch.empty(B, Hq, M, n, device="cuda") if stats else None
                uc.uc_attend_mixed(shape, segs, x, M, sm, o, lse, sl)
                assert uc.uc_last_kernel() == ("attend_valu" if path == "valu" else "attend_wide")
                torch.cuda.synchronize()
                _close(o.cpu(), o_ref)
                assert np.allclose(lse.cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-4)
                if stats:
                    got = sl.cpu().numpy()
                    assert np.array_equal(np.isfinite(got), np.isfinite(sl_ref))
                    fin = np.isfinite(sl_ref)
                    assert np.allclose(got[fin], sl_ref[fin], rtol=1e-5, atol=1e-4)
        scores = [torch.empty(B, Hkv, max(s.n_rows, 1), device="cuda") for s in segs]
        mass = torch.empty(B, Hkv, n, device="cuda")
        uc.uc_score_importance(shape, segs, qd, M, sm, [t if s.n_rows else None for t, s in zip(scores, segs)], mass)
        assert uc.uc_last_kernel() == ("score_valu" if path == "valu" else "score_wide")
        torch.cuda.synchronize()
    finally:
        uc.uc_set_path(prev)
    col = 0
    for s, t in zip(segs, scores):
        if s.n_rows:
            _close(t.cpu().numpy().reshape(B, Hkv, -1), sc_ref[:, :, col:col + s.n_rows])
        col += s.n_rows
    _close(mass.cpu(), ms_ref)


def test_scores_in_the_least_workspace():
    """Importance scores in a workspace that holds only a coarse cut of the keys
    (32 records per row and segment), and in the reported one."""
    Hq, W, n, D = 2, 16, 8192 + 5, 64
    print(f"CASE wide_least_ws n={n}", flush=True)
    k, v, q = (rand_rows(s, *x, D, "f32") for s, x in ((1, (1, n)), (2, (1, n)), (3, (Hq, W))))
    segs = [uc.dense_segment(dev(k, "f32").view(1, 1, n, D), dev(v, "f32").view(1, 1, n, D))]
    shape, sm = uc.make_shape(1, Hq, 1, D), sm_scale(D)
    want, _ = ref.score64(q.reshape(1, Hq, W, D), k[None], np.zeros(n, np.int32), 1, sm)
    full = uc.uc_score_workspace_size(shape, segs, W)
    parts = (Hq * W * ((n + 511) // 512) * 8, Hq * W * 8, (n + 63) // 64 * 8)  # records, normalisers, masses
    least = sum((p + 255) // 256 * 256 for p in parts)
    assert least < full
    for size in (least, full):
        out = torch.empty(1, 1, n, device="cuda")
        uc.uc_score_importance(shape, segs, dev(q, "f32").view(1, Hq, W, D), W, sm, [out],
                               ws=torch.empty(size, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        _close(out.cpu(), want)
    with pytest.raises(uc.UcError):
        uc.uc_score_importance(shape, segs, dev(q, "f32").view(1, Hq, W, D), W, sm, [out],
                               ws=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))
