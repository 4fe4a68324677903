"""GPU parity of short contexts, whose attention is one workgroup per head: both head widths, ranks 64 to 256, token
counts on both sides of a round of 128 rows and of the rounds asked for at once, whole eights of sequences and not,
grouped queries, one basis for all sequences, with and without an append (the fold in the launch before or in the same
one), 16-bit and fp32 outputs, log-sum-exps and logits."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2603_23914_amd import workloads as wl
from gpu_util import TORCH_DT, assert_close, to_dev, to_host64, workspace

pytestmark = pytest.mark.gpu

CASES = [  # dtype, B, H, H_kv, d, r, T, step, shared, 16-bit output
    ("bf16", 1, 32, 32, 128, 64, 321, True, False, False),
    ("f16", 2, 5, 5, 128, 64, 1, False, False, True),
    ("bf16", 3, 8, 8, 64, 64, 127, False, False, False),
    ("f16", 8, 32, 32, 64, 64, 512, True, False, True),
    ("bf16", 8, 16, 4, 128, 64, 513, False, False, False),
    ("f16", 1, 40, 40, 128, 64, 4096, False, False, False),
    ("bf16", 2, 32, 8, 128, 128, 129, True, True, False),
    ("f16", 16, 32, 32, 64, 128, 257, False, False, False),
    ("bf16", 4, 24, 24, 64, 128, 1000, True, False, False),
    ("f16", 3, 32, 32, 64, 192, 128, True, False, False),
    ("bf16", 5, 40, 40, 128, 192, 500, False, True, True),
    ("f16", 2, 33, 33, 128, 256, 2, True, False, False),
    ("bf16", 8, 32, 32, 64, 256, 700, False, False, False),
]


@pytest.mark.parametrize("dtype,B,H,H_kv,d,r,T,step,shared,half", CASES)
def test_short_contexts(dtype, B, H, H_kv, d, r, T, step, shared, half):
    from paper_2603_23914_amd import binding as ap
    print(f"short context {dtype} B={B} H={H}/{H_kv} d={d} r={r} T={T} step={step} shared={shared}", flush=True)
    case = wl.decode_case(dtype, B, H_kv, d, r, T - step, steps=int(step), seed=H * 5 + T, append=step)
    P = lambda x: oracle.promote(x, dtype)
    bits = (lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)) if dtype == "bf16" else (lambda t: t.cpu().numpy())
    q = torch.from_numpy(wl.rng_for(B, H, T, 3).standard_normal((B, H, d)).astype(np.float32)).to(TORCH_DT[dtype]).cuda()
    tail = torch.full((B, 7, r), 1.0e3, dtype=TORCH_DT[dtype], device="cuda")      # rows behind the tokens: never used
    dCk, dCv = (torch.cat([to_dev(x, dtype)[:, :T], tail], dim=1).contiguous() for x in (case.Ck, case.Cv))
    bases = [x[0] if shared else x for x in (case.Bk, case.Bv)]
    dBk, dBv = (to_dev(np.ascontiguousarray(x), dtype) for x in bases)
    out = torch.full((B, H, d), float("nan"), dtype=TORCH_DT[dtype] if half else torch.float32, device="cuda")
    lse = torch.full((B, H), float("nan"), dtype=torch.float32, device="cuda")
    scores = torch.full((B, T + 7, H), 123.0, dtype=torch.float32, device="cuda")
    ws = workspace(ap.ap_decode_workspace_bytes(B, H, d, T, r, ap._DT[TORCH_DT[dtype]]))
    kw = dict(T=T, sm_scale=1.0 / math.sqrt(d), lse=lse, scores=scores)
    if step:
        kn, vn = wl.step_new_token(case, 0, P(case.Bk), P(case.Bv))
        ap.ap_decode_step(q, to_dev(kn, dtype), to_dev(vn, dtype), dCk, dCv, dBk, dBv, out, ws, **kw)
    else:
        ap.ap_decode_attn(q, dCk, dCv, dBk, dBv, out, ws, **kw)
    torch.cuda.synchronize()
    Ck, Cv, qh, got_s = P(bits(dCk)), P(bits(dCv)), to_host64(q), to_host64(scores)
    assert (got_s[:, T:] == 123.0).all()
    eps = 2.0 ** -9 if dtype == "bf16" else 2.0 ** -12                             # half a unit of a 16-bit output
    for b in range(B):
        Bk, Bv = (P(x if shared else x[b]) for x in bases)
        if step:
            c_ref = P(kn)[b] @ Bk.T
            assert np.abs(Ck[b, T - 1] - c_ref).max() <= 2.0 ** -7 * np.abs(c_ref).max()
        for h in range(H):
            cols = slice(h // (H // H_kv) * d, h // (H // H_kv) * d + d)
            s = Ck[b, :T] @ (Bk[:, cols] @ qh[b, h]) / math.sqrt(d)
            w = np.exp(s - s.max())
            ref = (w / w.sum()) @ Cv[b, :T] @ Bv[:, cols]
            # q' carries at least 16 bits (two parts), everything after it is fp32: 1e-4 covers 2^-16 of the
            # largest logit (tens) in the weights; a 16-bit output adds its rounding
            top = np.abs(ref).max()
            assert np.abs(to_host64(out)[b, h] - ref).max() <= (1e-4 + (2 * eps if half else 0.0)) * top
            l_ref = s.max() + math.log(w.sum())
            assert abs(to_host64(lse)[b, h] - l_ref) <= 1e-4 * max(1.0, abs(l_ref))
            assert np.abs(got_s[b, :T, h] - s).max() <= 1e-4 * max(1.0, np.abs(s).max())
