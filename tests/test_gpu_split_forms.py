"""GPU parity of attention over token splits, in its forms.  Short contexts, where a split's heads are shared out to
workgroups: one, two, three and four head tiles, the last one partly filled, one tile of 16 heads or two per workgroup, batches whose splits make
whole eights and not, every coefficient format, gathered rows with the logits written, and the fused step whose
newest value row the expansion produces.  Longer splits, whose softmax has waves of its own: fewer tiles than that
pipeline is deep, as many as the value ring holds and more, for every coefficient format it serves."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2603_23914_amd import workloads as wl
from gpu_util import TORCH_DT, assert_close, to_dev, to_host64, workspace

pytestmark = pytest.mark.gpu

CASES = [  # dtype, B, H, H_kv, d, r, T, mode
    ("f16", 3, 17, 17, 64, 192, 33, "attend"),        # a second tile of one head; a workgroup per head tile
    ("bf16", 2, 40, 40, 32, 256, 200, "attend"),      # three tiles, one each
    ("f16", 1, 64, 8, 64, 320, 65, "attend"),         # four tiles, one each; grouped queries
    ("bf16", 8, 48, 48, 32, 192, 1100, "attend"),     # three tiles in groups of two and one, two tiles of tokens
    ("f16", 5, 33, 33, 32, 512, 4700, "attend"),      # three tiles of tokens at rank 512
    ("bf16", 64, 56, 8, 128, 640, 300, "attend"),     # four head tiles beyond rank 512, several tiles of tokens
    ("f16", 8, 24, 24, 64, 448, 1000, "step"),
    ("bf16", 3, 64, 64, 32, 640, 130, "step"),
    ("f16", 8, 32, 32, 32, 256, 1100, "late"),        # the newest token's weight comes from every head group
    ("bf16", 3, 40, 40, 32, 192, 97, "late"),
    ("f16", 4, 32, 32, 32, 256, 1000, "ragged"),
    ("bf16", 3, 41, 41, 32, 192, 150, "ragged"),
    ("f16", 8, 40, 40, 32, 192, 600, "i8"),
    ("f16", 3, 64, 64, 32, 640, 700, "i8"),
    ("f16", 8, 32, 32, 32, 256, 700, "i4"),
    ("bf16", 64, 40, 40, 32, 192, 520, "attend"),     # five tiles a split
    ("f16", 64, 24, 8, 64, 256, 1500, "late"),        # twelve, the last token's value row not there yet
    ("bf16", 32, 64, 8, 64, 256, 1100, "attend"),     # four head tiles: a ring of three tiles
    ("f16", 1, 16, 16, 64, 640, 20, "i8"),            # one tile
    ("f16", 64, 20, 20, 32, 512, 250, "i8"),          # two tiles a split
    ("f16", 64, 40, 8, 64, 448, 1100, "i8"),          # nine, three head tiles
    ("f16", 64, 32, 8, 128, 640, 900, "i4"),          # eight
    ("f16", 16, 16, 16, 64, 512, 1700, "ragged"),
    ("bf16", 32, 32, 8, 64, 256, 1300, "ragged"),
]


@pytest.mark.parametrize("dtype,B,H,H_kv,d,r,T,mode", CASES)
def test_forms_of_the_split_kernel(dtype, B, H, H_kv, d, r, T, mode):
    from paper_2603_23914_amd import binding as ap
    steps = 1 if mode in ("step", "late") else 0
    case = wl.decode_case(dtype, B, H_kv, d, r, T - steps, steps=steps, seed=H * 7 + T, append=steps > 0)
    P = lambda x: oracle.promote(x, dtype)
    bits = (lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)) if dtype == "bf16" else (lambda t: t.cpu().numpy())
    q = torch.from_numpy(wl.rng_for(B, H, T).standard_normal((B, H, d)).astype(np.float32)).to(TORCH_DT[dtype]).cuda()
    dCk, dCv, dBk, dBv = (to_dev(x, dtype) for x in (case.Ck, case.Cv, case.Bk, case.Bv))
    out = torch.full((B, H, d), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((B, H), float("nan"), dtype=torch.float32, device="cuda")
    ws = workspace(ap.ap_decode_workspace_bytes(B, H, d, T, r, ap._DT[TORCH_DT[dtype]]))
    kw = dict(T=T, sm_scale=1.0 / math.sqrt(d), lse=lse)
    rank = None
    Ck, Cv = P(case.Ck), P(case.Cv)
    if mode == "attend":
        ap.ap_decode_attn(q, dCk, dCv, dBk, dBv, out, ws, **kw)
    elif mode in ("step", "late"):
        kn, vn = wl.step_new_token(case, 0, P(case.Bk), P(case.Bv))
        ap.ap_set_fused_value_min_bytes(0 if mode == "late" else -1)
        try:
            ap.ap_decode_step(q, to_dev(kn, dtype), to_dev(vn, dtype), dCk, dCv, dBk, dBv, out, ws, **kw)
            torch.cuda.synchronize()
        finally:
            ap.ap_set_fused_value_min_bytes(-1)
        Ck, Cv = P(bits(dCk)), P(bits(dCv))
    elif mode == "ragged":
        mass = torch.from_numpy(wl.rng_for(T, r, H).random((B, T)).astype(np.float32)).cuda()
        rank, idx = (torch.empty((B, T), dtype=torch.int32, device="cuda") for _ in range(2))
        off = torch.empty((B, 4), dtype=torch.int32, device="cuda")
        ap.ap_select_ranks(mass, (r, 128, 64), (1, 2, 3), 3, rank, off, idx, workspace(ap.ap_select_workspace_bytes(B, T, 3)))
        scores = torch.full((B, dCk.shape[1], H), float("nan"), dtype=torch.float32, device="cuda")
        ap.ap_decode_attn(q, dCk, dCv, dBk, dBv, out, ws, rank_k=rank, rank_v=rank, bucket_off=off, bucket_idx=idx, F=3,
                          scores=scores, **kw)
    else:
        i4 = mode == "i4"
        codes, scales = [], []
        for C in (dCk, dCv):
            code = torch.zeros((*C.shape[:2], r // 2 if i4 else r), dtype=torch.uint8 if i4 else torch.int8, device="cuda")
            scale = torch.zeros((*C.shape[:2], r // 64), dtype=torch.float16, device="cuda")
            (ap.ap_quantize_i4 if i4 else ap.ap_quantize_i8)(C, code, scale, T=T)
            codes.append(code)
            scales.append(scale)
        ap.ap_decode_attn(q, *codes, dBk, dBv, out, ws, scale_k=scales[0], scale_v=scales[1], **kw)
        deq = []
        for code, scale in zip(codes, scales):
            v = code.cpu().numpy()
            if i4:
                v = np.stack([v & 15, v >> 4], axis=-1).reshape(*v.shape[:2], r).astype(np.int64) - 8
            deq.append(v.astype(np.float64) * np.repeat(scale.double().cpu().numpy(), 64, axis=-1))
        Ck, Cv = deq
    torch.cuda.synchronize()
    G = H // H_kv
    qh, Bk, Bv = to_host64(q), P(case.Bk), P(case.Bv)
    got_s = scores.double().cpu().numpy() if mode == "ragged" else None
    for b in range(B):
        ck, cv, bk, bv = Ck[b][:T], Cv[b][:T], Bk[b], Bv[b]
        if rank is not None:
            live = np.arange(r)[None, :] < rank[b].cpu().numpy()[:, None]
            ck, cv = ck * live, cv * live
        ref, ref_l = np.empty((H, d)), np.empty(H)
        for h in range(H):
            cols = slice(h // G * d, h // G * d + d)
            s = ck @ (bk[:, cols] @ qh[b, h]) / math.sqrt(d)
            m = s.max()
            w = np.exp(s - m)
            ref_l[h] = m + math.log(w.sum())
            ref[h] = (w / w.sum()) @ cv @ bv[:, cols]
            if got_s is not None:
                assert np.abs(got_s[b, :T, h] - s).max() <= 2e-3 * np.abs(s).max()
        assert_close(to_host64(out)[b], ref, dtype, f"{mode} sequence {b}")
        assert np.abs(to_host64(lse)[b] - ref_l).max() <= 2e-3 * np.abs(ref_l).max()


@pytest.mark.parametrize("dtype,B,H,r,T,scores", [
    ("bf16", 64, 40, 64, 1700, True),     # fourteen tiles a split, some waves with one more than others
    ("f16", 64, 17, 64, 1400, False),     # twelve
    ("bf16", 128, 9, 128, 800, True),     # fourteen, one head tile at rank 128
    ("f16", 128, 48, 64, 700, True),      # twelve, three head tiles
])
def test_gathered_small_ranks_over_long_splits(dtype, B, H, r, T, scores):
    """Ranks 64 and 128 by rank group where a split is a dozen tiles and more: eight waves share them."""
    from paper_2603_23914_amd import binding as ap
    d = 32
    case = wl.decode_case(dtype, B, H, d, r, T, steps=0, seed=H + T, append=False)
    P = lambda x: oracle.promote(x, dtype)
    q = torch.from_numpy(wl.rng_for(B, H, T).standard_normal((B, H, d)).astype(np.float32)).to(TORCH_DT[dtype]).cuda()
    dCk, dCv, dBk, dBv = (to_dev(x, dtype) for x in (case.Ck, case.Cv, case.Bk, case.Bv))
    out = torch.full((B, H, d), float("nan"), dtype=torch.float32, device="cuda")
    ws = workspace(ap.ap_decode_workspace_bytes(B, H, d, T, r, ap._DT[TORCH_DT[dtype]]))
    mass = torch.from_numpy(wl.rng_for(T, r, H).random((B, T)).astype(np.float32)).cuda()
    rank, idx = (torch.empty((B, T), dtype=torch.int32, device="cuda") for _ in range(2))
    off = torch.empty((B, 3), dtype=torch.int32, device="cuda")
    ap.ap_select_ranks(mass, (r, 16), (1, 4), 4, rank, off, idx, workspace(ap.ap_select_workspace_bytes(B, T, 2)))
    s_out = torch.full((B, dCk.shape[1], H), float("nan"), dtype=torch.float32, device="cuda") if scores else None
    ap.ap_decode_attn(q, dCk, dCv, dBk, dBv, out, ws, T=T, sm_scale=1.0 / math.sqrt(d), rank_v=rank, bucket_off=off,
                      bucket_idx=idx, F=2, scores=s_out)
    torch.cuda.synchronize()
    for b in range(0, B, 7):
        live = np.arange(r)[None, :] < rank[b].cpu().numpy()[:, None]
        ck, cv, bk, bv = P(case.Ck)[b][:T], P(case.Cv)[b][:T] * live, P(case.Bk)[b], P(case.Bv)[b]
        for h in range(H):
            cols = slice(h * d, h * d + d)
            s = ck @ (bk[:, cols] @ to_host64(q)[b, h]) / math.sqrt(d)
            w = np.exp(s - s.max())
            assert_close(to_host64(out)[b, h], (w / w.sum()) @ cv @ bv[:, cols], dtype, f"sequence {b} head {h}")
            if scores:
                assert np.abs(s_out[b, :T, h].double().cpu().numpy() - s).max() <= 2e-3 * np.abs(s).max()
