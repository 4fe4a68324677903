"""GPU parity: decode attention with several tiles per token split, more than the ring holds.

64 sequences give four splits each (one workgroup per CU), so 1200 tokens are nine or ten tiles of 32 per
split: the steady state of the two-role kernel, in which a tile is added up while the next one is scored,
ring slots are refilled and the buffers of weights and scales are used in turn.  The sequences are copies
of three, whose results are compared with the fp64 oracle; the copies' must be the same bits, whatever ran
next to them."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2603_23914_amd import workloads as wl
from gpu_util import TORCH_DT, assert_close, to_dev, to_host64, workspace

pytestmark = pytest.mark.gpu

B, T, DISTINCT = 64, 1200, 3
SRC = np.arange(B) % DISTINCT


def quantize(C, coef):
    """Codes, scales and the values they stand for."""
    q, dq = (oracle.quantize_i8, oracle.dequantize_i8) if coef == "i8" else (oracle.quantize_i4, oracle.dequantize_i4)
    codes, scales = zip(*(q(c) for c in C))
    return np.stack(codes), np.stack(scales), np.stack([dq(c, s) for c, s in zip(codes, scales)])


def select(ranks, cum, r):
    from paper_2603_23914_amd import binding as ap
    mass = wl.rng_for(61, r).random((DISTINCT, T)).astype(np.float32)[SRC]
    F = len(ranks)
    rank, off, idx = (torch.empty(s, dtype=torch.int32, device="cuda") for s in ((B, T), (B, F + 1), (B, T)))
    ap.ap_select_ranks(torch.from_numpy(mass).cuda(), ranks, cum, cum[-1], rank, off, idx,
                       workspace(ap.ap_select_workspace_bytes(B, T, F)))
    return dict(rank_k=rank, rank_v=rank, bucket_off=off, bucket_idx=idx, F=F)


def same_as_source(x):
    torch.cuda.synchronize()
    bits = x.view(torch.int32)
    assert torch.equal(bits, bits[torch.from_numpy(SRC).cuda()]), "copies of a sequence differ"


@pytest.mark.parametrize("gathered", [False, True])
@pytest.mark.parametrize("coef,H,d,r", [
    ("f16", 64, 32, 256),       # four head tiles
    ("bf16", 64, 32, 512),
    ("f16", 64, 32, 640),       # a ring of two tiles
    ("bf16", 64, 32, 640),
    ("bf16", 40, 32, 576),      # three
    ("f16", 16, 64, 256),       # one
    ("bf16", 16, 64, 640),
    ("i8", 64, 32, 512),
    ("i8", 64, 32, 640),
    ("i4", 64, 32, 640),
    ("i8", 40, 32, 320),        # five scale blocks
    ("i8", 16, 64, 192),
    ("i4", 16, 64, 256),
])
def test_many_tiles_per_split(coef, H, d, r, gathered):
    from paper_2603_23914_amd import binding as ap
    quant = coef in ("i8", "i4")
    dtype = "f16" if quant else coef
    P = lambda x: oracle.promote(x, dtype)
    case = wl.decode_case(dtype, DISTINCT, H, d, r, T, steps=0, seed=61, shared_basis=True, append=False)
    q = wl.step_query(case, 0)
    print(f"long splits {coef} H={H} r={r} gathered={gathered}", flush=True)
    kw = {}
    if quant:
        (ck, sk, ck64), (cv, sv, cv64) = quantize(case.Ck, coef), quantize(case.Cv, coef)
        C = [torch.from_numpy(x[SRC]).cuda() for x in (ck, cv)]
        kw = dict(scale_k=torch.from_numpy(sk[SRC]).cuda(), scale_v=torch.from_numpy(sv[SRC]).cuda())
    else:
        ck64, cv64 = P(case.Ck), P(case.Cv)
        C = [to_dev(x[SRC], dtype) for x in (case.Ck, case.Cv)]
    if gathered:
        kw.update(select((r, r // 128 * 64, 64), (1, 3, 8), r))       # whole scale blocks
    out = torch.full((B, H, d), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((B, H), float("nan"), dtype=torch.float32, device="cuda")
    ws = workspace(ap.ap_decode_workspace_bytes(B, H, d, T, r, ap._DT[TORCH_DT[dtype]]))
    ap.ap_decode_attn(to_dev(q[SRC], dtype), *C, to_dev(case.Bk, dtype), to_dev(case.Bv, dtype), out, ws, T=T,
                      sm_scale=1.0 / math.sqrt(d), lse=lse, **kw)
    same_as_source(out)
    same_as_source(lse)
    for b in range(DISTINCT):
        rank = kw["rank_k"][b].cpu().numpy() if gathered else None
        ref, ref_lse = oracle.decode_attn_absorbed(P(q)[b], ck64[b], cv64[b], P(case.Bk), P(case.Bv), rank_k=rank, rank_v=rank,
                                                   return_lse=True)
        assert_close(to_host64(out[b]), ref, dtype, f"b={b}")
        assert np.abs(to_host64(lse[b]) - ref_lse).max() <= 2e-3 * max(1.0, np.abs(ref_lse).max())


@pytest.mark.parametrize("dtype,H,d,r", [("bf16", 64, 32, 640), ("f16", 16, 128, 512)])
def test_fused_step_with_logits_over_many_tiles(dtype, H, d, r):
    """The fused step, whose newest token leaves the sum to the expansion, and its logits; a basis per
    sequence, long enough for the one-pass value path (160 MB, 128 MB)."""
    from paper_2603_23914_amd import binding as ap
    P = lambda x: oracle.promote(x, dtype)
    case = wl.decode_case(dtype, DISTINCT, H, d, r, T - 1, steps=1, seed=62)
    q = wl.step_query(case, 0)
    kn, vn = wl.step_new_token(case, 0, P(case.Bk), P(case.Bv))
    print(f"long splits, fused step {dtype} H={H} r={r}", flush=True)
    dCk, dCv = (to_dev(x[SRC], dtype) for x in (case.Ck, case.Cv))
    out = torch.full((B, H, d), float("nan"), dtype=torch.float32, device="cuda")
    scores = torch.full((B, T, H), float("nan"), dtype=torch.float32, device="cuda")
    ws = workspace(ap.ap_decode_workspace_bytes(B, H, d, T, r, ap._DT[TORCH_DT[dtype]]))
    ap.ap_decode_step(to_dev(q[SRC], dtype), to_dev(kn[SRC], dtype), to_dev(vn[SRC], dtype), dCk, dCv, to_dev(case.Bk[SRC], dtype),
                      to_dev(case.Bv[SRC], dtype), out, ws, T=T, sm_scale=1.0 / math.sqrt(d), scores=scores)
    same_as_source(out)
    same_as_source(scores)
    for b in range(DISTINCT):
        ck, cv = to_host64(dCk[b]), to_host64(dCv[b])
        for C, x, Bm in ((ck, kn, case.Bk), (cv, vn, case.Bv)):
            c_ref = oracle.compact(P(x)[b][None], P(Bm)[b])[0]
            assert np.abs(C[T - 1] - c_ref).max() <= (2.0 ** -10 if dtype == "f16" else 2.0 ** -7) * np.abs(c_ref).max()
        ref = oracle.decode_attn_absorbed(P(q)[b], ck, cv, P(case.Bk)[b], P(case.Bv)[b])
        assert_close(to_host64(out[b]), ref, dtype, f"b={b}")
        folded = np.einsum("jhe,he->hj", P(case.Bk)[b].reshape(r, H, d), P(q)[b]) / math.sqrt(d)
        s_ref = ck @ folded.T
        assert np.abs(to_host64(scores[b]) - s_ref).max() <= 2e-3 * np.abs(s_ref).max()
