"""GPU parity: one basis for all sequences (basis_batch_stride = 0).  From some size on the appends, the
fold and the expansion are matrix products over the batch (shared_basis.hip); checked against the fp64
oracle on some sequences and, on all, against the same call with the basis written out per sequence."""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_util import TORCH_DT, TOL, to_host64, workspace

pytestmark = pytest.mark.gpu


def run(ap, step, q, kn, vn, Ck, Cv, Bk, Bv, T, dt_out):
    B, H, d = q.shape
    Ck, Cv = Ck.clone(), Cv.clone()
    out = torch.full((B, H, d), float("nan"), device="cuda").to(dt_out)
    lse = torch.full((B, H), float("nan"), device="cuda")
    ws = workspace(ap.ap_decode_workspace_bytes(B, H, d, T, Ck.shape[2], ap._DT[q.dtype]))
    ws.fill_(255)                                    # padded heads of the folded query must be written
    if step:
        ap.ap_decode_step(q, kn, vn, Ck, Cv, Bk, Bv, out, ws, T=T, sm_scale=1.0 / math.sqrt(d), lse=lse)
    else:
        ap.ap_decode_attn(q, Ck, Cv, Bk, Bv, out, ws, T=T, sm_scale=1.0 / math.sqrt(d), lse=lse)
    torch.cuda.synchronize()
    return out, lse, Ck, Cv


@pytest.mark.parametrize("step", [False, True], ids=["attend", "step"])
@pytest.mark.parametrize("dtype,B,H,Hkv,d,r,T,scale", [
    ("bf16", 2, 40, 40, 64, 64, 33, 1.0),            # smallest fold: one column tile, half a rank block
    ("f16", 2, 7, 1, 256, 128, 5, 1.0),              # one key/value head
    ("bf16", 33, 40, 40, 128, 192, 40, 1.0),         # three column tiles, the last with one sequence
    ("f16", 17, 24, 8, 64, 320, 97, 1.0),            # grouped queries, ragged tiles, odd rank block
    ("bf16", 16, 33, 33, 32, 320, 64, 1.0),          # hidden axis of 1056: the last stage a quarter full
    ("f16", 65, 48, 48, 64, 640, 33, 1.0),           # expansion: ragged column tile, largest rank
    ("bf16", 65, 48, 48, 64, 640, 33, 1.0),
    ("f16", 64, 64, 4, 128, 256, 70, 1.0),           # expansion, sixteen heads per slice, several splits
    ("bf16", 80, 64, 64, 32, 640, 31, 1.0),          # expansion, narrow heads
    ("f16", 64, 32, 32, 256, 192, 300, 1.0),         # expansion, wide heads
    ("f16", 65, 48, 48, 64, 640, 33, 6.0e3),         # coefficients to the end of fp16, and down where
    ("f16", 65, 48, 48, 64, 640, 33, 2.0e-6),        # most of them are subnormal
    ("bf16", 65, 48, 48, 64, 640, 33, 1.0e30),
    ("bf16", 32, 40, 40, 128, 640, 257, 1.0),        # expansion, eight splits: two rounds of four
    ("bf16", 51, 40, 40, 128, 640, 150, 1.0),        # five splits, the second round with one
    ("bf16", 43, 64, 64, 64, 640, 170, 1.0),         # five, ragged column tile
    ("bf16", 37, 64, 32, 128, 640, 193, 1.0),        # six, grouped queries
    ("bf16", 64, 32, 32, 256, 256, 97, 1.0),         # expansion, wide heads
    ("f16", 64, 64, 64, 128, 256, 128, 1.0),         # fp16 has one round at most: four splits
    ("f16", 51, 40, 40, 128, 640, 150, 1.0),         # five: the expansion per sequence
])
def test_shared_basis(dtype, B, H, Hkv, d, r, T, scale, step):
    from paper_2603_23914_amd import binding as ap
    print(f"shared basis {dtype} B={B} H={H} Hkv={Hkv} d={d} r={r} T={T} scale={scale} step={step}", flush=True)
    dt, HD = TORCH_DT[dtype], Hkv * d
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 + B + r)
    N = lambda *s: torch.randn(s, generator=g, device="cuda")
    law = 4.0 * torch.arange(1, r + 1, device="cuda", dtype=torch.float32) ** -0.7
    Ck = (N(B, T + 7, r) * law).to(dt)
    Cv = (N(B, T + 7, r).clamp(-2.5, 2.5) * law * scale).to(dt)
    Bk, Bv = ((N(r, HD) / math.sqrt(HD)).to(dt) for _ in range(2))
    q, kn, vn = N(B, H, d).to(dt), N(B, HD).to(dt), (N(B, HD) * min(scale, 1.0)).to(dt)
    dt_out = dt if scale == 1.0 and B % 2 else torch.float32
    own = [x[None].expand(B, r, HD).contiguous() for x in (Bk, Bv)]
    out, lse, ck, cv = run(ap, step, q, kn, vn, Ck, Cv, Bk, Bv, T, dt_out)
    out2, lse2, ck2, cv2 = run(ap, step, q, kn, vn, Ck, Cv, *own, T, dt_out)
    rnd = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -11          # one rounding to storage
    sub = 0.0 if dtype == "bf16" else 2.0 ** -25               # and of an fp16 subnormal: half of 2^-24
    for name, a, b, tol in (("out", out, out2, TOL[dtype] + (rnd if dt_out == dt else 0)), ("lse", lse, lse2, TOL[dtype]),
                            ("Ck", ck, ck2, 2 * rnd), ("Cv", cv, cv2, 2 * rnd)):
        a, b = to_host64(a), to_host64(b)
        assert np.isfinite(a).all(), name
        assert np.abs(a - b).max() <= tol * np.abs(b).max() + (2 * sub if name[0] == "C" else 0), name
    for b in (0, B // 2, B - 1):
        P = lambda x: to_host64(x)
        ref = oracle.decode_attn_batched(P(q[b:b + 1]), P(ck[b:b + 1]), P(cv[b:b + 1]), P(Bk)[None], P(Bv)[None], T,
                                         absorbed=True, kv_heads=Hkv)
        err = np.abs(to_host64(out[b:b + 1]) - ref).max()
        assert err <= (TOL[dtype] + (rnd if dt_out == dt else 0)) * np.abs(ref).max(), (b, err)
        if step:
            for x, basis, c in ((kn, Bk, ck), (vn, Bv, cv)):
                row = oracle.compact(P(x[b:b + 1]), P(basis))[0]
                assert np.abs(P(c[b, T - 1]) - row).max() <= 2 * rnd * np.abs(row).max() + sub


def expansion_inputs(dtype, B, H, d, r, T, seed):
    """Inputs of a shared expansion with all logits zero: the merged sums are the tokens' mean."""
    dt, HD = TORCH_DT[dtype], H * d
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    N = lambda *s: torch.randn(s, generator=g, device="cuda")
    q = torch.zeros((B, H, d), dtype=dt, device="cuda")
    return q, N(B, T, r).to(dt), N(B, T, r), (N(r, HD) / 8).to(dt), (N(r, HD) / 8).to(dt)


def written_out(B, *bases):
    return [x[None].expand(B, *x.shape).contiguous() for x in bases]


@pytest.mark.parametrize("dtype,large,small,live", [("f16", 1.0e4, 1.0e-5, 4), ("f16", 1.0e4, 1.0e-3, 624),
                                                    ("bf16", 1.0e30, 1.0e-6, 4)])
def test_shared_expansion_of_small_sums(dtype, large, small, live):
    """Sixteen ranks hold large values that half of the hidden columns do not see: there the output is made of the
    `live` ranks behind them, 2^-20 to 2^-30 of their row's largest and less.  Either expansion is a sum of 640 fp32
    products of a mean of three: at most (640 + 4) 2^-24 of their magnitudes away."""
    from paper_2603_23914_amd import binding as ap
    B, H, d, r, T = 65, 48, 64, 640, 3
    print(f"small sums {dtype} {large} {small} {live}", flush=True)
    q, Ck, Cv, Bk, Bv = expansion_inputs(dtype, B, H, d, r, T, 77)
    Cv[:, :, :16] *= large
    Cv[:, :, 16:] *= small
    Cv[:, :, 16 + live:] = 0.0
    Cv = Cv.to(Bv.dtype)
    Bv[:16, 1::2] = 0.0
    c, b = to_host64(Cv), to_host64(Bv)
    ref, mag = c.mean(axis=1) @ b, np.abs(c).mean(axis=1) @ np.abs(b)
    for bases in ((Bk, Bv), written_out(B, Bk, Bv)):
        out = run(ap, False, q, None, None, Ck, Cv, *bases, T, torch.float32)[0]
        assert (np.abs(to_host64(out).reshape(B, H * d) - ref) <= 644 * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_shared_expansion_with_infinities(dtype):
    """Infinite and NaN elements in the basis, infinite coefficients: signed infinities and NaNs are where the call
    with the basis written out per sequence has them, and everything else is what it has."""
    from paper_2603_23914_amd import binding as ap
    B, H, d, r, T = 65, 48, 64, 640, 33
    print(f"infinities {dtype}", flush=True)
    q, Ck, Cv, Bk, Bv = expansion_inputs(dtype, B, H, d, r, T, 78)
    Cv[5, 3, 40], Cv[6, 32, 639], Cv[7, 0, 0] = float("inf"), float("-inf"), float("nan")
    Cv = Cv.to(Bv.dtype)
    Bv[0, 3], Bv[333, 70], Bv[639, 3071] = float("inf"), float("-inf"), float("inf")
    Bv[17, 200], Bv[400, 200] = float("inf"), float("-inf")               # both signs in one column
    Bv[100, 1000] = float("nan")
    Bv[40, 64:128] = 0.0                                                  # 0 x infinity
    out = to_host64(run(ap, False, q, None, None, Ck, Cv, Bk, Bv, T, torch.float32)[0])
    ref = to_host64(run(ap, False, q, None, None, Ck, Cv, *written_out(B, Bk, Bv), T, torch.float32)[0])
    assert np.isinf(ref[0]).sum() >= 3 and np.isnan(ref[7]).all() and np.isfinite(ref[0]).sum() > 3000
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert (kind(out) == kind(ref)).all(), kind.__name__
    ok = np.isfinite(ref)
    assert np.abs(out[ok] - ref[ok]).max() <= 2 * 644 * 2.0 ** -24 * 2.0 * np.abs(ref[ok]).max()


@pytest.mark.parametrize("case", ["above the largest bfloat16", "below parts of full length"])
def test_shared_expansion_at_the_ends_of_bfloat16(case):
    """Sums of two tokens between the largest bfloat16 and the largest fp32 value; sums so small that bfloat16 parts
    of them are subnormal.  Bounds as for small sums, and half of fp32's smallest value per product."""
    from paper_2603_23914_amd import binding as ap
    B, H, d, r, T = 65, 48, 64, 640, 3
    q, Ck, Cv, Bk, Bv = expansion_inputs("bf16", B, H, d, r, T, 79)
    if case[0] == "a":
        T = 2
        Cv[:, 0, 0], Cv[:, 1, 0] = 2.0 ** 127, 2.0 ** 127 * (1 - 2.0 ** -8)
    else:
        Cv *= 1.0e-37
        Cv[:, :, 4:] = 0.0
    Ck, Cv = Ck[:, :T].contiguous(), Cv[:, :T].bfloat16().contiguous()
    print(f"ends of bfloat16: {case}", flush=True)
    c, b = to_host64(Cv), to_host64(Bv)
    ref, mag = c.mean(axis=1) @ b, np.abs(c).mean(axis=1) @ np.abs(b)
    for bases in ((Bk, Bv), written_out(B, Bk, Bv)):
        out = to_host64(run(ap, False, q, None, None, Ck, Cv, *bases, T, torch.float32)[0]).reshape(B, H * d)
        assert (np.abs(out - ref) <= 644 * 2.0 ** -24 * mag + 640 * 2.0 ** -150).all()
