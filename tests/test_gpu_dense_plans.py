"""Dense path: every kernel and every way the items of an XCD are cut (run_dense), at lengths where the
32-key steps, the 64-key tiles and the unrolled loops end differently, against float32 attention of the
same bf16 inputs.  Tolerance: P and O are rounded to bf16 (2^-9 each, relative), which is 2.3e-3 of the
output's norm; twice that per 64 rows of a head (a wrong row shows as 1)."""
import math

import pytest
import torch

import paper_2509_22323_amd as ra

pytestmark = pytest.mark.gpu

# heads, tokens allocated: small kernel; whole items; pieces of 192 queries; full rounds with the rest in halves, in quarters; one round
# of whole items, of halves, of quarters (run_dense)
PLANS = {64: [("small", 3, 300), ("small, many", 200, 64), ("small, second round", 30, 1100), ("whole", 80, 1100),
              ("half", 70, 1100), ("quarter", 64, 1100), ("one round, whole", 40, 1100), ("one round of halves", 40, 1300),
              ("one round of quarters", 32, 1300)],
         128: [("small", 3, 300), ("small, many", 200, 64), ("whole", 45, 1100), ("pieces of 192", 30, 1100),
               ("a round and pieces of 192", 82, 1100), ("half", 24, 1100), ("quarter", 8, 1100)]}
CASES = [(D, plan, H, N, kv) for D in (64, 128) for plan, H, N in PLANS[D]
         for kv in (N, N - 13, N // 2 + 1, 257, 96, 65, 64, 33, 32, 31, 1) if kv <= N]


def reference(q, k, v, kv, scale):
    out = torch.zeros(q.shape, dtype=torch.float32, device=q.device)
    for h in range(q.shape[1]):
        s = (q[0, h, :kv].float() @ k[0, h, :kv].float().t()) * scale
        out[0, h, :kv] = torch.softmax(s, -1) @ v[0, h, :kv].float()
    return out


def check(o, ref, kv, what):
    assert (o[:, :, kv:] == 0).all(), what
    o = o.float()
    assert torch.isfinite(o).all(), what
    for r in range(0, kv, 64):
        a, b = o[0, :, r:min(r + 64, kv)], ref[0, :, r:min(r + 64, kv)]
        err = ((a - b).flatten(1).norm(dim=1) / b.flatten(1).norm(dim=1)).max().item()
        assert err <= 5e-3, f"{what}: rows {r}..: {err:.2e}"


@pytest.mark.parametrize("D,plan,H,N,kv", CASES)
def test_dense_plan_at_odd_lengths(D, plan, H, N, kv):
    g = torch.Generator(device="cuda").manual_seed(D + N + kv)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    for t in (q, k, v):
        t[:, :, kv:] = float("nan")
    o = torch.full_like(q, 7.0)
    ra.rapid_attn_dense(q, k, v, o, kv)
    check(o, reference(q, k, v, kv, D ** -0.5), kv, f"{plan} D={D} kv={kv}")


@pytest.mark.parametrize("D,plan,H,N", [(D, *p) for D in (64, 128) for p in PLANS[D]])
def test_reference_of_the_exponents_moves(D, plan, H, N):
    """Scores that climb by 72 (base 2) above a row's first keys, twice, at keys that lie in the
    first and in the second half of a step, and a row whose first keys are the largest by far."""
    g = torch.Generator(device="cuda").manual_seed(17 + D)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    q[..., 0] = 8.0
    q[:, :, 1::7, 0] = -8.0                                     # for these rows the first keys are the largest
    k[..., 0] = 0.0
    step = 50.0 * math.sqrt(D) / 8.0                            # 50 in the exponent of e = 72 in that of 2
    for i, at in enumerate((70, 150, 211)):
        k[:, :, at:, 0] = (i + 1) * step
    o = torch.empty_like(q)
    ra.rapid_attn_dense(q, k, v, o)
    check(o, reference(q, k, v, N, D ** -0.5), N, f"{plan} D={D}")


@pytest.mark.parametrize("D,plan,H,N", [(D, *p) for D in (64, 128) for p in PLANS[D]])
def test_dense_plan_on_joint_tensors_with_lengths(D, plan, H, N):
    """The same plans on fused projections, image and text apart, with a length per sample: full, a short prompt,
    none, inside the image."""
    pairs = H
    B = next(b for b in (4, 3, 2, 1) if pairs % b == 0)
    H = pairs // B
    n0 = (N - 1) // 128 * 128
    if n0 == 0:
        n0 = N
    lens = [N, min(n0 + 5, N), 0, n0 // 3][:B]
    g = torch.Generator(device="cuda").manual_seed(D + N)
    tokens = [n for n in (n0, N - n0) if n]
    fused = [torch.randn((B, n, 3, H, D), generator=g, device="cuda", dtype=torch.bfloat16) for n in tokens]
    segs = [tuple(f[:, :, i].transpose(1, 2) for i in range(3)) + (torch.full((B, n, H, D), 7.0, device="cuda", dtype=torch.bfloat16).transpose(1, 2),)
            for f, n in zip(fused, tokens)]
    ra.rapid_attn_joint(segs, kv_lens=torch.tensor(lens, dtype=torch.int32, device="cuda"))
    q, k, v, o = (torch.cat([s[i] for s in segs], 2) for i in range(4))
    for b, kv in enumerate(lens):
        if kv == 0:
            assert (o[b] == 0).all(), plan
        else:
            check(o[b:b + 1], reference(q[b:b + 1], k[b:b + 1], v[b:b + 1], kv, D ** -0.5), kv, f"{plan} D={D} sample {b}")
