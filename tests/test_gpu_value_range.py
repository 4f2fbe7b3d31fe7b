"""Attention over the range of its inputs: every output row is a weighted mean of values, so values scaled by a power
of two give outputs scaled by it, from near the bottom of bf16's exponents to near their top, on every dense plan and
every sparse kernel; and rows whose first keys have no finite score.  Against float32 attention of the unscaled bf16
inputs.  Tolerance: P and O are rounded to bf16 (2^-9 each, relative), 2.3e-3 of the output's norm; twice that per 64
rows of a head."""
import math

import pytest
import torch

import paper_2509_22323_amd as ra
from test_gpu_dense_plans import PLANS

pytestmark = pytest.mark.gpu

# A row's weights before the division by their sum are at most 2^-16 on the paths that take no row maximum, 2^-24 once
# its scores have climbed: subnormal sums leave bf16's precision down to V * 2^-120 and 2^-112.  The top is what the
# weights under climbing scores, up to 2^60 on the kernel of short rows at D = 64, leave room for.
SCALES = {False: [-118, -100, -80, 100], True: [-110, -100, -80, 50]}
# name, heads, blocks per side, block; the last is cut into 128-token rows of the kernel for many rows at D = 64
SPARSE = [("block 64", 3, 24, 64), ("block 128", 3, 24, 128), ("many rows", 100, 21, 128)]


def attention(q, k, v, mask=None, block=1):
    out = torch.zeros(q.shape, dtype=torch.float32, device=q.device)
    for h in range(q.shape[1]):
        s = (q[0, h].float() @ k[0, h].float().t()) * q.shape[3] ** -0.5
        if mask is not None:
            s = s.masked_fill(~mask[0, h].bool().repeat_interleave(block, 0).repeat_interleave(block, 1), -math.inf)
        out[0, h] = torch.softmax(s, -1) @ v[0, h].float()
    return out


def check(o, ref, power, what):
    scaled = o.float().double() * 2.0 ** -power
    assert torch.isfinite(scaled).all(), what
    N = o.shape[2]
    for r in range(0, N, 64):
        a, b = scaled[0, :, r:min(r + 64, N)].flatten(1), ref[0, :, r:min(r + 64, N)].flatten(1).double()
        err = ((a - b).norm(dim=1) / b.norm(dim=1)).max().item()
        assert err <= 5e-3, f"{what}, V * 2^{power}: rows {r}..: {err:.2e}"


def inputs(H, N, D, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return g, *(torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))


def climbing(q, k, D):
    """Later keys score up to 100 (base 2) above the first ones, in steps of 50; odd rows the other way round."""
    q[..., 0] = 8.0
    q[:, :, 1::7, 0] = -8.0
    k[..., 0] = 0.0
    for i, at in enumerate((70, k.shape[2] // 2 + 3)):
        k[:, :, at:, 0] = (i + 1) * 50.0 * math.log(2.0) * math.sqrt(D) / 8.0


def mask_of(g, H, nb):
    mask = (torch.rand((1, H, nb, nb), generator=g, device="cuda") < 0.3).to(torch.uint8)
    mask[:, :, :, 0] = 1
    mask[:, :, 5::9] = 1
    return mask


@pytest.mark.parametrize("climb", [False, True])
@pytest.mark.parametrize("D,plan,H,N", [(D, *p) for D in (64, 128) for p in PLANS[D]])
def test_dense_scales_with_v(D, plan, H, N, climb):
    _, q, k, v = inputs(H, N, D, 5 + D)
    if climb:
        climbing(q, k, D)
    ref = attention(q, k, v)
    for power in SCALES[climb]:
        o = torch.empty_like(q)
        ra.rapid_attn_dense(q, k, (v.double() * 2.0 ** power).to(torch.bfloat16), o)
        check(o, ref, power, f"{plan} D={D}")


@pytest.mark.parametrize("climb", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name,H,nb,block", SPARSE)
def test_sparse_scales_with_v(D, name, H, nb, block, climb):
    g, q, k, v = inputs(H, nb * block, D, 6 + D)
    if climb:
        climbing(q, k, D)
    mask = mask_of(g, H, nb)
    ref = attention(q, k, v, mask, block)
    for power in SCALES[climb]:
        o = torch.empty_like(q)
        ra.rapid_attn_block_sparse(q, k, (v.double() * 2.0 ** power).to(torch.bfloat16), o, mask, block)
        check(o, ref, power, f"{name} D={D}")


@pytest.mark.parametrize("climb", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("nb", [8, 24, 70])
def test_64_token_masks_keep_small_values(nb, D, climb):
    """A row's largest weight is at least 2^-5 there (the reference lies 4 above a first or a later maximum), so sums over
    V * 2^-120 lie 20 bits and more above the last subnormal of fp32; much below, the outputs, means of up to 1400 values,
    leave bf16's own normal numbers."""
    g, q, k, v = inputs(3, nb * 64, D, 6 + D)
    if climb:
        climbing(q, k, D)
    mask = mask_of(g, 3, nb)
    o = torch.empty_like(q)
    ra.rapid_attn_block_sparse(q, k, (v.double() * 2.0 ** -120).to(torch.bfloat16), o, mask, 64)
    check(o, attention(q, k, v, mask, 64), -120, f"D={D} nb={nb}")


@pytest.mark.parametrize("D", [64, 128])
def test_64_token_masks_largest_weights_of_peaked_rows(D):
    """Scores of standard deviation 4: one weight carries a row, and its rounding to bf16 (1.7e-3 in the mean) the row's
    error, unless it is a reference of the exponents and so a power of two.  With every reference at a row's first maximum
    the outputs are off by 1.91e-3, with references that follow within 8 of the running maximum by 1.86e-3, within 4
    by 1.81e-3 (24 x 2816 rows: the figure itself varies by 2e-6)."""
    H, N = 24, 2816
    g, q, k, v = inputs(H, N, D, 9 + D)
    q *= 4
    mask = torch.ones((1, H, N // 64, N // 64), dtype=torch.uint8, device="cuda")
    o = torch.empty_like(q)
    ra.rapid_attn_block_sparse(q, k, v, o, mask, 64)
    off = size = 0.0
    for h in range(H):
        w = torch.softmax(q[0, h].double() @ k[0, h].double().t() * D ** -0.5, -1) @ v[0, h].double()
        off += (o[0, h].double() - w).square().sum().item()
        size += w.square().sum().item()
    assert (off / size) ** 0.5 <= 1.86e-3, (off / size) ** 0.5


def without_finite_start(q, k, keys):
    """The first `keys` keys score -inf for every query (their products leave fp32), the others are ordinary."""
    q[..., 1] = 2.0 ** 80
    k[..., 1] = 0.0
    k[:, :, :keys, 1] = -(2.0 ** 80)


@pytest.mark.parametrize("keys", [32, 40])
@pytest.mark.parametrize("D,plan,H,N", [(D, *p) for D in (64, 128) for p in PLANS[D]])
def test_dense_first_keys_at_minus_infinity(D, plan, H, N, keys):
    _, q, k, v = inputs(H, N, D, 7 + D)
    without_finite_start(q, k, keys)
    o = torch.empty_like(q)
    ra.rapid_attn_dense(q, k, v, o)
    check(o, attention(q, k, v), 0, f"{plan} D={D}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("name,H,nb,block", SPARSE)
def test_sparse_first_keys_at_minus_infinity(D, name, H, nb, block):
    g, q, k, v = inputs(H, nb * block, D, 8 + D)
    without_finite_start(q, k, 40)
    mask = mask_of(g, H, nb)
    o = torch.empty_like(q)
    ra.rapid_attn_block_sparse(q, k, v, o, mask, block)
    check(o, attention(q, k, v, mask, block), 0, f"{name} D={D}")
