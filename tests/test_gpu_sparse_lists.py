"""Sparse path: kept lists of every short length (the list is read three blocks ahead), last blocks cut at
odd lengths and rows long enough to be split, against float32 attention of the same bf16 inputs under the
expanded mask.  Tolerance: P and O are rounded to bf16 (2^-9 each, relative), 2.3e-3 of the output's norm;
twice that per 64 rows of a head (a wrong row shows as 1)."""
import math

import pytest
import torch

import paper_2509_22323_amd as ra

pytestmark = pytest.mark.gpu


def reference(q, k, v, mask, block, kv, scale):
    N = q.shape[2]
    out = torch.zeros(q.shape, dtype=torch.float32, device=q.device)
    for h in range(q.shape[1]):
        keep = mask[0, h].bool().repeat_interleave(block, 0).repeat_interleave(block, 1)[:kv, :kv]
        s = (q[0, h, :kv].float() @ k[0, h, :kv].float().t()) * scale
        w = torch.nan_to_num(torch.softmax(s.masked_fill(~keep, -math.inf), -1), nan=0.0)
        out[0, h, :kv] = w @ v[0, h, :kv].float()
    return out


def check(o, ref, kv, what):
    assert (o[:, :, kv:] == 0).all(), what
    o = o.float()
    assert torch.isfinite(o).all(), what
    for r in range(0, kv, 64):
        a, b = o[0, :, r:min(r + 64, kv)].flatten(1), ref[0, :, r:min(r + 64, kv)].flatten(1)
        empty = b.norm(dim=1) == 0
        assert (a[empty] == 0).all(), what
        err = ((a - b).norm(dim=1) / b.norm(dim=1).clamp_min(1e-30))[~empty]
        assert err.numel() == 0 or err.max().item() <= 5e-3, f"{what}: rows {r}..: {err.max().item():.2e}"


def sparse(q, k, v, mask, block, kv):
    B, H, N, D = q.shape
    ws = torch.full((ra.rapid_attn_workspace_bytes(B, H, N, D, block),), 0xa5, dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, 7.0)
    ra.rapid_attn_block_sparse(q, k, v, o, mask, block, kv, workspace=ws)
    return o


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("cut", [0, 1, 31, 32, 33, 63, 64, 65, 127])
def test_every_list_length_and_odd_tails(D, block, cut):
    nb, H = 24, 3
    N = nb * block
    kv = N - min(cut, block - 1)
    g = torch.Generator(device="cuda").manual_seed(D + block + cut)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    for t in (q, k, v):
        t[:, :, kv:] = float("nan")
    rank = torch.rand((1, H, nb, nb), generator=g, device="cuda").argsort(-1).argsort(-1)
    length = torch.arange(nb, device="cuda").view(1, 1, nb, 1).expand(1, H, nb, 1) + torch.arange(H, device="cuda").view(1, H, 1, 1)
    mask = (rank < length).to(torch.uint8)        # rows of 0 .. nb kept blocks, the last block among them or not
    o = sparse(q, k, v, mask, block, kv)
    check(o, reference(q, k, v, mask, block, kv, D ** -0.5), kv, f"D={D} block={block} kv={kv}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("block", [64, 128])
def test_reference_of_the_exponents_moves(D, block):
    """Scores that climb by 72 (base 2) above a row's first keys, inside a block, in a later block
    and in another piece of a split row, and rows whose first keys are the largest by far."""
    nb, H = 40, 2
    N = nb * block
    g = torch.Generator(device="cuda").manual_seed(17 + D)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    q[..., 0] = 8.0
    q[:, :, 1::7, 0] = -8.0
    k[..., 0] = 0.0
    step = 50.0 * math.sqrt(D) / 8.0
    for i, at in enumerate((70, 150, N // 2 + 211)):
        k[:, :, at:, 0] = (i + 1) * step
    mask = (torch.rand((1, H, nb, nb), generator=g, device="cuda") < 0.2).to(torch.uint8)
    mask[:, :, :, 0] = 1
    mask[:, :, 5::9] = 1
    o = sparse(q, k, v, mask, block, N)
    check(o, reference(q, k, v, mask, block, N, D ** -0.5), N, f"D={D} block={block}")
