"""Sparse path: kept lists of every short length (the list is read ahead), last blocks cut at
odd lengths and rows long enough to be split, against float32 attention of the same bf16 inputs under the
expanded mask.  Tolerance: P and O are rounded to bf16 (2^-9 each, relative), 2.3e-3 of the output's norm;
twice that per 64 rows of a head (a wrong row shows as 1)."""
import math

import numpy as np
import pytest
import torch

import paper_2509_22323_amd as ra
from test_gpu_parity import check_plan, read_plan

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
def test_lists_longer_than_a_wavefront_holds(D):
    """64-token masks: a wavefront holds 64 entries of the list and reads on every 64, up to four entries ahead of their
    use; rows of every length from 50 to 132 kept blocks, the last block of all cut."""
    block, nb = 64, 132
    N, kv = nb * block, nb * block - 45
    g = torch.Generator(device="cuda").manual_seed(D)
    q, k, v = (torch.randn((1, 1, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    rank = torch.rand((1, 1, nb, nb), generator=g, device="cuda").argsort(-1).argsort(-1)
    length = (torch.arange(nb, device="cuda").view(1, 1, nb, 1) * 5) % 83 + 50
    mask = (rank < length).to(torch.uint8)
    o = sparse(q, k, v, mask, block, kv)
    check(o, reference(q, k, v, mask, block, kv, D ** -0.5), kv, f"D={D}")


@pytest.mark.parametrize("nb", [23, 24, 66])
@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("H", [1, 2, 3, 4, 5, 7, 8])
def test_pairs_dealt_out_over_the_chip(H, block, nb):
    """Fewer (sample, head) pairs than XCDs, on either side of the rows from which they are dealt out to all of them,
    with one planner launch and with two, long rows cut: every entry done once, lists and plan as ever."""
    D = 128 if (H + nb) % 2 else 64
    N, kv = nb * block, nb * block - 45
    g = torch.Generator(device="cuda").manual_seed(H * nb + block)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = (torch.rand((1, H, nb, nb), generator=g, device="cuda") < 0.2).to(torch.uint8)
    mask[:, :, -3:] = 1                            # (text rows)
    mask[:, 0, 5] = 0
    ws = torch.full((ra.rapid_attn_workspace_bytes(1, H, N, D, block),), 0xa5, dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, 7.0)
    ra.rapid_attn_block_sparse(q, k, v, o, mask, block, kv, workspace=ws)
    check(o, reference(q, k, v, mask, block, kv, D ** -0.5), kv, f"H={H} nb={nb} block={block}")
    counts, order, index, geo = read_plan(ws.cpu().numpy(), 1, H, nb, D, block)
    assert (counts == mask.sum(-1).flatten().cpu().numpy()).all()
    cut = check_plan(counts, order, geo, 1, H, nb, block, D)
    assert cut or block == 64


@pytest.mark.parametrize("H,nb,cut", [(4, 48, False), (7, 36, False), (8, 24, False), (4, 65, True), (7, 37, True), (8, 33, True), (24, 24, True)])
def test_rows_all_alike_are_cut_where_it_helps(H, nb, cut):
    """All ones, D = 128: with a CU for every row none is cut, as there are too few slots for the pieces of all of them."""
    D, block = 128, 128
    N = nb * block
    g = torch.Generator(device="cuda").manual_seed(H * nb)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = torch.ones((1, H, nb, nb), dtype=torch.uint8, device="cuda")
    ws = torch.full((ra.rapid_attn_workspace_bytes(1, H, N, D, block),), 0xa5, dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, 7.0)
    ra.rapid_attn_block_sparse(q, k, v, o, mask, block, N, workspace=ws)
    check(o, reference(q, k, v, mask, block, N, D ** -0.5), N, f"H={H} nb={nb}")
    counts, order, _, geo = read_plan(ws.cpu().numpy(), 1, H, nb, D, block)
    assert bool(check_plan(counts, order, geo, 1, H, nb, block, D)) == cut


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


# ---- D = 64, 128-token masks, more than 2048 rows of more than 8 blocks: 64 queries per wavefront
MANY = 96                                          # heads


@pytest.mark.parametrize("cut", [0, 1, 31, 32, 33, 63, 64, 65, 127])
def test_many_rows_every_list_length_and_odd_tails(cut):
    D, block, nb = 64, 128, 24
    N = nb * block
    kv = N - cut
    g = torch.Generator(device="cuda").manual_seed(cut)
    q, k, v = (torch.randn((1, MANY, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    for t in (q, k, v):
        t[:, :, kv:] = float("nan")
    rank = torch.rand((1, MANY, nb, nb), generator=g, device="cuda").argsort(-1).argsort(-1)
    length = (torch.arange(nb, device="cuda").view(1, 1, nb, 1) + torch.arange(MANY, device="cuda").view(1, MANY, 1, 1)) % (nb + 1)
    mask = (rank < length).to(torch.uint8)
    o = sparse(q, k, v, mask, block, kv)
    assert torch.equal(o.view(torch.int16), sparse(q, k, v, mask, block, kv).view(torch.int16))
    check(o, reference(q, k, v, mask, block, kv, D ** -0.5), kv, f"kv={kv}")


@pytest.mark.parametrize("nb", [8, 9])
def test_many_rows_on_either_side_of_the_rule(nb):
    D, block, H = 64, 128, 272                     # 2176 and 2448 rows
    N = nb * block
    g = torch.Generator(device="cuda").manual_seed(nb)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = (torch.rand((1, H, nb, nb), generator=g, device="cuda") < 0.3).to(torch.uint8)
    o = sparse(q, k, v, mask, block, N - 9)
    check(o, reference(q, k, v, mask, block, N - 9, D ** -0.5), N - 9, f"nb={nb}")


def test_many_rows_references_of_the_exponents_move():
    D, block, nb = 64, 128, 24
    N = nb * block
    g = torch.Generator(device="cuda").manual_seed(18)
    q, k, v = (torch.randn((1, MANY, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    q[..., 0] = 8.0
    q[:, :, 1::7, 0] = -8.0
    k[..., 0] = 0.0
    for i, at in enumerate((70, 150, N // 2 + 211)):
        k[:, :, at:, 0] = (i + 1) * 50.0 * math.sqrt(D) / 8.0
    mask = (torch.rand((1, MANY, nb, nb), generator=g, device="cuda") < 0.3).to(torch.uint8)
    mask[:, :, :, 0] = 1
    o = sparse(q, k, v, mask, block, N)
    check(o, reference(q, k, v, mask, block, N, D ** -0.5), N, "moving")


@pytest.mark.parametrize("climb", [False, True])
def test_many_rows_with_long_ones_cut_into_pieces(climb):
    """A few full rows among rows of one to four blocks: the plan cuts the full ones; every piece count,
    the merge of pieces whose references differ by up to 216 (base 2), and an odd last block."""
    D, block, nb, H = 64, 128, 260, 8
    N = nb * block
    kv = N - 37
    g = torch.Generator(device="cuda").manual_seed(21)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    if climb:
        q[..., 0] = 8.0
        q[:, :, 1::7, 0] = -8.0
        k[..., 0] = 0.0
        for i, at in enumerate((70, N // 3 + 5, N // 2 + 211)):
            k[:, :, at:, 0] = (i + 1) * 50.0 * math.sqrt(D) / 8.0
    mask = torch.zeros((1, H, nb, nb), dtype=torch.uint8, device="cuda")
    mask.diagonal(dim1=2, dim2=3).fill_(1)
    mask |= (torch.rand((1, H, nb, nb), generator=g, device="cuda") < 1.0 / nb).to(torch.uint8)
    full = {h: [3, 100 + h, nb - 1] for h in range(H)}
    for h, rows in full.items():
        for i, r in enumerate(rows):               # all of it, a third, all but the first blocks
            mask[0, h, r] = 1
            if i == 1:
                mask[0, h, r, nb // 3:] = 0
            if i == 2:
                mask[0, h, r, :40 + h] = 0
    ws = torch.zeros(ra.rapid_attn_workspace_bytes(1, H, N, D, block), dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, 7.0)
    ra.rapid_attn_block_sparse(q, k, v, o, mask, block, kv, workspace=ws)
    counts, order, _, geometry = read_plan(ws.cpu().numpy(), 1, H, nb, D, block)
    cut = check_plan(counts, order, geometry, 1, H, nb, block, D)
    assert {h * nb + r for h, rows in full.items() for r in rows} <= set(cut), sorted(cut)
    assert (o[:, :, kv:] == 0).all()
    for h in range(H):
        for r in full[h] + [0, 1, 50, nb - 2]:
            a, e = r * block, min((r + 1) * block, kv)
            keys = mask[0, h, r].bool().repeat_interleave(block)[:kv].nonzero()[:, 0]
            s = (q[0, h, a:e].float() @ k[0, h, keys].float().t()) * D ** -0.5
            want = torch.softmax(s, -1) @ v[0, h, keys].float()
            for i in range(0, e - a, 64):
                x, y = o[0, h, a + i:min(a + i + 64, e)].float(), want[i:i + 64]
                assert ((x - y).norm() / y.norm()).item() <= 5e-3, (h, r, i)


def test_many_rows_joint_tensors_and_lengths():
    """Image and text apart, fused projections, per-sample lengths: 2160 rows of 9 blocks."""
    B, H, D, block, n0, n1 = 4, 60, 64, 128, 1024, 100
    N, nb = n0 + n1, 9
    lens = [N, n0 + 5, 0, 300]
    g = torch.Generator(device="cuda").manual_seed(60)
    fused = [torch.randn((B, n, 3, H, D), generator=g, device="cuda", dtype=torch.bfloat16) for n in (n0, n1)]
    segs = [tuple(f[:, :, i].transpose(1, 2) for i in range(3)) + (torch.full((B, n, H, D), 7.0, device="cuda", dtype=torch.bfloat16).transpose(1, 2),)
            for f, n in zip(fused, (n0, n1))]
    mask = (torch.rand((B, H, nb, nb), generator=g, device="cuda") < 0.4).to(torch.uint8)
    ra.rapid_attn_joint(segs, mask, block, kv_lens=torch.tensor(lens, dtype=torch.int32, device="cuda"))
    q, k, v, o = (torch.cat([s[i] for s in segs], 2) for i in range(4))
    for b, kv in enumerate(lens):
        if kv == 0:
            assert (o[b] == 0).all()
            continue
        grown = [torch.nn.functional.pad(t[b:b + 1], (0, 0, 0, nb * block - N)) for t in (q, k, v, o)]
        ref = reference(*grown[:3], mask[b:b + 1], block, kv, D ** -0.5)
        check(grown[3], ref, kv, f"sample {b}")


# ---- where the plan comes from: every workgroup for itself (all rows on the chip at once), one planner launch from the
# mask, or compaction and a planner; sizes on either side of each, with per-sample lengths
def counts_lists_and_plan(block, B, H, nb, D):
    N = nb * block - 5
    g = torch.Generator(device="cuda").manual_seed(B + H + nb)
    q, k, v = (torch.randn((B, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    lens = torch.randint(0, N + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0], lens[-1] = N + 3, N - block // 2
    density = torch.rand((B, H, nb, 1), generator=g, device="cuda")
    mask = (torch.rand((B, H, nb, nb), generator=g, device="cuda") < density).to(torch.uint8) * 200
    mask[:, :, -1] = 1
    ws = torch.full((ra.rapid_attn_joint_workspace_bytes(B, H, N, D, block),), 0xa5, dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, 7.0)
    ra.rapid_attn_joint([(q, k, v, o)], mask, block, kv_lens=lens, workspace=ws)
    counts, order, index, geometry = read_plan(ws.cpu().numpy(), B, H, nb, D, block)
    kv = lens.clamp(0, N).view(B, 1, 1, 1)
    kept = (mask != 0) & (torch.arange(nb, device="cuda") * block < kv)
    assert (torch.from_numpy(counts.copy()) == kept.sum(-1).flatten().cpu()).all()
    kept = kept.reshape(-1, nb).cpu()
    for r in torch.randint(0, kept.shape[0], (300,)).tolist() + [0, kept.shape[0] - 1]:
        assert index[r, :counts[r]].tolist() == kept[r].nonzero()[:, 0].tolist(), r
    check_plan(counts, order, geometry, B, H, nb, block, D)
    for b in sorted({0, B // 2, B - 1}):
        n = int(kv[b])
        if n == 0:
            assert (o[b] == 0).all()
            continue
        for h in sorted({0, H - 1}):
            one = [torch.nn.functional.pad(t[b:b + 1, h:h + 1], (0, 0, 0, 5)) for t in (q, k, v, o)]
            check(one[3], reference(*one[:3], mask[b:b + 1, h:h + 1], block, n, D ** -0.5), n, f"sample {b} head {h}")
    return order


@pytest.mark.parametrize("block,B,H,nb,D", [
    (64, 1, 1, 1, 64), (64, 3, 5, 2, 128), (64, 3, 8, 21, 128), (64, 3, 8, 22, 128), (64, 4, 8, 24, 64), (64, 4, 8, 25, 64),
    (64, 2, 40, 64, 64), (64, 2, 40, 63, 128), (64, 1, 8, 65, 64), (64, 3, 8, 65, 128), (64, 300, 8, 2, 64), (64, 200, 40, 3, 64),
    (64, 9, 120, 33, 64), (128, 2, 32, 8, 128), (128, 5, 13, 8, 128), (128, 4, 32, 8, 64), (128, 3, 8, 15, 64), (128, 3, 8, 16, 64),
    (128, 64, 40, 1, 64), (128, 900, 40, 1, 64), (128, 8, 24, 36, 64), (128, 8, 40, 64, 64), (128, 2, 8, 65, 128)])
def test_counts_lists_and_plan_wherever_they_are_made(block, B, H, nb, D):
    counts_lists_and_plan(block, B, H, nb, D)


# the rules of run_sparse: more rows of an XCD than places (2 to 4 per CU), rows long enough to be cut, more than one (D = 128) or
# two rows per CU that are not short; fewer pairs than XCDs spread over the chip; from the list and from the mask
@pytest.mark.parametrize("block,B,H,nb,D,planned", [
    (64, 6, 8, 16, 64, False), (64, 7, 8, 14, 64, True), (64, 5, 8, 16, 64, False), (64, 5, 8, 17, 64, True), (64, 3, 8, 21, 64, False),
    (64, 2, 8, 32, 64, False), (64, 2, 8, 33, 64, True), (64, 2, 8, 24, 128, False), (64, 2, 8, 25, 128, True), (64, 1, 8, 32, 128, False),
    (64, 1, 8, 33, 128, True), (64, 1, 4, 128, 128, False), (64, 1, 4, 130, 128, True), (64, 1, 3, 172, 128, True), (64, 1, 2, 65, 64, False),
    (128, 21, 8, 6, 64, False), (128, 22, 8, 6, 64, True), (128, 9, 8, 7, 64, False), (128, 10, 8, 7, 64, True), (128, 4, 8, 15, 64, False),
    (128, 5, 8, 15, 64, True), (128, 1, 8, 15, 128, False), (128, 1, 8, 16, 128, True), (128, 4, 8, 15, 128, False), (128, 5, 8, 13, 128, True)])
def test_either_side_of_the_plan_rules(block, B, H, nb, D, planned):
    order = counts_lists_and_plan(block, B, H, nb, D)[..., 0]
    own = np.full(order.shape, -1)                 # a workgroup's row where there is no plan
    for x in range(8):
        for i in range(order.shape[1]):
            g = i // nb
            if (g * 8 + x) < B * H:
                own[x, i] = (g * 8 + x) * nb + (i + g * nb // 32 * ((3 * nb + 7) // 8)) % nb
    assert (order == own).all() == (not planned)


@pytest.mark.parametrize("D,H,nb", [(128, 16, 36), (128, 88, 13), (128, 24, 48), (128, 24, 49), (64, 16, 64), (64, 100, 8), (64, 32, 64), (64, 40, 52)])
@pytest.mark.parametrize("alike", [False, True])
def test_64_token_rows_looked_up_without_a_plan(D, H, nb, alike):
    """Either side of the line up to which workgroups look their rows up by themselves (more rows than places): every row
    done once, longest first, rows without a block and ties among them, lists, counts and plan left as ever."""
    block = 64
    N, kv = nb * block, nb * block - 29
    g = torch.Generator(device="cuda").manual_seed(H * nb + D)
    q, k, v = (torch.randn((1, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = (torch.rand((1, H, nb, nb), generator=g, device="cuda") < 0.3).to(torch.uint8) * 3
    mask[:, :, 4], mask[:, 1, 5], mask[:, :, -2:] = 0, 0, 255
    if alike:
        mask[:] = 1
    ws = torch.full((ra.rapid_attn_workspace_bytes(1, H, N, D, block),), 0xa5, dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, 7.0)
    ra.rapid_attn_block_sparse(q, k, v, o, mask, block, kv, workspace=ws)
    check(o, reference(q, k, v, mask, block, kv, D ** -0.5), kv, f"D={D} H={H} nb={nb}")
    counts, order, index, geo = read_plan(ws.cpu().numpy(), 1, H, nb, D, block)
    host = mask.cpu().numpy().reshape(H * nb, nb) != 0
    assert (counts == host.sum(-1)).all()
    check_plan(counts, order, geo, 1, H, nb, block, D)
    for x in range(8):                             # (the second round of 32 backwards)
        items = order[x][order[x][:, 0] >= 0, 0]
        lengths = counts[items]
        lengths[32:64] = lengths[32:64][::-1]
        assert (np.diff(lengths) <= 0).all(), x
    for r in range(H * nb):
        assert (index[r, :counts[r]] == np.flatnonzero(host[r])).all(), r


@pytest.mark.parametrize("D", [64, 128])
def test_64_token_rows_of_a_selected_mask_looked_up_without_a_plan(D):
    """Counts and lists from the selection, samples of different length (an empty one too): as under the mask it reports."""
    B, H, block = 3, 16, 64
    N = 22 * block - 5                             # 6 pairs of an XCD: 132 rows
    g = torch.Generator(device="cuda").manual_seed(D)
    q, k, v = (torch.randn((B, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    lens = torch.tensor([N, 0, N - 700], dtype=torch.int32, device="cuda")
    mask = torch.empty((B, H, 22, 22), dtype=torch.uint8, device="cuda")
    out = [torch.full_like(q, 7.0) for _ in range(2)]
    ws = [torch.full((ra.rapid_attn_joint_select_workspace_bytes(B, H, N, D, block),), 0xa5, dtype=torch.uint8, device="cuda") for _ in range(2)]
    ra.rapid_attn_joint_select([(q, k, v, out[0])], block, kv_lens=lens, text_start=20 * block, tau=0.7, mask_out=mask, workspace=ws[0])
    ra.rapid_attn_joint([(q, k, v, out[1])], mask=mask, block=block, kv_lens=lens, workspace=ws[1])
    assert torch.equal(out[0], out[1])
    plans = [read_plan(x.cpu().numpy(), B, H, 22, D, block) for x in ws]
    live = [(n + block - 1) // block for n in lens.tolist()]
    kept = torch.stack([mask[b, :, :, :n].sum(-1) for b, n in enumerate(live)]).flatten().cpu().numpy()
    for counts, order, index, geo in plans:        # counts of the selection, or the attention's own
        assert (counts == kept).all()
        check_plan(counts, order, geo, B, H, 22, block, D)
    assert (plans[0][1] == plans[1][1]).all()
    for b, n in enumerate(lens.tolist()):
        if n == 0:
            assert (out[0][b] == 0).all()
            continue
        pad = torch.zeros((1, H, 22 * block, D), dtype=torch.bfloat16, device="cuda")
        full = [torch.cat([x[b:b + 1], pad], 2)[:, :, :22 * block] for x in (q, k, v)]
        ref = reference(*full, mask[b:b + 1], block, n, D ** -0.5)
        check(torch.cat([out[0][b:b + 1], pad], 2)[:, :, :22 * block], ref, n, f"D={D} sample {b}")


@pytest.mark.parametrize("D,B,H,nb,alike", [(64, 3, 24, 8, False), (64, 2, 56, 15, True), (64, 3, 64, 10, False), (64, 5, 40, 11, False), (64, 3, 62, 11, False),
                                            (128, 2, 20, 8, False), (128, 4, 24, 12, True), (128, 2, 64, 12, False), (128, 1, 132, 12, False), (128, 1, 38, 15, False)])
def test_128_token_rows_looked_up_without_a_plan(D, B, H, nb, alike):
    """As above for rows of 8 to 15 blocks of 128 tokens, up to 2048 rows and beyond, either side of the line;
    samples of different length; the same lists from a mask that is given and from one that is selected."""
    block, N = 128, nb * 128
    g = torch.Generator(device="cuda").manual_seed(H * nb + D)
    q, k, v = (torch.randn((B, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = (torch.rand((B, H, nb, nb), generator=g, device="cuda") < 0.4).to(torch.uint8) * 3
    mask[:, :, 4], mask[:, 1, 5], mask[:, :, -2:] = 0, 0, 255
    if alike:
        mask[:] = 1
    host = mask.cpu().numpy().reshape(B * H * nb, nb) != 0
    lens = [N - 29 - 300 * b for b in range(B)]
    for kv_lens in (None, torch.tensor(lens, dtype=torch.int32, device="cuda")):
        ws = torch.full((ra.rapid_attn_workspace_bytes(B, H, N, D, block),), 0xa5, dtype=torch.uint8, device="cuda")
        o = torch.full_like(q, 7.0)
        if kv_lens is None:
            ra.rapid_attn_block_sparse(q, k, v, o, mask, block, N - 29, workspace=ws)
        else:
            ra.rapid_attn_joint([(q, k, v, o)], mask=mask, block=block, kv_lens=kv_lens)
        for b in range(B):
            n = N - 29 if kv_lens is None else lens[b]
            ref = reference(*(x[b:b + 1] for x in (q, k, v)), mask[b:b + 1], block, n, D ** -0.5)
            check(o[b:b + 1], ref, n, f"D={D} H={H} nb={nb} sample {b}")
        if kv_lens is None:
            counts, order, index, geo = read_plan(ws.cpu().numpy(), B, H, nb, D, block)
            assert (counts == host.sum(-1)).all()
            check_plan(counts, order, geo, B, H, nb, block, D)
            for r in range(B * H * nb):
                assert (index[r, :counts[r]] == np.flatnonzero(host[r])).all(), r
    chosen = torch.empty_like(mask)
    out = [torch.full_like(q, 7.0) for _ in range(2)]
    ra.rapid_attn_joint_select([(q, k, v, out[0])], block, kv_lens=kv_lens, text_start=(nb - 2) * block, tau=0.7, mask_out=chosen)
    ra.rapid_attn_joint([(q, k, v, out[1])], mask=chosen, block=block, kv_lens=kv_lens)
    assert torch.equal(out[0], out[1])
