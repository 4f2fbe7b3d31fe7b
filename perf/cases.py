"""The work whose speed counts here, as cases: joint attention calls (dense, block-sparse, on the
separate image and text tensors of a block, with per-sample lengths), block-mask selection and the
Cache-Reuse residual operations, from launch-bound calls to a 2048 x 2048 image.

Shapes are those of `workloads/` (token order [image | text | padding]; 64-wide heads for the sd3
shapes, 128-wide for the flux shapes) and of smaller images of the same models.  Everything a
program keeps between calls (output tensors, workspaces, masks) is made in `prepare`; `run` is one
call of a public entry point on torch's current stream.
"""
import math

import torch

import paper_2509_22323_amd as ra

# nominal densities of a group of rollouts whose samples drew different sparse actions
MIXED = (1.0, 0.5, 0.3, 0.15)
# share of the blocks that selection levels 1..3 keep of block-structured inputs, text blocks included
KEPT = {1: 0.77, 2: 0.58, 3: 0.41}
MOST_FLOPS = 4.0 * 24 * 16896.0 ** 2 * 128            # the largest listed case


def listed():
    return [
        # smallest call of the test workloads: launch latency and host time
        dict(name="dense_tiny", kind="dense", B=1, H=2, N=256, kv_len=256, D=64),
        # the same under a 4 x 4 block mask: two or three launches per call
        dict(name="sparse_tiny", kind="sparse", B=1, H=2, N=256, kv_len=256, D=64, block=64, text=0, density=0.5),
        # 512 x 512 image, guidance pair with prompts of different length, as the block's fused projections
        # hold it (1024 image tokens, up to 333 text tokens, joint length odd)
        dict(name="joint_dense_512", kind="joint", B=2, H=24, image=1024, text=333, D=64, block=128, density=0.0),
        # 1024 x 1024 image, 64-wide heads, guidance pair; last text block padded
        dict(name="dense_sd3_1024", kind="dense", B=2, H=24, N=4480, kv_len=4429, D=64),
        # 1024 x 1024 image, 128-wide heads: the benchmark's default workload
        dict(name="dense_flux_1024", kind="dense", B=1, H=24, N=4608, kv_len=4608, D=128),
        # 2048 x 2048 image: the largest call
        dict(name="dense_flux_2048", kind="dense", B=1, H=24, N=16896, kv_len=16896, D=128),
        # a sparse step at 1024 x 1024, strict level
        dict(name="sparse_flux_1024", kind="sparse", B=1, H=24, N=4608, kv_len=4608, D=128, block=128, text=4, density=0.2),
        # a rollout group of policy training: eight samples, each under the density it drew
        dict(name="sparse_grpo_sd3", kind="sparse", B=8, H=24, N=4480, kv_len=4429, D=64, block=128, text=3, density=-1.0),
        # 768 x 768 image under a mask of 64-token blocks
        dict(name="sparse64_flux_768", kind="sparse", B=1, H=24, N=2816, kv_len=2816, D=128, block=64, text=8, density=0.3),
        # selection of the mask alone, 2048 x 2048 image (the two-call form of a sparse layer)
        dict(name="select_flux_2048", kind="select", B=1, H=24, N=16896, kv_len=16896, D=128, block=128, text=4, level=2),
        # selection and attention of one layer in one call, on the block's own tensors
        dict(name="joint_select_flux_1024", kind="joint_select", B=1, H=24, image=4096, text=512, D=128, block=128, level=3),
        # a step that reuses the cache: residual added to the hidden states of a 1024 x 1024 image
        dict(name="cache_reuse_flux_1024", kind="cache", op="reuse", B=1, elems=4608 * 3072, flags=False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(["dense", "dense", "sparse", "sparse", "joint", "joint", "joint_select", "select", "cache"])
    if kind == "cache":
        B = rng.choice([1, 1, 2, 4, 8])
        return dict(kind=kind, op=rng.choice(["store", "reuse"]), B=B,
                    elems=_log_uniform(rng, 4096 * 16, 4608 * 3072 * 8) // B, flags=B > 1 and rng.random() < 0.5)
    D = rng.choice([64, 128])
    B, H = _log_uniform(rng, 1, 8), rng.choice([2, 8, 16, 24, 24, 24, 38])
    tokens = _log_uniform(rng, 256, 16896)
    if kind == "dense":
        pad = rng.choice([1, 1, 64, 128])
        return dict(kind=kind, B=B, H=H, N=-(-tokens // pad) * pad, kv_len=tokens, D=D)
    block = rng.choice([64, 128, 128, 128])
    nb = -(-tokens // block)
    text = min(rng.randint(0, 512 // block), nb // 3)      # trailing text blocks
    if kind == "sparse":
        return dict(kind=kind, B=B, H=H, N=nb * block, kv_len=tokens, D=D, block=block, text=text,
                    density=rng.choice([-1.0] if B > 1 else [1.0]) if rng.random() < 0.2 else round(rng.uniform(0.1, 0.9), 3))
    if kind == "select":
        return dict(kind=kind, B=B, H=H, N=nb * block, kv_len=tokens, D=D, block=block, text=text, level=rng.randint(1, 3))
    image, words = max(128, tokens // 128 * 128), rng.randint(1, 512)
    if kind == "joint":
        return dict(kind=kind, B=B, H=H, image=image, text=words, D=D, block=block,
                    density=rng.choice([0.0, round(rng.uniform(0.1, 0.9), 3)]))
    return dict(kind=kind, B=B, H=H, image=image, text=words, D=D, block=block, level=rng.randint(1, 3))


def draw(rng):
    """A case of the same ranges: 1 to 8 samples, 2 to 38 heads, 256 to 16896 tokens (odd numbers among
    them), both head sizes and mask tiles, densities 0.1 to 1, no more work than the largest listed one
    (half of it under a mask or with 64-wide heads, which cost more per operation) and at most 1 GB of tensors."""
    while True:
        case = _draw(rng)
        w = work(case)
        cheap = case["kind"] == "dense" and case["D"] == 128
        if w["flops"] <= MOST_FLOPS * (1.0 if cheap else 0.5) and w["bytes"] <= 1.0e9:
            return case


# ------------------------------------------------------------------------------- inputs
def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _structured(g, B, H, N, D, block, text_blocks):
    """Q, K [B,H,N,D] whose attention map has block structure, as the maps of a trained model have:
    every query-block looks at one key-block (text blocks at themselves); see
    workloads.make_qkv_block_structured, of which this is the GPU form."""
    nb = -(-N // block)
    n_image = nb - text_blocks
    centre = torch.randn((B, H, nb, D), generator=g, device="cuda") * math.sqrt(5.5 / math.sqrt(D))
    link = torch.rand((B, H, n_image), generator=g, device="cuda").argsort(-1)
    link = torch.cat([link, torch.arange(n_image, nb, device="cuda").expand(B, H, text_blocks)], -1)
    looks = centre.gather(2, link[..., None].expand(B, H, nb, D))
    looks = looks + 0.3 * torch.randn((B, H, nb, D), generator=g, device="cuda")
    made = []
    for c in (looks, centre):
        x = torch.randn((B, H, N, D), generator=g, device="cuda", dtype=torch.bfloat16) * 0.2
        x += c.to(torch.bfloat16).repeat_interleave(block, 2)[:, :, :N]
        made.append(x)
    return made


def _mask(g, B, H, nb, text, densities):
    """uint8 [B,H,nb,nb]: text rows and columns and the diagonal kept, further image tiles drawn without
    replacement until a share of densities[b] of the image tiles is kept."""
    n = nb - text
    m = torch.ones((B, H, nb, nb), dtype=torch.uint8, device="cuda")
    r = torch.rand((B, H, n, n), generator=g, device="cuda")
    r.diagonal(dim1=2, dim2=3).fill_(-1.0)
    rank = r.reshape(B, H, n * n).argsort(-1).argsort(-1).reshape(B, H, n, n)
    keep = torch.tensor([max(n, round(d * n * n)) for d in densities], device="cuda").reshape(B, 1, 1, 1)
    m[:, :, :n, :n] = rank < keep
    return m


def _densities(case):
    return [MIXED[b % 4] if case["density"] < 0 else case["density"] for b in range(case["B"])]


def _lens(case):
    """Valid tokens per sample of a joint call: all of the image, prompts of different length."""
    return [case["image"] + max(1, case["text"] * (b + 1) // case["B"]) for b in range(case["B"])]


def _segments(g, case, structured):
    """The image and the text stream as the fused projections [B, n, 3, H, D] of a block, outputs [B, n, H, D]."""
    B, H, D, n0, n1 = case["B"], case["H"], case["D"], case["image"], case["text"]
    fused = [_normal(g, B, n, 3, H, D) for n in (n0, n1)]
    if structured:
        text_blocks = -(-(n0 + n1) // case["block"]) - n0 // case["block"]
        for which, x in enumerate(_structured(g, B, H, n0 + n1, D, case["block"], text_blocks)):
            x = x.transpose(1, 2)
            fused[0][:, :, which] = x[:, :n0]
            fused[1][:, :, which] = x[:, n0:]
    made = []
    for f, n in zip(fused, (n0, n1)):
        q, k, v = (f[:, :, i].transpose(1, 2) for i in range(3))
        made.append((q, k, v, torch.empty((B, n, H, D), device="cuda", dtype=torch.bfloat16).transpose(1, 2)))
    return made


def _scratch(n):
    return torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind, B = case["kind"], case["B"]
    s = dict(kind=kind)
    if kind == "cache":
        s["a"], s["b"] = _normal(g, B, case["elems"]), _normal(g, B, case["elems"])
        s["out"] = torch.zeros_like(s["a"])
        s["flags"] = torch.tensor([b % 2 for b in range(B)], dtype=torch.uint8, device="cuda") if case["flags"] else None
        s["op"] = case["op"]
        return s
    H, D = case["H"], case["D"]
    if kind in ("joint", "joint_select"):
        block, N = case["block"], case["image"] + case["text"]
        nb = -(-N // block)
        s.update(block=block, segments=_segments(g, case, kind == "joint_select"), mask=None, workspace=None)
        s["lens"] = torch.tensor(_lens(case), dtype=torch.int32, device="cuda")
        if kind == "joint_select":
            s.update(text_start=case["image"], tau=ra.rapid_mask_level_tau(case["level"]),
                     mask=torch.empty((B, H, nb, nb), dtype=torch.uint8, device="cuda"),
                     workspace=_scratch(ra.rapid_attn_joint_select_workspace_bytes(B, H, N, D, block)))
        elif case["density"] > 0:
            s["mask"] = _mask(g, B, H, nb, nb - case["image"] // block, _densities(case))
            s["workspace"] = _scratch(ra.rapid_attn_joint_workspace_bytes(B, H, N, D, block))
        return s
    N, kv = case["N"], case["kv_len"]
    s["kv_len"] = kv
    if kind == "select":
        block, nb = case["block"], N // case["block"]
        s["q"], s["k"] = _structured(g, B, H, N, D, block, case["text"])
        s.update(block=block, text_start=(nb - case["text"]) * block, tau=ra.rapid_mask_level_tau(case["level"]),
                 mask=torch.empty((B, H, nb, nb), dtype=torch.uint8, device="cuda"),
                 workspace=_scratch(ra.rapid_mask_select_workspace_bytes(B, H, N, D, block)))
    else:
        for t in "qkv":
            s[t] = _normal(g, B, H, N, D)
        s["o"] = torch.empty_like(s["q"])
        if kind == "sparse":
            block, nb = case["block"], N // case["block"]
            s.update(block=block, mask=_mask(g, B, H, nb, case["text"], _densities(case)),
                     workspace=_scratch(ra.rapid_attn_workspace_bytes(B, H, N, D, block)))
    for t in "qk" if kind == "select" else "qkv":
        s[t][:, :, kv:] = 0                                # padding tokens
    return s


# ------------------------------------------------------------------------------- the call
def run(s):
    kind = s["kind"]
    if kind == "dense":
        return ra.rapid_attn_dense(s["q"], s["k"], s["v"], s["o"], s["kv_len"])
    if kind == "sparse":
        return ra.rapid_attn_block_sparse(s["q"], s["k"], s["v"], s["o"], s["mask"], s["block"], s["kv_len"],
                                          workspace=s["workspace"])
    if kind == "joint":
        return ra.rapid_attn_joint(s["segments"], mask=s["mask"], block=s["block"], kv_lens=s["lens"],
                                   workspace=s["workspace"])
    if kind == "joint_select":
        o = ra.rapid_attn_joint_select(s["segments"], s["block"], kv_lens=s["lens"], text_start=s["text_start"],
                                       tau=s["tau"], mask_out=s["mask"], workspace=s["workspace"])
        return [s["mask"]] + o
    if kind == "select":
        return ra.rapid_mask_select(s["q"], s["k"], s["mask"], s["block"], s["kv_len"], s["text_start"], s["tau"],
                                    workspace=s["workspace"])
    if s["op"] == "store":
        return ra.rapid_cache_store(s["a"], s["b"], s["out"], s["flags"])
    return ra.rapid_cache_reuse(s["a"], s["b"], s["out"], s["flags"])


# ------------------------------------------------------------------------------- what it cannot do without
def work(case):
    kind, B = case["kind"], case["B"]
    if kind == "cache":
        samples = B // 2 if case["flags"] else B
        return {"bytes": 6.0 * samples * case["elems"], "flops": 1.0 * samples * case["elems"]}
    H, D = case["H"], case["D"]
    joint = kind in ("joint", "joint_select")
    N = case["image"] + case["text"] if joint else case["N"]
    lens = _lens(case) if joint else [case["kv_len"]] * B
    read, written = 2.0 * H * D * sum(lens), 2.0 * B * H * N * D
    if kind == "dense" or (kind == "joint" and case["density"] == 0):
        return {"bytes": 3 * read + written, "flops": sum(4.0 * H * n * n * D for n in lens)}
    block = case["block"]
    nb = -(-N // block)
    grid = 1.0 * B * H * nb * nb                           # mask bytes
    if kind == "select":
        return {"bytes": 2 * read + grid, "flops": 2.0 * read + 2.0 * grid * D}
    if kind == "joint_select":
        return {"bytes": 3 * read + written + grid,
                "flops": KEPT[case["level"]] * sum(4.0 * H * n * n * D for n in lens)}
    text = nb - case["image"] // block if kind == "joint" else case["text"]
    image = nb - text
    kept = [max(image, d * image * image) + nb * nb - image * image for d in _densities(case)]
    return {"bytes": 3 * read + written + grid,
            "flops": sum(4.0 * H * n * n * D * k / (nb * nb) for n, k in zip(lens, kept))}


def tolerance(case):
    """Against the same attention in 64 bits every shape shows rel 2.1e-3 to 2.3e-3 (the weights and the
    output as bf16) and single values off by 0.015 of max(rms, |value|); four times that is allowed.  A
    selected mask decides single blocks by sums of fp32: one block in a thousand may lie on either side of
    the cut, and moves the 64 or 128 rows it belongs to."""
    kind = case["kind"]
    if kind == "cache":
        return "exact"
    if kind == "select":
        return {"rel": 0.0, "differ": 1e-3}
    if kind == "joint_select":
        return {"rel": 1e-2, "max": 0.8, "differ": 1e-3}
    return {"rel": 1e-2, "max": 0.08}
