"""The unrolled loops of the attention stream left after each of their steps, against the oracle: every residue of the number of
steps by the steps unrolled, for the dense kernels' whole items, halves, quarters and pieces of 192 queries, the small kernel and the
kernels of the block-sparse path, with last tiles that are whole and cut."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_22323_amd as ra
import workloads as wl
from gpu_common import assert_close, from_dev, to_dev

pytestmark = pytest.mark.gpu


def _inputs(seed, B, H, N, D, kv_len):
    rng = np.random.default_rng(seed)
    q, k, v = (wl.f32_to_bf16_bits(rng.standard_normal((B, H, N, D), dtype=np.float32)) for _ in range(3))
    for x in (q, k, v):
        x[:, :, kv_len:] = 0
    return q, k, v


@pytest.mark.parametrize("D,B,H,N,lens", [
    (128, 1, 96, 768, range(513, 769, 32)),        # 36 items of an XCD: 32 whole, the rest in quarters
    (128, 1, 112, 768, range(529, 769, 32)),       # 42: the rest in halves
    (128, 1, 24, 1300, range(1045, 1301, 32)),     # 18: all of them in pieces of 192 queries
    (128, 1, 2, 800, range(1, 801, 61)),           # the small kernel: 1 to 13 steps of the two key groups, 6 unrolled
    (64, 1, 96, 768, range(513, 769, 32)),         # 36: whole and quarters
    (64, 1, 128, 512, range(257, 513, 32)),        # one round of whole items
    (64, 1, 48, 1600, range(1313, 1601, 41)),      # 42: whole and halves
    (64, 1, 2, 800, range(1, 801, 61)),
])
def test_dense_every_residue(D, B, H, N, lens):
    for kv_len in lens:
        q, k, v = _inputs(7 + kv_len, B, H, N, D, kv_len)
        dq, dk, dv = to_dev(q), to_dev(k), to_dev(v)
        o = torch.full_like(dq, float("nan"))
        ra.rapid_attn_dense(dq, dk, dv, o, kv_len)
        heads = [0, H // 2, H - 1]
        ref = oracle.attention(q[:, heads], k[:, heads], v[:, heads], kv_len, None, 64)
        assert_close(from_dev(o[:, heads]), ref, f"D={D} H={H} N={N} kv_len={kv_len}")


# (D = 64, 128-token masks: the kernel of the stream is that for more than 2048 rows)
@pytest.mark.parametrize("D,block,H", [(64, 64, 3), (128, 64, 3), (64, 128, 3), (128, 128, 3), (64, 128, 108)])
def test_sparse_every_number_of_kept_blocks(D, block, H):
    """Row i of the mask keeps i + 1 blocks, so every number of steps up to three runs of the unrolled loop occurs at once."""
    nb = 19
    N = nb * block
    kv_len = N - 37
    q, k, v = _inputs(D + block, 1, H, N, D, kv_len)
    rng = np.random.default_rng(block)
    mask = np.zeros((1, H, nb, nb), np.uint8)
    for h in range(H):
        for i in range(nb):
            mask[0, h, i, rng.permutation(nb)[: i + 1]] = 1
    dq, dk, dv = to_dev(q), to_dev(k), to_dev(v)
    o = torch.full_like(dq, float("nan"))
    ra.rapid_attn_block_sparse(dq, dk, dv, o, torch.from_numpy(mask).cuda(), block, kv_len)
    heads = [0, H // 2, H - 1]
    assert_close(from_dev(o[:, heads]), oracle.attention(q[:, heads], k[:, heads], v[:, heads], kv_len, mask[:, heads], block),
                 f"D={D} block={block} H={H}")
