"""Block selection at the block counts where the kernel's layout changes: one value per lane of a wavefront, the number
of values per lane, rows per workgroup, the last partial tile of query blocks and of key blocks.  Masks and lists are
bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import jenga_inputs as ji
from oracle import jenga_oracle as jo
from paper_2505_16864_amd.layer import CarveLayer
from gpu_util import oracle_layout, lists_from_gpu, check_lists_against_mask

pytestmark = pytest.mark.gpu


def _workload(m, n_text_blocks, head_dim, topk, p, heads=2):
    # a line of m - n_text_blocks vision blocks of 32 tokens, all full, and full text blocks
    return dict(T=1, H=1, W=32 * (m - n_text_blocks), n_text=32 * n_text_blocks, batch=1, heads=heads,
                head_dim=head_dim, block=32, topk=topk, p=p)


def _select(w, q, k):
    layer = CarveLayer(w, "cuda:0", want_mask=True)
    layer.permute_in(q.cuda(), k.cuda(), k.cuda())
    layer.sel_index.fill_(-1)
    layer.select()
    torch.cuda.synchronize()
    return layer


def _check(w, q, k):
    layer = _select(w, q, k)
    lay = oracle_layout(w)
    qc, kc = [jo.bf16_bits_to_f64(jo.permute(ji.bits(x), lay)) for x in (q, k)]
    mask = jo.build_mask(qc, kc, lay, w["p"])
    assert np.array_equal(layer.mask.cpu().numpy().astype(bool), mask)
    cnt, idx = lists_from_gpu(layer)
    check_lists_against_mask(cnt, idx, mask)


@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 33, 63, 64, 65, 127, 128, 129, 255, 257, 511, 513, 1023, 1025, 2048])
@pytest.mark.parametrize("head_dim,topk,p", [(64, 0.1, 0.8), (128, 0.3, 0.3)])
def test_block_counts(m, head_dim, topk, p):
    w = _workload(m, min(m - 1, m % 3), head_dim, topk, p, heads=3 if m < 600 else 1)
    print("select", w, flush=True)
    q, k, _ = ji.make_qkv(w, 71 + m)
    _check(w, q, k)


# First and last block count of the numbers of values per lane between the powers of two.
@pytest.mark.parametrize("m", [192, 193, 320, 321, 384, 385, 448, 449, 512, 640, 641, 768, 769])
@pytest.mark.parametrize("head_dim,topk,p", [(128, 0.1, 0.8), (64, 0.3, 0.3)])
def test_block_counts_between(m, head_dim, topk, p):
    test_block_counts(m, head_dim, topk, p)


# Key blocks that repeat with period 7: groups of equal probabilities, larger than a wavefront from m = 512 on, resolved
# by index.  Small whole numbers, constant over a block, keep every score exact.
@pytest.mark.parametrize("m", [9, 64, 100, 200, 600, 1500])
@pytest.mark.parametrize("topk,p", [(0.05, 0.0), (0.2, 0.55), (0.4, 0.93), (1.0, 0.3)])
def test_equal_probabilities(m, topk, p):
    w = _workload(m, 0, 64, topk, p)
    print("ties", w, flush=True)
    rng = np.random.default_rng(m)
    rows = rng.integers(-1, 2, size=(2, 7, w["heads"], 64))
    block_of = np.arange(w["W"]) // 32
    q = torch.from_numpy(rows[0][block_of % 5].astype(np.float32)).to(torch.bfloat16)[None]
    k = torch.from_numpy(rows[1][block_of % 7].astype(np.float32)).to(torch.bfloat16)[None]
    _check(w, q, k)


# Logits so far apart that most probabilities underflow to zero; every block kept when the scores are undefined.
@pytest.mark.parametrize("m", [40, 150, 300, 1100])
def test_extreme_scores(m):
    w = _workload(m, 0, 64, 0.2, 0.6)
    print("extreme", w, flush=True)
    q, k, _ = ji.make_qkv(w, 5)
    _check(w, q * 64, k * 64)
    for bad in (float("nan"), float("inf")):
        q2, k2 = q.clone(), k.clone()
        q2[0, :, 0, 7] = q[0, :, 0, 7].abs() + 0.25   # head 0 only: the score of that block is +inf or NaN
        k2[0, 32 * (m // 2) + 3, 0, 7] = bad
        layer = _select(w, q2, k2)
        cnt, idx = lists_from_gpu(layer)
        assert (cnt[0, 0] == m).all() and (idx[0, 0] == np.arange(m)).all()
        assert (cnt[0, 1] < m).any()
