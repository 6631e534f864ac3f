"""A packed workspace depends on the grid and the shape alone: packed once, it serves plans with another walk."""
import pytest
import torch

import jenga_inputs as ji
from paper_2505_16864_amd import binding as jb
from paper_2505_16864_amd.layer import CarveLayer

pytestmark = pytest.mark.gpu


def _workload(block, head_dim, heads):
    return dict(T=1, H=1, W=block * 13 - 9, n_text=block + 5, batch=1, heads=heads, head_dim=head_dim, block=block,
                topk=0.3, p=0.3, text_bias=0.4)


# few heads: lists are cut in jenga_block_sparse_attn; many: they stay whole
@pytest.mark.parametrize("block,head_dim", [(128, 128), (128, 64), (64, 128), (64, 64), (32, 128), (32, 64)])
@pytest.mark.parametrize("heads", [2, 70])
@pytest.mark.parametrize("packed_by,read_by", [(15, 7), (7, 15)])
def test_packed_under_one_walk_read_under_the_other(block, head_dim, heads, packed_by, read_by):
    w = _workload(block, head_dim, heads)
    print("packed", w, packed_by, read_by, flush=True)
    first, second = CarveLayer(w, "cuda:0", flags=packed_by), CarveLayer(w, "cuda:0", flags=read_by)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 81)]
    for layer in (first, second):
        layer.permute_in(q, k, v)
        layer.select()
    second.pack()
    second.attend_packed()
    torch.cuda.synchronize()
    want = second.o_c.clone()
    first.pack()
    second.o_c.view(torch.int16).fill_(0x7FC1)
    jb.jenga_block_sparse_attn_packed(second.plan, second.q_c, first.ws_attn, first.ws_attn.numel(), second.sel_count,
                                      second.sel_index, second.o_c, None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    if read_by == 7 or block != 128:
        assert torch.equal(second.o_c, want)
    else:
        # The paced walk's last bits may differ between runs: one unit of the bf16 output, at most 2^-7 |o|, and the bf16
        # probabilities taken against another reference, 2^-8 max|v| (max|v| and max|o| are alike here).
        assert float((second.o_c.float() - want.float()).abs().max()) <= 2.0 ** -6 * float(want.float().abs().max())
