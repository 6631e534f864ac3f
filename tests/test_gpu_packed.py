"""A packed workspace depends on the grid and the shape alone: packed once, it serves plans with another walk, k or p,
and holds the packed tiles and 256 bytes, nothing else."""
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


# Grids whose lists jenga_block_sparse_attn cuts, so that it needs more workspace than the packed tiles take.
@pytest.mark.parametrize("block,head_dim,blocks,heads", [(128, 128, 9, 2), (64, 64, 20, 3), (32, 64, 1600, 2)])
def test_packed_entries_need_the_packed_tiles_only(block, head_dim, blocks, heads):
    w = dict(_workload(block, head_dim, heads), W=block * blocks - 9)
    print("packed size", w, flush=True)
    sparse, dense = CarveLayer(dict(w, topk=0.05), "cuda:0"), CarveLayer(dict(w, topk=1.0, p=0.9), "cuda:0")
    tiles = 2 * (-(-heads * dense.info.N_pad * head_dim * 2 // 256) * 256) + 256
    assert dense.info.attn_workspace_bytes > tiles
    ws = torch.empty(tiles, dtype=torch.uint8, device="cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 82)]
    for layer in (sparse, dense):
        layer.permute_in(q, k, v)
        layer.select()
        layer.pack()
        layer.attend_packed()
    jb.jenga_pack_kv(sparse.plan, sparse.k_c, sparse.v_c, ws, tiles, stream)
    for layer in (sparse, dense):                               # one pack, two k and two p
        torch.cuda.synchronize()
        want = layer.o_c.clone()
        layer.o_c.view(torch.int16).fill_(0x7FC1)
        jb.jenga_block_sparse_attn_packed(layer.plan, layer.q_c, ws, tiles, layer.sel_count, layer.sel_index, layer.o_c,
                                          None, stream)
        torch.cuda.synchronize()
        assert torch.equal(layer.o_c, want)
    for call in (lambda: jb.jenga_pack_kv(dense.plan, dense.k_c, dense.v_c, ws, tiles - 1, stream),
                 lambda: jb.jenga_block_sparse_attn_packed(dense.plan, dense.q_c, ws, tiles - 1, dense.sel_count,
                                                           dense.sel_index, dense.o_c, None, stream),
                 lambda: jb.jenga_block_sparse_attn(dense.plan, dense.q_c, dense.k_c, dense.v_c, dense.sel_count,
                                                    dense.sel_index, dense.o_c, None, ws, tiles, stream)):
        with pytest.raises(jb.JengaError) as err:
            call()
        assert err.value.status == -3
