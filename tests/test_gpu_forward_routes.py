"""jenga_forward on the routes that the small shapes of test_gpu_forward.py do not take: several launches, lists cut at the end and dealt
out by counters, the paced walk, batches beyond one grid; and tensors over each other, one by one, against the four calls."""
import pytest
import torch

import jenga_inputs as ji
from paper_2505_16864_amd.layer import CarveLayer
from test_gpu_forward import _results, _steps, _workload

pytestmark = pytest.mark.gpu


def _poison(layer):
    for t in (layer.q_c, layer.k_c, layer.v_c, layer.o_c, layer.out_thw):
        t.view(torch.int16).fill_(0x7FC1)
    for t in (layer.sel_count, layer.mask, layer.lse, layer.ws_select):
        t.fill_(77)


# Parts of the rows of one launch lie in the workspace, whatever the number of heads: three at a time here, so that four launches
# take ten (batch, head) pairs and the second one crosses from one batch to the next.
def test_several_launches():
    w = _workload(32, 64, 32 * 1600 - 9, 5, 2, 5)
    print("forward", w, flush=True)
    layer, one = CarveLayer(w, "cuda:0", want_mask=True, want_lse=True), CarveLayer(dict(w, heads=1, batch=1), "cuda:0")

    def parts(of):
        return of.info.attn_workspace_bytes - 256 - 4 * of.w["heads"] * of.w["batch"] * of.info.N_pad * 64
    assert 2.5 * parts(one) < parts(layer) < 3.5 * parts(one)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 91)]
    _steps(layer, q, k, v)
    want = _results(layer)
    _poison(layer)
    layer.forward(q, k, v)
    assert all(torch.equal(a, b) for a, b in zip(_results(layer), want))


# Vision rows whose last bits are not the packed entry's are rows that were cut, of lists at the end; likewise text rows.
# 64 tokens at head dim 128 without counters, in steps of 32 keys; 128 tokens with them; lists of uneven length.
@pytest.mark.parametrize("block,head_dim,blocks,heads,p,text_cut", [
    (64, 128, 121, 13, 0.3, True), (128, 128, 121, 14, 0.3, False), (64, 64, 301, 7, 0.97, False), (128, 64, 161, 7, 0.97, False)])
def test_lists_cut_at_the_end(block, head_dim, blocks, heads, p, text_cut):
    w = dict(_workload(block, head_dim, block * (blocks - 1) - 9, heads, 1, 5), p=p)
    print("forward", w, flush=True)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 91)]
    layer = CarveLayer(w, "cuda:0", want_mask=True, want_lse=True)
    _steps(layer, q, k, v)
    want = _results(layer)
    layer.pack()
    layer.attend_packed()
    torch.cuda.synchronize()
    differ = (want[6] != layer.o_c).any(dim=-1).view(heads, blocks, block).any(dim=-1)
    assert differ[:, :-1].any() and bool(differ[:, -1:].any()) == text_cut
    _poison(layer)
    layer.forward(q, k, v)
    assert all(torch.equal(a, b) for a, b in zip(_results(layer), want))


# The paced walk's last bits may differ between runs: the rows on the token-order side are those of the same call's curve side, and what
# comes before the attention is the same in any case.
@pytest.mark.parametrize("head_dim,blocks,heads,n_text,p", [
    (128, 17, 8, 64, 0.3), (128, 121, 14, 5, 0.3), (128, 61, 14, 300, 0.97), (64, 161, 7, 130, 0.97), (128, 40, 24, 0, 0.3)])
def test_paced_walk_writes_the_same_rows_to_both_sides(head_dim, blocks, heads, n_text, p):
    w = dict(_workload(128, head_dim, 128 * blocks - 9, heads, 1, n_text), p=p, flags=15)
    print("forward, paced", w, flush=True)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 92)]
    layer = CarveLayer(w, "cuda:0", want_mask=True, want_lse=True)
    _steps(layer, q, k, v)
    want = _results(layer)
    _poison(layer)
    layer.forward(q, k, v)
    got = _results(layer)
    assert all(torch.equal(a, b) for a, b in zip(got[:6], want[:6]))
    # one unit of the bf16 output, at most 2^-7 |o|, and the bf16 probabilities taken against another reference, 2^-8 max|v|
    assert float((got[6].float() - want[6].float()).abs().max()) <= 2.0 ** -6 * float(v.float().abs().max())
    layer.out_thw.view(torch.int16).fill_(0x7FC1)
    layer.permute_out()
    torch.cuda.synchronize()
    assert torch.equal(layer.out_thw, got[8])


# Three tensors of this many batches are more than the z of one grid.
def test_more_batches_than_one_grid_takes():
    w = _workload(32, 64, 1, 1, 21846, 0)
    print("forward", w, flush=True)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 93)]
    layer = CarveLayer(w, "cuda:0", want_mask=True, want_lse=True)
    _steps(layer, q, k, v)
    want = _results(layer)
    _poison(layer)
    layer.forward(q, k, v)
    assert all(torch.equal(a, b) for a, b in zip(_results(layer), want))


# Everything that a call leaves behind is what the four calls leave behind where the same tensors lie over each other.
@pytest.mark.parametrize("what", ["q_c over k", "q_c over v", "k_c over q", "out over k_c", "out over v_c", "out over attention workspace",
                                  "out over counts", "out over indices", "out over lse", "out over select workspace", "out over v"])
@pytest.mark.parametrize("block,heads", [(64, 3), (32, 3), (128, 5)])
def test_tensors_over_each_other_as_the_four_calls_take_them(what, block, heads):
    w = _workload(block, 64, block * 9, heads, 1, block)   # no pads: both sides have the same size
    print("overlap", what, w, flush=True)

    def run(forward):
        q, k, v = [x.cuda() for x in ji.make_qkv(w, 94)]
        layer = CarveLayer(w, "cuda:0", want_mask=True, want_lse=True)
        for t in (layer.ws_attn, layer.ws_select, layer.sel_count, layer.sel_index, layer.lse):
            t.zero_()
        for t in (layer.q_c, layer.k_c, layer.v_c, layer.o_c, layer.out_thw):
            t.zero_()
        if what.startswith("out over "):
            name = {"k_c": "k_c", "v_c": "v_c", "attention workspace": "ws_attn", "counts": "sel_count", "indices": "sel_index", "lse": "lse",
                    "select workspace": "ws_select", "v": None}[what[9:]]
            if name is None:
                layer.out_thw = v
            else:   # both at the start of one buffer
                old = getattr(layer, name)
                room = torch.zeros(max(old.numel() * old.element_size(), q.numel() * 2), dtype=torch.uint8, device="cuda:0")
                setattr(layer, name, room[:old.numel() * old.element_size()].view(old.dtype).view(old.shape))
                layer.out_thw = room[:q.numel() * 2].view(torch.bfloat16).view(q.shape)
        else:
            dst, src = what.split(" over ")
            setattr(layer, dst, {"q": q, "k": k, "v": v}[src].view(layer.q_c.shape))
        layer.forward(q, k, v) if forward else _steps(layer, q, k, v)
        return [t.contiguous().view(torch.uint8) for t in _results(layer) + [q, k, v]]
    assert all(torch.equal(a, b) for a, b in zip(run(True), run(False)))
