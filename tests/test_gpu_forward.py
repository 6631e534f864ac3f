"""jenga_forward against the four calls that it stands for: the same bits everywhere, whatever lies over what."""
import pytest
import torch

import jenga_inputs as ji
from paper_2505_16864_amd import binding as jb
from paper_2505_16864_amd.layer import CarveLayer

pytestmark = pytest.mark.gpu


def _workload(block, head_dim, tokens, heads, batch, n_text):
    return dict(T=1, H=1, W=tokens, n_text=n_text, batch=batch, heads=heads, head_dim=head_dim, block=block, topk=0.3,
                p=0.3, text_bias=0.4)


def _steps(layer, q, k, v):
    layer.permute_in(q, k, v)
    layer.select()
    layer.attend()
    layer.permute_out()


def _results(layer):
    torch.cuda.synchronize()
    return [t.clone() for t in (layer.q_c, layer.k_c, layer.v_c, layer.sel_count, layer.sel_index, layer.mask, layer.o_c,
                                layer.lse, layer.out_thw)]


# in place and packed, lists whole and all cut into parts, passes over key ranges; ragged blocks, no text, odd head counts (lists
# cut at the end, counters, the paced walk and several launches: test_gpu_forward_routes.py)
@pytest.mark.parametrize("block,head_dim,tokens,heads,batch,n_text", [
    (32, 64, 256, 2, 1, 32), (32, 64, 6, 1, 1, 0), (32, 128, 700, 3, 2, 37), (32, 64, 32 * 1600 - 9, 3, 1, 5),
    (64, 128, 64 * 20 - 1, 3, 2, 70), (64, 64, 64 * 9 + 1, 70, 1, 0), (128, 128, 128 * 16, 8, 1, 64),
    (128, 64, 128 * 13 - 100, 5, 2, 200), (128, 128, 128 * 33 + 5, 40, 1, 1), (128, 128, 1, 1, 1, 1)])
def test_same_bits_as_the_single_calls(block, head_dim, tokens, heads, batch, n_text):
    w = _workload(block, head_dim, tokens, heads, batch, n_text)
    print("forward", w, flush=True)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 91)]
    layer = CarveLayer(w, "cuda:0", want_mask=True, want_lse=True)
    _steps(layer, q, k, v)
    want = _results(layer)
    for t in (layer.q_c, layer.k_c, layer.v_c, layer.o_c, layer.out_thw):
        t.view(torch.int16).fill_(0x7FC1)
    for t in (layer.sel_count, layer.mask, layer.lse, layer.ws_select):
        t.fill_(77)
    assert layer.forward(q, k, v) is layer.out_thw
    assert all(torch.equal(a, b) for a, b in zip(_results(layer), want))


@pytest.mark.parametrize("what", ["out over q", "out over q_c", "q_c over k", "workspace over q"])
def test_tensors_over_each_other(what):
    w = _workload(64, 64, 64 * 9, 3, 1, 64)   # no pads: both sides have the same size
    print("overlap", what, flush=True)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 92)]
    layer, other = [CarveLayer(w, "cuda:0", want_mask=True, want_lse=True) for _ in range(2)]
    _steps(layer, q, k, v)
    want = _results(layer)
    if what == "out over q":
        other.out_thw = q
    elif what == "out over q_c":
        other.out_thw = other.q_c.view(q.shape)
    elif what == "q_c over k":   # Q moves first, and K is what is left there: as the single call does it
        other.q_c = k.view(other.q_c.shape)
        other.permute_in(q, k, v)
        torch.cuda.synchronize()
        k_c = other.k_c.clone()
        k.copy_(ji.make_qkv(w, 92)[1])
        other.forward(q, k, v)
        torch.cuda.synchronize()
        assert torch.equal(other.k_c, k_c)
        return
    else:
        n = q.numel() * 2
        other.ws_select = torch.empty(max(n, other.ws_select.numel()), dtype=torch.uint8, device="cuda:0")
        inside = other.ws_select[:n].view(torch.bfloat16).view(q.shape)
        inside.copy_(q)
        q = inside
    other.forward(q, k, v)
    got = _results(other)
    names = ["q_c", "k_c", "v_c", "count", "index", "mask", "o_c", "lse", "out"]
    for name, a, b in zip(names, got, want):
        if not (what == "out over q_c" and name == "q_c"):
            assert torch.equal(a.view(-1), b.view(-1)), name


def test_refusals_launch_nothing():
    w = _workload(64, 64, 64 * 9, 2, 1, 0)
    layer = CarveLayer(w, "cuda:0")
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 93)]
    for t in (layer.q_c, layer.out_thw):
        t.fill_(3.0)
    full = [layer.plan, q, k, v, layer.q_c, layer.k_c, layer.v_c, layer.sel_count, layer.sel_index, None, layer.ws_select,
            layer.ws_select.numel(), layer.o_c, None, layer.ws_attn, layer.ws_attn.numel(), layer.out_thw]
    for at, value, status in [(1, None, -1), (10, None, -1), (16, None, -1), (10, layer.ws_select[1:], -1),
                              (11, layer.info.select_workspace_bytes - 1, -3), (15, layer.info.attn_workspace_bytes - 1, -3)]:
        args = list(full)
        args[at] = value
        with pytest.raises(jb.JengaError) as err:
            jb.jenga_forward(*args, torch.cuda.current_stream().cuda_stream)
        assert err.value.status == status
    torch.cuda.synchronize()
    assert bool((layer.q_c == 3.0).all()) and bool((layer.out_thw == 3.0).all())
