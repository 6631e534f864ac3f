"""Attention with blocks of 32 and 64 tokens on lists of given lengths: shorter than the number of wavefronts that
share a list, empty, one off a multiple of it, and full, with the ragged blocks anywhere in them."""
import numpy as np
import pytest
import torch

import jenga_inputs as ji
from oracle import jenga_oracle as jo
from paper_2505_16864_amd.layer import CarveLayer
from gpu_util import oracle_layout, to_f64, check_output

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim,block,width", [(64, 32, 19), (128, 32, 19), (64, 64, 35), (128, 64, 35),
                                                  (64, 32, 13)])   # the last: 19 blocks, read in place
def test_list_lengths(head_dim, block, width):
    w = dict(T=3, H=13, W=width, n_text=2 * block + 5, batch=1, heads=2, head_dim=head_dim, block=block,
             topk=0.3, p=0.3, text_bias=0.4)
    print("list lengths", w, flush=True)
    q, k, v = ji.make_qkv(w, 51)
    layer = CarveLayer(w, "cuda:0", want_lse=True)
    lay = oracle_layout(w)
    rng = np.random.default_rng(7)
    lengths = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, lay.M]
    cnt = np.zeros((1, 2, lay.M), dtype=np.int32)
    idx = np.full((1, 2, lay.M, lay.M), -1, dtype=np.int32)
    mask = np.zeros((1, 2, lay.M, lay.M), dtype=bool)
    for h in range(2):
        for i in range(lay.M):
            n = min(lengths[(i + 5 * h) % len(lengths)], lay.M)
            chosen = rng.permutation(lay.M)[:n]
            if n > 1 and i % 2:
                chosen[0] = lay.M - 1       # the ragged text block first
            chosen = list(dict.fromkeys(chosen.tolist()))
            cnt[0, h, i] = len(chosen)
            idx[0, h, i, :len(chosen)] = chosen
            mask[0, h, i, chosen] = True
    layer.permute_in(q.cuda(), k.cuda(), v.cuda())
    layer.sel_count.copy_(torch.from_numpy(cnt))
    layer.sel_index.copy_(torch.from_numpy(idx))
    layer.o_c.view(torch.int16).fill_(0x7FC1)
    layer.attend()
    torch.cuda.synchronize()
    qc, kc, vc = [jo.permute(to_f64(x), lay) for x in (q, k, v)]
    want, want_lse = jo.block_sparse_attention(qc, kc, vc, mask, lay, beta=w["text_bias"], return_lse=True)
    check_output(to_f64(layer.o_c), want, "list lengths %d/%d" % (head_dim, block))
    got = layer.lse.cpu().numpy().astype(np.float64)
    alive = np.isfinite(want_lse)
    assert np.isneginf(got[~alive]).all()
    assert np.abs(got[alive] - want_lse[alive]).max() <= 1e-3     # float32 sums and one float32 logarithm


# Query blocks per head around the sizes at which the heads are dealt to 8, 4, 2 or 1 of the XCDs each, head counts
# that do not divide: every block has to be computed once, by somebody.
@pytest.mark.parametrize("m_v,heads,n_text", [(1, 1, 0), (7, 3, 40), (127, 3, 0), (129, 5, 70), (257, 3, 33), (513, 2, 5)])
def test_every_query_block_is_dealt_out(m_v, heads, n_text):
    w = dict(T=1, H=1, W=32 * m_v - 3, n_text=n_text, batch=1, heads=heads, head_dim=64, block=32, topk=0.3, p=0.3)
    print("dealt out", w, flush=True)
    q, k, v = ji.make_qkv(w, 52)
    layer = CarveLayer(w, "cuda:0")
    lay = oracle_layout(w)
    mask = np.zeros((1, heads, lay.M, lay.M), dtype=bool)
    mask[:, :, np.arange(lay.M), np.arange(lay.M)] = True
    mask[:, :, :, lay.M - 1] = True
    cnt, idx = jo.mask_to_lists(mask)
    layer.permute_in(q.cuda(), k.cuda(), v.cuda())
    layer.sel_count.copy_(torch.from_numpy(cnt))
    layer.sel_index.copy_(torch.from_numpy(idx))
    layer.o_c.view(torch.int16).fill_(0x7FC1)
    layer.attend()
    torch.cuda.synchronize()
    qc, kc, vc = [jo.permute(to_f64(x), lay) for x in (q, k, v)]
    # A row has a few dozen keys here and |o| reaches max |v|, so the bound is per rounding, not the one for long rows:
    # half a bf16 ulp (at most 2^-8 relative) on every probability and on the result, so 2^-8 (max |v| + |o|).
    err = np.abs(to_f64(layer.o_c) - jo.block_sparse_attention(qc, kc, vc, mask, lay))
    assert err.max() <= 2.0 ** -7 * np.abs(vc).max()


# Grids small enough that lists are cut into parts: lists shorter than one part, one off a multiple of it, empty and
# full, a block listed twice, with and without the paced walk (which visits it once), log-sum-exp included.
@pytest.mark.parametrize("head_dim,block", [(64, 64), (128, 64), (64, 128), (128, 128)])
@pytest.mark.parametrize("heads,paced", [(1, False), (2, True), (9, False)])
def test_lists_cut_into_parts(head_dim, block, heads, paced):
    if paced and block != 128:
        pytest.skip("the paced walk exists for blocks of 128 tokens")
    w = dict(T=1, H=1, W=block * 37 - 9, n_text=block + 5, batch=1, heads=heads, head_dim=head_dim, block=block,
             topk=0.3, p=0.3, text_bias=0.4, flags=15 if paced else 7)
    print("cut", w, flush=True)
    q, k, v = ji.make_qkv(w, 61)
    layer = CarveLayer(w, "cuda:0", want_lse=True)
    lay = oracle_layout(w)
    whole = 2 * (heads * layer.info.N_pad * head_dim * 2) + 256
    assert layer.info.attn_workspace_bytes > whole          # there is room for parts
    rng = np.random.default_rng(8)
    lengths = [0, 1, 2, 3, 4, 6, 7, 8, 9, 12, 13, 17, 24, 25, lay.M - 1, lay.M]
    cnt = np.zeros((1, heads, lay.M), dtype=np.int32)
    idx = np.full((1, heads, lay.M, lay.M), -1, dtype=np.int32)
    mask = np.zeros((1, heads, lay.M, lay.M), dtype=bool)
    for h in range(heads):
        for i in range(lay.M):
            chosen = rng.permutation(lay.M)[:lengths[(i + 5 * h) % len(lengths)]].tolist()
            mask[0, h, i, chosen] = True
            if paced and 0 < len(chosen) < lay.M:
                chosen.append(chosen[0])                     # listed twice, far apart
            cnt[0, h, i] = len(chosen)
            idx[0, h, i, :len(chosen)] = chosen
    layer.permute_in(q.cuda(), k.cuda(), v.cuda())
    layer.sel_count.copy_(torch.from_numpy(cnt))
    layer.sel_index.copy_(torch.from_numpy(idx))
    qc, kc, vc = [jo.permute(to_f64(x), lay) for x in (q, k, v)]
    want, want_lse = jo.block_sparse_attention(qc, kc, vc, mask, lay, beta=w["text_bias"], return_lse=True)
    alive = np.isfinite(want_lse)
    for attend in (layer.attend, layer.attend_packed):       # in parts, whole
        if attend == layer.attend_packed:
            layer.pack()
        layer.o_c.view(torch.int16).fill_(0x7FC1)
        layer.lse.fill_(7.0)
        attend()
        torch.cuda.synchronize()
        check_output(to_f64(layer.o_c), want, "%s %d/%d" % (attend.__name__, head_dim, block))
        got = layer.lse.cpu().numpy().astype(np.float64)
        assert np.isneginf(got[~alive]).all()
        assert np.abs(got[alive] - want_lse[alive]).max() <= 1e-3     # float32 sums and one float32 logarithm


# Heads larger than an L2: blocks of 32 tokens are visited in passes over ranges of key blocks.  Lists in any order,
# empty, of one block, inside one range, longer than the workgroup, full.
@pytest.mark.parametrize("head_dim,m_v", [(128, 385), (64, 1538)])
def test_passes_over_key_ranges(head_dim, m_v):
    w = dict(T=1, H=1, W=32 * m_v - 3, n_text=37, batch=1, heads=2, head_dim=head_dim, block=32, topk=0.5, p=0.3,
             text_bias=0.4)
    print("ranges", w, flush=True)
    q, k, v = ji.make_qkv(w, 62)
    # Most rows here see one block, where a row can come close to a single V row: the error is up to 2^-9 |o| (bf16
    # output) + 2^-9 |v| (bf16 probabilities) <= 2^-8 max|v|.  With V as drawn (max|v| above 5) that is beyond
    # check_output's 2e-2, which is meant for |o| of about 3; a quarter of it is below.
    v = v * 0.25
    assert float(v.abs().max()) < 2.0 ** 8 * 2e-2
    layer = CarveLayer(w, "cuda:0", want_lse=True)
    lay = oracle_layout(w)
    M = lay.M
    assert layer.info.attn_workspace_bytes > 2 * (2 * layer.info.N_pad * head_dim * 2) + 256
    rng = np.random.default_rng(9)
    cnt = np.ones((1, 2, M), dtype=np.int32)
    idx = np.zeros((1, 2, M, M), dtype=np.int32)
    idx[0, :, :, 0] = np.arange(M)
    mask = np.zeros((1, 2, M, M), dtype=bool)
    mask[0, :] = np.eye(M, dtype=bool)
    for h, i, chosen in [(0, 0, []), (0, 1, [M - 1]), (0, 2, rng.permutation(M)), (1, 3, rng.permutation(M)[:300]),
                         (1, 4, rng.permutation(M // 4)), (0, M - 1, np.arange(M)), (1, M - 2, rng.permutation(M)[:7]),
                         (0, 7, M - 1 - np.arange(65))]:
        cnt[0, h, i] = len(chosen)
        idx[0, h, i, :len(chosen)] = chosen
        mask[0, h, i] = False
        mask[0, h, i, list(chosen)] = True
    layer.permute_in(q.cuda(), k.cuda(), v.cuda())
    layer.sel_count.copy_(torch.from_numpy(cnt))
    layer.sel_index.copy_(torch.from_numpy(idx))
    qc, kc, vc = [jo.permute(to_f64(x), lay) for x in (q, k, v)]
    want, want_lse = jo.block_sparse_attention(qc, kc, vc, mask, lay, beta=w["text_bias"], return_lse=True)
    alive = np.isfinite(want_lse)
    for attend in (layer.attend, layer.attend_packed):       # in passes, whole
        if attend == layer.attend_packed:
            layer.pack()
        layer.o_c.view(torch.int16).fill_(0x7FC1)
        layer.lse.fill_(7.0)
        attend()
        torch.cuda.synchronize()
        check_output(to_f64(layer.o_c), want, "%s %d" % (attend.__name__, head_dim))
        got = layer.lse.cpu().numpy().astype(np.float64)
        assert np.isneginf(got[~alive]).all()
        assert np.abs(got[alive] - want_lse[alive]).max() <= 1e-3     # float32 sums and one float32 logarithm


# More heads than one launch has room for the results of: every head as in a plan that has it alone, bit for bit.
@pytest.mark.parametrize("head_dim,m_v,heads", [(64, 1538, 7), (128, 600, 9)])
def test_passes_over_key_ranges_in_several_launches(head_dim, m_v, heads):
    w = dict(T=1, H=1, W=32 * m_v - 3, n_text=37, batch=1, heads=heads, head_dim=head_dim, block=32, topk=0.2, p=0.3,
             text_bias=0.4)
    print("several launches", w, flush=True)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 64)]
    layer, one = CarveLayer(w, "cuda:0", want_lse=True), CarveLayer(dict(w, heads=1), "cuda:0", want_lse=True)

    def parts(of):
        return of.info.attn_workspace_bytes - 256 - 4 * of.w["heads"] * of.info.N_pad * head_dim
    assert 0 < parts(one) and parts(layer) < heads * parts(one)
    layer.permute_in(q, k, v)
    layer.select()
    layer.o_c.view(torch.int16).fill_(0x7FC1)
    layer.lse.fill_(7.0)
    layer.attend()
    for h in range(heads):
        for to, of in ((one.q_c, layer.q_c), (one.k_c, layer.k_c), (one.v_c, layer.v_c), (one.sel_count, layer.sel_count),
                       (one.sel_index, layer.sel_index)):
            to.copy_(of[:, h:h + 1])
        one.attend()
        torch.cuda.synchronize()
        assert torch.equal(one.o_c[:, 0].view(torch.int16), layer.o_c[:, h].view(torch.int16)), h
        assert torch.equal(one.lse[:, 0], layer.lse[:, h]), h


# K is read in place by some kernels: an output that lies over it must still see the K of before the call.
@pytest.mark.parametrize("block,flags", [(32, 7), (64, 7), (128, 7), (128, 15)])
@pytest.mark.parametrize("heads", [2, 90])
def test_output_over_an_input(block, flags, heads):
    from paper_2505_16864_amd import binding as jb
    w = dict(T=1, H=1, W=block * 11 - 9, n_text=block + 5, batch=1, heads=heads, head_dim=64, block=block, topk=0.4, p=0.3,
             flags=flags)
    print("over an input", w, flush=True)
    layer = CarveLayer(w, "cuda:0")
    layer.permute_in(*[x.cuda() for x in ji.make_qkv(w, 63)])
    layer.select()
    layer.attend()
    torch.cuda.synchronize()
    want = layer.o_c.clone()
    for over in range(3):
        t = [x.clone() for x in (layer.q_c, layer.k_c, layer.v_c)]
        jb.jenga_block_sparse_attn(layer.plan, t[0], t[1], t[2], layer.sel_count, layer.sel_index, t[over], None,
                                   layer.ws_attn, layer.ws_attn.numel(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        if flags & 8:
            # The paced walk's last bits may differ between runs: one unit of the bf16 output, at most 2^-7 |o|, and the
            # bf16 probabilities taken against another reference, 2^-8 max|v| (max|v| and max|o| are alike here).
            assert float((t[over].float() - want.float()).abs().max()) <= 2.0 ** -6 * float(want.float().abs().max())
        else:
            assert torch.equal(t[over], want)


# K and V anywhere in a buffer: the copies into LDS want 16-byte addresses, so either is copied or both are packed first.
@pytest.mark.parametrize("block,heads,flags", [(32, 2, 7), (64, 2, 7), (64, 90, 7), (128, 2, 7), (128, 90, 7), (128, 2, 15)])
@pytest.mark.parametrize("off_k,off_v", [(0, 1), (4, 0), (0, 4), (1, 4), (8, 8)])
def test_inputs_off_the_16_byte_grid(block, heads, flags, off_k, off_v):
    from paper_2505_16864_amd import binding as jb
    w = dict(T=1, H=1, W=block * 11 - 9, n_text=block + 5, batch=1, heads=heads, head_dim=64, block=block, topk=0.4, p=0.3,
             flags=flags)
    print("off the grid", w, off_k, off_v, flush=True)
    layer = CarveLayer(w, "cuda:0")
    layer.permute_in(*[x.cuda() for x in ji.make_qkv(w, 66)])
    layer.select()
    layer.attend()
    torch.cuda.synchronize()
    want = layer.o_c.clone()
    at = []
    for x, off in ((layer.k_c, off_k), (layer.v_c, off_v)):
        room = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
        at.append(room[off:off + x.numel()].view(x.shape).copy_(x))
        assert at[-1].data_ptr() % 16 == 2 * off % 16
    layer.o_c.view(torch.int16).fill_(0x7FC1)
    jb.jenga_block_sparse_attn(layer.plan, layer.q_c, at[0], at[1], layer.sel_count, layer.sel_index, layer.o_c, None,
                               layer.ws_attn, layer.ws_attn.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(layer.o_c, want)


# The direct entry twice, the second time with what the first left in the workspace, and the packed entry, which deals nothing
# out and cuts nothing: output and log-sum-exp of each, and the layer.  Lists of random blocks, of the given lengths.
def _direct_twice_and_packed(block, head_dim, blocks, heads, p, paced, lengths):
    w = dict(T=1, H=1, W=block * (blocks - 1) - 9, n_text=5, batch=1, heads=heads, head_dim=head_dim, block=block, topk=0.3,
             p=p, text_bias=0.4, flags=15 if paced else 7)
    print("dealt out", w, flush=True)
    layer = CarveLayer(w, "cuda:0", want_lse=True)
    M = layer.info.M
    assert M == blocks
    layer.permute_in(*[x.cuda() for x in ji.make_qkv(w, 62)])
    rng = np.random.default_rng(9)
    idx = np.argsort(rng.random((1, heads, M, M)), axis=-1).astype(np.int32)
    cnt = rng.choice([int(x) for x in lengths(M)], size=(1, heads, M)).astype(np.int32)
    layer.sel_count.copy_(torch.from_numpy(cnt))
    layer.sel_index.copy_(torch.from_numpy(idx))
    got = []
    layer.ws_attn.fill_(0xFF)
    for call in (layer.attend, layer.attend, layer.pack, layer.attend_packed):
        if call != layer.pack:
            layer.o_c.view(torch.int16).fill_(0x7FC1)
            layer.lse.fill_(7.0)
        call()
        torch.cuda.synchronize()
        if call != layer.pack:
            got.append((layer.o_c.float().clone(), layer.lse.clone()))
    (first, first_lse), _, (whole, whole_lse) = got
    assert torch.isfinite(first).all()
    # bf16 probabilities taken against another reference, 2^-8 max|v|, and one unit of the bf16 result
    for o, lse in got[:2]:
        assert float((o - whole).abs().max()) <= 2.0 ** -6 * float(layer.v_c.float().abs().max())
        alive = torch.isfinite(whole_lse)
        assert torch.equal(torch.isfinite(lse), alive) and torch.isneginf(lse[~alive]).all()
        assert float((lse[alive] - whole_lse[alive]).abs().max()) <= 1e-3      # float32 sums and one float32 logarithm
    if not paced:
        assert torch.equal(first, got[1][0]) and torch.equal(first_lse, got[1][1])
    differ = (first != whole).any(dim=-1).view(heads, M, block).any(dim=-1)
    return differ[:, :M - 1], differ[:, M - 1:]       # vision rows, text rows


# Workgroups of the first generation, half of which is how many vision lists are cut at most.
FIRST = {(128, 128): 768, (128, 64): 1024, (64, 128): 1024, (64, 64): 2048}


# More query blocks than resident workgroups, lists shorter than the number of parts, empty and full.
@pytest.mark.parametrize("block,head_dim,blocks,heads,p,paced", [
    # short lists: dealt out in the order of their numbers, whole
    (128, 128, 9, 86, 0.3, False), (128, 128, 13, 120, 0.3, False), (128, 128, 13, 61, 0.9, True),
    (128, 64, 37, 29, 0.9, False), (128, 64, 9, 230, 0.3, True), (64, 128, 29, 46, 0.9, False), (64, 64, 31, 67, 0.9, False),
    # text rows cut: in one generation, behind a counter, 64 tokens
    (128, 64, 67, 13, 0.3, True), (128, 64, 67, 13, 0.3, False), (128, 128, 113, 8, 0.3, False), (64, 64, 121, 14, 0.3, False),
    # long enough for the counters or about so: one to two generations, two and more, lists of uneven length, the paced walk
    (128, 128, 97, 9, 0.3, False), (128, 128, 97, 17, 0.3, True), (128, 128, 37, 24, 0.97, False), (128, 64, 97, 11, 0.97, True),
    (64, 128, 83, 16, 0.97, False), (64, 64, 193, 11, 0.97, False)])
def test_more_query_blocks_than_places(block, head_dim, blocks, heads, p, paced):
    vision, text = _direct_twice_and_packed(block, head_dim, blocks, heads, p, paced,
                                            lambda M: (0, 1, 2, 3, M // 2, M - 1, M))
    if not paced:   # at most half a generation of lists is cut, and the text rows
        assert int(vision.sum()) <= FIRST[(block, head_dim)] // 2


# Lists that last long enough for the counters: those at the end are cut, and text rows where they alone would last as long.
# With short lists on the same plan every vision list stays whole: the call's own lists decide.
@pytest.mark.parametrize("block,head_dim,blocks,heads,p,paced,vision_cut,text_cut", [
    (128, 128, 97, 9, 0.3, False, False, True), (128, 128, 97, 17, 0.3, False, True, False),
    (128, 128, 97, 17, 0.3, True, True, False), (128, 128, 61, 14, 0.97, False, True, False),
    (128, 64, 161, 7, 0.97, False, True, False), (128, 64, 161, 7, 0.97, True, True, False),
    (64, 128, 137, 10, 0.97, False, True, False), (64, 64, 301, 7, 0.97, False, True, False)])
def test_lists_decide_about_counters_and_cuts(block, head_dim, blocks, heads, p, paced, vision_cut, text_cut):
    vision, text = _direct_twice_and_packed(block, head_dim, blocks, heads, p, paced,
                                            lambda M: (0, 1, 2, M // 2, M - 1, M, M, M, M, M))
    if not paced:   # paced, last bits differ between runs
        assert (8 if vision_cut else 0) <= int(vision.sum()) <= (FIRST[(block, head_dim)] // 2 if vision_cut else 0)
        assert int(text.sum()) > heads // 3 if text_cut else not text.any()
    vision, _ = _direct_twice_and_packed(block, head_dim, blocks, heads, p, paced, lambda M: (0, 1, 2, 3, 8))
    if not paced:
        assert not vision.any()


# More text than vision blocks, text rows and the vision lists at the end both cut: every row comes from its own parts, also
# where the output lies over Q, which only the row itself may still read.
@pytest.mark.parametrize("block,vision,text,heads,topk,flags", [
    (64, 2333, 9726, 7, 0.1, 7), (128, 1003, 25540, 4, 0.2, 4), (64, 6754, 16434, 4, 0.05, 7)])
def test_more_text_than_vision(block, vision, text, heads, topk, flags):
    from paper_2505_16864_amd import binding as jb
    w = dict(T=1, H=1, W=vision, n_text=text, batch=1, heads=heads, head_dim=128, block=block, topk=topk, p=0.5, flags=flags)
    print("more text than vision", w, flush=True)
    layer = CarveLayer(w, "cuda:0", want_lse=True)
    layer.permute_in(*[x.cuda() for x in ji.make_qkv(w, 65)])
    layer.select()
    got = []
    layer.ws_attn.fill_(0xFF)
    for call in (layer.attend, layer.attend, layer.pack, layer.attend_packed):
        if call != layer.pack:
            layer.o_c.view(torch.int16).fill_(0x7FC1)
            layer.lse.fill_(7.0)
        call()
        torch.cuda.synchronize()
        if call != layer.pack:
            got.append((layer.o_c.clone(), layer.lse.clone()))
    (first, first_lse), (second, second_lse), (whole, whole_lse) = got
    assert torch.equal(first, second) and torch.equal(first_lse, second_lse)
    q = layer.q_c.clone()
    jb.jenga_block_sparse_attn(layer.plan, q, layer.k_c, layer.v_c, layer.sel_count, layer.sel_index, q, None,
                               layer.ws_attn, layer.ws_attn.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(q, first)
    # bf16 probabilities taken against another reference, 2^-8 max|v|, and one unit of the bf16 result
    err = (first.float() - whole.float()).abs()
    assert float(err.max()) <= 2.0 ** -6 * float(layer.v_c.float().abs().max())
    alive = torch.isfinite(whole_lse)
    assert torch.equal(torch.isfinite(first_lse), alive)
    assert float((first_lse[alive] - whole_lse[alive]).abs().max()) <= 1e-3      # float32 sums and one float32 logarithm
    n_v = layer.info.M_v * block
    assert bool((err[:, :, :n_v] > 0).any()) and bool((err[:, :, n_v:] > 0).any())   # of both some were cut


# Pad rows of K and V may hold anything: in place, V's reach the second product with probabilities of zero.  Ragged blocks
# of one row, one short, and around the 64 keys of a step.
@pytest.mark.parametrize("head_dim,block", [(64, 32), (64, 64), (128, 64), (64, 128), (128, 128)])
@pytest.mark.parametrize("tail_v,tail_c,heads,flags", [(1, 63, 2, 7), (127, 1, 2, 7), (64, 65, 95, 7), (5, 62, 95, 7),
                                                       (1, 63, 2, 15), (127, 1, 2, 15)])   # 15: short grids are not paced
def test_pad_rows_hold_anything(head_dim, block, tail_v, tail_c, heads, flags):
    w = dict(T=1, H=1, W=block * 8 + min(tail_v, block - 1), n_text=block + min(tail_c, block), batch=1, heads=heads,
             head_dim=head_dim, block=block, topk=0.9, p=0.3, flags=flags)
    print("pads", w, flush=True)
    layer = CarveLayer(w, "cuda:0", want_lse=True)
    layer.permute_in(*[x.cuda() for x in ji.make_qkv(w, 64)])
    layer.select()
    layer.attend()
    torch.cuda.synchronize()
    want, want_lse = layer.o_c.clone(), layer.lse.clone()
    i = layer.info
    assert i.pad_v > 0
    for x in (layer.k_c, layer.v_c):
        x[:, :, i.N_v:i.M_v * block] = float("nan")
        x[:, :, i.M_v * block + w["n_text"]:] = float("inf")
    layer.o_c.view(torch.int16).fill_(0x7FC1)
    layer.attend()
    torch.cuda.synchronize()
    assert torch.equal(layer.o_c, want) and torch.equal(layer.lse, want_lse)
    if block == 32:   # nothing is cut there: in place and packed give the same bits
        layer.pack()
        layer.o_c.view(torch.int16).fill_(0x7FC1)
        layer.attend_packed()
        torch.cuda.synchronize()
        assert torch.equal(layer.o_c, want) and torch.equal(layer.lse, want_lse)
