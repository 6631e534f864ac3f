"""GPU parity of jenga_curve_permute_rows (f_blk = G(f), appendix "Frequency re-ordering"): bit-exact."""
import numpy as np
import pytest
import torch

import jenga_inputs as ji
from oracle import jenga_oracle as jo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,cols", [("tiny", 4), ("tiny", 128), ("small", 32), ("hy_lowres", 128), ("small", 1024)])
def test_rows_follow_the_tokens(name, cols):
    from paper_2505_16864_amd import binding as jb
    w = ji.WORKLOADS[name]
    lay = jo.Layout(w["T"], w["H"], w["W"], w["n_text"], w["block"], w["topk"])
    n_src = lay.N_v + w["n_text"]
    g = torch.Generator().manual_seed(8100 + cols)
    table = torch.randn((n_src, cols), generator=g, dtype=torch.float32)
    cfg = jb.make_config(w["T"], w["H"], w["W"], w["n_text"], w["batch"], w["heads"], w["head_dim"], w["block"],
                         w["topk"], w["p"])
    plan = jb.jenga_plan_create(cfg)
    try:
        src = table.to("cuda:0")
        dst = torch.full((lay.N_pad, cols), float("nan"), device="cuda:0", dtype=torch.float32)
        jb.jenga_curve_permute_rows(plan, src, dst, cols * 4, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = dst.cpu().numpy()
    finally:
        jb.jenga_plan_destroy(plan)
    want = jo.permute(table.numpy().astype(np.float64)[None, :, None, :], lay)[0, 0]
    assert got.shape == want.shape
    assert np.array_equal(got.astype(np.float64), want)


def test_row_width_must_be_a_power_of_two():
    from paper_2505_16864_amd import binding as jb
    w = ji.WORKLOADS["tiny"]
    cfg = jb.make_config(w["T"], w["H"], w["W"], w["n_text"], w["batch"], w["heads"], w["head_dim"], w["block"],
                         w["topk"], w["p"])
    plan = jb.jenga_plan_create(cfg)
    try:
        buf = torch.zeros(1 << 16, device="cuda:0")
        for bad in (0, 8, 48, 8192):
            with pytest.raises(jb.JengaError) as err:
                jb.jenga_curve_permute_rows(plan, buf, buf, bad)
            assert err.value.status == -2
    finally:
        jb.jenga_plan_destroy(plan)


@pytest.mark.parametrize("name", ["tiny", "small"])
def test_three_tensors_in_one_launch(name):
    from paper_2505_16864_amd import binding as jb
    w = dict(ji.WORKLOADS[name], batch=2, heads=3)
    q, k, v = [x.cuda() for x in ji.make_qkv(w, 90)]
    plan = jb.jenga_plan_create(jb.make_config(w["T"], w["H"], w["W"], w["n_text"], w["batch"], w["heads"],
                                               w["head_dim"], w["block"], w["topk"], w["p"]))
    try:
        shape = (w["batch"], w["heads"], jb.jenga_plan_info(plan).N_pad, w["head_dim"])
        one = [torch.full(shape, 7.0, dtype=torch.bfloat16, device="cuda:0") for _ in range(3)]
        all3 = [torch.full(shape, 8.0, dtype=torch.bfloat16, device="cuda:0") for _ in range(3)]
        for src, dst in zip((q, k, v), one):
            jb.jenga_curve_permute(plan, src, dst)
        jb.jenga_curve_permute_qkv(plan, q, k, v, *all3)
        torch.cuda.synchronize()
    finally:
        jb.jenga_plan_destroy(plan)
    for a, b in zip(one, all3):
        assert np.array_equal(ji.bits(a), ji.bits(b))


# Results laid over tensors that three calls in a row have finished with: K's over Q, V's over K, all three results in
# one buffer (the last one stays).  Large enough for the three to be in flight together if they were launched as one.
@pytest.mark.parametrize("over", ["k over q, v over k", "v over q", "one buffer"])
def test_results_over_tensors_that_have_moved(over):
    from paper_2505_16864_amd import binding as jb
    w = dict(ji.WORKLOADS["small"], batch=2, heads=24, n_text=70)
    tensors = [x.cuda().reshape(-1) for x in ji.make_qkv(w, 91)]
    plan = jb.jenga_plan_create(jb.make_config(w["T"], w["H"], w["W"], w["n_text"], w["batch"], w["heads"],
                                               w["head_dim"], w["block"], w["topk"], w["p"]))
    try:
        n = w["batch"] * w["heads"] * jb.jenga_plan_info(plan).N_pad * w["head_dim"]
        room = [torch.cat([x, x.new_zeros(n - x.numel())]) for x in tensors]      # inputs in buffers a result fits in
        want = [x.new_empty(n) for x in room]
        for src, dst in zip(tensors, want):
            jb.jenga_curve_permute(plan, src, dst)
        own = [x.new_empty(n) for x in room]
        dst = {"k over q, v over k": [own[0], room[0], room[1]], "v over q": [own[0], own[1], room[0]],
               "one buffer": [own[0], own[0], own[0]]}[over]
        jb.jenga_curve_permute_qkv(plan, *room, *dst)
        torch.cuda.synchronize()
    finally:
        jb.jenga_plan_destroy(plan)
    for t in range(2 if over == "one buffer" else 0, 3):
        assert np.array_equal(ji.bits(dst[t]), ji.bits(want[t])), (over, t)


# More batches than a grid has in z for three tensors.
def test_three_tensors_of_many_batches():
    from paper_2505_16864_amd import binding as jb
    cfg = jb.make_config(1, 1, 3, 1, 21846, 1, 64, 32, 0.5, 0.3)
    plan = jb.jenga_plan_create(cfg)
    try:
        g = torch.Generator(device="cuda:0").manual_seed(92)
        src = [torch.randn((21846, 4, 1, 64), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(3)]
        shape = (21846, 1, jb.jenga_plan_info(plan).N_pad, 64)
        one = [src[0].new_full(shape, 7.0) for _ in range(3)]
        all3 = [src[0].new_full(shape, 8.0) for _ in range(3)]
        for a, b in zip(src, one):
            jb.jenga_curve_permute(plan, a, b)
        jb.jenga_curve_permute_qkv(plan, *src, *all3)
        torch.cuda.synchronize()
    finally:
        jb.jenga_plan_destroy(plan)
    for a, b in zip(one, all3):
        assert torch.equal(a, b)
