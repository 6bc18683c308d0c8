"""Products whose rows go out in two launches with different wave tiles (several rounds of workgroups, the last one partly empty):
a prefill of enough rows that every product of a layer is split, against the same prompts in passes with a pinned wave tile,
which is one launch: the same bits in every cached row and logit.  Rows that end inside a row tile and inside a row pass."""
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows", [776, 1328, 2600, 4841])
@pytest.mark.parametrize("opt", [False, True])
def test_two_launches_give_the_bits_of_one(opt, rows):
    from paper_2310_18813_amd import binding as B
    dtype = "fp16" if opt else "bf16"
    desc = si.opt_desc(2, 2048, 16, 5504, 500, 1024) if opt else si.llama_desc(2, 2048, 16, 5504, 500, 1024)
    w = si.make_weights(desc, dtype, 5, device=DEV, tag="tgt.")
    lengths, left = [], rows
    while left > 0:  # ragged prompts of `rows` rows in all
        m = min(left, 301 + 37 * len(lengths) % 200)
        lengths.append(m + 1)
        left -= m
    n = len(lengths)
    prompts = [torch.from_numpy(si.make_prompts(1, m, 500, 40 + i)[0]) for i, m in enumerate(lengths)]
    ctx = B.Context(desc, w, None, None, dtype, n, 0, 640, 40, B.PROPOSALS_EXTERNAL, DEV)
    got = []
    for tile in ((0, 0), (4, 6), (2, 3)):
        ctx.spec_set_gemm_tuning(*tile)
        ctx.spec_reset_ragged(prompts)
        k, v = ctx.spec_kv_export(B.MODEL_TARGET, 1, n, max(lengths) - 1)
        ctx.spec_set_gemm_tuning(0, 0)
        logits = ctx.spec_verify_step(0, want_logits=True).clone()
        ctx.spec_accept_commit(0)
        got.append((k.clone(), v.clone(), logits))
    ctx.close()
    for other in got[1:]:
        for i, m in enumerate(lengths):
            assert torch.equal(got[0][0][i, :m - 1], other[0][i, :m - 1]), (i, m)
            assert torch.equal(got[0][1][i, :m - 1], other[1][i, :m - 1]), (i, m)
        assert torch.equal(got[0][2], other[2])
