"""Prefill attention with four row groups to a workgroup, cache rows through LDS, against one wave per (group, head) (a pinned
launch shape): the same bits in every cached row and logit.  Prompts of all kinds of lengths, so that workgroups hold groups
of one, two and four sequences and a last one that is not full, and chunks end at 128, 512 and 768."""
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LENGTHS = [801, 33, 129, 5, 513, 17, 18, 260, 2, 128, 770, 64, 385]


@pytest.mark.parametrize("d,heads,opt", [(1024, 16, False), (1024, 8, False), (512, 8, True), (1024, 8, True)])
def test_prefill_shapes_give_identical_bits(d, heads, opt):
    from paper_2310_18813_amd import binding as B
    dtype = "fp16" if opt else "bf16"
    desc = si.opt_desc(2, d, heads, 2 * d, 500, 1024) if opt else si.llama_desc(2, d, heads, 2 * d, 500, 1024)
    w = si.make_weights(desc, dtype, 5, device=DEV, tag="tgt.")
    n = len(LENGTHS)
    prompts = [torch.from_numpy(si.make_prompts(1, m, 500, 40 + i)[0]) for i, m in enumerate(LENGTHS)]
    ctx = B.Context(desc, w, None, None, dtype, n, 0, 896, 40, B.PROPOSALS_EXTERNAL, DEV)
    assert sum((m + 14) // 16 for m in LENGTHS) * heads >= 768  # enough pairs for the shape with a wave each
    got = []
    for shape in (0, 2):
        ctx.spec_set_attention_shape(shape)
        ctx.spec_reset_ragged(prompts)
        k, v = ctx.spec_kv_export(B.MODEL_TARGET, 1, n, max(LENGTHS) - 1)
        ctx.spec_set_attention_shape(0)
        logits = ctx.spec_verify_step(0, want_logits=True).clone()
        ctx.spec_accept_commit(0)
        got.append((k.clone(), v.clone(), logits))
    ctx.close()
    for i, m in enumerate(LENGTHS):
        for a, b in zip(got[0][:2], got[1][:2]):
            assert torch.equal(a[i, :m - 1], b[i, :m - 1]), (i, m)
    assert torch.equal(got[0][2], got[1][2])
