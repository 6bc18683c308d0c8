"""The tiled kernel's epilogue against the streaming kernel's, with activations that leave the fp16 range and gates whose
exponential overflows: a batch of equal sequences has the logits of one alone, bit for bit, and clamps as many values a
sequence, whichever wave tile takes it and with the last row tile partly empty."""
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("shape", ["llama", "opt"])
@pytest.mark.parametrize("mtw,nbw", [(1, 2), (2, 3), (3, 4), (4, 6)])
def test_clamped_values_and_their_count_are_the_streaming_kernels(shape, mtw, nbw):
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(2, 256, 2, 416, 300, 64) if shape == "llama" else si.opt_desc(2, 256, 2, 416, 300, 64)
    w = si.make_weights(desc, "bf16", 11, device=DEV, emb_std=1.0, tag="tgt.")
    for L in w["layers"]:  # gates and up projections of several hundred, their products beyond 65504
        for k in ("w1", "w3"):
            if L.get(k) is not None:
                L[k] = (L[k].float() * 2000).to(torch.bfloat16) if shape == "llama" else (L[k].float() * 3e5).to(torch.bfloat16)
    n, s = 43, 2  # 129 rows
    prompt = si.make_prompts(1, 9, 300, 11)
    props = si.make_prompts(1, s, 300, 12)

    def run(count):
        ctx = B.Context(desc, w, None, None, "bf16", count, s, 32, 8, B.PROPOSALS_EXTERNAL, DEV)
        if count > 1:
            ctx.spec_set_gemm_tuning(mtw, nbw, 0)
        ctx.spec_reset_noprefill(prompt.repeat(count, axis=0))
        ctx.spec_set_proposals(torch.tensor(props.repeat(count, axis=0)))
        logits = ctx.spec_verify_step(s, want_logits=True).clone().reshape(count, s + 1, -1)
        clamped = ctx.spec_read_saturation()
        ctx.close()
        return logits, clamped

    one, clamped = run(1)
    many, clamped_many = run(n)
    assert clamped > 0 and clamped_many == n * clamped
    assert torch.equal(many.view(torch.int32), one.view(torch.int32).expand_as(many))
