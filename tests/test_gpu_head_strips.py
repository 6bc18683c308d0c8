"""The LM head with a wave per strip (up to 32 rows, d_model 256 to 1024, many strips) against the streaming kernel, which a
pinned wave tile selects at these row counts: the same bits in every logit, and the token of the largest one, at the
edges of its row tiles and with a vocabulary that ends inside a strip and inside a store of four."""
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("vocab", [16403, 28800, 33001])
@pytest.mark.parametrize("d,heads,opt", [(256, 4, False), (512, 8, True), (768, 12, False), (1024, 16, True)])
def test_strips_match_the_streaming_head(d, heads, opt, vocab):
    from paper_2310_18813_amd import binding as B
    dtype = "fp16" if opt else "bf16"
    desc = si.opt_desc(1, d, heads, 2 * d, vocab, 128) if opt else si.llama_desc(1, d, heads, 2 * d, vocab, 128)
    w = si.make_weights(desc, dtype, 5, device=DEV, tag="tgt.")
    for rows in (1, 15, 16, 17, 32):
        ctx = B.Context(desc, w, None, None, dtype, rows, 0, 96, 40, B.PROPOSALS_EXTERNAL, DEV)
        prompts = si.make_prompts(rows, 9, vocab, 7)
        got = []
        for tile in ((0, 0), (1, 4)):
            ctx.spec_set_gemm_tuning(*tile)
            ctx.spec_reset(prompts)
            logits = ctx.spec_verify_step(0, want_logits=True).clone()
            ctx.spec_accept_commit(0)
            got.append((logits.cpu(), [int(t[-1]) for t in ctx.spec_read_output()[0]]))
        ctx.close()
        assert torch.equal(got[0][0], got[1][0]), (rows, (got[0][0] != got[1][0]).sum())
        want = got[0][0].reshape(rows, vocab).numpy().argmax(-1)  # the first of equal ones, as the kernels take it
        assert got[0][1] == got[1][1] == list(want), rows
