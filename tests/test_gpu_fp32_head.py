"""The fp32 LM head with three row tiles and four strips to a workgroup (33 to 48 rows, many strips): every row of a batch of
equal prompts has the logits of the prompt alone, bit for bit, and the token of the largest one."""
import numpy as np
import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows", [33, 40, 48])
@pytest.mark.parametrize("vocab", [16000, 16003])
def test_rows_of_a_batch_are_the_row_alone(vocab, rows):
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(1, 256, 4, 512, vocab, 128)
    w = si.make_weights(desc, "fp32", 5, device=DEV, tag="tgt.")
    prompt = si.make_prompts(1, 7, vocab, 7)
    got = []
    for n in (1, rows):
        ctx = B.Context(desc, w, None, None, "fp32", n, 0, 96, 40, B.PROPOSALS_EXTERNAL, DEV)
        ctx.spec_reset(np.repeat(prompt, n, 0))
        logits = ctx.spec_verify_step(0, want_logits=True).clone()
        ctx.spec_accept_commit(0)
        got.append((logits.reshape(n, vocab).cpu(), [int(t[-1]) for t in ctx.spec_read_output()[0]]))
        ctx.close()
    assert torch.equal(got[1][0], got[0][0].expand(rows, vocab))
    assert got[1][1] == [int(got[0][0][0].numpy().argmax())] * rows
