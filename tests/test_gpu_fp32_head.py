"""The fp32 LM head with three row tiles and four strips to a workgroup (33 to 48 rows, many strips): every row of a batch of
equal prompts has the logits of the prompt alone, bit for bit, and the token of the largest one."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from launches import launched_kernels, template_ints

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


@pytest.mark.parametrize("d,rows,product,tiles", [(1024, 40, "head", 12), (1024, 72, "head", 4), (768, 784, "down", 6), (768, 784, "o", 6),
                                                  (1024, 704, "qkv", 12), (1024, 1920, "gate-up", 12)])
def test_twelve_tiles_to_a_workgroup_only_where_they_are_faster(d, rows, product, tiles):
    """The head at 72 rows and the residual products of 768 at 784 rows took 1.3 and 1.7 times as long with twelve."""
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(1, d, d // 64, 4 * d, 32000, 1024)
    w = si.make_weights(desc, "fp32", 5, device=DEV, tag="tgt.")
    prefill = rows > 100
    n, length = (rows // 16, 17) if prefill else (rows // 8, 2)
    prompts = torch.randint(0, 32000, (n, length), dtype=torch.int32, device=DEV)
    table = torch.randint(0, 32000, (n, 64), dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    ctx = B.Context(desc, w, None, None, "fp32", n, 7, 64, 16, B.PROPOSALS_EXTERNAL, DEV, stream)
    ctx.spec_set_proposal_table(table)
    ctx.spec_reset(prompts)
    kernels = launched_kernels(B.lib, stream, (lambda: ctx.spec_reset(prompts)) if prefill else (lambda: ctx.spec_verify_step(7)))
    torch.cuda.synchronize()
    ctx.close()
    got = [template_ints(name)[:2] for name, _, _ in kernels if "k_gemm_f32" in name]
    assert len(got) == (4 if prefill else 5), kernels
    mt, nb = got[["qkv", "o", "gate-up", "down", "head"].index(product)]
    assert mt * nb == tiles, got
