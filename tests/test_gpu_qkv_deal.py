"""QKV products of decoding rounds over several row passes, whose strip groups go to the XCDs whole unless that takes more rounds: every sequence's logits and
cached rows are those of the same sequence in a small batch (one row pass), bit for bit, at numbers of groups that eight
divides and does not."""
import pytest
import torch

import synth_inputs as si
from launches import launched_kernels, template_ints

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPI_QKV = 1


@pytest.mark.parametrize("d,heads,opt,n,in_turn", [(1536, 12, False, 64, True), (1536, 12, False, 97, False), (2048, 32, True, 48, True),
                                                  (1280, 10, True, 128, True)])
def test_rows_of_several_passes_are_those_of_small_batches(d, heads, opt, n, in_turn):
    from paper_2310_18813_amd import binding as B
    s, dtype = 7, "fp16" if opt else "bf16"
    desc = si.opt_desc(1, d, heads, 2 * d, 500, 64) if opt else si.llama_desc(1, d, heads, 2 * d, 500, 64)
    w = si.make_weights(desc, dtype, 5, device=DEV, tag="tgt.")
    prompts = torch.from_numpy(si.make_prompts(n, 9, 500, 3)).to(DEV)
    table = torch.from_numpy(si.make_prompts(n, 48, 500, 4)).to(DEV)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()

    def run(b0, b1, names=None):
        ctx = B.Context(desc, w, None, None, dtype, b1 - b0, s, 48, 16, B.PROPOSALS_EXTERNAL, DEV, stream)
        part = table[b0:b1].contiguous()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            ctx.spec_set_proposal_table(part)
            ctx.spec_reset(prompts[b0:b1])
            logits = ctx.spec_verify_step(s, want_logits=True)
            k, v = ctx.spec_kv_export(B.MODEL_TARGET, 0, b1 - b0, 9 + s)
            ctx.spec_accept_commit(s)
        if names is not None:
            names += launched_kernels(B.lib, stream, lambda: ctx.spec_verify_step(s))
        torch.cuda.synchronize()
        ctx.close()
        return logits, k, v

    kernels = []
    whole = run(0, n, kernels)
    mine = [(template_ints(name), grid[0]) for name, grid, _ in kernels if "k_gemm_tile" in name and template_ints(name)[2] == EPI_QKV]
    assert len(mine) == 1, kernels
    (mtw, nbw, *_), blocks = mine[0]
    groups, passes = -(-(3 * d // 16) // (2 * nbw)), -(-n * (s + 1) // (64 * mtw))
    assert passes > 1 and blocks == (-(-groups // 8) * 8 * passes if in_turn else -(-groups * passes // 8) * 8), (mine, groups, passes)
    for b in range(0, n, 6):
        e = min(n, b + 6)
        for got, want in zip(whole, run(b, e)):
            assert torch.equal(got[b:e], want), b
