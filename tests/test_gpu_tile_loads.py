"""The tiled kernel's weights of a single row pass: read non-temporally where the model is larger than the memory-side cache, plainly
where it fits.  The same layer below a small LM head and below one of 200 copies of its rows takes the one kernel and the other: the
same bits in every cached row and logit, at every wave tile whose one row pass holds the rows."""
import pytest
import torch

import synth_inputs as si
from launches import launched_kernels, template_ints

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SINGLE_NT, SINGLE_KEPT = 1, 2
COPIES = 200  # 1000 x 1024 in 16 bits: 2 MB a copy


@pytest.mark.parametrize("opt", [False, True])
@pytest.mark.parametrize("n,s", [(5, 8), (16, 3), (11, 15), (16, 15)])
def test_both_kinds_of_loads_give_the_same_bits(n, s, opt):
    from paper_2310_18813_amd import binding as B
    dtype, d = ("fp16" if opt else "bf16"), 1024
    desc = si.opt_desc(2, d, 16, 8192, 1000, 64) if opt else si.llama_desc(2, d, 16, 8192, 1000, 64)
    small = si.make_weights(desc, dtype, 7, device=DEV, tag="tgt.")
    large = dict(small, tok_emb=small["tok_emb"].repeat(COPIES, 1), lm_head=small["lm_head"].repeat(COPIES, 1))
    prompts = torch.from_numpy(si.make_prompts(n, 9, 1000, 3)).to(DEV)
    table = torch.from_numpy(si.make_prompts(n, 64, 1000, 4)).to(DEV)
    got = {}
    for kind, w, vocab in ((SINGLE_KEPT, small, 1000), (SINGLE_NT, large, 1000 * COPIES)):
        torch.cuda.synchronize()
        stream = torch.cuda.Stream()
        ctx = B.Context(dict(desc, vocab=vocab), w, None, None, dtype, n, s, 64, 16, B.PROPOSALS_EXTERNAL, DEV, stream)
        with torch.cuda.stream(stream):
            ctx.spec_set_proposal_table(table)
            for mt in range((n * (s + 1) + 63) // 64, 5):
                for nb in (2, 3, 4, 6):
                    ctx.spec_set_gemm_tuning(0, 0)
                    ctx.spec_reset(prompts)
                    ctx.spec_set_gemm_tuning(mt, nb)
                    logits = ctx.spec_verify_step(s, want_logits=True)
                    ctx.spec_accept_commit(s)
                    out = [logits[..., :1000].clone()] + [t for layer in (0, 1) for t in ctx.spec_kv_export(B.MODEL_TARGET, layer, n, 9)]
                    stream.synchronize()
                    if kind == SINGLE_KEPT:
                        got[mt, nb] = out
                    else:
                        for i, (a, b) in enumerate(zip(out, got[mt, nb])):
                            assert torch.equal(a, b), (mt, nb, i)
                    ctx.spec_set_gemm_tuning(0, 0)
                    ctx.spec_reset(prompts)
                    ctx.spec_set_gemm_tuning(mt, nb)
                    stream.synchronize()
                    kernels = [template_ints(name) for name, _, _ in launched_kernels(B.lib, stream, lambda: ctx.spec_verify_step(s))
                               if "k_gemm_tile" in name]
                    assert kernels and all(k[:2] == [mt, nb] and k[4] == kind for k in kernels), kernels
        ctx.close()
