"""A round by itself against the same round in steps: inside a round the last proposal's arg-max is the second stage of the embedding kernel
of the pass behind it, and nothing a caller can read may differ."""
import pytest
import torch

import synth_inputs as si
from launches import launched_kernels

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,tgt,drf,n", [
    ("fp32", si.llama_desc(2, 128, 2, 352, 333, 64), si.llama_desc(1, 64, 1, 96, 333, 64), 3),
    ("fp32", si.opt_desc(1, 128, 2, 256, 5000, 64), si.opt_desc(1, 128, 2, 192, 5000, 64), 1),
    ("bf16", si.llama_desc(1, 256, 2, 416, 1000, 64), si.llama_desc(1, 128, 2, 160, 1000, 64), 5),
    ("bf16", si.llama_desc(1, 256, 2, 416, 33000, 64), si.llama_desc(1, 256, 4, 512, 33000, 64), 2),   # the head's partials by workgroup
    ("bf16", si.llama_desc(1, 128, 2, 160, 600, 64), si.llama_desc(1, 128, 2, 160, 600, 64), 40),
    ("fp16", si.opt_desc(1, 256, 4, 384, 777, 64), si.opt_desc(1, 128, 2, 192, 777, 64), 2),
    ("fp16", si.llama_desc(1, 256, 4, 448, 900, 64), si.llama_desc(1, 96, 2, 96, 900, 64), 2)])         # a draft on the plain kernels
@pytest.mark.parametrize("caps,table", [(False, False), (True, False), (False, True)])
def test_round_equals_its_steps(dtype, tgt, drf, n, caps, table):
    from paper_2310_18813_amd import binding as B
    wt = si.make_weights(tgt, dtype, 5, device=DEV, emb_std=1.0, tag="tgt.")
    wd = si.make_weights(drf, dtype, 5, device=DEV, emb_std=1.0, tag="drf.")
    torch.cuda.synchronize()
    ctx = B.Context(tgt, wt, drf, wd, dtype, n, 4, 40, 20, B.PROPOSALS_EXTERNAL if table else B.PROPOSALS_DRAFT, DEV)
    prompts = torch.from_numpy(si.make_prompts(n, 6, tgt["vocab"], 5)).to(DEV)
    torch.cuda.synchronize()

    def run(whole):
        ctx.spec_reset(prompts)
        if table:
            ctx.spec_set_proposal_table(si.make_prompts(n, 40, tgt["vocab"], 6))
        ctx.spec_set_seq_s([(3 * b + 1) % 5 for b in range(n)] if caps else None)
        seen = []
        for s in (4, 1, 0, 2, 0, 0, 3, 4):
            if whole:
                ctx.spec_round(s, 1)
            else:
                for j in range(1, s + 1):
                    ctx.spec_draft_step(j)
                ctx.spec_verify_step(s)
                ctx.spec_accept_commit(s)
            seen.append((ctx.spec_read_proposals(), ctx.spec_read_state(), ctx.spec_read_output()))
        return seen

    steps = run(False)
    assert run(True) == steps
    ctx.close()


@pytest.mark.parametrize("dtype,tgt,drf", [
    ("fp32", si.llama_desc(1, 128, 2, 352, 333, 64), si.llama_desc(1, 64, 1, 96, 333, 64)),
    ("bf16", si.llama_desc(1, 256, 2, 416, 1000, 64), si.llama_desc(1, 128, 2, 160, 1000, 64))])
def test_timed_draft_passes_are_whole(dtype, tgt, drf):
    """While launches are timed, a draft pass (SPEC_KCLASS_DRAFT_PASS) takes its own arg-max to the end: a round of three draft steps
    launches four second stages (one of them the verification's), as its steps by themselves do, and emits the same tokens."""
    from paper_2310_18813_amd import binding as B
    wt = si.make_weights(tgt, dtype, 5, device=DEV, emb_std=1.0, tag="tgt.")
    wd = si.make_weights(drf, dtype, 5, device=DEV, emb_std=1.0, tag="drf.")
    stream = torch.cuda.Stream()
    ctx = B.Context(tgt, wt, drf, wd, dtype, 2, 3, 40, 20, B.PROPOSALS_DRAFT, DEV, stream)
    prompts = torch.from_numpy(si.make_prompts(2, 6, tgt["vocab"], 5)).to(DEV)
    torch.cuda.synchronize()

    def second_stages(timed):
        ctx.spec_reset(prompts)
        ctx.spec_kernel_timing(timed)
        names = [k for k, _, _ in launched_kernels(B.lib, stream, lambda: B._check(B.lib.spec_round(ctx.h, 3, 1), ctx.h))]
        ctx.spec_kernel_timing(False)
        return sum("k_argmax_partials" in k for k in names)

    assert second_stages(False) == 1
    assert second_stages(True) == 4

    def tokens(timed):
        ctx.spec_reset(prompts)
        ctx.spec_kernel_timing(timed)
        ctx.spec_round(3, 3)
        ctx.spec_kernel_timing(False)
        return ctx.spec_read_output()

    assert tokens(True) == tokens(False)
    ctx.close()
