"""Products whose rows go out in two launches with different wave tiles (several rounds of workgroups, the last one partly empty)
against the same passes with a pinned wave tile, which is one launch: the same bits in every cached row and logit."""
import pytest
import torch

import synth_inputs as si
from launches import launched_kernels, template_ints

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPI = {"residual": 0, "qkv": 1, "swiglu": 2, "relu": 3}


def _tiled(names):
    """-> {epilogue: number of tiled launches}"""
    epis = [template_ints(name)[2] for name in names if "k_gemm_tile" in name]
    return {k: epis.count(v) for k, v in EPI.items() if epis.count(v)}


# rows of a prefill's groups of 16 and of 8, and of decoding rounds (no table of groups: the cache pointers move by whole
# sequences); 3464 and 3495 rows end inside a row tile, 3495 are no multiple of 15 rows behind any row pass but the QKV product's
# own, which stays whole
@pytest.mark.parametrize("opt", [False, True])
@pytest.mark.parametrize("n,length,s,rows,whole", [(24, 145, None, 3456, ()), (433, 9, None, 3464, ()), (216, 3, 15, 3456, ()),
                                                   (233, 3, 14, 3495, ("qkv",))])
def test_every_product_in_two_launches(opt, n, length, s, rows, whole):
    from paper_2310_18813_amd import binding as B
    dtype = "fp16" if opt else "bf16"
    desc = si.opt_desc(1, 4096, 32, 4096, 500, 256) if opt else si.llama_desc(1, 4096, 32, 4096, 500, 256)
    w = si.make_weights(desc, dtype, 5, device=DEV, tag="tgt.")
    prompts = torch.from_numpy(si.make_prompts(n, length, 500, 3)).to(DEV)
    table = torch.from_numpy(si.make_prompts(n, length + 40, 500, 4)).to(DEV)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    ctx = B.Context(desc, w, None, None, dtype, n, s or 0, length + 40, 16, B.PROPOSALS_EXTERNAL, DEV, stream)
    act = "relu" if opt else "swiglu"
    got = []
    with torch.cuda.stream(stream):
        if s:
            ctx.spec_set_proposal_table(table)
        for tile in ((0, 0), (4, 6), (2, 3)):
            ctx.spec_set_gemm_tuning(0, 0)
            ctx.spec_reset(prompts)
            ctx.spec_set_gemm_tuning(*tile)
            if s:
                logits = ctx.spec_verify_step(s, want_logits=True)
                call = lambda: ctx.spec_verify_step(s)
            else:
                ctx.spec_reset(prompts)
                ctx.spec_set_gemm_tuning(0, 0)
                logits = ctx.spec_verify_step(0, want_logits=True)
                ctx.spec_set_gemm_tuning(*tile)
                call = lambda: ctx.spec_reset(prompts)
            k, v = ctx.spec_kv_export(B.MODEL_TARGET, 0, n, length + (s or 0))
            ctx.spec_accept_commit(s or 0)
            if s:
                ctx.spec_rewind()
            launches = _tiled([name for name, _, _ in launched_kernels(B.lib, stream, call)])
            ctx.spec_rewind()
            if tile == (0, 0):
                assert launches == {"qkv": 1 if "qkv" in whole else 2, act: 2, "residual": 4}, launches
            else:
                assert launches["qkv"] == 1 and launches[act] == 1, launches
            got.append((logits, k, v))
    torch.cuda.synchronize()
    ctx.close()
    live = length - 1 if s is None else length + s
    for other in got[1:]:
        assert torch.equal(got[0][0], other[0])
        assert torch.equal(got[0][1][:, :live], other[1][:, :live]) and torch.equal(got[0][2][:, :live], other[2][:, :live])


@pytest.mark.parametrize("rows", [776, 1328, 2600, 4841])
@pytest.mark.parametrize("opt", [False, True])
def test_ragged_prefills_have_the_bits_of_a_pinned_tile(opt, rows):
    """Some hundred to some thousand rows of ragged prompts; none of the products, or one, takes two launches."""
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
