"""Which launch shape a decoding pass of three or four chunks takes: a wave per (sequence, head) from more than two workgroups a CU on
for heads of 128, a workgroup per pair up to seven eighths of a round of waves for heads of 64; and that the shape changes no bit."""
import pytest
import torch

import synth_inputs as si
from launches import launched_kernels

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("hd,heads,n,kv,kernel", [
    (128, 32, 16, 300, "k_attn_group"), (128, 32, 17, 300, "k_attn_seq"), (128, 32, 17, 400, "k_attn_group"),
    (64, 32, 24, 300, "k_attn_group"), (64, 32, 24, 500, "k_attn_group"), (64, 32, 24, 200, "k_attn_seq"),
    (64, 32, 28, 300, "k_attn_group"), (64, 32, 29, 300, "k_attn_seq"), (64, 32, 32, 500, "k_attn_seq")])
def test_launch_shape_of_three_and_four_chunks(hd, heads, n, kv, kernel):
    from paper_2310_18813_amd import binding as B
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the pair counts are those of 256 compute units")
    d = hd * heads
    desc = si.llama_desc(1, d, heads, 64, 300, 600)
    w = si.make_weights(desc, "bf16", 3, device=DEV, emb_std=1.0, tag="tgt.")
    stream = torch.cuda.Stream()
    ctx = B.Context(desc, w, None, None, "bf16", n, 1, kv + 8, 4, B.PROPOSALS_EXTERNAL, DEV, stream)
    K, V = si.make_kv(n, d, kv, "bf16", 3, DEV)
    torch.cuda.synchronize()
    ctx.spec_kv_import(B.MODEL_TARGET, 0, K, V)
    prompts = torch.from_numpy(si.make_prompts(n, kv + 1, 300, 3)).to(DEV)
    props = torch.from_numpy(si.make_prompts(n, 1, 300, 4)).to(DEV)
    logits = []
    for shape in (0, 1, 2, 3):
        ctx.spec_set_attention_shape(shape)
        ctx.spec_reset_noprefill(prompts)
        ctx.spec_set_proposals(props)
        torch.cuda.synchronize()
        if shape == 0:
            names = [k for k, _, _ in launched_kernels(B.lib, stream, lambda: B._check(B.lib.spec_verify_step(ctx.h, 1, None), ctx.h))]
            assert sum("k_attn" in k for k in names) == 1 and sum(kernel in k for k in names) == 1, names
            ctx.spec_accept_commit(1)
            ctx.spec_reset_noprefill(prompts)
            ctx.spec_set_proposals(props)
        logits.append(ctx.spec_verify_step(1, want_logits=True))
        ctx.spec_accept_commit(1)
        torch.cuda.synchronize()
    assert all(torch.equal(logits[0], x) for x in logits[1:])
    ctx.close()
