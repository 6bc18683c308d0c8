"""The tiled kernel's epilogue against the streaming kernel's, with activations that leave the fp16 range and gates whose
exponential overflows: a batch of equal sequences has the (finite) logits of one alone, bit for bit, and clamps as many values a
sequence, whichever wave tile takes it and with the last row tile partly empty.  Both share SwiGLU's quotient, which is compared with
64 bits by itself."""
import numpy as np
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
    assert torch.isfinite(one).all()
    assert clamped > 0 and clamped_many == n * clamped
    assert torch.equal(many.view(torch.int32), one.view(torch.int32).expand_as(many))


# Gates of -400 to 400 in steps of 0.5 up to 104: the exponential overflows below -88.7, and from -87.3 on the divisor's reciprocal is
# below the smallest normal float.  (All of them exact in bf16.)
GATES = np.concatenate([np.arange(-104, 104, 0.5), np.linspace(-400, -105, 16).round() // 2 * 2, np.linspace(105, 400, 16).round() // 2 * 2])


@pytest.mark.parametrize("log2_up", [0, 27])
@pytest.mark.parametrize("n,tile", [(1, (0, 0)), (4, (0, 0)), (43, (1, 2)), (43, (2, 3)), (43, (4, 6))])  # 3, 12 and 129 rows
def test_swiglu_of_known_gates(n, tile, log2_up):
    """One layer whose attention adds nothing and whose gate and up projections each read one channel of value +-1: activation i is
    swiglu(GATES[i] r, +-2^log2_up r), r the norm's 1 / rms, and the down projection (the identity) adds it to channel i of the
    row.  Allowed: fp16's rounding of the activation, 2^-11, beside 4e-5 for the exponential of an argument of up to 90 (the gate's
    and the scaled argument's fp32 roundings); half fp16's smallest number; the fp32 rounding of the row's sum."""
    from paper_2310_18813_amd import binding as B
    d, f, s = 512, len(GATES), 2
    assert f == 448
    desc = si.llama_desc(1, d, 4, f, 300, 64)
    w = si.make_weights(desc, "bf16", 3, device="cpu", tag="tgt.")
    sign = torch.where(torch.rand(d, generator=torch.Generator().manual_seed(5)) < 0.5, -1.0, 1.0)
    sign[0] = 1.0
    L = w["layers"][0]
    w["tok_emb"][:] = sign.to(torch.bfloat16)
    L["wo"].zero_()
    for name in ("w1", "w3", "w2"):
        L[name].zero_()
    L["w1"][:, 0] = torch.from_numpy(GATES).to(torch.bfloat16)
    assert np.array_equal(L["w1"][:, 0].double().numpy(), GATES)
    up = torch.where(torch.arange(f) % 3 == 0, -1.0, 1.0) * 2.0 ** log2_up
    L["w3"][:, 0] = up.to(torch.bfloat16)
    L["w2"][:f, :f] = torch.eye(f).to(torch.bfloat16)
    dev = lambda t: None if t is None else t.to(DEV)
    wg = {k: dev(v) for k, v in w.items() if k != "layers"}
    wg["layers"] = [{k: dev(v) for k, v in L.items()}]
    ctx = B.Context(desc, wg, None, None, "bf16", n, s, 32, 8, B.PROPOSALS_EXTERNAL, DEV)
    if tile[0]:
        ctx.spec_set_gemm_tuning(*tile, 0)
    ctx.spec_reset_noprefill(si.make_prompts(n, 9, 300, 11))
    ctx.spec_set_proposals(torch.tensor(si.make_prompts(n, s, 300, 12)))
    dump = ctx.spec_set_hidden_dump(True)
    ctx.spec_verify_step(s)
    M = n * (s + 1)
    rows = dump[:2 * M * d].view(2, M, d).cpu().double().numpy()
    ctx.close()
    x = sign.double().numpy()
    assert np.array_equal(rows[0], np.broadcast_to(x, (M, d)))
    r = 1.0 / np.sqrt(1.0 + 1e-5)
    g = GATES * r
    with np.errstate(over="ignore"):
        act = np.clip(g / (1.0 + np.exp(-g)) * up.double().numpy() * r, -65504.0, 65504.0)
    want = x.copy()
    want[:f] += act
    bound = np.zeros(d)
    bound[:f] = np.abs(act) * (2.0 ** -11 + 4e-5) + 2.0 ** -25
    bound += np.abs(want) * 2.0 ** -24
    err = np.abs(rows[1] - want)
    assert np.isfinite(rows[1]).all() and (err <= bound).all(), (np.nanargmax((err / np.maximum(bound, 1e-30)).max(0)), (err / np.maximum(bound, 1e-30)).max())
