"""Models the matrix-core kernels do not take (heads of neither 64 nor 128, widths that are no multiple of 32, of 16 in
fp32) run on the generic kernels: logits of a verification and behind ragged prompts against the fp64 oracle, within the
dtype's logit tolerance.  (Draft and target on different paths: test_gpu_draft.py.)"""
import numpy as np
import pytest
import torch

import synth_inputs as si
from helpers import LOGIT_TOL, build_pair
from test_gpu_prefill_groups import LENGTHS

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

DESCS = {
    "hd32_fp32": ("fp32", si.llama_desc(2, 96, 3, 100, 211, 2400)),
    "hd80_odd_ffn_fp32": ("fp32", si.opt_desc(2, 160, 2, 45, 203, 2400)),
    "hd96_bf16": ("bf16", si.llama_desc(2, 192, 2, 160, 211, 2400)),
    "hd64_ffn72_fp16": ("fp16", si.opt_desc(2, 128, 2, 72, 1001, 2400)),
}


def _context(name, n, s, longest, random_norms):
    from oracle import oracle as om
    from paper_2310_18813_amd import binding as B
    dtype, desc = DESCS[name]
    ot, _, gt, _ = build_pair(om.Oracle("f64"), desc, None, dtype, 23, DEV, random_norms=random_norms)
    return dtype, desc, ot, B.Context(desc, gt, None, None, dtype, n, s, longest + s + 8, 4, B.PROPOSALS_EXTERNAL, DEV)


@pytest.mark.parametrize("name", list(DESCS))
@pytest.mark.parametrize("n,s,longest", [(1, 0, 1), (3, 4, 17), (5, 15, 70)])
def test_verification_logits(name, n, s, longest):
    dtype, desc, ot, ctx = _context(name, n, s, longest, True)
    rng = np.random.default_rng(n * 100 + longest)
    V = desc["vocab"]
    prompts = [rng.integers(0, V, size=max(1, longest - 3 * b)).astype(np.int32) for b in range(n)]
    table = rng.integers(0, V, size=(n, ctx.L_max), dtype=np.int32)
    ctx.spec_set_proposal_table(table)
    ctx.spec_reset_ragged([torch.from_numpy(p) for p in prompts])
    got = ctx.spec_verify_step(s, want_logits=True).cpu().numpy()
    for b, p in enumerate(prompts):
        seq = list(p) + list(table[b, len(p):len(p) + s])
        want = ot.forward(ot.cache(len(seq)), seq, 0)[len(p) - 1:]
        assert np.abs(got[b] - want).max() <= LOGIT_TOL[dtype], b
    ctx.close()


@pytest.mark.parametrize("lengths", list(LENGTHS))
@pytest.mark.parametrize("name", list(DESCS))
def test_ragged_prompts(name, lengths):
    lens = LENGTHS[lengths]
    dtype, desc, ot, ctx = _context(name, len(lens), 2, max(lens), False)
    rng = np.random.default_rng(len(name))
    prompts = [rng.integers(0, desc["vocab"], size=n).astype(np.int32) for n in lens]
    ctx.spec_reset_ragged([torch.from_numpy(p) for p in prompts])
    got = ctx.spec_verify_step(0, want_logits=True).cpu().numpy()[:, 0]
    for b, p in enumerate(prompts):
        if len(p) > 1600 and b != 3:
            continue  # one long sequence across the pass boundary is enough of the oracle's time
        want = ot.forward(ot.cache(len(p)), list(p), 0)[-1]
        assert np.abs(got[b] - want).max() <= LOGIT_TOL[dtype], (b, len(p))
    ctx.close()
