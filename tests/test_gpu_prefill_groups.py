"""Prefill row groups: prompts of very different lengths cut into groups of 16 or 8 positions and packed into passes.
The logits behind every prompt (they see its whole cache) against the fp64 oracle, within the dtype's logit tolerance."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from helpers import LOGIT_TOL, build_pair

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

LENGTHS = {
    "groups_of_8": [1, 2, 9, 8, 5, 10, 3],            # half groups leave fewer dead rows; a prompt without rows
    "groups_of_16": [17, 1, 33, 16, 49, 18, 64],      # exact and ragged last groups
    "two_passes": [2111, 1, 2100, 2049, 1025, 1500],  # more rows than a pass takes: a boundary inside a sequence
}


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("dtype", ["fp32", "bf16", "fp16"])
def test_ragged_prompts_leave_the_caches_the_oracle_expects(name, dtype):
    from oracle import oracle as om
    from paper_2310_18813_amd import binding as B
    lens = LENGTHS[name]
    desc = si.llama_desc(2, 128, 2, 160, 211, 2400)
    ot, _, gt, _ = build_pair(om.Oracle("f64"), desc, None, dtype, 91, DEV)
    rng = np.random.default_rng(len(name))
    prompts = [rng.integers(0, 211, size=n).astype(np.int32) for n in lens]
    ctx = B.Context(desc, gt, None, None, dtype, len(lens), 2, max(lens) + 8, 4, B.PROPOSALS_EXTERNAL, DEV)
    ctx.spec_reset_ragged([torch.from_numpy(p) for p in prompts])
    got = ctx.spec_verify_step(0, want_logits=True).cpu().numpy()[:, 0]
    for b, p in enumerate(prompts):
        if len(p) > 1600 and b != 3:
            continue  # one long sequence across the pass boundary is enough of the oracle's time
        want = ot.forward(ot.cache(len(p)), list(p), 0)[-1]
        assert np.abs(got[b] - want).max() <= LOGIT_TOL[dtype], (b, len(p))


# heads of 128: more than four thousand rows a pass (every row a live one of some prompt or of its last group), so that the
# products take more than eight row passes and their largest tiles
WIDE = {
    "llama_bf16": ("bf16", si.llama_desc(2, 4096, 32, 11008, 512, 2048)),
    "opt_fp16": ("fp16", si.opt_desc(2, 5120, 40, 20480, 512, 2048)),
}
WIDE_LENGTHS = [1100, 37, 2, 1021, 17, 1500, 9, 1005]


@pytest.mark.parametrize("tile", [(0, 0), (4, 6), (2, 6), (1, 4)])
@pytest.mark.parametrize("name", list(WIDE))
def test_a_large_ragged_prefill_leaves_the_rows_of_prompts_admitted_one_by_one(name, tile):
    """Cache rows bit for bit, prompts of a few rows (other kernels) among them."""
    from paper_2310_18813_amd import binding as B
    dtype, desc = WIDE[name]
    w = si.make_weights(desc, dtype, 5, device=DEV, emb_std=1.0, tag="tgt.")
    rng = np.random.default_rng(12)
    prompts = [torch.from_numpy(rng.integers(0, desc["vocab"], size=n).astype(np.int32)) for n in WIDE_LENGTHS]
    n, longest = len(prompts), max(WIDE_LENGTHS)

    def context():
        return B.Context(desc, w, None, None, dtype, n, 1, longest + 8, 4, B.PROPOSALS_EXTERNAL, DEV)

    whole, single = context(), context()
    whole.spec_set_gemm_tuning(*tile)
    whole.spec_reset_ragged(prompts)
    single.spec_reset_ragged([p[:1] for p in prompts])
    for b, p in enumerate(prompts):
        single.spec_admit(b, p.to(DEV))
    for layer in range(desc["n_layers"]):
        got, want = whole.spec_kv_export(B.MODEL_TARGET, layer, n, longest), single.spec_kv_export(B.MODEL_TARGET, layer, n, longest)
        for b, p in enumerate(prompts):
            for g, x in zip(got, want):
                assert torch.equal(g[b, :len(p) - 1], x[b, :len(p) - 1]), (layer, b)
    assert torch.equal(whole.spec_verify_step(0, want_logits=True), single.spec_verify_step(0, want_logits=True))
    whole.close()
    single.close()
