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
