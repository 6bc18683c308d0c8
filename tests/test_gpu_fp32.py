"""The fp32 matrix-core path at the edges of its tiles, against the fp64 oracle within the fp32 logit tolerance: vocabularies
that are no multiple of 4 or 16, one k-slice and eight, heads of 64 and 128, LayerNorm with biases, rows of 1 to 4 tiles
and beyond, contexts around the 16-key tiles and the eight waves' turn."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from helpers import LOGIT_TOL, build_pair

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

DESCS = {
    "hd64": si.llama_desc(2, 128, 2, 160, 211, 320),
    "hd64_one_slice": si.llama_desc(1, 192, 3, 48, 1001, 320),
    "hd128": si.llama_desc(1, 256, 2, 512, 500, 320),
    "opt": si.opt_desc(2, 128, 2, 256, 203, 320),
}


def _context(name, n, s, longest):
    from oracle import oracle as om
    from paper_2310_18813_amd import binding as B
    desc = DESCS[name]
    ot, _, gt, _ = build_pair(om.Oracle("f64"), desc, None, "fp32", 17, DEV, random_norms=True)
    return ot, B.Context(desc, gt, None, None, "fp32", n, s, longest + s + 8, 4, B.PROPOSALS_EXTERNAL, DEV), desc


@pytest.mark.parametrize("name", list(DESCS))
@pytest.mark.parametrize("n,s,longest", [(1, 0, 1), (3, 4, 17), (8, 7, 129), (5, 15, 145), (16, 8, 40)])
def test_verification_logits(name, n, s, longest):
    ot, ctx, desc = _context(name, n, s, longest)
    rng = np.random.default_rng(n * 100 + longest)
    V = desc["vocab"]
    prompts = [rng.integers(0, V, size=max(1, longest - 3 * b)).astype(np.int32) for b in range(n)]
    table = rng.integers(0, V, size=(n, ctx.L_max), dtype=np.int32)
    ctx.spec_set_proposal_table(table)
    ctx.spec_reset_ragged([torch.from_numpy(p) for p in prompts])
    got = ctx.spec_verify_step(s, want_logits=True).cpu().numpy()
    for b in sorted({0, n // 2, n - 1}):
        m = len(prompts[b])
        seq = list(prompts[b]) + list(table[b, m:m + s])
        want = ot.forward(ot.cache(len(seq)), seq, 0)[m - 1:]
        assert np.abs(got[b] - want).max() <= LOGIT_TOL["fp32"], b


def test_a_later_row_that_is_not_finite_leaves_the_rows_before_it_alone():
    """Keys and values behind a row's position do not reach it, infinite and NaN ones (weight zero) included."""
    from paper_2310_18813_amd import binding as B
    desc = DESCS["hd64"]
    w = si.make_weights(desc, "fp32", 3, device=DEV, tag="tgt.")
    w["tok_emb"][7] = float("inf")
    prompt = np.arange(8, 30, dtype=np.int32)
    rows = []
    for last in (9, 7):
        ctx = B.Context(desc, w, None, None, "fp32", 1, 3, 64, 4, B.PROPOSALS_EXTERNAL, DEV)
        table = np.full((1, ctx.L_max), 5, dtype=np.int32)
        table[0, len(prompt) + 2] = last
        ctx.spec_set_proposal_table(table)
        ctx.spec_reset_ragged([torch.from_numpy(prompt)])
        rows.append(ctx.spec_verify_step(3, want_logits=True)[0].cpu().numpy().copy())
    assert np.array_equal(rows[0][:3], rows[1][:3])
    assert np.isfinite(rows[0]).all() and not np.isfinite(rows[1][3]).any()


@pytest.mark.parametrize("d,heads,ffn", [(128, 2, 416), (320, 5, 1232), (640, 10, 1024), (1024, 16, 4096)])
def test_a_row_alone_has_the_bits_of_the_row_among_many(d, heads, ffn):
    """One row's products keep more steps of a k-slice under way than those of many rows do (slices of 1 to 77 steps here, odd
    ones among them): the same sums, for batches on either side of the row counts where that changes."""
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(2, d, heads, ffn, 700, 128)
    w = si.make_weights(desc, "fp32", 5, device=DEV, tag="tgt.")
    prompt = si.make_prompts(1, 21, 700, 7)
    got = {}
    for n in (1, 5, 17, 40, 130):
        ctx = B.Context(desc, w, None, None, "fp32", n, 0, 64, 8, B.PROPOSALS_EXTERNAL, DEV)
        ctx.spec_reset(np.repeat(prompt, n, 0))
        got[n] = ctx.spec_verify_step(0, want_logits=True).reshape(n, 700).cpu()
        ctx.close()
    for n, rows in got.items():
        assert torch.equal(rows, got[1].expand(n, 700)), n
