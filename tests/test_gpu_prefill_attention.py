"""Prefill attention with four row groups to a workgroup, cache rows through LDS, against one wave per (group, head) (a pinned
launch shape): the same bits in every cached row and logit, for workgroups that hold groups of one, two, three and four
sequences and a last one that is not full, groups of 16 and of 8 rows, chunks that end at 128, 512 and 768.  And that it is taken
only where the groups of a workgroup share cache rows."""
import math

import pytest
import torch

import synth_inputs as si
from launches import launched_kernels

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# groups of 16; groups of 8 (they leave clearly fewer dead rows)
MIXED = [801, 33, 129, 5, 513, 17, 18, 260, 2, 128, 770, 64, 385, 700, 640, 130, 257, 515, 20, 300]
SHORT = [9] * 40 + [1000, 7, 1001, 3, 2] + [9] * 30 + [900, 3]


def _groups(lengths):
    """-> rows of a group, and the last position and the sequence of every group, as a prefill cuts them."""
    rows16, rows8 = (sum(-(-(m - 1) // q) * q for m in lengths) for q in (16, 8))
    q = 8 if 8 * rows8 < 7 * rows16 else 16
    return q, [(b, min((i + 1) * q - 1, m - 2)) for b, m in enumerate(lengths) for i in range(-(-(m - 1) // q))]


def _expected(lengths, heads, hd, n_cu):
    """Whether the automatic choice takes the kernel: pairs enough for a wave per (group, head) in well filled rounds, and
    cache rows that a workgroup's groups share."""
    q, groups = _groups(lengths)
    pairs, slots = len(groups) * heads, 4 * n_cu
    rounds = -(-pairs // slots)
    longest = max(last for _, last in groups)
    chunks = 1 + (longest // 128 if longest < 512 else 4 + (longest - 512) // 256)
    assert 1 < chunks <= 8
    own = sum(last // 32 + 1 for _, last in groups)
    shared = 0
    for i in range(0, len(groups), 4):
        steps = dict(groups[i:i + 4])  # the last group of each sequence
        shared += sum(last // 32 + 1 + 2 for last in steps.values())
    enough = (1.5 if rounds > 1 else 3.0) if hd == 128 else (2.5 if rounds > 1 else math.inf)
    return pairs >= 768 and (rounds == 1 or pairs >= 0.85 * rounds * slots) and own >= enough * shared


def _context(B, d, heads, opt, lengths, stream=None):
    dtype = "fp16" if opt else "bf16"
    desc = si.opt_desc(2, d, heads, 2 * d, 500, 1152) if opt else si.llama_desc(2, d, heads, 2 * d, 500, 1152)
    w = si.make_weights(desc, dtype, 5, device=DEV, tag="tgt.")
    torch.cuda.synchronize()
    return B.Context(desc, w, None, None, dtype, len(lengths), 0, 1088, 40, B.PROPOSALS_EXTERNAL, DEV, stream)


@pytest.mark.parametrize("d,heads,opt", [(1024, 16, False), (1024, 8, False), (1024, 16, True), (1024, 8, True)])
@pytest.mark.parametrize("lengths,rows", [(MIXED, 16), (SHORT, 8)])
def test_prefill_shapes_give_identical_bits(d, heads, opt, lengths, rows):
    from paper_2310_18813_amd import binding as B
    n, hd = len(lengths), d // heads
    q, groups = _groups(lengths)
    assert q == rows and len(groups) % 4 and _expected(lengths, heads, hd, torch.cuda.get_device_properties(0).multi_processor_count)
    prompts = [torch.from_numpy(si.make_prompts(1, m, 500, 40 + i)[0]) for i, m in enumerate(lengths)]
    ctx = _context(B, d, heads, opt, lengths)
    got = []
    for shape in (0, 2):
        ctx.spec_set_attention_shape(shape)
        ctx.spec_reset_ragged(prompts)
        k, v = ctx.spec_kv_export(B.MODEL_TARGET, 1, n, max(lengths) - 1)
        ctx.spec_set_attention_shape(0)
        logits = ctx.spec_verify_step(0, want_logits=True).clone()
        ctx.spec_accept_commit(0)
        got.append((k.clone(), v.clone(), logits))
    ctx.close()
    for i, m in enumerate(lengths):
        for a, b in zip(got[0][:2], got[1][:2]):
            assert torch.equal(a[i, :m - 1], b[i, :m - 1]), (i, m)
    assert torch.equal(got[0][2], got[1][2])


@pytest.mark.parametrize("d,heads,n,length,taken", [(1024, 16, 16, 513, True), (1024, 16, 48, 130, False), (1024, 16, 1, 777, False),
                                                    (2048, 16, 16, 513, True), (2048, 16, 48, 130, True), (4096, 32, 1, 500, True)])
def test_the_kernel_is_taken_where_groups_share_cache_rows(d, heads, n, length, taken):
    """Equal prompts in one pass; heads of 64 and of 128."""
    from paper_2310_18813_amd import binding as B
    assert taken == _expected([length] * n, heads, d // heads, torch.cuda.get_device_properties(0).multi_processor_count)
    stream = torch.cuda.Stream()
    ctx = _context(B, d, heads, False, [length] * n, stream)
    prompts = torch.from_numpy(si.make_prompts(n, length, 500, 3)).to(DEV)
    torch.cuda.synchronize()
    ctx.spec_reset(prompts)
    names = [name for name, _, _ in launched_kernels(B.lib, stream, lambda: ctx.spec_reset(prompts)) if "k_attn" in name]
    torch.cuda.synchronize()
    ctx.close()
    assert len(names) == 2 and all(("k_attn_prefill" in name) == taken for name in names), names


@pytest.mark.parametrize("d,heads", [(2048, 16), (1024, 16)])
def test_short_prompts_beside_a_long_one_are_not_slowed_down(d, heads):
    """200 prompts of 9 tokens and one of 200 (groups of different sequences in most workgroups): 1.4 times as long through LDS."""
    from paper_2310_18813_amd import binding as B
    lengths = [200] + [9] * 200
    prompts = [torch.from_numpy(si.make_prompts(1, m, 500, 40 + i)[0]) for i, m in enumerate(lengths)]
    ctx = _context(B, d, heads, False, lengths)
    best = {}
    for rep in range(12):
        for shape in (0, 2):
            ctx.spec_set_attention_shape(shape)
            ctx.spec_kernel_timing(True)
            ctx.spec_reset_ragged(prompts)
            ms = ctx.spec_read_kernel_timing()["attention"][1]
            ctx.spec_kernel_timing(False)
            best[shape] = min(best.get(shape, 1e9), ms)
    ctx.close()
    assert best[0] <= 1.15 * best[2], best
