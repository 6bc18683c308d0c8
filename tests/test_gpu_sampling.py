"""Speculative sampling (the non-greedy acceptance rule that Sec. 2 cites) on the GPU against the numpy oracle,
through the C ABI.

The GPU decides in fp32, the oracle in fp64, and a decision is an integer: where the oracle reports that the random
number fell within MARGIN of a decision boundary, either outcome is legitimate and that row or sequence is left out
of the comparison (and counted: the share must stay tiny).  Everything else must agree exactly.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import synth_inputs as si
from helpers import build_pair, truth_table
from launches import launched_kernels, template_ints
from oracle import sampling as osm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
MARGIN = 1e-5   # fp32 sums over a vocabulary, added chunk by chunk: the cumulative weights are good to about 1e-6 of the total


@pytest.fixture(scope="module")
def B():
    from paper_2310_18813_amd import binding
    return binding


@pytest.mark.parametrize("V,T", [(32000, 0.7), (32000, 1.3), (50272, 1.0), (1003, 0.9), (37, 1.0), (5, 2.0)])
def test_token_draws_match_the_oracle(B, V, T):
    rng = np.random.default_rng(V)
    rows = 48
    z = _peaky(rng, (rows, V))
    u = rng.random(rows).astype(np.float32)
    u[0], u[1] = 0.0, np.float32(1.0 - 2 ** -24)      # the ends of the range
    got = B.spec_sample_tokens(torch.from_numpy(z).to(DEV), torch.from_numpy(u).to(DEV), T).cpu().numpy()
    skipped = 0
    for r in range(rows):
        tok, margin = osm.sample_token(z[r], T, float(u[r]))
        if margin < MARGIN:
            skipped += 1
            continue
        assert got[r] == tok, (r, got[r], tok, margin)
    assert skipped <= 4


def _peaky(rng, shape):
    """Logits with the shape of a language model's: a broad bulk and a few tokens far above it that carry the mass
    (with a flat distribution over 32000 tokens most draws land within rounding of a boundary and say nothing)."""
    z = rng.normal(size=shape) * 2.0
    z += (rng.random(shape) < 24.0 / shape[-1]) * rng.uniform(8.0, 14.0, size=shape)
    return z.astype(np.float32)


def _round_inputs(rng, nB, s, V, point_mass, T):
    tl = _peaky(rng, (nB, s + 1, V))
    u = rng.random((nB, s + 1, 3)).astype(np.float32)
    if point_mass:
        dl = None
        props = np.where(rng.random((nB, s)) < 0.6, tl[:, :s].argmax(-1), rng.integers(V, size=(nB, s))).astype(np.int32)
    else:
        # a draft near the target, so that keeping and rejecting both happen; step-major as the entry point wants it
        dl = (tl[:, :s] + rng.normal(size=(nB, s, V)) * 1.2).astype(np.float32).transpose(1, 0, 2).copy()
        props = np.array([[osm.sample_token(dl[j, b], T, float(u[b, j, 0]))[0] for j in range(s)] for b in range(nB)],
                         dtype=np.int32).reshape(nB, s)
    return tl, dl, props, u


@pytest.mark.parametrize("V", [32000, 1003])
@pytest.mark.parametrize("s", [0, 1, 4, 8])
@pytest.mark.parametrize("point_mass", [False, True])
def test_acceptance_rule_matches_the_oracle(B, V, s, point_mass):
    rng = np.random.default_rng(1000 * s + V + point_mass)
    nB, T = 40, 0.9
    tl, dl, props, u = _round_inputs(rng, nB, s, V, point_mass, T)
    dev = lambda a: None if a is None else torch.from_numpy(a).to(DEV)
    chosen, acc, em = B.spec_sample_accept(dev(tl), dev(dl) if s else None, dev(props) if s else None, dev(u), T)
    chosen, acc, em = chosen.cpu().numpy(), acc.cpu().numpy(), em.cpu().numpy()
    skipped, ls = 0, []
    for b in range(nB):
        l, emitted, margin = osm.spec_sample_round(tl[b], None if dl is None else dl[:, b], props[b], u[b, :s, 1], u[b, :, 2], T)
        if margin < MARGIN:
            skipped += 1
            continue
        ls.append(l)
        assert acc[b] == l, (b, acc[b], l, margin)
        assert list(em[b, :l + 1]) == emitted and all(x == -1 for x in em[b, l + 1:]), (b, em[b], emitted)
        assert list(chosen[b, :l + 1]) == emitted
    assert skipped <= 4
    if s >= 4:
        assert 0 < np.mean(ls) < s, "the inputs should exercise both keeping and rejecting"


@pytest.mark.parametrize("V", [1, 5, 256, 260, 1024, 1028, 2048, 2052, 4095, 4100, 32772, 70001])
@pytest.mark.parametrize("offset", [0, 1])
def test_draws_and_rule_at_the_edges_of_steps_segments_and_alignment(B, V, offset):
    """Vocabularies around a wave's step (256), a segment per wave (4096), a register tile (32768) and beyond, rows that
    end inside a float4, and buffers that start 4 bytes off a 16-byte boundary; masked tokens, rows of NaN and of -inf."""
    rng = np.random.default_rng(V + offset)
    nB, s, T = 12, 3, 0.8
    tl, dl, props, u = _round_inputs(rng, nB, s, V, False, T)
    if V > 8:   # a masked prefix that covers whole steps: weight 0 in the target, so never emitted unless kept
        tl[0, :, :V // 2] = -np.inf

    def dev(a):
        buf = torch.empty(a.size + offset, dtype=torch.from_numpy(a).dtype, device=DEV)
        buf[offset:] = torch.from_numpy(a.ravel()).to(DEV)
        return buf[offset:].view(a.shape)

    skipped = 0
    for draft in (dl, None):
        chosen, acc, em = (x.cpu().numpy() for x in B.spec_sample_accept(dev(tl), None if draft is None else dev(draft),
                                                                         dev(props), dev(u), T))
        for b in range(nB):
            l, emitted, margin = osm.spec_sample_round(tl[b], None if draft is None else draft[:, b], props[b], u[b, :s, 1],
                                                       u[b, :, 2], T)
            if margin < MARGIN:
                skipped += 1
                continue
            want = emitted + [-1] * (s - l)
            assert acc[b] == l and list(em[b]) == want and list(chosen[b]) == want, (b, draft is None, chosen[b], emitted, margin)
    assert skipped <= 3
    z = tl[:, 0].copy()
    z[1], z[2] = np.nan, -np.inf   # no distribution: the lowest index
    got = B.spec_sample_tokens(dev(z), dev(u[:, 0, 0].copy()), T).cpu().numpy()
    assert got[1] == 0 and got[2] == 0
    for b in [0] + list(range(3, nB)):
        tok, margin = osm.sample_token(z[b], T, float(u[b, 0, 0]))
        assert got[b] == tok or margin < MARGIN, (b, got[b], tok, margin)


@pytest.mark.parametrize("V", [5, 1003, 4100, 8192, 8200, 32000, 50272, 70001])
@pytest.mark.parametrize("T", [1e30, float(np.finfo(np.float32).max), float("inf")])
def test_very_large_and_infinite_temperatures_draw_uniformly(B, V, T):
    """1 / T so small that every finite logit has a weight of 1 in fp32 (sums of ones are exact), masked tokens none; rows that do
    not fill their last step group.  The uniform numbers lie in the middle of a token's share, half a share from either
    boundary: several thousand times what rounding u * V moves it by."""
    rng = np.random.default_rng(V)
    rows, lo = 16, V // 3
    z = (rng.normal(size=(rows, V)) * 4.0).astype(np.float32)
    z[1::2, :lo] = -np.inf                                        # odd rows: a masked prefix
    first = np.where(np.arange(rows) % 2, lo, 0)
    want = np.concatenate([first[:2], np.full(2, V - 1), rng.integers(first[4:], V)])
    u = ((want - first + 0.5) / (V - first)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    assert B.spec_sample_tokens(dev(z), dev(u), T).cpu().tolist() == want.tolist()
    # the rule, a round of one proposal per row: a point mass is kept below 1 / V and replaced otherwise
    zz = np.stack([z, z], axis=1)                                 # [rows][2][V]
    props = np.full((rows, 1), V - 1, dtype=np.int32)
    un = np.zeros((rows, 2, 3), dtype=np.float32)
    un[:, 0, 1], un[:, 1, 2] = 0.5 / V, u                         # kept, then the bonus draw
    _, acc, em = (x.cpu().numpy() for x in B.spec_sample_accept(dev(zz), None, dev(props), dev(un), T))
    assert acc.tolist() == [1] * rows and em[:, 0].tolist() == [V - 1] * rows and em[:, 1].tolist() == want.tolist()
    props[:, 0] = first                                           # the residual is every live token but the first
    un[:, 0, 1] = 2.0 / (V - first)
    got = np.maximum(want, first + 1)
    un[:, 0, 2] = (got - first - 1 + 0.5) / (V - first - 1)
    _, acc, em = (x.cpu().numpy() for x in B.spec_sample_accept(dev(zz), None, dev(props), dev(un), T))
    assert acc.tolist() == [0] * rows and em[:, 0].tolist() == got.tolist()
    # a draft without the mask: its masked proposals are rejected, and the residual is uniform over the live tokens
    odd = np.arange(1, rows, 2)
    q = np.where(np.isinf(z[odd]), np.float32(0.0), z[odd])
    un[odd, 0, 1], un[odd, 0, 2] = 0.5, u[odd]
    _, acc, em = (x.cpu().numpy() for x in B.spec_sample_accept(dev(zz[odd]), dev(q[None]), dev(np.zeros((len(odd), 1), np.int32)), dev(un[odd]), T))
    assert acc.tolist() == [0] * len(odd) and em[:, 0].tolist() == want[odd].tolist()


@pytest.mark.parametrize("V,steps", [(256, 1), (1024, 1), (1028, 2), (2048, 2), (2052, 4), (8192, 4), (8196, 8), (1003, 1), (2047, 2), (8191, 2)])
def test_a_wave_loads_no_more_steps_than_its_segment_has(B, V, steps):
    """Rows of up to 1024 logits are one step a wave: with four in flight a draw took 1.08 of the time of the loop before it."""
    z, u, out = torch.zeros((3, V), device=DEV), torch.zeros(3, device=DEV), torch.zeros(3, dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    stream, p = torch.cuda.Stream(), lambda x: C.c_void_p(x.data_ptr())
    kernels = launched_kernels(B.lib, stream, lambda: B.lib.spec_sample_tokens(C.c_void_p(stream.cuda_stream), p(z), 3, V, C.c_float(1.0), p(u), p(out)))
    (name, _, threads), = kernels
    waves, loads = template_ints(name)[:2]
    assert threads == 64 * waves == (256 if V <= 8192 else 1024) and loads >> 1 == steps and (loads & 1) == (V % 4 == 0), name


def _on_device_round(nB, s, V, sigma, seed, T):
    """Peaked target rows, a draft `sigma` away from them, proposals drawn from the draft, uniform numbers."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    tl = torch.empty((nB, s + 1, V), device=DEV).normal_(0.0, 3.0, generator=g)
    dl = (tl[:, :s].transpose(0, 1) + sigma * torch.empty((s, nB, V), device=DEV).normal_(generator=g)).contiguous()
    gum = torch.empty((s, nB, V), device=DEV).exponential_(generator=g).log_().neg_()
    props = (dl / T + gum).argmax(-1).transpose(0, 1).to(torch.int32).contiguous()
    return tl, dl, props, torch.rand((nB, s + 1, 3), device=DEV, generator=g)


@pytest.mark.parametrize("nB,s,V", [(257, 1, 8196), (300, 5, 9001), (130, 15, 8448), (1025, 3, 1000), (600, 8, 1003), (300, 6, 8192)])
@pytest.mark.parametrize("sigma", [0.0, 1.0, 3.0])
def test_rounds_too_large_for_a_workgroup_per_place_are_the_sum_of_small_ones(B, nB, s, V, sigma):
    """Large rounds decide several places per workgroup in turn, small ones a place per workgroup: same bits for a
    sequence either way, whether its proposals are all kept, some or none; vocabularies on both sides of the change of
    the workgroup's size."""
    T = 0.9
    tl, dl, props, u = _on_device_round(nB, s, V, sigma, nB + s, T)
    if sigma == 3.0:
        props = (props + 1) % V   # mostly rejected at the first place
    for draft in (dl, None):
        whole = B.spec_sample_accept(tl, draft, props, u, T)
        for i in range(0, nB, 14):   # 14 * 16 places: a workgroup each
            part = B.spec_sample_accept(tl[i:i + 14].contiguous(), None if draft is None else draft[:, i:i + 14].contiguous(),
                                        props[i:i + 14].contiguous(), u[i:i + 14].contiguous(), T)
            for w, p in zip(whole, part):
                assert torch.equal(w[i:i + 14], p), (i, draft is None)


def test_a_large_round_does_not_pay_for_places_behind_the_first_rejection(B):
    """512 sequences x 9 places of 16000 logits: when every round ends at its first place, one place in nine is needed.
    A workgroup per place would take about as long as with every proposal kept (ratio 0.9 to 1.1); in turn 0.15 to 0.3."""
    nB, s, V, T = 512, 8, 16000, 0.8
    tl, _, _, u = _on_device_round(nB, s, V, 1.0, 3, T)
    best = tl[:, :s].argmax(-1).to(torch.int32)
    tl[:, :s].scatter_(2, best.long()[..., None], 60.0)   # the arg-max has probability 1: kept whatever u is
    ms = {}
    for name, props in (("kept", best.contiguous()), ("rejected", ((best + 1) % V).contiguous())):
        run = lambda: B.spec_sample_accept(tl, None, props, u, T)
        assert run()[1].unique().tolist() == [s if name == "kept" else 0]
        times = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                run()
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        ms[name] = min(times)
    assert ms["rejected"] < 0.6 * ms["kept"], ms


def test_identical_draft_keeps_everything_and_bad_arguments_are_refused(B):
    rng = np.random.default_rng(5)
    nB, s, V, T = 16, 5, 2048, 1.1
    tl = (rng.normal(size=(nB, s + 1, V)) * 2).astype(np.float32)
    dl = tl[:, :s].transpose(1, 0, 2).copy()
    u = rng.random((nB, s + 1, 3)).astype(np.float32)
    props = np.array([[osm.sample_token(dl[j, b], T, float(u[b, j, 0]))[0] for j in range(s)] for b in range(nB)], dtype=np.int32)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    _, acc, em = B.spec_sample_accept(dev(tl), dev(dl), dev(props), dev(u), T)
    assert acc.cpu().tolist() == [s] * nB          # p = q bit for bit: the ratio is 1, every u < 1 keeps
    assert np.array_equal(em.cpu().numpy()[:, :s], props)
    with pytest.raises(B.SpecError):
        B.spec_sample_accept(dev(tl), dev(dl), dev(props), dev(u), 0.0)
    with pytest.raises(B.SpecError):
        B.spec_sample_tokens(dev(tl[:, 0]), dev(u[:, 0, 0].copy()), -1.0)


PAIRS = {
    "tiny_fp32": ("fp32", 1000, si.CONFIGS["tiny_fp32"][2], si.CONFIGS["tiny_fp32"][3]),
    "small_bf16": ("bf16", 77, si.llama_desc(2, 256, 2, 416, 1000, 128), si.llama_desc(1, 128, 2, 160, 1000, 128)),
}


def _context(B, name, mode, nB, P, N, s_max, twin=False):
    from oracle import oracle as om
    dtype, seed, tdesc, ddesc = PAIRS[name]
    L_max = P + N + s_max + 3
    tdesc = dict(tdesc, max_pos=max(L_max, tdesc["max_pos"]))
    ddesc = dict(tdesc) if twin else dict(ddesc, max_pos=max(L_max, ddesc["max_pos"]))
    ot, od, gt, gd = build_pair(om.Oracle("f64"), tdesc, ddesc, dtype, seed, DEV, random_norms=True, emb_std=1.0)
    if twin:
        gd = gt
    ctx = B.Context(tdesc, gt, ddesc, gd, dtype, nB, s_max, L_max, N, mode, DEV)
    return ctx, si.make_prompts(nB, P, tdesc["vocab"], seed), L_max, tdesc["vocab"]


@pytest.mark.parametrize("name", list(PAIRS))
@pytest.mark.parametrize("mode", ["draft", "table", "draft_caps"])
def test_rounds_inside_a_context_follow_the_rule_on_their_own_logits(B, name, mode):
    """Sampling switched on in a context: every round's proposals, acceptance count and committed tokens must be
    what the oracle's rule gives on the logits the GPU itself produced in that round (the library leaves them in the
    caller's buffers) and the caller's table of uniform numbers, indexed by sequence and absolute position.  This
    checks the wiring -- which random number decides which token, which draft step's logits meet which target row,
    the hand-over to the commit step -- independently of the models' numerics."""
    nB, P, N, s_max = 5, 9, 40, 4
    T = 0.9 if mode != "table" else 0.2
    ctx, prompts, L_max, V = _context(B, name, B.PROPOSALS_DRAFT if mode != "table" else B.PROPOSALS_EXTERNAL, nB, P, N, s_max)
    rng = np.random.default_rng(3)
    u = rng.random((nB, L_max, 3)).astype(np.float32)
    ctx.spec_reset(prompts)
    if mode == "table":
        # the table holds the target's greedy continuation: at a low temperature the sampled sequences follow it for
        # a while, so proposals are kept as well as rejected
        ctx.spec_round(0, N)
        greedy, _ = ctx.spec_read_output()
        ctx.spec_set_proposal_table(truth_table(np.array(greedy), P, L_max))
        ctx.spec_reset(prompts)
    caps = None
    if mode == "draft_caps":   # a speculation length per sequence: the bonus draw moves to row s_b
        mode, caps = "draft", [0, 1, 2, 3, 4]
        ctx.spec_set_seq_s(caps)
    tl, dl = ctx.spec_set_sampling(T, torch.from_numpy(u).to(DEV))
    skipped, ls, checked = 0, [], 0
    for rnd, s in enumerate([3, 4, 1, 0, 2, 4, 3, 3]):
        n0 = list(ctx.spec_read_state()[0])
        out0, _ = ctx.spec_read_output()
        ctx.spec_round(s, 1)
        n1, _, l_last, _ = ctx.spec_read_state()
        out1, _ = ctx.spec_read_output()
        props = ctx.spec_read_proposals()
        tln = tl[:nB * (s + 1)].view(nB, s + 1, V).cpu().numpy()
        dln = dl.cpu().numpy() if mode == "draft" else None
        s_round = s
        for b in range(nB):
            s = min(s_round, caps[b]) if caps else s_round
            ub = u[b, n0[b]:n0[b] + s + 1]
            margin = 1.0
            if mode == "draft":
                for j in range(s):
                    tok, m = osm.sample_token(dln[j, b], T, float(ub[j, 0]))
                    margin = min(margin, m)
                    if margin >= MARGIN:
                        assert props[b][j] == tok, (rnd, b, j)
            l, emitted, m = osm.spec_sample_round(tln[b][:s + 1], None if dln is None else dln[:s, b], props[b][:s], ub[:s, 1],
                                                  ub[:, 2], T)
            if min(margin, m) < MARGIN:
                skipped += 1
                continue
            checked += 1
            ls.append(l / max(1, s))
            assert l_last[b] == l and n1[b] - n0[b] == l + 1, (rnd, b, l_last[b], l, n1[b] - n0[b])
            assert out1[b][len(out0[b]):] == emitted, (rnd, b)
    assert skipped <= 3 and checked >= 30
    assert 0.0 < np.mean(ls) < 1.0, "the rounds should exercise both keeping and rejecting"
    # back to the greedy rule: the next round's tokens are the arg-max of their rows again
    ctx.spec_set_sampling(0.0, None)
    if caps:
        ctx.spec_set_seq_s(None)
    lg = None
    out0, _ = ctx.spec_read_output()
    if mode == "draft":
        for j in range(1, 3):
            ctx.spec_draft_step(j)
    lg = ctx.spec_verify_step(2, want_logits=True).cpu().numpy()
    a = ctx.spec_read_state()[3]
    assert [list(r[:3]) for r in a] == [list(lg[b].argmax(-1)) for b in range(nB)]
    ctx.spec_accept_commit(2)
    ctx.close()


@pytest.mark.parametrize("mode", ["draft", "table"])
def test_a_large_batch_with_caps_samples_what_a_small_one_does(B, mode):
    """300 sequences that repeat five, with a speculation length each: more places than workgroups, so they are decided
    in turn; every sequence must emit what it emits in a batch of five."""
    P, N, s_max, T, caps = 9, 24, 4, 0.9, [0, 1, 2, 3, 4]
    outs = []
    for nB in (5, 300):
        ctx, prompts, L_max, V = _context(B, "tiny_fp32", B.PROPOSALS_DRAFT if mode == "draft" else B.PROPOSALS_EXTERNAL, nB, P, N, s_max)
        rep = nB // 5
        rng = np.random.default_rng(6)
        u, table = rng.random((5, L_max, 3)).astype(np.float32), rng.integers(V, size=(5, L_max), dtype=np.int32)
        if mode == "table":
            ctx.spec_set_proposal_table(np.tile(table, (rep, 1)))
        ctx.spec_reset(np.tile(np.asarray(prompts)[:5], (rep, 1)))
        ctx.spec_set_seq_s(caps * rep)
        ctx.spec_set_sampling(T, torch.from_numpy(np.tile(u, (rep, 1, 1))).to(DEV))
        for s in (3, 4, 1, 0, 2, 4):
            ctx.spec_round(s, 1)
        outs.append(ctx.spec_read_output()[0])
        ctx.close()
    small, large = outs
    assert any(len(t) > 6 for t in small) or mode == "table"
    for b in range(300):
        assert list(large[b]) == list(small[b % 5]), b


@pytest.mark.parametrize("name", list(PAIRS))
def test_draft_equal_to_target_keeps_every_proposal_when_sampling(B, name):
    """The draft is the target: a row's bits do not depend on the pass it sits in, so q = p bit for bit, the ratio is
    1 and every proposal is kept whatever the random numbers -- any slip in which draft step's logits meet which
    target row would break it."""
    nB, P, N, s_max, T = 4, 8, 36, 5, 1.0
    ctx, prompts, L_max, V = _context(B, name, B.PROPOSALS_DRAFT, nB, P, N, s_max, twin=True)
    rng = np.random.default_rng(4)
    ctx.spec_reset(prompts)
    ctx.spec_set_sampling(T, torch.from_numpy(rng.random((nB, L_max, 3)).astype(np.float32)).to(DEV))
    for s in (5, 3, 4, 1, 5):
        ctx.spec_round(s, 1)
        assert list(ctx.spec_read_state()[2]) == [s] * nB
    ctx.close()
