"""The choice between the streaming and the tiled kernel: at the sizes where the two are furthest apart, the automatic
choice takes no more than 1.15 of the time of a tiled launch that suits the size (least of interleaved launches, HIP
events around each; the streaming kernel takes 1.2 to 1.8 of it there)."""
import pytest
import torch

import synth_inputs as si
from launches import launched_kernels, template_ints

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# width, heads, feed-forward width, vocabulary, rows, the tile to compare with, the product
SIZES = [(768, 12, 1536, 32000, 48, (1, 4), "gemm_head"), (2048, 16, 4096, 32000, 48, (1, 4), "gemm_head"),
         (2048, 16, 4096, 32000, 112, (2, 4), "gemm_head"), (4096, 32, 8192, 8192, 80, (1, 2), "gemm_head"),
         (1024, 16, 4096, 1000, 256, (1, 4), "gemm_ffn_in"), (768, 12, 3072, 1000, 192, (1, 4), "gemm_ffn_in")]


@pytest.mark.parametrize("d,heads,ffn,vocab,rows,tile,product", SIZES)
def test_the_automatic_choice_is_not_the_slow_kernel(d, heads, ffn, vocab, rows, tile, product):
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(1, d, heads, ffn, vocab, 256)
    w = si.make_weights(desc, "bf16", 3, device=DEV, tag="tgt.")
    ctx = B.Context(desc, w, None, None, "bf16", rows, 0, 256, 80, B.PROPOSALS_EXTERNAL, DEV)
    ctx.spec_reset_noprefill(si.make_prompts(rows, 65, vocab, 3))
    best = {}
    for rep in range(30):
        for shape in ((0, 0), tile):
            ctx.spec_set_gemm_tuning(*shape)
            ctx.spec_kernel_timing(True)
            ctx.spec_round(0, 1)
            n, ms = ctx.spec_read_kernel_timing()[product]
            ctx.spec_kernel_timing(False)
            if rep:
                best[shape] = min(best.get(shape, 1e9), ms / n)
    ctx.close()
    assert best[(0, 0)] <= 1.15 * best[tile], best


@pytest.mark.parametrize("d,heads,ffn,rows,product", [(1024, 16, 4096, 224, "gate-up"), (512, 8, 1024, 192, "gate-up"), (2048, 16, 5504, 80, "qkv"),
                                                        (2560, 20, 5120, 64, "gate-up"), (3072, 24, 6144, 64, "qkv"), (3072, 24, 6144, 64, "gate-up"),
                                                        (5120, 40, 5120, 64, "gate-up")])
def test_short_products_are_tiled_and_take_their_row_sums_in_the_loop(d, heads, ffn, rows, product):
    """With larger wave tiles and k_row_inv_x in front, or streaming, these took 1.07 to 1.4 times as long."""
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(1, d, heads, ffn, 500, 64)
    w = si.make_weights(desc, "bf16", 3, device=DEV, tag="tgt.")
    n, s = rows // 16, 15
    prompts = torch.randint(0, 500, (n, 2), dtype=torch.int32, device=DEV)
    table = torch.randint(0, 500, (n, 48), dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    ctx = B.Context(desc, w, None, None, "bf16", n, s, 48, 16, B.PROPOSALS_EXTERNAL, DEV, stream)
    ctx.spec_set_proposal_table(table)
    ctx.spec_reset(prompts)
    names = [name for name, _, _ in launched_kernels(B.lib, stream, lambda: ctx.spec_verify_step(s))]
    torch.cuda.synchronize()
    ctx.close()
    products = [i for i, name in enumerate(names) if "k_gemm" in name]
    at = products[{"qkv": 0, "gate-up": 2}[product]]
    assert len(products) == 5 and "k_gemm_tile" in names[at] and template_ints(names[at])[0] == 1 and "k_row_inv_x" not in names[at - 1], names
