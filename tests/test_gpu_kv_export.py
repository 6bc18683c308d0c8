"""The export of cached rows by eight channels and eight positions against the one by elements, which buffers that are not
aligned to 16 bytes take: the same bits, at lengths around a block of positions, for heads of 64, 80 and 128."""
import ctypes as C

import pytest
import torch

import synth_inputs as si

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("length", [1, 7, 8, 9, 33])
@pytest.mark.parametrize("d,heads", [(256, 4), (256, 2), (160, 2)])
def test_export_by_blocks_is_the_export_by_elements(d, heads, length):
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(2, d, heads, 2 * d, 300, 256)
    w = si.make_weights(desc, "bf16", 3, device=DEV, tag="tgt.")
    n = 3
    ctx = B.Context(desc, w, None, None, "bf16", n, 0, 96, 40, B.PROPOSALS_EXTERNAL, DEV)
    ctx.spec_reset(si.make_prompts(n, length + 1, 300, 3))
    k, v = ctx.spec_kv_export(B.MODEL_TARGET, 1, n, length)
    size = n * length * d
    room = torch.zeros((2, size + 64), dtype=torch.bfloat16, device=DEV)
    odd = [room[i, 1:1 + size] for i in range(2)]  # two bytes off
    B._check(B.lib.spec_kv_export(ctx.h, B.MODEL_TARGET, 1, n, length, C.c_void_p(odd[0].data_ptr()), C.c_void_p(odd[1].data_ptr())), ctx.h)
    torch.cuda.synchronize()
    assert torch.equal(k.flatten().view(torch.int16), odd[0].view(torch.int16)) and torch.equal(v.flatten().view(torch.int16), odd[1].view(torch.int16))
    assert k.abs().sum() > 0 and v.abs().sum() > 0
    ctx.close()
