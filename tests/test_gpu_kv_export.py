"""The export of cached rows by eight channels and eight positions against the one by elements, which buffers that are not
aligned to 16 bytes take: the same bits, at lengths around a block of positions, for heads of 64, 80 and 128, with as many
sequences as the export by blocks needs; and that short exports go by elements."""
import ctypes as C

import pytest
import torch

import synth_inputs as si
from launches import launched_kernels

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BLOCKS_FROM = 3 << 18   # elements


def _export(B, ctx, n, length, buf, off):
    """A call that exports layer 1 to the parts of buf that start `off` elements behind a 16-byte boundary."""
    size = n * length * ctx.tgt_desc["d_model"]
    k, v = (buf[i, off:off + size] for i in range(2))

    def call():
        B._check(B.lib.spec_kv_export(ctx.h, B.MODEL_TARGET, 1, n, length, C.c_void_p(k.data_ptr()), C.c_void_p(v.data_ptr())), ctx.h)
    return call, k.view(torch.int16), v.view(torch.int16)


@pytest.mark.parametrize("length", [1, 7, 8, 9, 33])
@pytest.mark.parametrize("d,heads", [(256, 4), (256, 2), (320, 4)])
def test_export_by_blocks_is_the_export_by_elements(d, heads, length):
    from paper_2310_18813_amd import binding as B
    desc = si.llama_desc(2, d, heads, 2 * d, 300, 256)
    w = si.make_weights(desc, "bf16", 3, device=DEV, tag="tgt.")
    n = -(-BLOCKS_FROM // (length * d))
    room = torch.zeros((4, n * length * d + 64), dtype=torch.bfloat16, device=DEV)
    prompts = torch.from_numpy(si.make_prompts(n, length + 1, 300, 3)).to(DEV)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    ctx = B.Context(desc, w, None, None, "bf16", n, 0, length + 8, 4, B.PROPOSALS_EXTERNAL, DEV, stream)
    ctx.spec_reset(prompts)
    by_blocks, k, v = _export(B, ctx, n, length, room[:2], 0)
    by_elements, ke, ve = _export(B, ctx, n, length, room[2:], 1)  # two bytes off
    short, _, _ = _export(B, ctx, n - 1, length, room[:2], 0)
    for call, kernel in ((by_blocks, "k_kv_export16"), (by_elements, "k_kv_convert"), (short, "k_kv_convert")):
        names = [name for name, _, _ in launched_kernels(B.lib, stream, call)]
        assert len(names) == 1 and kernel in names[0], names
    by_blocks()
    by_elements()
    torch.cuda.synchronize()
    assert torch.equal(k, ke) and torch.equal(v, ve)
    assert k.count_nonzero() > 0 and v.count_nonzero() > 0
    ctx.close()
