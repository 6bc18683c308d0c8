"""What the compiler says each kernel of the built library uses (its metadata notes; no GPU): a kernel that takes more than
64 KB of LDS gets it only as dynamic LDS that the launch states and the set-up has asked for, and no kernel spills."""
import os
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2310_18813_amd", "libspecdec.so")
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _notes(blob, at, size):
    end = at + size
    while at < end:
        name, desc, kind = struct.unpack_from("<III", blob, at)
        body = at + 12 + (name + 3) // 4 * 4
        yield kind, blob[body:body + desc]
        at = body + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """name -> metadata of every kernel: the device ELFs embedded in the library."""
    blob, out, at = open(LIB, "rb").read(), {}, 0
    while (at := blob.find(b"\x7fELF\x02\x01", at)) >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == EM_AMDGPU:
            table = at + struct.unpack_from("<Q", blob, at + 40)[0]
            entry, count = struct.unpack_from("<HH", blob, at + 58)
            for i in range(count):
                if struct.unpack_from("<I", blob, table + i * entry + 4)[0] != SHT_NOTE:
                    continue
                offset, size = struct.unpack_from("<QQ", blob, table + i * entry + 24)
                for kind, desc in _notes(blob, at + offset, size):
                    if kind == NT_AMDGPU_METADATA:
                        out.update({k[".name"]: k for k in msgpack.unpackb(desc)["amdhsa.kernels"]})
        at += 4
    assert len(out) > 100
    return out


def test_kernels_whose_dynamic_lds_can_fill_64_kb_have_no_lds_besides(kernels):
    """Nor may the tiled products and the prefill attention have any: their loads straight to LDS count from its start."""
    products = {n: k for n, k in kernels.items() if any(x in n for x in ("k_gemm_f32", "k_gemm_tile", "k_gemm_strips", "k_attn_prefill", "k_attn_group"))}
    assert all(sum(x in n for n in products) >= 4 for x in ("k_gemm_f32", "k_gemm_tile", "k_gemm_strips", "k_attn_prefill", "k_attn_group"))
    assert {n: k[".group_segment_fixed_size"] for n, k in products.items() if k[".group_segment_fixed_size"]} == {}


def test_no_kernel_spills_or_has_more_static_lds_than_comes_unasked(kernels):
    assert [n for n, k in kernels.items() if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]] == []
    assert [n for n, k in kernels.items() if k[".group_segment_fixed_size"] > 64 * 1024] == []
