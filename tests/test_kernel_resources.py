"""The matrix-core kernels (attention, products) keep everything in registers: read from the metadata of the built library's own
code objects.  A spilled register is reloaded inside the tile loop, where the reload waits for every tile load in flight."""
import struct

import paper_2506_06472_amd as tio
from paper_2506_06472_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + name].decode()
            p += 24 + name
            if "gfx950" in triple and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def _kernels(obj):
    """The kernel descriptions in the note section of a code object (note type 32: msgpack)."""
    import msgpack
    shoff, shentsize, shnum = struct.unpack_from("<Q", obj, 0x28)[0], *struct.unpack_from("<HH", obj, 0x3A)
    for i in range(shnum):
        kind, _, _, off, size = struct.unpack_from("<IQQQQ", obj, shoff + i * shentsize + 4)
        end = off + size
        while kind == 7 and off < end:
            nlen, dlen, ntype = struct.unpack_from("<III", obj, off)
            desc = off + 12 + (nlen + 3) // 4 * 4
            if ntype == 32:
                yield from msgpack.unpackb(obj[desc:desc + dlen])["amdhsa.kernels"]
            off = desc + (dlen + 3) // 4 * 4


def test_matrix_core_kernels_do_not_spill():
    tio.binding.lib()
    with open(build.LIB, "rb") as f:
        blob = f.read()
    found = {k[".name"]: k for obj in _code_objects(blob) for k in _kernels(obj)}
    mfma = {n: k for n, k in found.items() if "attn_" in n or "gemm_" in n}
    for family in ("attn_fwd_mfma_k", "attn_bwd_dq_mfma_k", "attn_bwd_dkv_mfma_k", "gemm_bf16_dl_k", "gemm_f32_mfma_k"):
        assert any(family in n for n in mfma), family
    spilled = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in mfma.items()
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled, spilled
