"""The built library's kernels against the register file: the kernels of the
default sweeps, and the launches of their own that replace them, keep every
value in registers (a spilled one costs a scratch store and load per thread)."""
import os
import re
import struct
import subprocess

import pytest

import paper_1611_06765_amd

LIB = os.path.join(os.path.dirname(paper_1611_06765_amd.__file__), "libccd.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _registers(tmp_path):
    """{kernel symbol: (vector registers, spilled ones)} of the gfx950 code in the library."""
    b = open(LIB, "rb").read()
    out, at = {}, b.find(MAGIC)
    while at >= 0:
        o = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", b, at + len(MAGIC))[0]):
            off, size, length = struct.unpack_from("<QQQ", b, o)
            triple = b[o + 24:o + 24 + length]
            o += 24 + length
            if size and triple.endswith(b"gfx950"):
                f = tmp_path / "code.elf"
                f.write_bytes(b[at + off:at + off + size])
                s = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
                names = re.findall(r"\.symbol:\s+(\S+)\.kd", s)
                used = re.findall(r"\.vgpr_count:\s+(\d+)", s)
                spilled = re.findall(r"\.vgpr_spill_count:\s+(\d+)", s)
                assert len(names) == len(used) == len(spilled)
                out.update(zip(names, zip(map(int, used), map(int, spilled))))
        at = b.find(MAGIC, at + 1)
    return out


needs_readelf = pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")


@needs_readelf
def test_sweep_kernels_do_not_spill(tmp_path):
    regs = _registers(tmp_path)
    for name in ("k_front", "k_mid", "k_mid64", "k_update", "k_direct", "k_live_lists", "k_nm_ring", "k_nm_mid",
                 "k_nm_update", "k_mlp_fwd", "k_mlp_grad", "k_warm", "k_dense_one"):
        found = {k: v for k, v in regs.items() if re.search(r"\d" + name + r"(I|E|7DevPtrs)", k)}
        assert found, (name, sorted(regs))
        assert not any(spilled for _, spilled in found.values()), found


@needs_readelf
@pytest.mark.parametrize("variant,waves", [((0, 32, 4), 6), ((1, 32, 4), 6), ((2, 32, 4), 6), ((0, 64, 16), 8),
                                           ((1, 64, 16), 8)])
def test_ring_launches_keep_their_waves(tmp_path, variant, waves):
    """Registers of a pair launch that leave it this many waves a SIMD (512 registers,
    given out by eights)."""
    symbol = "_Z7k_ringpILi%dELi%dELi%dEEv7DevPtrsijii" % variant
    used, spilled = _registers(tmp_path)[symbol]
    assert spilled == 0 and (used + 7) // 8 * 8 * waves <= 512, (used, spilled)
