"""Kernels keep their values in registers: the code objects in the built library say how much
scratch memory a lane has, and only the kernels named here, whose spills are known, have any."""
import os
import re
import struct
import subprocess

from paper_1603_04339_amd import sparc as sp

READELF = "/opt/rocm/llvm/bin/llvm-readelf"

# the 32 x 32 tiles (1024 threads, 128 registers; only the autotuner picks them), the register
# tridiagonalisations of complex matrices and of the largest real ones, the plans of
# several chunk widths in complex single, and a few words of two small solvers
KNOWN = [r"hstep_(batched_)?kernelI\S*Li32ELi32E", r"hetrd_reg_kernelI(N\S*cplxId|dLi3E)",
         r"hrow_mixed_kernelINS_4cplxIfE", r"latrd_kernelINS_4cplxIdE", r"anderson_gamma_kernel"]


def _code_objects(path):
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            p += 24
            if b"gfx950" in data[p:p + length]:
                yield data[at + off:at + off + size]
            p += length
        at = data.find(magic, at + 1)


def test_scratch_only_where_known(tmp_path):
    scratch = {}
    for i, obj in enumerate(_code_objects(sp.LIB_PATH)):
        f = tmp_path / f"{i}.co"
        f.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for name, size in re.findall(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, flags=re.S):
            scratch[name] = int(size)
    assert len(scratch) > 1000
    assert any("force_nl_kernel" in n for n in scratch)
    extra = {n: s for n, s in scratch.items() if s and not any(re.search(k, n) for k in KNOWN)}
    assert not extra, extra
