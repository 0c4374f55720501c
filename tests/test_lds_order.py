"""The GEMM kernels that refill LDS by direct loads: the fragment reads in front of the main loop are complete, for every wave that
shares the place, before a load into it is requested.  Nothing but the order of instructions shows this (a load is slow enough
that results come out right without it), so that order is read from the library's own gfx950 code."""
import os
import re
import struct
import subprocess

import pytest

from paper_2104_04473_amd import binding as B
from paper_2104_04473_amd import build as Bld


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel symbol: [instruction, ..]} of every GEMM kernel in the built library."""
    objdump = os.path.join(os.path.dirname(os.path.realpath(Bld.HIPCC)), "..", "lib", "llvm", "bin", "llvm-objdump")
    blob, at, out = open(B.LIB_PATH, "rb").read(), 0, {}
    while (at := blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            start, size, n = struct.unpack_from("<QQQ", blob, p)
            target, p = blob[p + 24:p + 24 + n], p + 24 + n
            code = blob[at + start:at + start + size]
            if b"gfx950" not in target or b"gemm_bf16" not in code:
                continue
            obj = tmp_path_factory.mktemp("code") / "gemm.o"
            obj.write_bytes(code)
            text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(obj)], capture_output=True, text=True, check=True).stdout
            for part in re.split(r"\n(?=[0-9a-f]{16} <)", text):
                head = re.match(r"[0-9a-f]{16} <(\S*gemm_bf16\S*)>:", part)
                if head:
                    out[head.group(1)] = [line.split("//")[0].strip() for line in part.splitlines()[1:]]
        at += 24
    return out


def position(code, pattern, start=0):
    return next(i for i in range(start, len(code)) if re.search(pattern, code[i]))


READ, WAIT, BARRIER, REQUEST = r"^ds_read", r"^s_waitcnt.*lgkmcnt\(0\)", r"^s_barrier", r"^buffer_load\S* .* lds$"


def test_256x128_tiles_first_reads_are_complete_before_their_place_is_refilled(kernels):
    """A group of waves reads its first half-tile and refills that place in the phase behind: a wait and a barrier lie between."""
    found = [k for k in kernels if "gemm_bf16_wide_kernel" in k]
    assert len(found) == 2
    for name in found:
        code = kernels[name]
        first = position(code, READ)
        request, wait = position(code, REQUEST, first), position(code, WAIT, first)
        assert position(code, BARRIER, wait) < request, name


def test_256x256_tiles_first_reads_are_complete_at_the_second_groups_first_barrier(kernels):
    """Both groups of waves share every place.  The first refills the half-tile that all read in front of the loop two barriers after
    those reads, while the second multiplies for the first time: the second has waited for them before its extra barrier."""
    found = [k for k in kernels if any(x in k for x in ("gemm_bf16_dp_kernel", "gemm_bf16_dp_multi_kernel", "gemm_bf16_split_kernel"))]
    assert len(found) > 3
    for name in found:
        code = kernels[name]
        first = position(code, READ)
        assert position(code, WAIT, first) < position(code, BARRIER, first), name


def test_256x192_tiles_first_reads_are_complete_before_their_place_is_refilled(kernels):
    """The first phase refills what was read in front of the loop: both groups wait for those reads, and a barrier lies between."""
    found = [k for k in kernels if "gemm_bf16_mid_kernel" in k]
    assert len(found) == 2
    for name in found:
        code = kernels[name]
        first = position(code, READ)
        request, wait = position(code, REQUEST, first), position(code, WAIT, first)
        assert position(code, BARRIER, wait) < request, name
