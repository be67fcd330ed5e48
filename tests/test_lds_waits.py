"""The built kernels that fill LDS by DMA in several stages: before each barrier
after which a stage is filled again, the wave waits for its own LDS reads (they
may be of that stage) in the barrier's own wait, not wherever the compiler
happened to put the multiplications that use them."""
import os
import re
import struct
import subprocess

import pytest

from paper_2509_22462_amd import build

LLVM = "/opt/rocm/llvm/bin"


def code_objects(lib, tmp):
    """Paths of the bundled gfx950 code objects that hold the staged kernels."""
    fat = tmp / "fatbin"
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", lib, os.devnull], check=True)
    data = fat.read_bytes()
    out = []
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.end()
        count, = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            off, size, tl = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + tl]
            at += 24 + tl
            code = data[m.start() + off:m.start() + off + size]
            if b"gfx950" in triple and (b"gemm_pk_kernel" in code or b"gemm_dma_kernel" in code):
                p = tmp / f"co{len(out)}"
                p.write_bytes(code)
                out.append(p)
    return out


def kernels(path):
    """(name, instructions) of each kernel that loads LDS by DMA."""
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                          check=True, capture_output=True, text=True).stdout
    name, ins = None, []
    for line in text.splitlines():
        m = re.match(r"^(?:[0-9a-f]+ )?<(.+)>:", line)
        if m:
            if any(" lds" in i for i in ins):
                yield name, ins
            name, ins = m.group(1), []
        elif line.strip():
            ins.append(line.split("//")[0].strip())
    if any(" lds" in i for i in ins):
        yield name, ins


def test_barriers_before_a_refill_wait_for_the_reads(tmp_path):
    if not os.path.exists(build.LIB):
        pytest.fail("libnnc.so is not built: run python -m paper_2509_22462_amd.build")
    seen = 0
    for co in code_objects(build.LIB, tmp_path):
        for name, ins in kernels(co):
            bars = [i for i, t in enumerate(ins) if t.startswith("s_barrier")]
            for i, nxt in zip(bars, bars[1:] + [len(ins)]):
                if not any(t.startswith("buffer_load") and t.endswith(" lds") for t in ins[i:nxt]):
                    continue
                wait = next(t for t in reversed(ins[:i]) if t.startswith("s_waitcnt"))
                assert "lgkmcnt(0)" in wait, (name, i, wait)
                seen += 1
    if seen == 0:
        pytest.fail("no DMA-staged kernel found in the library")
