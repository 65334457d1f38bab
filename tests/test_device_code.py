"""The gfx950 instructions of the built library: waits that the hardware asks of
the code and that neither the assembler (inside inline assembly) nor a result
that happens to be right would show."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2502_15524_amd", "_lib", "libhs.so")
OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP) and shutil.which("llvm-objdump") is None,
                                reason="needs llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name: [instruction, ...]} of every device function in the library."""
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    data = open(LIB, "rb").read()
    d = tmp_path_factory.mktemp("code")
    out = {}
    for n, m in enumerate(re.finditer(MAGIC, data)):
        at = m.start() + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            off, size, tl = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + tl].decode()
            at += 24 + tl
            if "gfx950" not in triple or not size:
                continue
            path = str(d / f"{n}.co")
            with open(path, "wb") as f:
                f.write(data[m.start() + off:m.start() + off + size])
            exe = OBJDUMP if os.path.exists(OBJDUMP) else "llvm-objdump"
            text = subprocess.run([exe, "-d", "-C", "--no-show-raw-insn", "--no-leading-addr", path],
                                  capture_output=True, text=True, check=True).stdout
            name = None
            for line in text.splitlines():
                h = re.match(r"^(?:[0-9a-f]+ )?<(.*)>:$", line.strip())
                if h:
                    name = h.group(1)
                    out[name] = []
                elif name and line.strip():
                    out[name].append(line.split("//")[0].strip())
    assert any("gemm_ring" in k for k in out) and any("attn_prefill" in k for k in out), list(out)[:5]
    return out


def test_m0_is_written_a_wait_state_before_a_load_into_lds(kernels):
    """A load into LDS takes its LDS address from M0, and a scalar write of M0
    needs one wait state before such a load (gfx9): at least one instruction
    between the two. Without it the load may land at the previous address."""
    loads, bad = 0, []
    for name, ins in kernels.items():
        for i, x in enumerate(ins):
            if re.match(r"(buffer|global)_load\w*\b.*\blds\b", x):
                loads += 1
                if re.match(r"s_\w+\s+m0\b", ins[i - 1]):
                    bad.append(name)
    assert loads > 100
    assert not bad, {n: bad.count(n) for n in sorted(set(bad))}


def test_no_lds_read_is_outstanding_when_its_stage_is_given_up(kernels):
    """The pipelined kernels refill a stage of LDS from any wave right after the
    barrier that ends its use, so each wave's reads of it have to be complete at
    that barrier (lgkmcnt 0 after the last read), not merely issued. The
    ping-pong loop (last template argument true) refills two barriers after a
    read: its reads may pass one."""
    seen = 0
    for name, ins in kernels.items():
        if "gemm_ring<" in name:
            passes = 1 if re.search(r"true>\(", name) else 0
        elif "attn_prefill_wide_kernel" in name:
            passes = 0
        else:
            continue
        seen += 1
        out = None  # barriers passed since the oldest read that may be outstanding
        barriers = 0
        for x in ins:
            if x.startswith("ds_read"):
                out = 0 if out is None else out
            elif x.startswith("s_waitcnt") and "lgkmcnt(0)" in x:
                out = None
            elif x.startswith("s_barrier"):
                barriers += 1
                if out is not None:
                    out += 1
                    assert out <= passes, (name, barriers)
        assert barriers, name
    assert seen > 50
