"""Static checks of the generated gfx950 code (CPU only: compiles the kernel
source to assembly).  Stores and atomics must go through vector memory: the
scalar data cache is never written, and no kernel spills to scratch."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2106_11286_amd", "csrc")


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    """Assembly of every device source, compiled with the library's own flags."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    import sys

    sys.path.insert(0, ROOT)
    from concurrent.futures import ThreadPoolExecutor

    from paper_2106_11286_amd import build as B

    common, dev = B.compile_flags()
    d = tmp_path_factory.mktemp("isa")

    def one(src):
        out = str(d / (src + ".s"))
        subprocess.check_call([hipcc] + common + dev + ["--offload-device-only", "-S", "-o", out,
                                                        os.path.join(CSRC, src)],
                              stderr=subprocess.DEVNULL)
        return open(out).read()

    with ThreadPoolExecutor(max_workers=len(B.KERNEL_SOURCES)) as pool:
        return "\n".join(pool.map(one, B.KERNEL_SOURCES))


def test_no_scalar_memory_writes(asm):
    bad = re.compile(r"^\s*(s_store_|s_buffer_store|s_scratch_store|s_atomic_|s_buffer_atomic|"
                     r"s_dcache_wb|s_dcache_discard)", re.M)
    hits = bad.findall(asm)
    assert not hits, sorted(set(hits))


def test_no_scratch_spills(asm):
    spills = [int(v) for v in re.findall(r"\.vgpr_spill_count:\s+(\d+)", asm)]
    assert spills and max(spills) == 0
    for m in re.finditer(r"\.private_segment_fixed_size:\s+(\d+)", asm):
        assert int(m.group(1)) == 0


def _registers(operand):
    m = re.match(r"v\[(\d+):(\d+)\]$", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"v(\d+)$", operand)
    return {int(m[1])} if m else set()


def wide_store_overwrites(text):
    """Stores of more than 8 bytes whose data registers a vector instruction
    writes within two wait states: such a store can take the new values."""
    code = [ln.strip() for ln in text.splitlines() if re.match(r"\s+[a-z]\w*(\s|$)", ln)]
    hits = []
    for i, ln in enumerate(code):
        m = re.match(r"(buffer|global|flat)_store_dwordx[34]\s+(.*)", ln)
        if not m:
            continue
        ops = [o.strip().split()[0] for o in m[2].split(",")]
        data = _registers(ops[0] if m[1] == "buffer" else ops[1])
        assert len(data) > 2, ln
        waits = 0
        for nxt in code[i + 1:i + 3]:
            if waits >= 2 or nxt.startswith(("s_branch", "s_endpgm")):
                break
            if nxt.startswith("v_") and _registers(nxt.split(None, 1)[1].split(",")[0].strip()) & data:
                hits.append((ln, nxt))
            nop = re.match(r"s_nop (\d+)", nxt)
            waits += 1 + int(nop[1]) if nop else 1
    return hits


def test_wide_store_data_not_overwritten(asm):
    # the check itself: a hit at one wait state, none behind a wait of two
    store, write = "\tbuffer_store_dwordx4 v[8:11], v1, s[0:3], s4 offen", "\tv_mov_b32_e32 v9, v2"
    assert wide_store_overwrites("\n".join((store, write)))
    assert not wide_store_overwrites("\n".join((store, "\ts_nop 1", write)))
    assert re.search(r"buffer_store_dwordx4", asm)
    assert not wide_store_overwrites(asm), wide_store_overwrites(asm)[:8]
