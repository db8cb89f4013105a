"""Static check of the generated gfx950 code along its control flow (CPU only:
compiles every device source to assembly): no vector register that a store of
more than 8 bytes still reads is written within two wait states of it, on any
path, also across branches and by instructions with two results."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2106_11286_amd", "csrc")

WIDE = re.compile(r"(buffer|global|flat|scratch)_store_dwordx[34]$")
TWO_RESULTS = re.compile(r"v_(permlane(16|32)_swap|swap)_b\d+")


def registers(operand):
    """Vector registers of an operand, as ("v" or "a", index)."""
    m = re.match(r"([va])\[(\d+):(\d+)\]$", operand)
    if m:
        return {(m[1], i) for i in range(int(m[2]), int(m[3]) + 1)}
    m = re.match(r"([va])(\d+)$", operand)
    return {(m[1], int(m[2]))} if m else set()


def parse(text):
    """Instructions [(name, operands)] in order and {label: index of the next one}."""
    code, labels = [], {}
    for ln in text.splitlines():
        ln = ln.split(";")[0].rstrip()
        m = re.match(r"([.\w$]+):$", ln)
        if m:
            labels[m[1]] = len(code)
            continue
        m = re.match(r"\s+([a-z]\w+)(?:\s+(.*))?$", ln)
        if m:
            ops = [o.strip().split()[0] for o in (m[2] or "").split(",") if o.strip()]
            code.append((m[1], ops))
    return code, labels


def written(name, ops):
    """Vector registers that a vector ALU instruction writes."""
    if not name.startswith("v_") or not ops:
        return set()
    out = registers(ops[0])
    return out | registers(ops[1]) if TWO_RESULTS.match(name) else out


def successors(code, labels, i):
    name, ops = code[i]
    if name in ("s_endpgm", "s_setpc_b64"):
        return []
    if name == "s_branch":
        return [labels[ops[0]]]
    nxt = [i + 1] if i + 1 < len(code) else []
    return nxt + [labels[ops[0]]] if name.startswith("s_cbranch_") else nxt


def overwrites(text, states=2):
    """(store, later instruction) pairs where the latter writes the store's data
    with fewer than `states` wait states between them."""
    code, labels = parse(text)
    hits, stores = [], 0
    for i, (name, ops) in enumerate(code):
        m = WIDE.match(name)
        if not m:
            continue
        stores += 1
        data = registers(ops[0] if m[1] == "buffer" else ops[1])
        assert len(data) > 2, (name, ops)
        todo = [(s, 0) for s in successors(code, labels, i)]
        while todo:
            j, waits = todo.pop()
            n2, o2 = code[j]
            if written(n2, o2) & data:
                hits.append((" ".join([name] + ops), " ".join([n2] + o2)))
                continue
            waits += 1 + int(o2[0]) if n2 == "s_nop" else 1
            if waits < states:
                todo += [(s, waits) for s in successors(code, labels, j)]
    return hits, stores


STORE = "\tbuffer_store_dwordx4 v[8:11], v1, s[0:3], s4 offen\n"
END = "\ts_endpgm\n"


@pytest.mark.parametrize("body,hit", [
    (STORE + "\tv_mov_b32_e32 v9, v2\n", True),
    (STORE + "\tv_mov_b32_e32 v3, v2\n\tv_mov_b32_e32 v11, v2\n", True),
    (STORE + "\ts_nop 1\n\tv_mov_b32_e32 v9, v2\n", False),
    # the second result of a swap, and an accumulator register's data
    (STORE + "\tv_permlane32_swap_b32_e32 v2, v10\n", True),
    ("\tglobal_store_dwordx4 v0, a[4:7], s[0:1]\n\tv_accvgpr_write_b32 a5, v1\n", True),
    # the taken side of a conditional branch and an unconditional one
    (STORE + "\ts_cbranch_vccnz .L1\n\ts_nop 1\n.L1:\n\tv_mov_b32_e32 v8, v2\n", True),
    ("\ts_branch .L2\n.L1:\n\tv_mov_b32_e32 v8, v2\n" + END + ".L2:\n" + STORE + "\ts_branch .L1\n",
     True),
    # a loop whose head writes the data of the store at its end
    (".L3:\n\tv_add_u32_e32 v9, v9, v1\n\ts_nop 1\n" + STORE + "\ts_cbranch_scc1 .L3\n", True),
    # reads, scalar results and other registers
    (STORE + "\tv_add_u32_e32 v12, v9, v10\n\tv_readlane_b32 s8, v9, 0\n", False),
])
def test_the_check_itself(body, hit):
    hits, stores = overwrites(body + END)
    assert stores == 1 and bool(hits) == hit


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    """{source: assembly}, compiled with the library's own flags."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    import sys

    sys.path.insert(0, ROOT)
    from concurrent.futures import ThreadPoolExecutor

    from paper_2106_11286_amd import build as B

    common, dev = B.compile_flags()
    d = tmp_path_factory.mktemp("isa_flow")
    sources = B.KERNEL_SOURCES + B.MIXED_SOURCES

    def one(src):
        out = str(d / (src + ".s"))
        subprocess.check_call([hipcc] + common + dev + ["--offload-device-only", "-S", "-o", out,
                                                        os.path.join(CSRC, src)],
                              stderr=subprocess.DEVNULL)
        return open(out).read()

    with ThreadPoolExecutor(max_workers=8) as pool:
        return dict(zip(sources, pool.map(one, sources)))


def test_wide_store_data_kept_on_every_path(asm):
    found = 0
    for src, text in asm.items():
        hits, stores = overwrites(text)
        found += stores
        assert not hits, (src, hits[:8])
    assert found
