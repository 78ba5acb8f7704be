"""Hazards of inline assembly that the compiler does not see, checked in the
generated gfx950 code (CPU only) with the helpers of test_asm_hazards_cpu.py:

 - head-dim-64 attention: no inline LDS read writes a register that a recent
   MFMA still reads as its accumulator input (these 16x16x32 MFMAs take 4 passes
   of 4 cycles, the 32x32x16 ones of the other kernels 8: twice that is scanned);
 - MFMAs issued inline (GEMM, head-dim-64 backward): on every control-flow path
   no vector instruction writes an operand in the 2 wait states before one, and
   no instruction but another MFMA touches the result in the 11 wait states after
   (a 4-pass MFMA's result needs 7, one more on gfx950)."""
import os
import re
import subprocess

import pytest

from paper_2503_03182_amd import build as B

from test_asm_hazards_cpu import _blocks, _functions, _preds, _regs, _wait_states, scan

BEFORE, AFTER = 2, 11
STORES = ("ds_write", "buffer_store", "global_store", "flat_store", "scratch_store", "v_cmp", "v_readfirstlane",
          "v_readlane")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("asm")
    out, procs = {}, []
    for src in ("attention_fwd16.hip", "attention_bwd16.hip", "gemm_nt.hip", "gemm_nn.hip", "gemm_tn.hip"):
        dst = str(tmp / (src + ".s"))
        cmd = [B.hipcc(), "-x", "hip", *B.COMMON, *B.DEVICE_FLAGS, "--cuda-device-only", "-S",
               os.path.join(B.CSRC, src), "-o", dst]
        procs.append((src, dst, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE)))
    for src, dst, p in procs:
        _, err = p.communicate()
        assert p.returncode == 0, (src, err.decode()[-2000:])
        out[src] = open(dst).read()
    return out


def _written(ins):
    mn, ops, _ = ins
    if not ops or mn.startswith(STORES) or not mn.startswith(("v_", "ds_read", "ds_bpermute", "buffer_load", "global_load",
                                                              "scratch_load")):
        return set()
    if mn.startswith("buffer_load") and "lds" in " ".join(ops):
        return set()
    return _regs(ops[0].split()[0])


def _touched(ins):
    return set().union(*[_regs(t) for o in ins[1] for t in o.split()]) if ins[1] else set()


def _walk(blocks, nexts, b, j, step, limit, visit):
    """visit(instruction, wait states between) along every path from (b, j)."""
    stack, seen = [(b, j, 0)], set()
    while stack:
        b, j, d = stack.pop()
        if (b, j, d) in seen:
            continue
        seen.add((b, j, d))
        ins = blocks[b][1]
        if not 0 <= j < len(ins):
            stack += [(n, len(blocks[n][1]) - 1 if step < 0 else 0, d) for n in nexts[b]]
            continue
        if visit(ins[j], d):
            continue
        nd = d + _wait_states(ins[j])
        if nd < limit:
            stack.append((b, j + step, nd))


def mfma_hits(text):
    """(kernel, "before"|"after", wait states, instruction) for every inline MFMA
    with an operand written too late or a result touched too early."""
    hits, n = [], 0
    for name, lines in _functions(text):
        blocks = _blocks(lines)
        preds = _preds(blocks)
        succs = {i: [k for k in range(len(blocks)) if i in preds[k]] for i in range(len(blocks))}
        for bi, (_, ins) in enumerate(blocks):
            for ii, (mn, ops, inline) in enumerate(ins):
                if not (inline and mn.startswith("v_mfma")):
                    continue
                n += 1
                src = _regs(ops[1]) | _regs(ops[2]) | _regs(ops[3])
                dst = _regs(ops[0])

                def late(i, d):
                    if i[0].startswith("v_") and not i[0].startswith("v_mfma") and _written(i) & src:
                        hits.append((name, "before", d, i))
                    return False

                def early(i, d):
                    if i[0].startswith("v_mfma"):
                        return bool(_regs(i[1][0]) & dst)   # the accumulator's next MFMA takes over
                    if _touched(i) & dst:
                        hits.append((name, "after", d, i))
                    return False
                _walk(blocks, preds, bi, ii - 1, -1, BEFORE, late)
                _walk(blocks, succs, bi, ii + 1, 1, AFTER, early)
    return hits, n


def test_scanner_finds_planted_hazards():
    text = "\n".join([
        "k:",
        "\tv_mov_b32_e32 v20, v1",
        "\ts_nop 0",
        "\t;;#ASMSTART",
        "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[16:19], v[20:23], v[0:3]",
        "\t;;#ASMEND",
        "\ts_nop 3",
        "\tv_add_f32_e32 v9, v3, v8",
        "\ts_nop 15",
        "\tv_add_f32_e32 v9, v2, v8",
        ".Lfunc_end0:",
    ])
    hits, n = mfma_hits(text)
    assert n == 1
    assert {(h[1], h[2]) for h in hits} == {("before", 1), ("after", 4)}


@pytest.mark.parametrize("src", ["attention_fwd16.hip", "attention_bwd16.hip"])
def test_inline_lds_reads_never_overwrite_mfma_accumulator_inputs(assembly, src):
    assert len(re.findall(r";;#ASMSTART\s*\n\s*ds_read", assembly[src])) > 100
    bad = [h for h in scan(assembly[src], 8) if h[1] and h[2] == "C"]
    assert not bad, bad[:5]


@pytest.mark.parametrize("src", ["attention_bwd16.hip", "gemm_nt.hip", "gemm_nn.hip", "gemm_tn.hip"])
def test_inline_mfmas_have_their_wait_states(assembly, src):
    hits, n = mfma_hits(assembly[src])
    assert n > 100
    assert not hits, (len(hits), hits[:6])
