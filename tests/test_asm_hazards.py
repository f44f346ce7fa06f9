"""Host-side check of the wait states around inline assembly. The GEMM kernels issue their MFMAs and their direct
global -> LDS loads as inline assembly, and the compiler's hazard recognizer does not look inside it: what the CDNA3/4
instruction set leaves to software has to hold by the way the code around it is written, and this is where it shows if
it does not. Checked in program order and, for loops, from the end of the body to its beginning:
  * a memory instruction reads a scalar register at least 5 wait states after a vector instruction wrote it
  * a direct-to-LDS load follows a write of M0 by at least 1 wait state
  * an MFMA reads a vector register at least 2 wait states after an ordinary vector instruction wrote it
  * an ordinary vector instruction reads an MFMA's result at least 11 wait states after the MFMA (8 passes or fewer), and
    so does a memory instruction that stores it
  * a vector instruction overwrites the data registers of a store of more than 64 bits at least 2 wait states after the
    store, on the way past a branch as on the way through it
"""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2512_10236_amd import _build


def _regs(tok):
    """Registers named by an operand: {'s12', 'a3', ...}."""
    tok = tok.strip().split()[0] if tok.strip() else ""
    m = re.fullmatch(r"([sva])\[(\d+):(\d+)\]", tok)
    if m:
        return {m.group(1) + str(i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    if re.fullmatch(r"[sva]\d+", tok):
        return {tok}
    return {"vcc": {"vcc_lo", "vcc_hi"}, "vcc_lo": {"vcc_lo"}, "vcc_hi": {"vcc_hi"}, "m0": {"m0"}}.get(tok, set())


def _parse(line):
    t = line.split(";")[0].strip()
    if not t or t.startswith(".") or t.endswith(":"):
        return None
    op = t.split()[0]
    args = [_regs(a) for a in t[len(op):].split(",")]
    mfma = op.startswith("v_mfma")
    valu = op.startswith("v_") and not mfma
    memory = op.startswith(("global_", "buffer_", "flat_", "scratch_"))
    store = memory and "store" in op
    to_lds = memory and "_lds_" in op
    # registers of the data of a store of three or four words: the first operand of a buffer store, else the second
    wide = args[0 if op.startswith("buffer_") else 1] if store and op.endswith(("x3", "x4")) else set()
    nop = int(t.split()[1]) + 1 if op == "s_nop" else 1
    n_dst = 0 if (store or to_lds or op.startswith(("s_cmp", "s_waitcnt", "s_barrier", "s_branch", "s_cbranch", "s_nop", "ds_write"))) else 1
    writes = set().union(*args[:n_dst]) if n_dst else set()
    reads = set().union(*args[n_dst:]) if len(args) > n_dst else set()
    if op == "v_permlane16_swap_b32":
        writes, reads = set().union(*args), set().union(*args)
    return dict(op=op, writes=writes, reads=reads, mfma=mfma, valu=valu, memory=memory, to_lds=to_lds, wide=wide, states=nop, text=t)


def _check(name, body, bad):
    """`body`: parsed instructions in the order they run."""
    for n, x in enumerate(body):
        if x is None:
            continue
        states = 0
        for y in reversed(body[max(0, n - 24):n]):
            if y is None:
                continue
            if x["memory"] and y["valu"] and states < 5:
                hit = {r for r in y["writes"] & x["reads"] if r[0] == "s" or r.startswith("vcc")}
                if hit:
                    bad.add((name, "scalar written by a vector instruction %d states before" % states, y["text"], x["text"]))
            if x["to_lds"] and "m0" in y["writes"] and states < 1:
                bad.add((name, "M0", y["text"], x["text"]))
            if x["mfma"] and y["valu"] and states < 2 and y["writes"] & x["reads"]:
                bad.add((name, "MFMA operand written %d states before" % states, y["text"], x["text"]))
            if x["valu"] and y["mfma"] and states < 11 and y["writes"] & (x["reads"] | x["writes"]):
                bad.add((name, "MFMA result touched after %d states" % states, y["text"], x["text"]))
            if x["memory"] and y["mfma"] and states < 11 and y["writes"] & x["reads"]:
                bad.add((name, "MFMA result stored after %d states" % states, y["text"], x["text"]))
            if (x["valu"] or x["mfma"]) and states < 2 and y["wide"] & x["writes"]:
                bad.add((name, "store data overwritten after %d states" % states, y["text"], x["text"]))
            states += y["states"]


def _taken(parsed, i, k, head):
    """What runs around a branch at line k of the function at line i to the label at line head, when it is taken."""
    return parsed[max(0, k - i - 40):k - i + 1] + parsed[head - i:head - i + 40]


def hazards(asm):
    bad, seen = set(), 0
    lines = asm.split("\n")
    starts = [i for i, l in enumerate(lines) if re.match(r"^_Z\w+:", l)]
    for i in starts:
        end = next((k for k in range(i, len(lines)) if lines[k].startswith(".Lfunc_end")), len(lines))
        name = lines[i].split(":")[0]
        labels = {m.group(1): k for k in range(i, end) for m in [re.match(r"^(\.L\w+):", lines[k])] if m}
        parsed = [_parse(l) for l in lines[i:end]]
        seen += sum(1 for x in parsed if x and x["mfma"])
        _check(name, parsed, bad)
        for k in range(i, end):
            m = re.search(r"s_c?branch\w*\s+(\.L\w+)", lines[k])
            if m and labels.get(m.group(1), end) < k:
                head = labels[m.group(1)]
                _check(name + " (loop)", parsed[max(head - i, k - i - 40):k - i] + parsed[head - i:head - i + 40], bad)
            elif m and m.group(1) in labels:
                _check(name + " (branch)", _taken(parsed, i, k, labels[m.group(1)]), bad)
    return bad, seen


def test_checker_sees_what_it_is_for():
    """The checker itself, on hand-written sequences: one for each rule, too close and far enough."""
    far = {"v_readfirstlane_b32 s4, v0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 v1, s[4:5]", "s_add_i32 m0, s1, 4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v1, s[4:5]",
           "v_mov_b32_e32 v8, v0\n\ts_nop 1\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[4:7], a[0:3]",
           "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[4:7], a[0:3]\n\ts_nop 10\n\tv_accvgpr_read_b32 v0, a2",
           "v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[4:7], a[0:3]\n\ts_nop 10\n\tglobal_store_dwordx4 v[0:1], a[0:3], off",
           "global_store_dwordx4 v[0:1], v[4:7], off sc0 sc1\n\ts_nop 1\n\tv_mov_b32_e32 v7, v0",
           "global_store_dwordx3 v0, v[4:6], s[2:3]\n\ts_or_b64 exec, exec, s[0:1]\n\ts_nop 0\n\tv_cvt_pk_bf16_f32 v4, v0, v1",
           "buffer_store_dwordx4 v[4:7], v0, s[0:3], 0 offen\n\ts_nop 1\n\tv_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], 0"}
    for text in far:
        near = "\n".join(l for l in text.split("\n") if "s_nop" not in l)
        assert not hazards("_Zf:\n\t%s\n.Lfunc_end0:" % text)[0], text
        assert hazards("_Zf:\n\t%s\n.Lfunc_end0:" % near)[0], near
    loop = "_Zf:\n.LBB0_1:\n\tglobal_load_lds_dwordx4 v1, s[4:5]\n\tv_readfirstlane_b32 s4, v0\n\ts_cbranch_scc1 .LBB0_1\n.Lfunc_end0:"
    assert hazards(loop)[0]
    past = "_Zf:\n\tglobal_store_dwordx4 v[0:1], v[4:7], off\n\ts_cbranch_scc1 .LBB0_1\n\ts_nop 4\n.LBB0_1:\n\tv_mov_b32_e32 v7, v0\n.Lfunc_end0:"
    assert hazards(past)[0]
    assert not hazards(past.replace("scc1 .", "scc1  .").replace("off\n", "off\n\ts_nop 0\n"))[0]
    short = "_Zf:\n\tglobal_store_dwordx2 v[0:1], v[4:5], off\n\tv_mov_b32_e32 v5, v0\n.Lfunc_end0:"
    assert not hazards(short)[0]


def test_wait_states_around_inline_assembly():
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "gemm.s")
        cmd = [hipcc] + _build.FLAGS + ["-S", "--cuda-device-only", os.path.join(_build.CSRC, "ficco_gemm.hip"), "-o", out]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert r.returncode == 0, r.stdout[-2000:]
        with open(out) as f:
            bad, seen = hazards(f.read())
    assert seen > 1000, "no MFMAs found in the assembly"
    assert not bad, "\n".join(map(str, sorted(bad)[:20]))
