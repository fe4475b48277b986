"""Checks on the gfx950 assembly of the window attentions (attn_kl, attn_ct).

attn_kl loads the next query tile's Q with inline-assembly global loads that
it does not wait for at once: the registers are written when the loads land,
and the kernel's own waits (a stage count of steps later) cover them.  That is
only correct while the compiler leaves those registers alone until the copy
at the query-tile boundary (no spill, no move, no other use).  Its global ->
LDS copies are inline assembly too, so the compiler inserts no wait of its own
in front of the step loop's LDS reads.  These tests compile the source to
assembly (no GPU needed) and check both facts, so a compiler change that
breaks them fails here before anything runs on a GPU.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2511_14694_amd import build as B

# head_dim -> (symbol, waves per workgroup, LDS stages) of the instantiations
KERNELS = {
    128: ("_ZN12_GLOBAL__N_17attn_klILi128ELi4ELi4EEEv15focus_attn_descfl", 4, 4),
    64: ("_ZN12_GLOBAL__N_17attn_klILi64ELi4ELi4EEEv15focus_attn_descfl", 4, 4),
}


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not available")
    out = tmp_path_factory.mktemp("isa") / "window_attn.s"
    src = os.path.join(B.CSRC, "window_attn.hip")
    cmd = [hipcc, *B.HIPCC_FLAGS, *B.EXTRA_FLAGS.get("window_attn.hip", []), "--cuda-device-only", "-S", src,
           "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text().split("\n")


def _body(lines, name):
    start = next(i for i, line in enumerate(lines) if line.startswith(name + ":"))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return start, end


def _regs(text):
    used = set()
    for m in re.finditer(r"v\[(\d+):(\d+)\]", text):
        used |= set(range(int(m.group(1)), int(m.group(2)) + 1))
    for m in re.finditer(r"\bv(\d+)\b", text):
        used.add(int(m.group(1)))
    return used


@pytest.mark.parametrize("head_dim", [128, 64])
def test_prefetched_q_registers_untouched_until_copied(asm, head_dim):
    name, waves, stages = KERNELS[head_dim]
    start, end = _body(asm, name)
    # the asynchronous Q loads: inline-assembly blocks of plain global loads
    # with no wait inside
    prefetch, blocks = set(), 0
    i = start
    while i < end:
        if "ASMSTART" in asm[i]:
            j = i
            while "ASMEND" not in asm[j]:
                j += 1
            body = [x.strip() for x in asm[i + 1:j] if x.strip()]
            if body and all(b.startswith("global_load_dwordx4") for b in body):
                blocks += 1
                for b in body:
                    prefetch |= _regs(b.split(",")[0])
            i = j
        i += 1
    assert blocks > 0, "no asynchronous Q load found"
    assert len(prefetch) == 4 * (head_dim // 16)
    # Copies of the tiles in flight at a query-tile boundary: (stages - 1)
    # steps' copies of 2 x (tile bytes / 1 KB / waves) each.
    in_flight = (stages - 1) * 2 * (32 * head_dim * 2 // 1024 // waves)
    uses = 0
    in_asm = False
    last_wait = None  # vmcnt of the latest s_waitcnt in layout order
    for line in asm[start:end]:
        s = line.strip()
        if "ASMSTART" in s or "ASMEND" in s:
            in_asm = "ASMSTART" in s
            continue
        if not s or s.startswith((";", ".")) or s.endswith(":"):
            continue
        if in_asm and s.startswith("global_load_dwordx4") and _regs(s.split(",")[0]) & prefetch:
            last_wait = None  # a new prefetch: no wait covers it yet
            continue
        m = re.match(r"s_waitcnt\b.*vmcnt\((\d+)\)", s)
        if m:
            last_wait = int(m.group(1))
        if not in_asm and _regs(s) & prefetch:
            # the only other access: the copy into the working Q registers,
            # reading them as a source, after the wait that covers the loads
            assert s.startswith("v_mov_b"), s
            assert not (_regs(s.split(None, 1)[1].split(",", 1)[0]) & prefetch), s
            assert last_wait is not None and last_wait <= in_flight, (s, last_wait)
            uses += 1
    assert uses, "the prefetched Q is never copied"


@pytest.mark.parametrize("head_dim", [128, 64])
def test_no_spills_and_no_compiler_wait_before_lds_reads(asm, head_dim):
    name = KERNELS[head_dim][0]
    # kernel metadata: the fields after .name are in alphabetical order
    i = next(k for k, line in enumerate(asm) if re.search(r"\.name:\s+" + re.escape(name) + r"$", line))
    spill = next(line for line in asm[i:] if ".vgpr_spill_count:" in line)
    assert int(spill.split(":")[1]) == 0, spill
    start, end = _body(asm, name)
    prev, in_asm = None, False
    for line in asm[start:end]:
        s = line.strip()
        if "ASMSTART" in s or "ASMEND" in s:
            in_asm = "ASMSTART" in s
            prev = None
            continue
        if in_asm or not s or s.startswith((";", ".")) or s.endswith(":"):
            continue
        if prev is not None and prev.startswith("s_waitcnt") and "vmcnt" in prev:
            assert not s.startswith(("ds_read", "v_mfma")), f"compiler wait before an LDS read: {prev} -> {s}"
        prev = s


# attn_ct keeps its output accumulators in AGPRs through inline-assembly MFMAs,
# whose latency the compiler does not know: any other access to an AGPR must
# come after the kernel's own wait states (s_nop 15), and the phases (blocks with
# a row of MFMAs) must leave the AGPRs, the copies' counter and scratch alone.
CT_KERNELS = ["_ZN12_GLOBAL__N_17attn_ctILi128EEEv15focus_attn_descfliNS_5SplitE",
              "_ZN12_GLOBAL__N_17attn_ctILi64EEEv15focus_attn_descfliNS_5SplitE"]


@pytest.mark.parametrize("name", CT_KERNELS)
def test_ct_accumulators_touched_only_behind_wait_states(asm, name):
    i = next(k for k, line in enumerate(asm) if re.search(r"\.name:\s+" + re.escape(name) + r"$", line))
    spill = next(line for line in asm[i:] if ".vgpr_spill_count:" in line)
    assert int(spill.split(":")[1]) == 0, spill
    start, end = _body(asm, name)
    pending, blocks, block = False, 0, []

    def close():
        mfmas = [x for x in block if x.startswith("v_mfma")]
        if len(mfmas) < 8 or any(x.startswith("s_barrier") for x in block):
            return 0
        bad = [x for x in block if x.startswith(("v_accvgpr", "scratch_", "s_nop 15")) or "vmcnt" in x]
        assert not bad, bad
        return 1

    for line in asm[start:end]:
        s = line.strip()
        if s.startswith(".LBB"):
            blocks += close()
            block = []
        if not s or s.startswith((";", ".")) or s.endswith(":"):
            continue
        block.append(s)
        if s.startswith("v_mfma") and s.split()[1].startswith("a["):
            pending = True
        elif s.startswith("s_nop 15"):
            pending = False
        elif s.startswith("v_accvgpr"):
            assert not pending, s
    blocks += close()
    assert blocks >= 12, blocks  # four clean phases, eight masked ones


def _sets(text):
    """Registers of an operand list, as names (v1, a7)."""
    out = set()
    for kind, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text):
        out |= {f"{kind}{x}" for x in range(int(lo), int(hi) + 1)}
    out |= {m.group(0) for m in re.finditer(r"\b[va]\d+\b", text)}
    return out


@pytest.mark.parametrize("name", CT_KERNELS)
def test_ct_output_products_read_settled_registers(asm, name):
    """An inline-assembly MFMA gets no compiler wait states: a vector instruction's
    result (a probability, an operand copied by the register allocator, an
    accumulator written back) may be its source only from the third instruction on.
    Checked against the two instructions before every such MFMA along all paths."""
    start, end = _body(asm, name)
    code, label_at = [], {}      # instructions; label -> index of the next one
    for line in asm[start:end]:
        s = line.split(";")[0].strip()
        if s.endswith(":"):
            label_at[s[:-1]] = len(code)
        elif s and not s.startswith("."):
            code.append(s)
    jumps = {}                   # index -> branches that lead there
    for i, s in enumerate(code):
        if s.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(label_at[s.split()[1]], []).append(i)

    def writers(i, left):
        """Vector instructions that end fewer than `left` wait states before code[i]."""
        found = []
        before = list(jumps.get(i, []))
        if i > 0 and not code[i - 1].startswith(("s_branch", "s_endpgm", "s_setpc")):
            before.append(i - 1)
        for j in before:
            s = code[j]
            if s.startswith("v_") and not s.startswith("v_mfma"):
                found.append(s)
            states = int(s.split()[1], 0) + 1 if s.startswith("s_nop") else 1
            if left > states:
                found += writers(j, left - states)
        return found

    seen = 0
    for i, s in enumerate(code):
        if not (s.startswith("v_mfma") and s.split()[1].startswith("a[")):
            continue
        seen += 1
        read = _sets(s.split(None, 1)[1])
        for w in writers(i, 2):
            ops = w.split(None, 1)[1]
            dst = _sets(ops.split(",")[0]) | (_sets(ops) if "swap" in w.split()[0] else set())
            assert not dst & read, (w, s)
    assert seen >= 64
