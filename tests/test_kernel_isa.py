"""Host-side check of what the compiler made of the attention kernel's streaming loops.

The decode kernel lives on counting its outstanding loads exactly: one `s_waitcnt vmcnt(0)`
inside a streaming loop drains the whole KV pipeline every step and costs several per cent
of bandwidth, without any test of results noticing.  Small source changes have flipped the
compiler into that mode before, so the generated code itself is checked: in the innermost
MFMA loops of k_attention there is no full wait on vector memory, no scratch traffic, and
the kernel keeps two waves per SIMD (at most 256 VGPRs).  The prefill kernel counts its
requests into LDS by hand: the compiler may add no wait to its steps beside those for the
block ids and scales of the next 64 page pairs."""
import functools
import os
import re
import subprocess
import tempfile

from paper_2505_04021_amd import build as B


@functools.lru_cache(maxsize=None)
def device_assembly(source="attn_kernels.hip"):
    out = os.path.join(tempfile.mkdtemp(prefix="pkv_isa_"), "attn.s")
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-shared")]
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["--cuda-device-only", "-S",
                                                                      os.path.join(B.CSRC, source), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return open(out).read()


def kernel_body(asm, mangled_part):
    lines = asm.split("\n")
    start = [i for i, l in enumerate(lines) if re.match(r"^_Z\w*" + mangled_part + r"\w*:", l)][0]
    end = [i for i, l in enumerate(lines) if ".end_amdhsa_kernel" in l and i > start][0]
    labels, insn = {}, []
    for l in lines[start:end]:
        m = re.match(r"^(\.LBB\d+_\d+):", l)
        if m:
            labels[m.group(1)] = len(insn)
            continue
        t = l.strip()
        if t and not t.startswith((";", ".", "//")):
            insn.append(t)
    meta = "\n".join(lines[end:end + 400])
    return insn, labels, meta


def innermost_mfma_loops(insn, labels, min_mfma=20):
    mf = [i for i, t in enumerate(insn) if t.startswith("v_mfma")]
    loops = []
    for i, t in enumerate(insn):
        m = re.match(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", t)
        if m and m.group(1) in labels and labels[m.group(1)] < i:
            a = labels[m.group(1)]
            if sum(1 for x in mf if a <= x <= i) >= min_mfma:
                loops.append((a, i))
    return [l for l in loops if not any(o != l and o[0] >= l[0] and o[1] <= l[1] for o in loops)]


def test_streaming_loops_keep_exact_load_counts():
    asm = device_assembly()
    # both forms (two waves per SIMD / one wave per SIMD), each with bf16 / e4m3 x head dim 128 / 64
    for name, n_loops, max_vgpr in (("11k_attentionE", 4, 256), ("16k_attention_deepE", 4, 512)):
        insn, labels, _ = kernel_body(asm, name)
        loops = innermost_mfma_loops(insn, labels)
        assert len(loops) == n_loops, (name, loops)
        for a, b in loops:
            seg = insn[a:b]
            assert sum(t.startswith("buffer_load_dwordx4") for t in seg) >= 12
            full = [t for t in seg if t.startswith("s_waitcnt") and re.search(r"vmcnt\(0\)", t)]
            assert not full, f"{name} loop {a}..{b} drains vector memory: {full[:3]}"
            assert not any(t.startswith("scratch_") for t in seg), f"{name} loop {a}..{b} spills to scratch"
        vg = [int(x) for x in re.findall(r"\.name:\s+\S*" + name + r"\S*\s*\n(?:.*\n){0,40}?\s+\.vgpr_count:\s+(\d+)", asm)]
        assert vg and max(vg) <= max_vgpr, (name, vg)


def test_small_launches_keep_exact_load_counts():
    """The loops of k_attention_small, two page pairs a turn: nothing is read but the pages, no full wait, no scratch traffic; only a
    turn that looks up the next 32 pairs, and then goes on in the loop, waits for them."""
    asm = device_assembly()
    for name in ("17k_attention_smallINS_7AttnOne", "17k_attention_smallI9AttnGroup"):
        insn, labels, _ = kernel_body(asm, name)
        loops = innermost_mfma_loops(insn, labels)
        tight = [l for l in loops if not any(t.startswith("global_load") for t in insn[l[0]:l[1]])]
        shapes = sorted((sum(t.startswith("v_mfma") for t in insn[a:b]), sum(t.startswith("buffer_load_dwordx4") for t in insn[a:b])) for a, b in tight)
        assert shapes == [(24, 8), (24, 16), (48, 16), (48, 32)], (name, shapes)      # 64- and 128-wide heads, e4m3 and bf16
        for a, b in loops:
            full = [t for t in insn[a:b] if t.startswith("s_waitcnt") and re.search(r"vmcnt\(0\)", t)]
            assert len(full) <= (0 if (a, b) in tight else 1), (name, a, b, full)
            assert not any(t.startswith("scratch_") for t in insn[a:b]), f"{name} loop {a}..{b} spills to scratch"
        vg = [int(x) for x in re.findall(r"\.name:\s+\S*" + name + r"\S*\s*\n(?:.*\n){0,40}?\s+\.vgpr_count:\s+(\d+)", asm)]
        assert vg and max(vg) <= 256, (name, vg)


def test_prefill_steps_wait_only_where_written():
    asm = device_assembly("prefill_kernels.hip")
    for seqs in (127, 447):                                     # sequences of the launch's plan
        for d, dtype, mfma in ((128, 0, 24), (64, 0, 12), (128, 1, 16), (64, 1, 8)):
            name = f"9k_prefillILi{d}ELi{dtype}ELi{seqs}E"
            insn, labels, _ = kernel_body(asm, name)
            loops = innermost_mfma_loops(insn, labels, min_mfma=mfma)
            assert len(loops) == 2, (name, loops)               # steps without masks, and the others
            for a, b in loops:
                seg = insn[a:b]
                assert sum(t.startswith("v_mfma") for t in seg) == mfma and seg.count("s_barrier") == 1
                assert not any(t.startswith("scratch_") for t in seg), f"{name} loop {a}..{b} spills to scratch"
                full = [t for t in seg if t.startswith("s_waitcnt") and "vmcnt(0)" in t]
                # the meeting point, the two places where it may ask for the next ids; e4m3: both pages' ids and scales
                assert len(full) <= (3 if dtype == 0 else 5), (name, full)
            vg = [int(x) for x in re.findall(r"\.name:\s+\S*" + name + r"\S*\s*\n(?:.*\n){0,40}?\s+\.vgpr_count:\s+(\d+)", asm)]
            assert vg and max(vg) <= 256, (name, vg)


def test_prefill_steps_down_only_where_two_work_groups_share_a_cu():
    """Priority levels help the two work-groups a CU has on 128-wide heads; the three of 64-wide heads lost up to a tenth."""
    asm = device_assembly("prefill_kernels.hip")
    for seqs in (127, 447):
        for d, dtype in ((128, 0), (64, 0), (128, 1), (64, 1)):
            insn, _, _ = kernel_body(asm, f"9k_prefillILi{d}ELi{dtype}ELi{seqs}E")
            levels = {t.split()[1] for t in insn if t.startswith("s_setprio")}
            assert levels == ({"0", "1", "2", "3"} if d == 128 else set()), (d, dtype, levels)


def test_prefill_sums_leave_their_lanes_in_order():
    """A lane's sums are four output elements in a row, sixteen bytes a store, and no lane exchanges any with another."""
    asm = device_assembly("prefill_kernels.hip")
    for seqs in (127, 447):
        for d, dtype in ((128, 0), (64, 0), (128, 1), (64, 1)):
            name = f"9k_prefillILi{d}ELi{dtype}ELi{seqs}E"
            insn, _, _ = kernel_body(asm, name)
            stores = [i for i, t in enumerate(insn) if t.startswith("global_store_dwordx4")]
            assert len(stores) == 2 * d // 8, name                  # a part's sums, and rows
            for at in (stores[:len(stores) // 2], stores[len(stores) // 2:]):
                assert not any("permlane" in t for t in insn[at[0]:at[-1]]), name


def test_prefill_rings_of_short_walks_leave_room():
    """The e4m3 kernel whose waves meet once in two pairs holds half the LDS of the other one, so that a third work-group fits on a
    CU beside two; both keep to the registers of two."""
    asm = device_assembly("prefill_kernels.hip")
    for seqs in (127, 447):
        lds = {}
        for meet in (2, 4):
            name = f"9k_prefillILi128ELi1ELi{seqs}ELi{meet}E"
            found = re.findall(r"\.group_segment_fixed_size:\s+(\d+)(?:(?!\.group_segment_fixed_size)[\s\S])*?\.name:\s+\S*" + name, asm)
            vg = re.findall(r"\.name:\s+\S*" + name + r"\S*\s*\n(?:.*\n){0,40}?\s+\.vgpr_count:\s+(\d+)", asm)
            assert len(found) == 1 and len(vg) == 1 and int(vg[0]) <= 256, (name, found, vg)
            lds[meet] = int(found[0])
        assert 3 * lds[2] <= 160 * 1024 < 3 * lds[4], lds
