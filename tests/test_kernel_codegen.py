"""Properties of the compiled gfx950 code that the kernels' timing rests on and that a change
elsewhere in the source can silently undo (the compiler decides them, not the source text).

The device code of the library is compiled to assembly text (no GPU needed, about half a minute) and
read as text:

* the GEMM kernels that feed B fragments through LDS issue their global -> LDS transfers from
  assembly statements the compiler cannot see.  A wait for outstanding vector memory operations that
  the compiler places BETWEEN two such transfers (for a load of its own that it moved up) makes the
  wave wait for every transfer in turn; the kernels start their filling code with a wait the compiler
  does see, so that it has nothing left to wait for.  Measured cost when it went wrong: 49 -> 65 us per
  gate/up launch at 56 rows.  In bat_gemm_wide the transfers are spread over the products of a k-step: there the loop of
  products may hold the kernel's own counted waits, one per k-step, and no other wait for vector memory.
* the products of bat_gemm_wide's three- and four-wave tiles are assembly too, so the compiler does not know when their results
  are there: nothing in the loop may move an accumulator (the kernel waits before it reads them at the end).
* the GEMM kernels of the per-layer hot path use no scratch memory (register spills cost about 3 us per
  launch on the 8-row kernels).  For the persistent whole-step kernel this is the property that decides
  whether it works at all: a reload from scratch is a vector memory operation that returns behind every
  weight fragment the wave has in flight, and what forced its descriptors and loop-invariant per-lane
  values into scratch (a descriptor copied out of global memory, a load through a selected address,
  values hoisted out of the loop over phases) is invisible in the source.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def device_asm(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    from paper_2603_17573_amd import build as b
    out = str(tmp_path_factory.mktemp("asm") / "heisd_device.s")
    flags = [f for f in b.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    cmd = [HIPCC] + flags + ["--cuda-device-only", "-S"] + b.SOURCES + ["-o", out]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert proc.returncode == 0, proc.stdout
    return open(out).read()


def kernel_bodies(asm, pattern):
    """{mangled name: [instructions]} of the kernels whose name matches pattern."""
    out = {}
    for m in re.finditer(r"^(_Z\w+):", asm, flags=re.M):
        name = m.group(1)
        if not re.search(pattern, name):
            continue
        end = asm.find("s_endpgm", m.end())
        lines = [ln.strip() for ln in asm[m.end():end].split("\n")]
        out[name] = [ln for ln in lines if ln and not ln.startswith(";") and not ln.startswith(".")]
    return out


def waits_between_transfers(instr):
    """Count the vector-memory waits that are followed, within a few instructions, by another
    global -> LDS transfer of the same run of transfers."""
    bad = 0
    for i, ins in enumerate(instr):
        if not ins.startswith("global_load_lds"):
            continue
        nxt = instr[i + 1:i + 12]
        for k, t in enumerate(nxt):
            if t.startswith("global_load_lds"):
                break
            if t.startswith("s_waitcnt") and "vmcnt" in t:
                if any(x.startswith("global_load_lds") for x in nxt[k + 1:k + 8]):
                    bad += 1
                break
    return bad


def test_scanner_sees_a_planted_wait():
    good = ["s_mov_b32 m0, s1", "global_load_lds_dwordx4 v[0:1], off", "s_mov_b32 m0, s2",
            "global_load_lds_dwordx4 v[2:3], off", "s_waitcnt vmcnt(0)", "s_barrier"]
    bad = good[:2] + ["s_waitcnt vmcnt(0)"] + good[2:]
    assert waits_between_transfers(good) == 0
    assert waits_between_transfers(bad) == 1


def test_no_compiler_wait_between_lds_transfers(device_asm):
    bodies = kernel_bodies(device_asm, r"bat_gemm_(ns|wide)|persist_forward")
    assert len(bodies) >= 10, sorted(bodies)
    for name, instr in bodies.items():
        assert any(i.startswith("global_load_lds") for i in instr), name
        assert waits_between_transfers(instr) == 0, name


def product_blocks(asm):
    """{name: (waves, AW, CW, OCC, [instructions of every basic block with matrix products])} of the bat_gemm_wide kernels."""
    out = {}
    for m in re.finditer(r"^(_Z\w*bat_gemm_wideI\w*TileShapeILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E\w*):", asm, flags=re.M):
        wa, wc, aw, cw, occ = (int(m.group(k)) for k in range(2, 7))
        blocks = [[]]
        for ln in asm[m.end():asm.find(".Lfunc_end", m.end())].split("\n"):
            ln = ln.strip()
            if re.match(r"\.LBB\w+:", ln):
                blocks.append([])
            elif ln and ln[0] not in ";.":
                blocks[-1].append(ln)
                if ln.startswith(("s_cbranch", "s_branch")):
                    blocks.append([])
        out[m.group(1)] = (wa, wc, aw, cw, occ, [b for b in blocks if any(i.startswith("v_mfma") for i in b)])
    return out


def loop_faults(wa, wc, aw, cw, occ, block):
    """What a block of whole k-steps of products must not hold: see the module's docstring."""
    slots = min(8, (78 if occ == 2 else 156) // (wa * aw + wc * cw))          # the ring, and transfers per wave and k-step
    ops = -(-(wa * aw + wc * cw) // (wa * wc))
    steps, rest = divmod(sum(i.startswith("v_mfma") for i in block), aw * cw)
    faults = ["part of a k-step"] if rest else []
    if sum(i.startswith("global_load_lds") for i in block) != steps * ops:
        faults.append("transfers")
    waits = [i for i in block if i.startswith("s_waitcnt") and "vmcnt" in i]
    if waits != ["s_waitcnt vmcnt(%d)" % ((slots - 3) * ops)] * steps:
        faults.append("waits %s" % waits)
    if any("accvgpr" in i for i in block):
        faults.append("accumulators moved")
    return faults


def test_loop_of_spread_transfers(device_asm):
    kernels = product_blocks(device_asm)
    assert len(kernels) >= 32, sorted(kernels)
    for name, (*shape, blocks) in kernels.items():
        assert len(blocks) == 2, name                                         # two k-steps, and an odd last one
        for b in blocks:
            assert loop_faults(*shape, b) == [], name
        # a wait planted anywhere among the products is seen, and so is a moved accumulator
        b = blocks[0]
        for at in [k for k, i in enumerate(b) if i.startswith("v_mfma")][1::3]:
            assert loop_faults(*shape, b[:at] + ["s_waitcnt vmcnt(0)"] + b[at:]), (name, at)
            assert loop_faults(*shape, b[:at] + ["s_waitcnt vmcnt(0) lgkmcnt(0)"] + b[at:]), (name, at)
            assert loop_faults(*shape, b[:at] + ["v_accvgpr_read_b32 v0, a0"] + b[at:]), (name, at)


def test_only_lds_reads_write_fragments_in_the_loop(device_asm):
    """Among the products of the three- and four-wave tiles, which the compiler does not know to be products, the only vector instructions are
    address sums: a fragment moved by the vector ALU would need wait states in front of the product that reads it."""
    kernels = product_blocks(device_asm)
    seen = 0
    for name, (wa, wc, aw, cw, occ, blocks) in kernels.items():
        if wa * wc > 4:
            continue
        seen += 1
        for b in blocks:
            inside = b[next(k for k, i in enumerate(b) if i.startswith("v_mfma")):len(b) - next(k for k, i in enumerate(b[::-1]) if i.startswith("v_mfma"))]
            other = [i for i in inside if i.startswith("v_") and not i.startswith(("v_mfma", "v_add_u32"))]
            assert not other, (name, other[:3])
    assert seen >= 30, seen


def test_hot_kernels_use_no_scratch(device_asm):
    strict = r"(fast_gemm_kernel|fast_gemm_short_kernel|fast_gemm_stream_kernel|fast_lmhead_accept|argmax_accept|fast_attn_kernel|persist_forward|bat_gemm_ns|bat_gemm_wide|bat_split_finish|retrieve_scores|retrieve_scan_mfma|pair_similarity|skip_decide|attn_verifyI)"
    lenient = r"heisd8bat_gemmILi"          # a few set-up values outside the loop of products: at most 64 bytes
    seen = 0
    for m in re.finditer(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", device_asm, flags=re.S):
        name, block = m.group(1), m.group(2)
        size = int(re.search(r"\.amdhsa_private_segment_fixed_size\s+(\d+)", block).group(1))
        if re.search(strict, name):
            seen += 1
            assert size == 0, (name, size)
        elif re.search(lenient, name):
            seen += 1
            assert size <= 64, (name, size)
    assert seen >= 117, seen                # all instantiations of today: fewer means that a pattern no longer matches
