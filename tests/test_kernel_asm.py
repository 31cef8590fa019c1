"""Checks on the assembly of the persistent GEMM kernels (compiled here, no GPU needed).

The kernels issue their LDS-direct loads from inline assembly, which hides three things from the compiler that it
would otherwise take care of; each is checked on the generated code:

* a scalar register written by a vector instruction (a base address reloaded with v_readlane, made uniform with
  v_readfirstlane) must not be read by a vector memory instruction within the next five wait states;
* a load that reuses M0 (the runs of pieces that move by the instruction offset) must follow the load that set
  M0 with no other M0 write in between;
* no basic block of the K loops of the kernels the default dispatch takes may hold a wait for ALL outstanding
  vector memory operations: the compiler puts one in front of any copy of a pending atomic's reply (the tile
  draw), and inside the loop that undoes the load pipeline (it has: twice the time per slice).

The accumulators of the wide kernels are AGPRs that only inline assembly names.  To the compiler they are free: short of
vector registers it spills into them, silently and with wrong results (it has, at 256 VGPRs, without a count of spills).
"""
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_18663_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = ["w4ax_gemm_wide.hip", "w4a4_fp6_gemm.hip", "w4ax_gemm.hip"]

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")


def _flags():
    import importlib.util
    spec = importlib.util.spec_from_file_location("dvdq_build", os.path.join(ROOT, "paper_2505_18663_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return [f for f in mod.HIPCC_FLAGS if f not in ("-Wall",)]


@pytest.fixture(scope="module")
def listings():
    """{kernel symbol: its assembly} of every GEMM kernel in SOURCES"""
    out = {}
    with tempfile.TemporaryDirectory() as tmp:
        procs = []
        for src in SOURCES:
            asm = os.path.join(tmp, src + ".s")
            cmd = [HIPCC, *_flags(), "-w", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-S",
                   os.path.join(CSRC, src), "-o", asm]
            procs.append((src, asm, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        for src, asm, proc in procs:
            log, _ = proc.communicate()
            assert proc.returncode == 0, f"{src}:\n{log}"
            text = open(asm).read()
            for part in re.split(r"\n(?=\S+:\s*; @)", text):
                m = re.match(r"(\S+):", part)
                if not m or "gemm" not in m.group(1) or "prepack" in m.group(1):
                    continue
                out[m.group(1)] = part
    assert len(out) >= 10, sorted(out)
    return out


@pytest.fixture(scope="module")
def kernels(listings):
    """{kernel symbol: list of instruction lines and labels}"""
    out = {}
    for name, part in listings.items():
        lines = []
        for line in part.split("\n")[1:]:
            t = line.strip()
            if not t or t.startswith(";"):
                continue
            if re.match(r"\.LBB\d+_\d+:", t):
                lines.append(t.split(":")[0] + ":")
            elif not t.startswith("."):
                lines.append(t.split(";")[0].strip())
        out[name] = lines
    return out


def _sregs(token):
    m = re.match(r"s\[(\d+):(\d+)\]", token)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"s(\d+)$", token)
    return {int(m.group(1))} if m else set()


def _blocks(lines):
    blocks, cur = [], []
    for t in lines:
        if t.endswith(":"):
            if cur:
                blocks.append(cur)
            cur = []
            continue
        cur.append(t)
        if t.startswith(("s_cbranch", "s_branch", "s_endpgm", "s_setpc")):
            blocks.append(cur)
            cur = []
    if cur:
        blocks.append(cur)
    return blocks


def test_no_vector_written_scalar_register_is_read_by_a_memory_instruction_too_early(kernels):
    for name, lines in kernels.items():
        ins = [t for t in lines if not t.endswith(":")]
        for i, x in enumerate(ins):
            if not re.match(r"(global_|buffer_|flat_|scratch_)", x):
                continue
            need = set()
            for op in x.split(None, 1)[1].split(","):
                need |= _sregs(op.strip().split()[0]) if op.strip() else set()
            states, j = 0, i - 1
            while need and j >= 0 and states < 5:
                y = ins[j]
                op = y.split()[0]
                if op.startswith(("v_readlane", "v_readfirstlane")):
                    dst = y.split(None, 1)[1].split(",")[0].strip()
                    assert not (_sregs(dst) & need), f"{name}: {' | '.join(ins[j:i + 1])}"
                states += int(y.split()[1]) + 1 if op == "s_nop" else 1
                j -= 1


def test_loads_that_reuse_m0_follow_the_load_that_set_it(kernels):
    chained = 0
    for name, lines in kernels.items():
        for block in _blocks(lines):
            m0_fresh = False   # M0 was set for an LDS-direct load earlier in this block and not written since
            for t in block:
                if re.search(r"\bm0\b", t) and not t.startswith("global_load_lds"):
                    m0_fresh = t.startswith("s_mov_b32 m0")
                    continue
                if t.startswith("global_load_lds_dwordx4") and "offset:" in t:
                    chained += 1
                    # (a run may span blocks -- the common path between two MFMA slots has no M0 write at all -- so
                    # only a foreign M0 write inside the block is an error here; the sequence test below covers order)
                    assert m0_fresh or not any(re.search(r"\bm0\b", u) and not u.startswith(("global_load_lds", "s_mov_b32 m0"))
                                               for u in block), f"{name}: {t}"
        # in program text every run reads: M0 write, first load, then its offset loads in ascending order
        seq = [t for t in lines if t.startswith("s_mov_b32 m0") or t.startswith("global_load_lds_dwordx4")]
        last_off = None
        for t in seq:
            if t.startswith("s_mov_b32 m0"):
                last_off = -1
            elif "offset:" in t:
                off = int(t.split("offset:")[1].split()[0], 0)
                assert last_off is not None and last_off >= 0 and off == last_off + 1024, f"{name}: {t} after offset {last_off}"
                last_off = off
            else:
                assert last_off == -1, f"{name}: a first load of a run without its M0 write: {t}"
                last_off = 0
    assert chained > 0


# every persistent GEMM kernel of the three files
HOT = ("w4ax_gemm_wide_kernel", "w4a4_fp6_gemm_kernel", "w4ax_gemm_native_kernel")


def test_no_wait_for_all_memory_operations_inside_the_k_loops(kernels):
    for name, lines in kernels.items():
        bad = [b for b in _blocks(lines) if any("v_mfma" in t for t in b) and any(re.search(r"s_waitcnt.*vmcnt\(0\)", t) for t in b)]
        if any(h in name for h in HOT):
            assert not bad, f"{name}: {bad[0][:12]}"
        elif bad:
            print(f"{name}: {len(bad)} block(s) with MFMAs and a full vmcnt wait")


def test_only_inline_assembly_touches_the_accumulators_of_the_wide_kernels(listings):
    wide = {name: part for name, part in listings.items() if "w4ax_gemm_wide_kernel" in name}
    assert len(wide) == 6
    for name, part in wide.items():
        inside, seen = False, 0
        for line in part.split("\n")[1:]:
            if "#ASMSTART" in line or "#ASMEND" in line:
                inside = "#ASMSTART" in line
                continue
            t = line.split(";")[0].strip()
            if t.startswith(".") or not re.search(r"accvgpr|\ba\d+\b|\ba\[", t):
                continue
            assert inside, f"{name}: {t}"
            seen += 1
        assert seen > 256, name
