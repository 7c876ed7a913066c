"""Wait states around the instructions that the kernels write out themselves.

The compiler places the wait states that the hardware does not enforce, but it does not look into inline
assembly.  The backward kernels and the wide forward write out matrix instructions with accumulation registers,
all tile loops write out direct-to-LDS loads.  These tests compile the sources to assembly and walk it backwards and
forwards from each such instruction, over branches too:

  a vector instruction that writes an operand of a written-out MFMA: 2 wait states before it
  anything but an MFMA that touches its result:                      19 after it (the longest MFMA)
  a vector instruction that writes the scalar base of a load:        5 before it

The same listings show what else a kernel must not do: write M0 between the loads of a tile, spill vector registers, read its
arguments through vector memory.
"""

import os
import re
import subprocess

import pytest

from paper_2508_10774_amd import build

MFMA_SRC, MFMA_DST, LOAD_BASE = 2, 19, 5


def _regs(text):
    """The registers named in an operand list: {"v4", "a0", "s20", ...}."""
    out = set()
    for kind, lo, hi, one in re.findall(r"\b([vas])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out.update(f"{kind}{i}" for i in (range(int(lo), int(hi) + 1) if lo else [int(one)]))
    if re.search(r"\bvcc\b", text):
        out.add("vcc")
    return out


class Listing:
    """Instructions of one function with their predecessors and successors."""

    def __init__(self, lines):
        self.ins, labels, pending = [], {}, []
        for line in lines:
            inline = "ASMSTART" in line
            line = line.split(";")[0].split("//")[0].strip()
            if inline or not line or line.startswith("."):
                if re.match(r"\.LBB\w+:", line):
                    pending.append(line.split(":")[0])
                continue
            for name in pending:
                labels[name] = len(self.ins)
            pending = []
            op, _, rest = line.partition(" ") if " " in line else line.partition("\t")
            self.ins.append((op.strip(), rest.strip()))
        n = len(self.ins)
        self.succ, self.pred = [[] for _ in range(n)], [[] for _ in range(n)]
        for i, (op, rest) in enumerate(self.ins):
            to = []
            if op.startswith(("s_branch", "s_cbranch")):
                to += [labels[x] for x in re.findall(r"\.LBB\w+", rest) if x in labels]
            if op not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < n:
                to.append(i + 1)
            for t in to:
                self.succ[i].append(t)
                self.pred[t].append(i)

    def _within(self, start, steps, states, stop=lambda j: False):
        """(instruction, wait states between it and `start`) for everything closer than `states`; no further
        than an instruction at which stop() holds."""
        todo, best = [(j, 0) for j in steps[start]], {}
        while todo:
            j, ws = todo.pop()
            if ws >= states or best.get(j, states) <= ws:
                continue
            best[j] = ws
            if stop(j):
                continue
            op, rest = self.ins[j]
            ws += int(rest, 0) + 1 if op == "s_nop" else 1
            todo += [(t, ws) for t in steps[j]]
        return best

    def _writes(self, j):
        op, rest = self.ins[j]
        first = rest.split(",")[0]
        if op.startswith(("v_cmp", "v_div_scale")) or "_co_" in op:
            return _regs(",".join(rest.split(",")[:2]))
        return _regs(first)

    def faults(self):
        found, seen = [], {"mfma": 0, "load": 0}
        for i, (op, rest) in enumerate(self.ins):
            ops = [x.strip() for x in rest.split(",")]
            if op.startswith("v_mfma") and ops[0].startswith("a"):
                seen["mfma"] += 1
                for j in self._within(i, self.pred, MFMA_SRC):
                    o = self.ins[j][0]
                    if o.startswith("v_") and not o.startswith("v_mfma") and self._writes(j) & _regs(rest):
                        found.append(f"{' '.join(self.ins[j])} too close in front of {op} {rest}")
                for j in self._within(i, self.succ, MFMA_DST):
                    o, r = self.ins[j]
                    if not o.startswith("v_mfma") and _regs(r) & _regs(ops[0]):
                        found.append(f"{o} {r} too close behind {op} {rest}")
            if op.startswith("global_load_lds") and "s[" in rest:
                seen["load"] += 1
                for base in (x for x in _regs(rest) if x[0] == "s"):
                    # (a scalar instruction that sets the register anew has waited for the vector one)
                    def anew(j):
                        return self.ins[j][0].startswith("s_") and base in self._writes(j)
                    for j in self._within(i, self.pred, LOAD_BASE, anew):
                        if self.ins[j][0].startswith("v_") and base in self._writes(j):
                            found.append(f"{' '.join(self.ins[j])} too close in front of {op} {rest}")
        return found, seen


def _functions(text):
    for m in re.finditer(r"^(_Z\w+):.*?^\.Lfunc_end\d+:", text, re.M | re.S):
        yield m.group(1), m.group(0).splitlines()[1:]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    running = {src: subprocess.Popen([hipcc, *build.HIPCC_FLAGS, "-S", "--cuda-device-only",
                                      os.path.join(build.CSRC, src), "-o", str(out / src)],
                                     stderr=subprocess.DEVNULL) for src in ("asa_bwd.hip", "asa_fwd.hip", "asa_mask.hip")}
    for src, p in running.items():
        assert p.wait() == 0, src
    return {src: (out / src).read_text() for src in running}


@pytest.mark.parametrize("src,kinds", [("asa_bwd.hip", ("mfma", "load")), ("asa_fwd.hip", ("mfma", "load")),
                                       ("asa_mask.hip", ("load",))])
def test_wait_states_around_written_out_instructions(assembly, src, kinds):
    total = dict.fromkeys(("mfma", "load"), 0)
    for name, lines in _functions(assembly[src]):
        found, seen = Listing(lines).faults()
        assert not found, f"{name}: {found[:4]}"
        for k in total:
            total[k] += seen[k]
    print(src, total)
    assert all(total[k] > 0 for k in kinds)


def _m0_outside_inline_code(text):
    """Instructions of the compiler's own that name M0."""
    inline, found = False, []
    for line in text.splitlines():
        inline = (inline or "ASMSTART" in line) and "ASMEND" not in line
        code = line.split(";")[0]
        if not inline and re.search(r"\bm0\b", code):
            found.append(code.strip())
    return found


def test_only_the_written_out_loads_of_a_tile_set_m0(assembly):
    """Several loads in a row share one write of M0 (lds_dma_begin): the compiler must not use it in between."""
    for name, lines in [*_functions(assembly["asa_fwd.hip"]), *_functions(assembly["asa_bwd.hip"])]:
        if any(x in name for x in ("fwd_wide_kernel", "fwd_pipe_kernel", "fwd_kernel", "dkv_kernel", "dq_kernel")):
            assert not _m0_outside_inline_code("\n".join(lines)), name
    planted = "\t;;#ASMSTART\n\ts_mov_b32 m0, s1\n\t;;#ASMEND\n\ts_mov_b32 m0, s2"
    assert _m0_outside_inline_code(planted) == ["s_mov_b32 m0, s2"]


# (at the ends of its walk, two groups of wavefronts with a walk each)
SPILLS_ALLOWED = {"fwd_pp_kernelILi128ELi128ELb0E": 5}


@pytest.mark.parametrize("src,kernels", [("asa_mask.hip", 4), ("asa_fwd.hip", 20), ("asa_bwd.hip", 12)])
def test_no_vector_registers_are_spilled(assembly, src, kernels):
    """A reload waits for the copies that a loop over tiles has in flight."""
    spills = re.findall(r"\.name:\s+(\S+)[\s\S]*?\.vgpr_spill_count:\s+(\d+)", assembly[src])
    assert sum(any(x in name for x in ("probe_", "fwd_", "dq_", "dkv_")) for name, _ in spills) >= kernels
    for name, n in spills:
        assert int(n) <= sum(v for k, v in SPILLS_ALLOWED.items() if k in name), name


def _argument_loads(lines):
    """Vector loads from the kernel's arguments (s[0:1] until something else is put there)."""
    found = []
    for line in lines:
        code = line.split(";")[0].strip()
        if re.match(r"global_load_(?!lds)\w+ .*, s\[0:1\]", code):
            found.append(code)
        if re.match(r"s_\w+ s(0|1|\[0:\d+\])\s*,", code):
            break
    return found


def test_kernel_arguments_are_read_by_scalar_loads(assembly):
    """An argument array that is indexed per lane becomes a load from the memory that holds the arguments, and all that
    depends on it waits for that: the probe's sample positions come out of scalar registers."""
    for src in assembly:
        for name, lines in _functions(assembly[src]):
            assert not _argument_loads(lines), (src, name)
    planted = ["\ts_load_dword s3, s[0:1], 0x78", "\tglobal_load_dword v1, v6, s[0:1] offset:156"]
    assert _argument_loads(planted) and not _argument_loads(["\ts_mov_b64 s[0:1], s[4:5]", *planted])


LOOP = """.LBB0_1:
\tds_read_b128 v[4:7], v20
\t{front}
\t{wait}
\t;;#ASMSTART
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]
\t;;#ASMEND
\ts_cbranch_scc1 .LBB0_1
\t{behind}
\tv_accvgpr_read_b32 v30, a3
\ts_endpgm"""


@pytest.mark.parametrize("front,wait,behind,faults", [
    ("v_mov_b32_e32 v12, v1", "s_nop 0", "s_nop 15\n\ts_nop 3", 0),
    ("v_mov_b32_e32 v9, v1", "s_nop 0", "s_nop 15\n\ts_nop 3", 1),       # one state in front
    ("v_cvt_pk_bf16_f32 v8, v1, v2", "s_nop 1", "s_nop 15\n\ts_nop 3", 0),
    ("v_mov_b32_e32 v12, v1", "s_nop 0", "s_nop 15", 1),                 # 17 behind (branch included)
    ("v_mov_b32_e32 v12, v1", "s_nop 0", "s_nop 15\n\ts_nop 1", 0),      # 19
])
def test_the_walk_finds_planted_matrix_hazards(front, wait, behind, faults):
    found, seen = Listing(LOOP.format(front=front, wait=wait, behind=behind).splitlines()).faults()
    assert seen["mfma"] == 1 and len(found) == faults, found


@pytest.mark.parametrize("between,faults", [("s_nop 0", 1), ("s_nop 1", 0), ("s_mov_b64 s[8:9], s[4:5]", 0)])
def test_the_walk_finds_planted_load_hazards_over_a_branch(between, faults):
    text = f"""\tv_readfirstlane_b32 s8, v1
\t{between}
\ts_branch .LBB0_2
.LBB0_1:
\ts_endpgm
.LBB0_2:
\ts_mov_b32 m0, s3
\ts_nop 0
\tglobal_load_lds_dwordx4 v2, s[8:9]
\ts_branch .LBB0_1"""
    found, seen = Listing(text.splitlines()).faults()
    assert seen["load"] == 1 and len(found) == faults, found
