"""Static check of the two kernels whose matrix products and waits are written by hand: the direct-load prefill
contraction (prefill_mma_kernel) and the direct-load down-projection GEMM (down_gemm_dma_kernel).

Their products are inline assembly, so the compiler adds no wait states between a product and what writes its operands or
reads its result, and their operands are loaded straight into LDS, so every wait for them is counted by hand.  The test
compiles both files to assembly and follows every instantiation's instructions along all branches:

* a register with a load in flight (global memory or LDS, in-order counters vmcnt and lgkmcnt) is neither read nor written;
* no vector instruction writes a register that a product reads within the next two wait states;
* no other instruction reads or writes a product's result before the product has left the pipe;
* each k-step of the main loops issues the direct loads that its tile calls for, and its one counted wait leaves no load
  in flight that the next step, by the schedule of the LDS rings, reads.

The batched gate/up kernels are read for the kind of their weight rows' loads.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_06822_amd", "csrc")

WRITE_TO_PRODUCT = 2                       # wait states between a vector write and a product that reads it
PRODUCT_TO_READ = {"16x16x32": 11, "32x32x16": 19}  # between a product and another instruction that touches its result


# ---------------------------------------------------------------- instructions

_REG = re.compile(r"(?<![\w.$])([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _registers(text):
    out = set()
    for m in _REG.finditer(text):
        lo, hi = (m.group(2), m.group(3)) if m.group(2) else (m.group(4), m.group(4))
        out.update((m.group(1), i) for i in range(int(lo), int(hi) + 1))
    return out


class Ins:
    def __init__(self, line):
        self.text = line
        self.op = line.split()[0]
        args = [a.strip() for a in line[len(self.op):].split(",")]
        op = self.op
        no_result = op.startswith(("global_store", "ds_write", "buffer_store", "scratch_store", "global_load_lds", "s_",
                                   "v_cmpx", "global_atomic")) or (op.startswith("ds_") and "_rtn" not in op and
                                                                  not op.startswith(("ds_read", "ds_bpermute", "ds_permute")))
        self.dst = set() if no_result else _registers(args[0])
        self.src = _registers(line[len(op):]) if no_result else _registers(",".join(args[1:]))
        if op.startswith("v_swap"):
            self.src, self.dst = self.src | self.dst, self.src | self.dst
        self.mfma = op.startswith("v_mfma")
        self.valu = op.startswith("v_") and not self.mfma
        self.states = int(args[0]) + 1 if op == "s_nop" else 1
        # in-order counters
        self.vm = op.startswith(("global_load", "global_store", "global_atomic", "buffer_", "scratch_"))
        self.lgkm = op.startswith(("ds_", "s_load", "s_buffer_load"))
        self.loads = self.dst if (self.vm or self.lgkm) else set()
        self.wait = {}
        if op == "s_waitcnt":
            for name in ("vmcnt", "lgkmcnt"):
                m = re.search(name + r"\((\d+)\)", line)
                if m:
                    self.wait[name] = int(m.group(1))
        self.next = []


def parse(lines):
    """Instructions of one function with their successors."""
    code, labels = [], {}
    for raw in lines:
        line = raw.split(";")[0].strip()
        m = re.match(r"([\w.$]+):$", line)
        if m:
            labels[m.group(1)] = len(code)
        elif line and line[0] != ".":
            code.append(Ins(line))
    for i, ins in enumerate(code):
        if ins.op.startswith(("s_branch", "s_cbranch")):
            ins.target = labels[ins.text.split()[1]]
            ins.next.append(ins.target)
        if ins.op not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(code):
            ins.next.append(i + 1)
    return code


# ---------------------------------------------------------------- registers with a load in flight

def loads_in_flight(code):
    """(number of register loads, instructions that touch one before its wait)."""
    bad, n = [], 0
    for i, load in enumerate(code):
        if not load.loads:
            continue
        n += 1
        kind = "vm" if load.vm else "lgkm"
        seen, todo = set(), [(j, 0) for j in load.next]
        while todo:
            j, younger = todo.pop()
            if (j, younger) in seen:
                continue
            seen.add((j, younger))
            ins = code[j]
            if ins.wait.get(kind + "cnt", 1 << 30) <= younger:
                continue
            # (the counter returns loads of one kind in order: a younger load of the same kind may overwrite)
            if (ins.src | (set() if getattr(ins, kind) else ins.dst)) & load.loads:
                bad.append(ins.text)
                continue
            younger = min(younger + (1 if getattr(ins, kind) else 0), 64)
            todo.extend((k, younger) for k in ins.next)
    return n, bad


# ---------------------------------------------------------------- wait states around products

def _within(code, start, states, hit):
    """Instructions reached from `start` after fewer than `states` wait states for which hit(instruction) holds."""
    out, best, todo = [], {}, [(j, 0) for j in code[start].next]
    while todo:
        j, passed = todo.pop()
        if passed >= states or best.get(j, 1 << 30) <= passed:
            continue
        best[j] = passed
        if hit(code[j]):
            out.append(code[j].text)
            continue
        todo.extend((k, passed + code[j].states) for k in code[j].next)
    return out


def product_hazards(code):
    """(products, pairs of instructions that are too close)."""
    bad, n = [], 0
    for i, ins in enumerate(code):
        if ins.mfma:
            n += 1
            shape = re.search(r"(\d+x\d+x\d+)", ins.op).group(1)
            if shape not in PRODUCT_TO_READ:
                continue  # (FP64 products: intrinsics, the compiler's own)
            res = ins.dst
            # another product may add to exactly this result (the pipe forwards it), nothing else may touch it
            bad += [(ins.text, t) for t in _within(code, i, PRODUCT_TO_READ[shape], lambda o: not (
                o.mfma and o.dst == res and not _registers(",".join(o.text.split(",")[1:3])) & res) and (o.src | o.dst) & res)]
        elif ins.valu and ins.dst:
            bad += [(ins.text, t) for t in _within(code, i, WRITE_TO_PRODUCT, lambda o: o.mfma and o.src & ins.dst)]
    return n, bad


# ---------------------------------------------------------------- the counted waits of the main loops

def counted_waits(code):
    """Per main loop (a backward branch around products with one wait of the form vmcnt(n) lgkmcnt(0) + barrier): loads into
    LDS before and after that wait within a k-step, n, and the products of a k-step."""
    out = []
    for end, br in enumerate(code):
        if not br.op.startswith(("s_branch", "s_cbranch")) or br.target > end:
            continue
        body = code[br.target:end + 1]
        if any(b.op.startswith(("s_branch", "s_cbranch")) and b is not br for b in body):
            continue  # (an outer loop, or none of the pipelined ones)
        waits = [k for k, b in enumerate(body[:-1]) if b.wait.get("vmcnt", 0) > 0 and b.wait.get("lgkmcnt") == 0
                 and body[k + 1].op == "s_barrier"]
        if not waits:
            continue
        assert len(waits) == 1, "one counted wait per k-step"
        w = waits[0]
        assert not [b for k, b in enumerate(body) if k != w and "vmcnt" in b.wait], "no other wait for loads in a k-step"
        assert sum(b.op == "s_barrier" for b in body) == 1
        lds = [b.op.startswith("global_load_lds") for b in body]
        assert not [b for b, l in zip(body, lds) if b.vm and not l], "no other vector memory traffic in a k-step"
        out.append((sum(lds[:w]), sum(lds[w:]), body[w].wait["vmcnt"], sum(b.mfma for b in body)))
    return out


def most_left_in_flight(na, nb, pa, pb, channels):
    """The largest vmcnt for the wait in the middle of a k-step.  Step s requests the weight rows of step s + nb - 1 (and,
    with `channels`, first the channel numbers of the weight rows it will request two steps on), waits, and requests the
    token rows of step s + na; after the wait step s + 1 reads its rows, and requests weight rows by their channel numbers."""
    order = []
    for s in range(-8, 9):
        if channels:
            order.append(("c", s + nb + 1))
        order += [("b", s + nb - 1)] * pb
        order.append(("wait", s))
        order += [("a", s + na)] * pa
    best = None
    for i, (what, s) in enumerate(order):
        if what != "wait" or not 0 <= s < 4:
            continue
        needed = [k for k in range(i) if order[k] in (("a", s + 1), ("b", s + 1), ("c", s + 1 + nb - 1))]
        left = sum(o[0] != "wait" for o in order[max(needed) + 1:i])
        best = left if best is None else min(best, left)
    return best


# ---------------------------------------------------------------- the same in the order of the listing

def _regs(tok):
    out = set()
    for m in re.finditer(r"v\[(\d+):(\d+)\]", tok):
        out.update(range(int(m.group(1)), int(m.group(2)) + 1))
    for m in re.finditer(r"(?<![\w\[:])v(\d+)\b", tok):
        out.add(int(m.group(1)))
    return out


def replay(lines):
    """Returns (number of loads seen, list of offending instructions)."""
    vmq, lgq, bad, n_loads = [], [], [], 0
    for raw in lines:
        line = raw.strip()
        if not line or line[0] in ";.":
            continue
        op = line.split()[0]
        parts = [a.strip() for a in line[len(op):].split(",")]
        if op == "s_waitcnt":
            for name, queue in (("vmcnt", vmq), ("lgkmcnt", lgq)):
                m = re.search(name + r"\((\d+)\)", line)
                if m:
                    del queue[:max(0, len(queue) - int(m.group(1)))]
            continue
        dst = _regs(parts[0]) if parts else set()
        src = set().union(*[_regs(a) for a in parts[1:]]) if len(parts) > 1 else set()
        if op.startswith(("global_store", "ds_write")):
            src, dst = src | dst, set()
        pending = set().union(*vmq, *lgq) if (vmq or lgq) else set()
        if op.startswith("global_load_lds"):          # direct load: no register result
            if (src | dst) & pending:
                bad.append(line)
            vmq.append(set())
        elif op.startswith("global_load"):
            if src & pending:
                bad.append(line)
            vmq.append(dst)
            n_loads += 1
        elif op.startswith("ds_read"):
            if src & pending:
                bad.append(line)
            lgq.append(dst)
            n_loads += 1
        elif op.startswith(("s_load", "s_buffer_load")):
            lgq.append(set())
        elif (src | dst) & pending:
            bad.append(line)
    return n_loads, bad


def test_replay_flags_a_planted_hazard():
    ok = ["global_load_dword v5, v[6:7], off", "s_waitcnt vmcnt(0)", "v_add_u32_e32 v1, v5, v2"]
    assert replay(ok) == (1, [])
    early = ["global_load_dword v5, v[6:7], off", "v_add_u32_e32 v1, v5, v2", "s_waitcnt vmcnt(0)"]
    assert replay(early)[1] == ["v_add_u32_e32 v1, v5, v2"]
    reused = ["ds_read_b128 v[8:11], v3", "ds_read_b128 v[12:15], v4", "s_waitcnt lgkmcnt(1)",
              "v_mov_b32_e32 v12, 0", "v_mov_b32_e32 v8, 0"]
    assert replay(reused)[1] == ["v_mov_b32_e32 v12, 0"]


# ---------------------------------------------------------------- planted mistakes

def test_a_register_with_a_load_in_flight_is_found():
    def run(*lines):
        return loads_in_flight(parse(list(lines)))
    assert run("global_load_dword v5, v[6:7], off", "s_waitcnt vmcnt(0)", "v_add_u32_e32 v1, v5, v2") == (1, [])
    assert run("global_load_dword v5, v[6:7], off", "v_add_u32_e32 v1, v5, v2", "s_waitcnt vmcnt(0)")[1] == \
        ["v_add_u32_e32 v1, v5, v2"]
    assert run("ds_read_b128 v[8:11], v3", "ds_read_b128 v[12:15], v4", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v12, 0",
               "v_mov_b32_e32 v8, 0")[1] == ["v_mov_b32_e32 v12, 0"]
    # the wait stands on the fall-through path only
    assert run("global_load_dword v5, v[6:7], off", "s_cbranch_scc1 .L1", "s_waitcnt vmcnt(0)", ".L1:",
               "v_add_u32_e32 v1, v5, v2")[1] == ["v_add_u32_e32 v1, v5, v2"]


def test_an_operand_written_just_before_its_product_is_found():
    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"

    def run(*lines):
        return len(product_hazards(parse(list(lines) + ["s_endpgm"]))[1])
    assert run("v_perm_b32 v4, v8, v9, s0", "s_nop 1", mfma) == 0
    assert run("v_perm_b32 v4, v8, v9, s0", "s_nop 0", mfma) == 1
    assert run("v_accvgpr_write_b32 a3, v8", mfma) == 1
    assert run("v_mov_b32_e32 v9, 0", mfma) == 0
    assert run("v_mov_b32_e32 v3, 0", "s_branch .L2", "s_nop 1", ".L2:", mfma) == 1


def test_a_result_read_before_its_product_is_done_is_found():
    mfma = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"

    def run(*lines):
        return len(product_hazards(parse(list(lines) + ["s_endpgm"]))[1])
    assert run(mfma, mfma) == 0
    assert run(mfma, "s_nop 15", "v_accvgpr_read_b32 v8, a2") == 0
    assert run(mfma, "s_nop 7", "v_accvgpr_read_b32 v8, a2") == 1
    assert run(mfma, "v_accvgpr_write_b32 a0, 0") == 1
    assert run(mfma, "v_mfma_f32_16x16x32_bf16 a[4:7], v[0:3], a[0:3], a[4:7]") == 1
    # round a loop
    assert run(".L1:", "v_accvgpr_read_b32 v8, a2", mfma, "s_cbranch_scc1 .L1") == 1


def test_the_schedule_of_the_rings():
    # two buffers of token rows: the rows of step s + 1 are requested in step s - 1, right before the weight rows of step s
    assert most_left_in_flight(2, 4, 4, 6, False) == 6
    # deeper rings leave whole k-steps in flight
    assert most_left_in_flight(4, 5, 2, 6, False) == min(3 * 6 + 2 * 2, 3 * (2 + 6))
    assert most_left_in_flight(3, 3, 6, 4, True) == min(2 * 5 + 6, 6 + 5, 6 + 2 * 4 + 1)


# ---------------------------------------------------------------- the kernels

needs_hipcc = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """The listings of every instantiation of the two kernels."""
    found = {}
    for src, kernel in (("pop_down_gemm.hip", "down_gemm_dma_kernel"), ("pop_prefill.hip", "prefill_mma_kernel")):
        out = tmp_path_factory.mktemp("asm") / (src + ".s")
        cmd = ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
               os.path.join(CSRC, src), "-o", str(out)]
        subprocess.run(cmd, check=True, capture_output=True, timeout=900)
        bodies, name = {}, None
        for line in out.read_text().split("\n"):
            m = re.match(r"(_ZN3pop\d+" + kernel + r"I\w+):", line)
            if m:
                name = m.group(1)
                bodies[name] = []
            elif line.startswith(".Lfunc_end"):
                name = None
            elif name:
                bodies[name].append(line)
        found[src] = bodies
    return found


@needs_hipcc
def test_direct_load_gemm_touches_no_register_with_a_load_in_flight(assembly):
    """In the order of the listing, every instantiation of the GEMM (the walks along all branches are further down)."""
    bodies = assembly["pop_down_gemm.hip"]
    assert len(bodies) == 5
    for name, body in bodies.items():
        n_loads, bad = replay(body)
        assert n_loads > 40, "the kernel's loads (LDS fragments, channel numbers) were not found"
        assert not bad, (name, bad[:5])


@needs_hipcc
def test_down_projection_gemm(assembly):
    found = {name: parse(body) for name, body in assembly["pop_down_gemm.hip"].items()}
    assert len(found) == 5
    for name, code in found.items():
        mf = int(re.search(r"ILi(\d)E", name).group(1))
        assert not loads_in_flight(code)[1], name
        n, bad = product_hazards(code)
        assert n == 2 * mf * 8 and not bad, (name, n, bad[:4])
        na, nb = {5: 2, 4: 3, 3: 3}.get(mf, 4), 3 if mf == 4 else 4
        loops = counted_waits(code)
        assert len(loops) == 1, name
        before, after, left, products = loops[0]
        assert (before, after, products) == (5, 2 * mf, 16 * mf), (name, loops)
        assert left == most_left_in_flight(na, nb, 2 * mf, 4, True), (name, left)


@needs_hipcc
def test_prefill_contraction(assembly):
    found = {name: parse(body) for name, body in assembly["pop_prefill.hip"].items()}
    assert len(found) == 5 * 3 + 2
    for name, code in found.items():
        mf, mode = (int(v) for v in re.search(r"ILi(\d)ELi(\d)E", name).groups())
        assert not loads_in_flight(code)[1], name
        bad = product_hazards(code)[1]
        assert not bad, (name, bad[:4])
        na, nb = 2 if mf >= 4 else (3 if mf >= 2 else 4), 3 if mf >= 3 else (4 if mf == 2 else 5)
        loops = counted_waits(code)
        assert sorted(p // (2 * mf) for _, _, _, p in loops) == [4, 6, 7, 8, 10, 11, 12], (name, loops)
        for before, after, left, products in loops:
            pb = (products // (2 * mf) + 1) // 2
            assert (before, after) == (pb, 2 * mf), (name, loops)
            assert left == most_left_in_flight(na, nb, 2 * mf, pb, False), (name, before, left)


@needs_hipcc
def test_prefill_contraction_with_three_steps_of_token_rows(tmp_path):
    out = tmp_path / "pop_prefill.s"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
                    os.path.join(CSRC, "pop_prefill.hip"), "-o", str(out)], check=True, capture_output=True, timeout=900)
    bodies = re.findall(r"^_ZN3pop\d+prefill_deep_kernelI\w+:(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S)
    assert len(bodies) == 2
    for body in bodies:
        code = parse(body.split("\n")[1:])
        assert not loads_in_flight(code)[1]
        assert not product_hazards(code)[1]
        loops = counted_waits(code)
        assert sorted(p // 8 for _, _, _, p in loops) == [4, 6, 7, 8]
        for before, after, left, products in loops:
            pb = (products // 8 + 1) // 2
            assert (before, after, left) == (pb, 8, most_left_in_flight(3, 3, 8, pb, False))


@needs_hipcc
def test_batched_gate_up_rows_are_global_loads(tmp_path):
    """The weight rows of the batched gate/up kernels are read by global loads (a flat load counts as an LDS operation too, and the
    kernels read x from LDS between the rows); the decode step's kernel of bf16 layers requests a group of 2 U row vectors
    together and the first wait behind them leaves some of the group in flight."""
    out = tmp_path / "pop_gemv.s"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
                    os.path.join(CSRC, "pop_gemv.hip"), "-o", str(out)], check=True, capture_output=True, timeout=900)
    bodies = re.findall(r"^_ZN3pop\d+(gateup_(?:select_)?kernel)INS_\d+(VecBF16|VecF32)ELi(\d)\w+:(.*?)^\.Lfunc_end", out.read_text(),
                        re.M | re.S)
    assert len(bodies) == 2 * (8 + 7)
    for kernel, vec, batch, body in bodies:
        code = parse(body.split("\n")[1:])
        assert not [i.text for i in code if i.op.startswith("flat_")], (kernel, vec, batch)
        if kernel == "gateup_kernel" or vec == "VecF32":  # (float32 rows: spilled registers come back in between)
            continue
        together, waits = 0, []
        for i in code:
            together += i.op == "global_load_dwordx4"
            if "vmcnt" in i.wait:
                if together >= 2 * (8 if int(batch) < 5 else 4):
                    waits.append(i.wait["vmcnt"])
                together = 0
        assert waits and max(waits) > 0, (vec, batch, waits)
