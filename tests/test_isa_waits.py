"""What the assembly statements of the kernels take for granted about the code around them, checked in the
compiler's output for gfx950 (CPU only).

The loads straight into LDS are assembly, so the compiler neither sees a buffer load in them nor keeps the
distances the hardware asks for: a load that reads a scalar register which a vector instruction wrote must issue at
least five wait states later, or it may see the register's old value.  Their LDS address has 16 bits, so the staged
tiles have to lie in the first 64 KB of a kernel's LDS: they are the start of its only object.  And they overwrite
m0, which the compiler does not save for them."""
import os
import re
import subprocess

import pytest

from paper_2502_01776_amd import build as B

WAIT_STATES = 5
INF = 1 << 20

pytestmark = pytest.mark.skipif(not os.path.exists(B.hipcc_path()), reason="needs hipcc")


def registers(operand):
    """Scalar registers named by an operand: s7, s[4:7], vcc."""
    operand = operand.strip()
    m = re.fullmatch(r"s(\d+)", operand)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else set()


class Kernel:
    def __init__(self, name):
        self.name, self.ins, self.labels = name, [], {}      # ins: (mnemonic, [operands], inside an assembly statement)

    def predecessors(self):
        pred = [[] for _ in self.ins]
        for i, (op, args, _) in enumerate(self.ins):
            if op.startswith(("s_branch", "s_cbranch")):
                at = self.labels[args[0]]
                if at < len(self.ins):
                    pred[at].append(i)
            if i + 1 < len(self.ins) and op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                pred[i + 1].append(i)
        return pred

    def direct_loads(self):
        return [i for i, (op, args, asm) in enumerate(self.ins) if asm and op.startswith("buffer_load") and args[-1].endswith(" lds")]

    def nearest_vector_write(self, at, pred):
        """Fewest wait states between a vector instruction that writes one of the load's scalar registers and the load."""
        wanted = set().union(*(registers(a) for arg in self.ins[at][1] for a in arg.split()))
        best, seen, work = INF, {}, [(p, 0) for p in pred[at]]
        while work:
            i, passed = work.pop()
            if passed >= best or seen.get(i, INF) <= passed:
                continue
            seen[i] = passed
            op, args, _ = self.ins[i]
            written = set().union(*(registers(a) for a in args[:2 if "_co_" in op or "div_scale" in op else 1])) if args else set()
            if op.startswith("v_") and written & wanted:
                best = passed
                continue
            passed += int(args[0], 0) + 1 if op == "s_nop" else 1
            if passed < WAIT_STATES:
                work += [(p, passed) for p in pred[i]]
        return best


def parse(text):
    kernels, k, asm = [], None, False
    for line in text.splitlines():
        m = re.match(r"(\w+):\s*; @", line)
        if m:
            k = Kernel(m.group(1))
            kernels.append(k)
        elif k is None:
            continue
        elif line.startswith(".Lfunc_end"):
            k = None
        elif "#ASMSTART" in line or "#ASMEND" in line:
            asm = "#ASMSTART" in line
        elif re.match(r"\.LBB\w+:", line):
            k.labels[line.split(":")[0]] = len(k.ins)
        else:
            code = line.split(";")[0].strip()
            if code and not code.startswith("."):
                op, *rest = code.split(None, 1)
                k.ins.append((op, [a.strip() for a in rest[0].split(",")] if rest else [], asm))
    return kernels


@pytest.fixture(scope="module", params=["svg_attn.hip", "svg_fp8.hip"])
def compiled(request, tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "kernels.s")
    res = subprocess.run([B.hipcc_path(), *B.compile_flags(), "--offload-device-only", "-S", os.path.join(B.CSRC, request.param),
                          "-o", out], check=True, capture_output=True, text=True)
    text = open(out).read()
    kernels = parse(text)
    assert sum(len(k.direct_loads()) for k in kernels) > 0
    return text, kernels, res.stderr


def test_reader_of_the_listing_finds_a_missing_wait():
    """The check itself: a register written four wait states ahead of a load is reported, also across a
    branch; five are enough; the address and offset registers count as well."""
    def listing(gap, written="s6", branch=""):
        return (f"kern:  ; @kern\n.LBB0_1:\n\tv_readfirstlane_b32 {written}, v1\n{branch}\ts_nop {gap}\n\t;;#ASMSTART\n"
                "\ts_mov_b32 m0, s9\n\tbuffer_load_dwordx4 v0, s[4:7], s8 offen lds\n\t;;#ASMEND\n\ts_endpgm\n.Lfunc_end0:\n")
    def nearest(text):
        k, = parse(text)
        at, = k.direct_loads()
        return k.nearest_vector_write(at, k.predecessors())
    assert nearest(listing(2)) == 4 and nearest(listing(2, "s8")) == 4
    assert nearest(listing(3)) == INF and nearest(listing(0, "s9")) == INF
    assert nearest(listing(1, branch="\ts_branch .LBB0_2\n.LBB0_2:\n")) == 4


def test_direct_loads_read_settled_scalar_registers(compiled):
    for k in compiled[1]:
        pred = k.predecessors()
        for at in k.direct_loads():
            n = k.nearest_vector_write(at, pred)
            lines = "; ".join(f"{op} {', '.join(args)}" for op, args, _ in k.ins[max(0, at - 8):at + 1])
            assert n >= WAIT_STATES, f"{k.name}: {n} wait states in front of load {at}: {lines}"


def test_staged_tiles_are_the_only_object_in_lds(compiled):
    """Anything else the compiler puts into LDS could stand in front of the tiles and move them out of reach."""
    text, kernels, _ = compiled
    size = dict(re.findall(r"\.amdhsa_kernel (\w+)\n\s*\.amdhsa_group_segment_fixed_size (\d+)", text))
    for k in kernels:
        if k.direct_loads():
            m = re.search(r"11attn_kernelILi(\d+)ELi\d+ELi(\d+)E", k.name)
            D, keys = map(int, m.groups()) if m else (128, 64)
            tiles = 2 * 2 * keys * D * 2 if m else 8 * keys * D       # two stages of K and V in bf16; four in FP8
            assert tiles <= 65536 and int(size[k.name]) == tiles, k.name


def test_no_accumulator_is_moved_between_the_halves_of_the_register_file(compiled):
    """With more than 256 registers allowed the compiler keeps the accumulators in the second half and moves
    them around every softmax, a third of a tile's instructions."""
    for k in compiled[1]:
        if k.direct_loads():
            moves = [op for op, _, _ in k.ins if op.startswith("v_accvgpr")]
            assert not moves, f"{k.name}: {len(moves)} moves"


def test_m0_is_used_by_the_direct_loads_only(compiled):
    for k in compiled[1]:
        if k.direct_loads():
            other = [(op, args) for op, args, asm in k.ins if not asm and "m0" in args]
            assert not other, f"{k.name}: {other[:3]}"


def test_three_passes_of_profiling_carry_nothing_of_the_pieces(compiled):
    """The loops of either kernel know nothing of each other's walk: without pieces all scalars stay in registers (14 and 10 spilled at 128-row tiles
    otherwise, as one kernel with the pieces 36 and 20), with them 14 are spilled at 128-row tiles (32)."""
    names = [k.name for k in compiled[1] if re.search(r"11attn_kernelILi\d+ELi\d+ELi\d+ELi2E", k.name)]
    spilled = dict(re.findall(r"\.name: +(\w+)\n(?:(?!\.name:).*\n)*?\s*\.sgpr_spill_count: (\d+)", compiled[0]))
    assert len(names) in (0, 8) and 2 * sum("ELb1E" in n for n in names) == len(names)      # (none in the FP8 file)
    for n in names:
        assert int(spilled[n]) <= (16 if "ELi4ELi64ELi2E" in n and "ELb1E" in n else 0), n


def test_kernels_of_profiling_take_no_arguments_of_their_launch(compiled):
    """blockDim and gridDim come in 256 bytes of arguments behind the own ones, which short launches notice."""
    sizes = dict((n, int(b)) for b, n in re.findall(r"\.kernarg_segment_size: (\d+)\n(?:(?!\.name:).*\n)*?\s*\.name: +(\w+)\n", compiled[0]))
    for n in [n for n in sizes if "attn_kernel" in n or "profile_error_kernel" in n]:
        assert sizes[n] <= 352, (n, sizes[n])


def test_two_blocks_of_the_largest_magnitudes_fit_a_compute_unit(compiled):
    """1024 threads each, for heads of up to 1024 rows: 64 vector registers."""
    used = dict(re.findall(r"\.name: +(\w+)\n(?:(?!\.name:).*\n)*?\s*\.vgpr_count: +(\d+)", compiled[0]))
    for n in [n for n in used if "fp8_amax_kernelILi1024E" in n]:
        assert int(used[n]) <= 64


def test_loops_that_notice_where_they_begin(compiled, tmp_path):
    """Four bytes behind a multiple of eight, where these three forms are up to 8 % faster than on one: a line of assembly in front of them sees to it."""
    tools = os.path.join(os.path.dirname(os.path.dirname(B.hipcc_path())), "llvm", "bin")
    (tmp_path / "k.s").write_text(compiled[0])
    subprocess.run([os.path.join(tools, "clang"), "-x", "assembler", "-target", "amdgcn-amd-amdhsa", "-mcpu=gfx950", "-c", "k.s", "-o", "k.o"], cwd=tmp_path, check=True)
    listing = subprocess.run([os.path.join(tools, "llvm-objdump"), "-d", "--no-show-raw-insn", "k.o"], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
    heads = {}
    for block in re.split(r"(?m)^(?=[0-9a-f]+ <\w+>:)", listing):
        form = re.match(r"[0-9a-f]+ <\w*11attn_kernelILi(\d+)ELi(\d)ELi\d+ELi(\d)ELi1ELi1E", block)
        if not form:
            continue
        ins = [(int(at, 16), op, args) for op, args, at in re.findall(r"(?m)^\s+(\S+) *(.*?) *// ([0-9A-F]+):", block)]
        for at, op, args in ins:
            if op.startswith(("s_cbranch", "s_branch")):
                words = int(args.split()[0])
                to = at + 4 + 4 * (words - 65536 if words >= 32768 else words)
                if to < at and 16 <= sum("mfma" in o for a, o, _ in ins if to <= a <= at) <= 64:
                    heads.setdefault(tuple(int(x) for x in form.groups()), to)
                    break
    for form in ((64, 4, 4), (64, 4, 3), (128, 1, 1)):      # gathering, exact masks, 32-row tiles
        assert not heads or heads[form] % 8 == 4, (form, hex(heads[form]))


def test_the_compiler_has_nothing_to_say(compiled):
    """(a warning per inlined load, 600 of them, once hid whatever else there was)"""
    lines = [l for l in compiled[2].splitlines() if "warning" in l and "--hip-link" not in l]
    assert not lines, lines[:3]
