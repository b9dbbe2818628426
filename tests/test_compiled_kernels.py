"""What the compiler does not look after in inline assembly, checked in the code that it makes of it."""
import collections
import os
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2604_16734_amd import build as B


def _sources():
    """The sources whose inline assembly loads from memory."""
    found = []
    for src in B.SOURCES:
        with open(os.path.join(B.CSRC, src)) as f:
            if re.search(r'asm volatile\("[^;]*_load_', f.read()):
                found.append(src)
    return found


SOURCES = _sources()


@pytest.fixture(scope="module")
def texts(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("assembly"))
    with ThreadPoolExecutor(max_workers=4) as ex:
        paths = list(ex.map(lambda src: B.assembly(src, out), SOURCES))
    return {src: open(path).read() for src, path in zip(SOURCES, paths)}


def functions(text):
    """(name, lines) of every function; a line is an instruction, a label, or #ASMSTART / #ASMEND around a statement of inline assembly."""
    name, lines = None, []
    for line in text.splitlines():
        start = re.match(r"(_Z\w+):", line)
        if start:
            name, lines = start.group(1), []
        elif name and line.startswith(".Lfunc_end"):
            yield name, lines
            name = None
        elif name:
            line = line.strip() if "#ASM" in line else line.split(";")[0].strip()
            line = line.lstrip(";").strip()
            if line and (not line.startswith(".") or line.endswith(":")):
                lines.append(line)


def loads_without_their_own_m0(lines):
    """Loads into LDS in inline assembly whose statement does not set M0 before them."""
    bad, inside, own = [], False, False
    for line in lines:
        if line in ("#ASMSTART", "#ASMEND"):
            inside, own = line == "#ASMSTART", False
        elif inside and re.match(r"s_mov_b32 m0,", line):
            own = True
        elif inside and (line.endswith(" lds") or "_load_lds_" in line) and not own:
            bad.append(line)
    return bad


def test_the_check_of_m0():
    assert loads_without_their_own_m0(["#ASMSTART", "s_mov_b32 m0, s4", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3]",
                                       "buffer_load_dwordx4 v2, s[4:7], 0 offen offset:1024 lds", "#ASMEND"]) == []
    late = "buffer_load_dwordx4 v2, s[4:7], 0 offen offset:1024 lds"
    assert loads_without_their_own_m0(["#ASMSTART", "s_mov_b32 m0, s4", "#ASMEND", "#ASMSTART", late, "#ASMEND"]) == [late]


@pytest.mark.parametrize("src", SOURCES)
def test_m0_is_set_where_it_is_used(texts, src):
    """Between two statements the compiler may use M0 for itself."""
    n_loads = n_statements = 0
    for name, lines in functions(texts[src]):
        assert loads_without_their_own_m0(lines) == [], name
        n_statements += lines.count("#ASMSTART")
        n_loads += sum(line.endswith(" lds") or "_load_lds_" in line for line in lines)
    assert n_loads > 0 and n_statements > 0


# A load or store may read a scalar register only so many wait states after a vector instruction has written it
WAIT_STATES = 5
CARRY = ("v_add_co", "v_sub_co", "v_subrev_co", "v_addc", "v_subb", "v_div_scale", "v_mad_u64", "v_mad_i64")


def _scalars(operands):
    found = set()
    for first, last, one, vcc in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b|\b(vcc)(?:_lo|_hi)?\b", operands):
        if first:
            found.update(range(int(first), int(last) + 1))
        elif one:
            found.add(int(one))
        else:
            found.add(vcc)
    return found


def early_reads(lines):
    """(instruction, the one before it that wrote a register of it, wait states between them), over all ways through the function."""
    code, labels, before = [], {}, collections.defaultdict(set)
    for line in lines:
        if line.endswith(":"):
            labels[line[:-1]] = len(code)
        elif not line.startswith("#"):
            code.append(line.partition(" ")[::2] if " " in line else (line, ""))
    for i, (op, operands) in enumerate(code):
        if op.startswith(("s_branch", "s_cbranch")):
            before[labels[operands]].add(i)
        if op not in ("s_branch", "s_endpgm"):
            before[i + 1].add(i)
    bad = []
    for i, (op, operands) in enumerate(code):
        reads = _scalars(operands) if op.startswith(("buffer_", "global_", "flat_", "scratch_")) else None
        if not reads:
            continue
        least, todo = {}, [(j, 0) for j in before[i]]
        while todo:
            j, waits = todo.pop()
            if waits >= WAIT_STATES or least.get(j, WAIT_STATES) <= waits:
                continue
            least[j] = waits
            op_j, operands_j = code[j]
            if op_j.startswith("v_"):
                results = operands_j.split(",")[:2 if op_j.startswith(CARRY) else 1]
                if reads & _scalars(",".join(results)):
                    bad.append((" ".join(code[i]), " ".join(code[j]), waits))
                    continue
            todo += [(k, waits + (int(operands_j, 0) + 1 if op_j == "s_nop" else 1)) for k in before[j]]
    return bad


def test_the_check_of_wait_states():
    write, load = "v_readfirstlane_b32 s6, v1", "buffer_load_dwordx4 v2, s[4:7], 0 offen lds"
    assert early_reads([write, "#ASMSTART", "s_mov_b32 m0, s8", "s_nop 3", load, "#ASMEND"]) == []
    assert early_reads([write, "s_mov_b32 m0, s8", "s_nop 0", load]) == [(load, write, 2)]
    assert early_reads(["L1:", "s_mov_b32 m0, s8", load, "v_add_u32_e32 v1, s6, v1", write, "s_cbranch_scc1 L1", "s_endpgm"]) == [(load, write, 2)]
    assert early_reads(["v_add_u32_e32 v1, s6, v1", load]) == []
    carry = "v_add_co_u32_e64 v1, s[4:5], v2, v3"
    assert early_reads([carry, load]) == [(load, carry, 0)]


@pytest.mark.parametrize("src", SOURCES)
def test_scalar_registers_of_loads_have_settled(texts, src):
    """The compiler sees to this, but not where the load is in inline assembly."""
    for name, lines in functions(texts[src]):
        assert early_reads(lines) == [], name
