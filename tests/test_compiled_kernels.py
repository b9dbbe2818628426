"""What the compiler does not look after in inline assembly, checked in the code that it makes of it."""
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
