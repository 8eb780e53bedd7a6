"""Inline assembly under csrc/: a statement that writes a register by name says so to the compiler, which may otherwise keep a value of its
own there (the destination of an LDS load that it places itself, say), and one that loads to LDS says that it writes memory.  A wait for
loads to LDS counts those behind the awaited ones only, never loads that the compiler issues, in whatever number."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1511_05950_amd", "csrc")
STATEMENT = re.compile(r"\basm\s+volatile\s*\((.*?)\);", re.S)
# first operand of an instruction that is a register by name; stores and waits have none
WRITES = re.compile(r"(?:^|\\n\\t|\\n|;)\s*[sv]_\w+\s+(m0|vcc(?:_lo|_hi)?|exec(?:_lo|_hi)?|scc|s\d+|v\d+|a\d+|[sva]\[\d+:\d+\])\b")


def written_and_named(source):
    for m in STATEMENT.finditer(source):
        parts = m.group(1).split(":")
        text = "".join(re.findall(r'"([^"]*)"', parts[0]))
        yield set(WRITES.findall(text)), set(re.findall(r'"([^"]*)"', parts[-1])) if len(parts) >= 4 or "::" in m.group(1) else set()


def test_registers_written_by_name_are_clobbers():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        for written, named in written_and_named(open(path).read()):
            seen += bool(written)
            assert written <= named, (os.path.basename(path), written, named)
    assert seen                                  # the strip kernel's loads to LDS


def test_the_scan_sees_a_missing_clobber():
    bad = r'asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(a), "v"(b), "s"(c) : "memory");'
    good = bad.replace('"memory"', '"memory", "m0"')
    assert [w <= n for w, n in written_and_named(bad)] == [False] and [w <= n for w, n in written_and_named(good)] == [True]


LDS_LOAD = re.compile(r"\b(?:buffer|global)_load_\w+.*\blds\b|\bglobal_load_lds_\w+")


def lds_loads(source):
    for m in STATEMENT.finditer(source):
        parts = m.group(1).split(":")
        if LDS_LOAD.search(re.sub(r"\\[nt]", " ", "".join(re.findall(r'"([^"]*)"', parts[0])))):
            yield '"memory"' in parts[-1]


def test_loads_to_lds_clobber_memory():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        for named in lds_loads(open(path).read()):
            seen += 1
            assert named, os.path.basename(path)
    assert seen >= 5                             # the strip kernel's, two of the fully connected product, two of the update from factors
    bad = r'asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(a), "v"(b), "s"(c) : "m0");'
    assert list(lds_loads(bad)) == [False] and list(lds_loads(bad.replace('"m0");', '"memory", "m0");'))) == [True]


def test_the_staged_update_waits_for_its_own_loads_only():
    """vmcnt is the number of loads still on their way that a wait allows.  In the staged update from factors a stage is eight loads to LDS, of which
    the next stage's are behind it: more may only be allowed where more of the kernel's own are certain to be."""
    source = open(os.path.join(CSRC, "update.hip")).read()
    kernel = source[source.index("void apply_update_fc_deep_kernel("):source.index("hipError_t launch_apply_update_fc(")]
    allowed = [int(n) for n in re.findall(r"vmcnt\((\d+)\)", kernel)]
    assert allowed and max(allowed) <= 8
