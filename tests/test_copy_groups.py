"""The order of the direct global->LDS copies in the kernels that wait for a count of them: a wait for the
first group that leaves the second in flight is right only if no copy of the second was issued before one of
the first.  In the compiler's intermediate form of every such kernel, a compiler barrier must stand between
copies into one LDS variable and copies into the next."""
import os
import re
import subprocess

import pytest

from paper_2406_11626_amd import build

GLOBAL = re.compile(r"@\w+")
DEST = re.compile(r"@llvm\.amdgcn\.global\.load\.lds\(ptr addrspace\(1\) [^,]*, ptr addrspace\(3\) (?:\w+ )*([%@][\w.]+)")
DEFINED = re.compile(r"^\s+(%[\w.]+) = (?:getelementptr|phi|select|bitcast)\b(.*)")


def _functions(source, tmp_path):
    out = str(tmp_path / "k.ll")
    subprocess.check_call([build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "--cuda-device-only", "-S", "-emit-llvm",
                           "-O1", "-std=c++17", os.path.join(build.CSRC, source), "-o", out], stderr=subprocess.DEVNULL)
    for text in re.split(r"^define ", open(out).read(), flags=re.M)[1:]:
        body = text[:text.index("\n}")]
        if "load.lds(" in body:
            yield re.search(r"@(\w+)\(", body).group(1), body.split("\n")


def _variable(value, defs, depth=0):
    """The LDS variable that a destination points into."""
    if value.startswith("@") or depth > 20:
        return value
    text = defs.get(value, "")
    found = GLOBAL.search(text)
    if found:
        return found.group(0)
    base = re.search(r"ptr addrspace\(3\) (%[\w.]+)", text)
    return _variable(base.group(1), defs, depth + 1) if base else value


@pytest.mark.parametrize("source,least", [("ccz4_kernels.hip", 5), ("ccz4_lds_fp64.hip", 4)])
def test_a_barrier_between_groups(source, least, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    seen = 0
    for name, lines in _functions(source, tmp_path):
        defs = {m.group(1): m.group(2) for m in map(DEFINED.match, lines) if m}
        into, groups = None, 0
        for line in lines:
            if 'asm sideeffect "", "~{memory}"' in line:
                into = None
                continue
            m = DEST.search(line)
            if not m:
                continue
            to = _variable(m.group(1), defs)
            assert to.startswith("@"), (name, line)
            assert into in (None, to), f"{name}: copies into {into} and {to} with no barrier between them"
            groups += into is None
            into = to
        seen += groups > 1
    assert seen >= least
