"""Requests from memory straight into LDS are inline assembly, inside which the compiler inserts no wait states and tracks no
register that is not named.  Read from the sources: no GPU, no compiler."""
import glob
import os
import re

from paper_2603_09555_amd import build


def statements():
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*.h*"))):
        for m in re.finditer(r'asm volatile\((.*?)\);', open(path).read(), re.S):
            yield os.path.basename(path), m.group(1)


def test_requests_into_lds_wait_for_their_scalar_registers():
    """A vector memory instruction reads a scalar register at the earliest five wait states after a vector instruction wrote it
    (a move to a uniform register, a spilled one reloaded), and m0 one after a scalar instruction did."""
    requests = [(f, s) for f, s in statements() if re.search(r"buffer_load\w* .* lds", s)]
    assert len(requests) >= 2
    for name, s in requests:
        text = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', s.split("::")[0]))
        lines = [q.strip() for q in re.split(r"(?:\\n|\\t)+", text) if q.strip()]
        first = next(i for i, q in enumerate(lines) if q.startswith("buffer_load"))
        waits = sum(int(q.split()[1]) + 1 if q.startswith("s_nop") else 1 for q in lines[:first])
        assert waits >= 5, (name, lines)
        m0 = next(i for i, q in enumerate(lines) if q.startswith("s_mov_b32 m0"))
        assert m0 + 1 < first and lines[m0 + 1].startswith("s_nop"), (name, lines)
        assert '"m0"' in s.rsplit(":", 1)[1], (name, "m0 is written and not named as clobbered")
