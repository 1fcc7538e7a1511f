"""What the compiled device code has to hold that no run can show for sure: a
wave waits for its own LDS accesses before it reports at a barrier.  The
compiler puts that wait before the barriers of the accesses it knows; those
inside an asm statement it does not know."""
import os
import re
import subprocess

import pytest

from paper_2608_09225_amd import build

HERE = os.path.dirname(os.path.abspath(build.__file__))


def device_asm(source: str) -> str:
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [build.hipcc(), *flags, "--offload-device-only", "-S", "-o", "-",
           os.path.join(HERE, source)]
    return subprocess.run(cmd, capture_output=True, text=True, check=True).stdout


def kernels(asm: str) -> dict:
    """Instructions and labels per function, comments left out."""
    out, name = {}, None
    for line in asm.splitlines():
        s = line.split(";")[0].strip()
        m = re.fullmatch(r"(_Z\w+):", s)
        if m:
            name = m.group(1)
            out[name] = []
        elif s.startswith(".Lfunc_end"):
            name = None
        elif name and s and (s.endswith(":") or not s.startswith(".")):
            out[name].append(s)
    return out


def late_barriers(body: list) -> list:
    """Barriers that some path reaches with LDS accesses not waited for: the
    number of accesses in flight is carried along every branch."""
    at = {s[:-1]: i for i, s in enumerate(body) if s.endswith(":")}
    seen, todo, late = {}, [(0, 0)], set()
    while todo:
        i, flying = todo.pop()
        while i < len(body):
            s = body[i]
            if s.endswith(":"):
                if seen.get(i, -1) >= flying:
                    break
                seen[i] = flying
            op = s.split()[0]
            if op.startswith("ds_") and not re.match(r"ds_(b?permute|swizzle|nop)", op):
                flying = min(flying + 1, 16)
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", s)
                flying = min(flying, int(m.group(1))) if m else flying
            elif op == "s_barrier" and flying:
                late.add(i)
            elif op.startswith("s_cbranch"):
                todo.append((at[s.split()[1]], flying))
            elif op == "s_branch":
                i = at[s.split()[1]]
                continue
            elif op == "s_endpgm":
                break
            i += 1
    return sorted(late)


@pytest.mark.parametrize("source", build.LIBS["libkvgov.so"])
def test_lds_accesses_are_waited_for_before_barriers(source):
    found = kernels(device_asm(source))
    assert found
    bad = {name: late_barriers(body) for name, body in found.items()}
    assert not {name: len(late) for name, late in bad.items() if late}


def test_late_barriers_are_found():
    """The walk itself, on code written for it."""
    wait, bar = "s_waitcnt lgkmcnt(0)", "s_barrier"
    assert late_barriers(["ds_write_b32 v0, v1", bar, "s_endpgm"]) == [1]
    assert late_barriers(["ds_write_b32 v0, v1", wait, bar, "s_endpgm"]) == []
    assert late_barriers(["ds_write_b32 v0, v1", "ds_read_b32 v2, v3", "s_waitcnt lgkmcnt(1)", bar,
                          "s_endpgm"]) == [3]
    # around a loop, and past a branch that skips the wait
    assert late_barriers([".L:", bar, "ds_write_b32 v0, v1", "s_cbranch_scc1 .L", "s_endpgm"]) == [1]
    assert late_barriers(["ds_write_b32 v0, v1", "s_cbranch_scc1 .L", wait, ".L:", bar,
                          "s_endpgm"]) == [4]
    assert late_barriers(["ds_bpermute_b32 v0, v1, v2", bar, "s_endpgm"]) == []
