"""Memory ordering in the gfx950 assembly of the kernels (CPU: cross-compiles, runs nothing).

k_feas combines the feasibility masks of a group's banks over workgroups: every wave ANDs its words into
global memory, and after a workgroup barrier one thread counts the bank as arrived; the last bank reads the
masks.  The barrier waits for no vector-memory operation and the count's release for those of its own wave
only, so each wave has to wait for its ANDs itself.
"""

import os
import re
import subprocess

import pytest

from paper_2608_27922_amd import build


@pytest.fixture(scope="module")
def update_asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "dkv_update.s"
    subprocess.run([build._hipcc(), "-x", "hip", *build.FLAGS, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "dkv_update.hip"), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


def unwaited(lines, op):
    """Occurrences of instruction `op` that some straight or branching path takes to an s_barrier, or to the
    end of the kernel, without an s_waitcnt vmcnt(0) between."""
    label = {m.group(1): i for i, x in enumerate(lines) if (m := re.match(r"(\.L\w+):", x))}
    bad = []
    for start in (i for i, x in enumerate(lines) if x.split()[:1] == [op]):
        todo, seen = [start + 1], set()
        while todo:
            i = todo.pop()
            if i in seen or i >= len(lines):
                continue
            seen.add(i)
            x = lines[i].split(";")[0].split()
            if not x or x[0].endswith(":") or x[0].startswith("."):
                todo.append(i + 1)
            elif x[0] == "s_waitcnt" and "vmcnt(0)" in lines[i]:
                continue
            elif x[0] in ("s_barrier", "s_endpgm"):
                bad.append(lines[start])
                break
            elif x[0].startswith("s_cbranch"):
                todo += [i + 1, label[x[1]]]
            elif x[0] == "s_branch":
                todo.append(label[x[1]])
            else:
                todo.append(i + 1)
    return bad


def test_the_path_search_finds_a_missing_wait():
    """On listings of a few lines: a wait on one of two branches is not enough, one on both is."""
    head = ["global_atomic_and v[0:1], v2, off", "s_cbranch_execz .LBB0_1"]
    tail = [".LBB0_1:", "s_barrier", "s_endpgm"]
    assert unwaited(head + ["s_waitcnt vmcnt(0)"] + tail, "global_atomic_and")
    assert not unwaited(head[:1] + ["s_waitcnt vmcnt(0) lgkmcnt(0)"] + head[1:] + tail, "global_atomic_and")


def test_feasibility_masks_are_done_before_the_count(update_asm):
    m = re.search(r"^(_ZN\w*6k_feas\w*):.*?^\.Lfunc_end", update_asm, re.S | re.M)
    assert m, "k_feas not found"
    lines = [x.strip() for x in m.group(0).splitlines()]
    assert any(x.startswith("global_atomic_and") for x in lines)
    assert not unwaited(lines, "global_atomic_and")
