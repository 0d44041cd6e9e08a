"""The prompt kernel's LDS tiles are filled by loads the compiler does not know of and handed over by bare barriers, so the
waits around them are the source's own.  These tests compile the kernel for gfx950 and follow them through the assembly."""
import os
import re
import subprocess

import pytest

from paper_2311_01282_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


class Code:
    """Basic blocks of one kernel: lists of (instruction, whether it stands in inline assembly), and their successors."""

    def __init__(self, text, name):
        lines = text[re.search(r"^\S*%s\S*:" % name, text, re.M).start():].split("\n")
        self.blocks, self.next, labels = [[]], [], {}
        inline = False
        for line in lines[1:]:
            if line.startswith(".Lfunc_end"):
                break
            label = re.match(r"(\.LBB\w+):", line)
            if label:
                if self.blocks[-1]:
                    self.blocks.append([])
                labels[label.group(1)] = len(self.blocks) - 1
                continue
            if "#ASMSTART" in line or "#ASMEND" in line:
                inline = "#ASMSTART" in line
                continue
            ins = line.split(";")[0].strip()
            if not ins or ins.startswith("."):
                continue
            self.blocks[-1].append((ins, inline))
            if ins.startswith(("s_cbranch", "s_branch", "s_endpgm")):
                self.blocks.append([])
        for i, block in enumerate(self.blocks):
            last = block[-1][0] if block else ""
            after = [] if last.startswith(("s_branch", "s_endpgm")) or i + 1 == len(self.blocks) else [i + 1]
            if last.startswith(("s_branch", "s_cbranch")):
                after.append(labels[last.split()[-1]])
            self.next.append(after)


def lds_reads_at_barriers(code):
    """For every s_barrier the number of this wavefront's LDS reads that can still be in flight there: the largest over
    all paths (LDS operations return in order; lgkmcnt(N) leaves N at most)."""
    entry = [-1] * len(code.blocks)              # -1: not reached
    entry[0] = 0
    found, todo = {}, [0]
    while todo:
        i = todo.pop()
        n = entry[i]
        for at, (ins, _) in enumerate(code.blocks[i]):
            if ins.startswith("ds_") and not ins.startswith("ds_write"):
                n = min(n + 1, 16)               # (the counter ends at 15)
            wait = re.search(r"lgkmcnt\((\d+)\)", ins)
            if wait:
                n = min(n, int(wait.group(1)))
            if ins.startswith("s_barrier"):
                found[i, at] = max(n, found.get((i, at), 0))
        for j in code.next[i]:
            if n > entry[j]:
                entry[j] = n
                todo.append(j)
    return found


def waits_over_tile_fetches(code):
    """The compiler's own waits for vector loads that a tile fetch in inline assembly can be in flight at: such a wait is
    for an older load, but loads return in order and the compiler counts only those it knows, so it waits for the tile too."""
    entry = [None] * len(code.blocks)            # False: no such fetch in flight
    entry[0] = False
    found, todo = set(), [0]
    while todo:
        i = todo.pop()
        flying = entry[i]
        for at, (ins, inline) in enumerate(code.blocks[i]):
            if inline and ins.startswith("buffer_load") and ins.endswith(" lds"):
                flying = True
            if "vmcnt(" in ins:
                if flying and not inline:
                    found.add((i, at, ins))
                flying = flying and "vmcnt(0)" not in ins
        for j in code.next[i]:
            if entry[j] is None or flying and not entry[j]:
                entry[j] = flying
                todo.append(j)
    return found


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("prefill") / "prefill.s")
    subprocess.check_call([build.hipcc()] + build.FLAGS + ["-S", "--cuda-device-only", "-o", out,
                           os.path.join(build.CSRC, "fd_prefill_kernels.hip")], stderr=subprocess.DEVNULL)
    with open(out) as f:
        return f.read()


def test_the_walk_finds_a_read_across_a_barrier():
    text = "k:\n ds_read_b128 v[0:3], v4\n ds_read_b128 v[4:7], v4\n s_cbranch_scc1 .LBB0_2\n s_waitcnt lgkmcnt(%d)\n" \
           ".LBB0_2:\n %s s_barrier\n s_endpgm\n.Lfunc_end0:\n"
    assert list(lds_reads_at_barriers(Code(text % (1, ""), "k")).values()) == [2]        # over the branch
    assert list(lds_reads_at_barriers(Code(text % (1, "s_waitcnt vmcnt(0) lgkmcnt(1)\n"), "k")).values()) == [1]
    assert list(lds_reads_at_barriers(Code(text % (1, "s_waitcnt lgkmcnt(0)\n"), "k")).values()) == [0]


def test_no_lds_read_is_in_flight_at_a_barrier(assembly):
    """A tile's place in the ring is filled again after the barrier that ends the step: its reads have to have returned."""
    found = lds_reads_at_barriers(Code(assembly, "prefill_kernel"))
    assert len(found) >= 8
    assert not any(found.values()), found


def test_no_inline_assembly_writes_m0(assembly):
    """m0 holds the LDS address of a tile fetch.  The compiler uses it for the fetches it knows and is not told of a write
    inside a statement, so it has to set m0 itself, for every fetch."""
    code = Code(assembly, "prefill_kernel")
    fetches = 0
    for block in code.blocks:
        for ins, inline in block:
            if not inline:
                continue
            assert not re.match(r"[sv]_\w+ m0\b", ins), ins
            fetches += ins.startswith("buffer_load") and ins.endswith(" lds")
    assert fetches >= 16


def test_tile_fetches_are_waited_for_by_the_source_alone(assembly):
    """A tile is fetched two steps ahead: nothing but the wait at the end of the next step may wait for it."""
    text = "k:\n;#ASMSTART\n buffer_load_dwordx4 v1, s[0:3], s4 offen lds\n;#ASMEND\n%s s_waitcnt vmcnt(3)\n s_endpgm\n.Lfunc_end0:\n"
    assert len(waits_over_tile_fetches(Code(text % "", "k"))) == 1
    assert not waits_over_tile_fetches(Code(text % ";#ASMSTART\n s_waitcnt vmcnt(0)\n;#ASMEND\n", "k"))
    assert not waits_over_tile_fetches(Code(assembly, "prefill_kernel"))


@pytest.mark.parametrize("split", [0, 1])
def test_both_forms_of_the_kernel(assembly, split):
    """The three rules for the form with a query tile per wavefront and for the one whose wavefronts share the keys."""
    code = Code(assembly, "prefill_kernelILb%dE" % split)
    found = lds_reads_at_barriers(code)
    assert len(found) >= 8 and not any(found.values()), found
    assert not any(inline and re.match(r"[sv]_\w+ m0\b", ins) for block in code.blocks for ins, inline in block)
    assert sum(inline and ins.startswith("buffer_load") and ins.endswith(" lds") for block in code.blocks for ins, inline in block) >= 16
    assert not waits_over_tile_fetches(code)
