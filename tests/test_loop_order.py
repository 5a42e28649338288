"""The resident loop's LDS words between the units of a block, on the CPU.

A block of k_icp_loop takes its units one after the other.  Each unit's waves
write records that wave 0 reads, and count misses that every wave reads, so a
barrier has to stand between those reads and the next unit's writes.  This
reads the unit loop's body from the source, follows the path on which no query
misses (the one with the fewest barriers) over two consecutive units, and
checks that every read of a word and another wave's write of it, in either
order, have a barrier between them."""
import os
import re

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(os.path.dirname(HERE), "paper_2512_04996_amd", "csrc", "k_loop.hip")

TOKENS = [("barrier", r"__syncthreads\(\)"),
          ("add misses", r"atomicAdd\(&sh\.misses"),
          ("read misses", r"=\s*sh\.misses\b"),
          ("read rec", r"=\s*sh\.rec\["),
          ("write rec", r"sh\.rec\[[^\]]*\]\[[^\]]*\]\s*=(?!=)")]


def braces(text, at):
    """The block that opens at the first brace from `at` on, and where it ends."""
    a = text.index("{", at)
    depth = 0
    for i in range(a, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[a + 1:i], i + 1
    raise AssertionError("unbalanced braces")


def tokens(text):
    found = [(m.start(), name) for name, pat in TOKENS for m in re.finditer(pat, text)]
    return [name for _, name in sorted(found)]


def unit_path(src):
    """The tokens of one unit without misses, and those between two units."""
    src = re.sub(r"//[^\n]*", "", src)
    body, _ = braces(src, src.index("for (int u = job.u0; u < U; u += job.stride)"))
    at = body.index("for (int pass = 0;")
    passes, end = braces(body, at)
    leave = passes.index("if (pass == 1 || nmiss == 0) break;")
    rest = body[end:]
    # a barrier that stands only where another unit follows
    between = re.search(r"if \(u \+ job\.stride < U\) __syncthreads\(\);", rest)
    one = tokens(body[:at]) + tokens(passes[:leave]) + tokens(rest[:between.start()] if between else rest)
    return one, ["barrier"] if between else []


def ordered(path, first, then):
    """Every `first` and every later `then` have a barrier between them."""
    return all("barrier" in path[i:j] for i, a in enumerate(path) if a == first
               for j, b in enumerate(path) if b == then and j > i)


def test_units_of_a_block_are_ordered():
    one, between = unit_path(open(SRC).read())
    for t in ("add misses", "read misses", "write rec", "read rec", "barrier"):
        assert t in one, t
    two = one + between + one
    assert ordered(one, "write rec", "read rec") and ordered(one, "add misses", "read misses")
    assert ordered(two, "read rec", "write rec"), two
    assert ordered(two, "read misses", "add misses"), two
