"""The union queue of the kernel that sweeps small lattices whole, by its own
source: with every row offering as many entries as a wave can push, no push goes
past the queue's end (random draws never come near that, so no run shows it)."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1208_2080_amd", "csrc",
                   "sw_whole.hip")
TEXT = open(SRC).read()
FORMS = sorted({(int(m[1]), int(m[2])) for m in re.finditer(r"\bk_whole<(\d+), (\d+)>", TEXT)})


def steps(text):
    """The queue's checks, drains and pushes of a piece of the kernel, in order."""
    for m in re.finditer(r"if \(qn > ([^;]*?)\) (?:drain|draw)\(\);|push\((\w+)|qn \+= popc64\(m\);|(?:drain|draw)\(\);", text):
        if m[1]:
            yield "check", m[1]
        elif m[2] or m[0].startswith("qn +="):
            yield "push", m[2] or "m"
        else:
            yield "drain", None


@pytest.mark.parametrize("lmax,nw", FORMS)
def test_union_queue_holds_all_that_is_pushed(lmax, nw):
    sizes = {"CH": (lmax + 63) // 64, "RP": lmax // nw,
             "QCAP": int(re.search(r"constexpr uint32_t QCAP = (\d+);", TEXT)[1])}
    marks = [TEXT.index(f"// ---- {i}. ") for i in (1, 2, 3, 4)]
    rows_end = TEXT.index("(a run's first site is its node")   # behind the loop over the rows

    def run(text, fill, times):
        """Fill after `times` passes over a piece of the kernel in which every
        push by column pass adds a wave's 64, a push by row one for each row."""
        for _ in range(times):
            for what, arg in steps(text):
                if what == "drain":
                    fill = 0
                elif what == "check":
                    fill = min(fill, eval(arg, {}, sizes))
                elif arg in ("wrap", "join"):
                    fill += sizes["RP"] if arg == "wrap" or sizes["CH"] > 1 else 0
                else:
                    fill += 64 * sizes["CH"]
                assert fill <= sizes["QCAP"], (lmax, nw, what, arg, fill)
        return fill

    fill = run(TEXT[marks[0]:rows_end], 0, sizes["RP"])
    assert fill > sizes["QCAP"] - 64 * sizes["CH"]            # the rows can fill it
    assert run(TEXT[rows_end:marks[1]], fill, 1) == 0         # across passes and edges, and the drain
    assert run(TEXT[marks[1]:marks[2]], 0, 1) == 0            # seams
    roots = TEXT[marks[2]:marks[3]]
    loop = roots[roots.index("uint32_t p[RP][CH];"):]
    run(loop[:loop.index("draw();\n#pragma")], 0, sizes["RP"])
