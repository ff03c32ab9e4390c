"""Rules on the error word of a context that the kernels' source has to keep,
checked on the text: a launch that runs out of a capacity raises the word
while others of its blocks and waves are still to start, and what those then
do cannot be shown by running it."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _functions():
    """Body of every function of kernels.hip, comments left out, by name."""
    with open(os.path.join(ROOT, "paper_2504_12858_amd", "csrc", "kernels.hip")) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    out = {}
    for m in re.finditer(r"(\w+)\(([^;{}()]*)\)\s*\{", text):
        if m.group(1) in ("if", "for", "while", "switch"):
            continue
        depth, k = 1, m.end()
        while depth:
            depth += {"{": 1, "}": -1}.get(text[k], 0)
            k += 1
        out.setdefault(m.group(1), "")
        out[m.group(1)] += text[m.end():k]
    return out


def test_places_of_stops_are_all_written():
    """The stop linking forms its places by sums over the regions of the stop
    lists, and the end of the step counts them all: no block may leave by the
    error word, which the launch itself raises when the store is full."""
    body = _functions()["k_stoplink"]
    assert "stopped_put" in body
    assert "dead(" not in body and "->err" not in body
