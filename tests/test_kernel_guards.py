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


def _closure(functions, direct):
    """Names of the functions whose body, or that of one they call, matches."""
    found = {n for n, b in functions.items() if re.search(direct, b)}
    while True:
        more = {n for n, b in functions.items() if n not in found and
                any(re.search(r"\b%s(<[^;()]*>)?\(" % f, b) for f in found)}
        if not more:
            return found
        found |= more


def test_blocks_take_the_error_word_as_a_whole():
    """A kernel whose own launch can raise the capacity error, and whose waves
    share LDS, reads the word once per block: taken wave by wave, some waves
    of a block could leave and the others read what those had not written."""
    functions = _functions()
    functions = {n: b for n, b in functions.items() if n not in ("dead", "block_dead")}
    raises = _closure(functions, r"\bERR_CAPACITY\b")
    shares = _closure(functions, r"__syncthreads\(|\bblock_dead\(")
    assert {"k_advance", "k_branch", "k_scan", "k_stoplink", "k_finish"} <= raises & shares
    assert "k_scatter" in shares - raises and "k_classify_new" in raises - shares
    for name in sorted(raises & shares):
        assert not re.search(r"(?<!block_)\bdead\(", functions[name]), name
