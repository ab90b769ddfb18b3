"""Vector types of the FP64 passes by pairs of columns (CPU, on the source).

Rows of the per-particle workspaces hold (n + 1)^2 doubles, an odd number, and a caller's state may start
on any double: a pair of doubles loaded or stored there is aligned to 8 bytes, and its type has to say so (a
wider promise is undefined, whatever the hardware makes of it).
"""
import os
import re

from conftest import ROOT

SOURCE = os.path.join(ROOT, "paper_2503_16028_amd", "csrc", "k_solve.hip")


def test_pairs_of_doubles_promise_eight_bytes():
    text = open(SOURCE).read()
    bodies = re.findall(r"\b(pair_\w+)\(const double\*|\b(pair_\w+)\(double\*", text)
    names = {a or b for a, b in bodies}
    assert {"pair_refine", "pair_residual", "pair_update", "pair_setup"} <= names
    for name in names:
        body = re.search(r"__noinline__ \w+ %s\(.*?\n}\n" % name, text, re.S).group(0)
        pairs = re.findall(r"typedef double (\w+) __attribute__\(\((.*?)\)\);", body)
        used = set(re.findall(r"(?:at|put)_off<(\w+)>", body))
        assert any(t in used for t, _ in pairs), name
        for t, attributes in pairs:
            assert t not in used or "aligned(8)" in attributes, (name, t)
