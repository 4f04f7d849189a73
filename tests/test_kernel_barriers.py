"""No kernel returns from inside a loop ahead of a workgroup barrier (CPU only, reads the sources).

The trip count of a grid-stride loop differs between the threads of a workgroup, down to zero, so a
return inside it is taken by some of them only, and a barrier behind it is then not reached by the
whole workgroup: undefined, whatever the hardware makes of waves that have ended.  Tests of a flag
that is the same for every thread belong outside the loop."""

import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2112_03370_amd", "csrc")
BARRIER = re.compile(r"\b(__syncthreads\w*|block_sum|reduce_partials|group_total)\s*\(")


def _matching(text, at):
    """Index past the brace or parenthesis that closes the one at `at`."""
    depth = 0
    for i in range(at, len(text)):
        depth += text[i] in "{("
        depth -= text[i] in "})"
        if depth == 0:
            return i + 1
    raise AssertionError("unbalanced source")


def _kernels(text):
    """(name, body) of every kernel defined in a source without comments."""
    for m in re.finditer(r"__global__[^;{]*?\bvoid\b.*?\b(k_\w+)\s*\(", text, re.S):
        end = _matching(text, m.end() - 1)
        brace = text.find("{", end)
        if text[end:brace].strip() == "":
            yield m.group(1), text[brace:_matching(text, brace)]


def returns_ahead_of_barrier(text):
    text = re.sub(r"//[^\n]*|/\*.*?\*/", "", text, flags=re.S)
    bad = []
    for name, body in _kernels(text):
        for loop in re.finditer(r"\b(?:for|while)\s*\(", body):
            head = _matching(body, loop.end() - 1)
            if body[head:].lstrip()[:1] != "{":
                continue
            start = body.index("{", head)
            stop = _matching(body, start)
            if re.search(r"\breturn\b", body[start:stop]) and BARRIER.search(body, start):
                bad.append(name)
    return bad


def test_scan_finds_a_return_ahead_of_a_barrier():
    kernel = "__global__ void k_a(int n) { for (int i = t; i < n; i += s) { %s } %s }"
    assert returns_ahead_of_barrier(kernel % ("if (done) return;", "__syncthreads();")) == ["k_a"]
    assert returns_ahead_of_barrier(kernel % ("if (done) return;", "")) == []
    assert returns_ahead_of_barrier(kernel % ("v += 1; /* return */", "__syncthreads();")) == []


@pytest.mark.parametrize("source", sorted(map(os.path.basename,
                                              glob.glob(os.path.join(CSRC, "*.hip")))))
def test_no_return_ahead_of_a_barrier(source):
    with open(os.path.join(CSRC, source)) as f:
        assert returns_ahead_of_barrier(f.read()) == []
