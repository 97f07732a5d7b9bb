"""A wave of k_round_end that reads the control block after thread 0 has begun
to rewrite it for the next range search may take a branch with barriers that
thread 0 does not take.  Such a race shows on no CPU and seldom on a GPU, so
the kernel's source is checked: the round's kind is read before the first
barrier only, and a barrier stands between the last branch and the rewrite."""

import os
import re

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2304_01660_amd", "csrc", "kernels.hip")


def _body(name):
    text = re.sub(r"//[^\n]*", "", open(SRC).read())
    at = re.search(r"__global__[^;{]*\b%s\([^{;]*\)\s*\{" % name, text)
    depth, q = 1, at.end()
    while depth:
        depth += {"{": 1, "}": -1}.get(text[q], 0)
        q += 1
    return text[at.end():q - 1]


def test_round_end_reads_the_rounds_kind_before_its_first_barrier():
    head, _, tail = _body("k_round_end").partition("__syncthreads()")
    for field in ("c->handled", "c->nlive", "lean_round(c)"):
        conditions = [x for x in re.findall(r"\bif\s*\(([^{;]*)\)", tail) if field in x]
        assert not conditions, (field, conditions)
    assert "c->handled" in head and "lean_round(c)" in head


def test_round_end_rewrites_the_control_block_after_a_barrier():
    body = _body("k_round_end")
    before = body[:body.index("next_range(")]
    last = before.rindex("__syncthreads()")
    assert before[last:].count("{") == before[last:].count("}") == 0, "the barrier is conditional"
    assert "c->" not in before[last:]
