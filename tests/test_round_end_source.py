"""A wave of k_round_end that reads the control block after thread 0 has begun
to rewrite it for the next range search may take a branch with barriers that
thread 0 does not take.  Such a race shows on no CPU and seldom on a GPU, so
the kernel's source is checked: the round's kind is read before the first
barrier only, and once thread 0 rewrites it no other thread reads it."""

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


def test_only_thread_0_reads_the_control_block_once_it_is_rewritten():
    body = _body("k_round_end")
    at = body.index("c->rounds += 1")
    start = body.rindex("if (tid == 0) {", 0, at)
    assert body[:start].rstrip().endswith("}"), "the part of thread 0 follows the parts' return"
    rest = body[start:]
    while "if (tid == 0) {" in rest:  # leave out what only thread 0 runs
        a = rest.index("if (tid == 0) {")
        q, depth = rest.index("{", a) + 1, 1
        while depth:
            depth += {"{": 1, "}": -1}.get(rest[q], 0)
            q += 1
        rest = rest[:a] + rest[q:]
    assert "c->" not in rest, [x for x in rest.splitlines() if "c->" in x]
    assert "tid == 0) next_range(" in rest
    # a barrier stands between the last read by any other thread and that part
    head = body[:start]
    assert "c->" not in head[head.rindex("__syncthreads()"):].replace("c->pcnt[tid] = 0", "").replace(
        "c->ncand = ", "").replace("c->cand_at = ", "").replace("c->pending = ", "")
