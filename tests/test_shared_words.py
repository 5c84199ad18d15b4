"""Words of device memory that several blocks of one launch use: which stores
the kernels may make to them, checked on the sources (a wrong order shows
neither on the CPU nor, reliably, on the GPU)."""
import os
import re

import pytest

import paper_2105_00115_amd as q

CSRC = os.path.join(os.path.dirname(os.path.abspath(q.__file__)), "csrc")


def _body(name, file):
    """The function or kernel `name`: from its parameter list to the brace
    that closes it, without comments."""
    text = open(os.path.join(CSRC, file)).read()
    text = re.sub(r"//[^\n]*", "", text)
    m = re.search(r"\b%s\(" % name, text)
    assert m, name
    i = text.index("{", text.index(")", m.end()))
    depth, j = 0, i
    while True:
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        j += 1
        if depth == 0:
            return text[i:j]


def test_one_block_of_a_launch_stores_the_guess_verdict():
    """The verdict that k_sel_sweep reads is set in k_spec_sweep by the last
    block to finish and by no other block (each XCD writes its L2 back when it
    likes, so a plain store of another block could land after it), and cleared
    in the launch before."""
    store = re.compile(r"\bdone\s*=[^=]")
    sweep = _body("k_spec_sweep", "qdot_fused.hip")
    stores = [m.start() for m in store.finditer(sweep)]
    assert len(stores) == 1
    assert stores[0] > sweep.index("if (!last_block(")
    assert len(store.findall(_body("k_key_sample", "qdot_fused.hip"))) == 1
    assert not store.search(_body("sel_sweep", "qdot_fused.hip"))


def test_fp64_gang_dot_waits_for_every_block_before_it_takes_a_value_back():
    """Block 0 of a gang takes back the previous inner product's value once
    every block has contributed to this one (they have all read it then).  Its
    waves wait for 64 blocks each, so a barrier has to stand between the waits
    and the store: without it, wave 0 takes the value back while a block past
    the 64th may still poll for it, and the gang waits until it gives up."""
    body = _body("gang_dot64", "qdot_cg.hpp")
    wait, retract = body.index("gang_take("), body.index("gang_retract(")
    assert wait < retract
    assert re.search(r"__syncthreads(_and)?\(", body[wait:retract])
    # and the store is complete before the new value can be seen
    assert "vmem_drain()" in body[retract:]


def test_gang_qdot_takes_a_value_back_behind_a_barrier_of_the_gang():
    """The same order in the two-pass inner product: behind its counting
    barrier, which no block passes before it has read the other value."""
    body = _body("gang_qdot", "qdot_cg.hpp")
    assert body.index("gang_barrier_with<true>(") < body.index("gang_retract(")


def test_a_block_whose_gang_gives_up_leaves_its_counts_clean():
    """cg_solve is the one way out of a gang: where it has given up, the LDS
    counts (which the launch's next item takes for zero) are cleared, after
    the last place that fills them."""
    body = _body("cg_solve", "qdot_cg.hpp")
    clear = re.search(r"else\s+for \(int j = threadIdx.x; j < 4 \* FQ; j \+= NT\) L\.h\[j\] = 0u;",
                      body)
    assert clear
    assert clear.start() > max(body.rindex("dot("), body.rindex("scan_pair("))
    assert not re.search(r"\breturn;", body)


def test_a_gang_with_a_launch_of_its_own_comes_together_before_it_begins():
    """Another solve's launch may hold CUs that the gang waits for, and the
    other way round: the blocks meet first (a bounded wait that all of them
    leave the same way), before any of them stores a result."""
    body = _body("k_cg_gangs", "qdot_cg.hip")
    assert body.index("gang_join(") < body.index("cg_solve<")
    join = _body("gang_join", "qdot_cg.hpp")
    assert join.count("compare_exchange") == 1 and "spins >= limit" in join
    reset = _body("gang_reset", "qdot_cg.hpp")
    assert "gg->join.v = 0u;" in reset and "gg->verdict.v = 0u;" in reset
