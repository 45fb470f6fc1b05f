"""Kernels of many workgroups that both read and write the solve's control
block: the fields they read and the fields they write are disjoint.

The waves of a workgroup read a field one by one, so a kernel whose workgroup 0
sets the flag that the others return on can split a later workgroup: one wave
leaves, the rest go on past barriers to LDS contents (row pointers, partial
sums) that it never wrote.  Read from the source (CPU only)."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_09001_amd", "csrc",
                   "solve.hip")


def _body(text, head):
    """The brace-matched block that follows `head`."""
    at = text.index("{", text.index(head))
    depth, i = 0, at
    while True:
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        i += 1
        if depth == 0:
            return text[at:i]


def _source():
    return re.sub(r"//[^\n]*", "", open(SRC).read())


def _fields(body):
    reads, writes = set(), set()
    for m in re.finditer(r"ctl->(\w+(?:\[[^\]]*\])?)\s*(\+=|=(?!=))?", body):
        (writes if m.group(2) else reads).add(re.sub(r"\s", "", m.group(1)))
    return reads, writes


@pytest.mark.parametrize("kernel", ["k_cg_update", "k_bi_dir", "k_bi_half", "k_bi_full"])
def test_vector_kernels_do_not_write_what_they_read(kernel):
    reads, writes = _fields(_body(_source(), f" {kernel}("))
    assert reads and writes
    assert not reads & writes, reads & writes


def test_product_sweep_does_not_write_what_it_reads():
    text = _source()
    reads, writes = _fields(_body(text, "struct OpSpmvXpay"))
    assert reads and writes
    assert not reads & writes, reads & writes
    # the sweep around it returns on this flag
    assert "done" not in writes
    assert re.search(r"sweep\([^;]*OpSpmvXpay\{[^}]*\}, done,", text), "the product's stop flag"


@pytest.mark.parametrize("kernel", ["k_sum_update", "k_sum_half", "k_fin_chunk", "k_bfin_chunk"])
def test_kernels_that_test_and_set_a_flag_are_one_workgroup(kernel):
    text = _source()
    reads, writes = _fields(_body(text, f" {kernel}("))
    assert reads & writes <= {"done", "gate[1]"}
    launches = re.findall(rf"hipLaunchKernelGGL\({kernel}, (dim3\(\w+\)), (dim3\(\w+\))", text)
    assert launches and set(launches) == {("dim3(1)", "dim3(kFinBlock)")}
    # set by one thread, after the barrier inside fold_partials
    body = _body(text, f" {kernel}(")
    assert body.index("fold_partials") < body.index("if (threadIdx.x != 0) return;") < body.rindex("= 1;")
