"""Host-only, on the sources: a workgroup of a launch that does the routing steps says that it has read the call number only
behind a barrier that all of its wavefronts reach, each having read it.  (The workgroup that steps the number waits for these
words and for nothing else that ties a wavefront without a dot product; a late one would take the next call's number.)"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_09983_amd", "csrc")


def _said_behind_a_barrier(source, number, said):
    """number, said: patterns of the read of the call number and of the store of the workgroup's word.  What holds the read in
    front of the barrier takes a vector register: the number may be in one, and a copy to a scalar register does not compile then."""
    source = re.sub(r"//[^\n]*", "", source)
    first, store = re.search(number, source), re.search(said, source)
    assert first and store and first.start() < store.start()
    used, barrier, stack, n = False, [], [], 0
    for m in re.finditer(r"[{}]|asm volatile\(\"\" : : \"v\"\(r?tag\)\)|__syncthreads\(\)", source[:store.start()]):
        if m.group() == "{":
            stack.append(n)
            n += 1
        elif m.group() == "}":
            stack.pop()
        elif m.start() > first.start():
            if m.group() == "__syncthreads()":
                barrier.append((used, tuple(stack)))
            else:
                used = True
    # a barrier in a block that the store is in too: not in a branch or a loop that some may not enter
    return any(read and inside == tuple(stack[:len(inside)]) for read, inside in barrier)


@pytest.mark.parametrize("name,number,said", [
    ("stream.hip", r"rtag = ctrl\[kCtrlEpoch\]",
     r"__hip_atomic_store\((seen \+ b|glob\(R->lists_pub\) \+ \(size_t\)kListReplicas \* list_pub_entries\(T, a\.k, C\) \+ b),"),
    ("layer.hip", r"epoch0 = a\.ctrl\[kCtrlEpoch\]", r"store_entry\((seen \+ b|ra\.lists_pub \+ \(size_t\)kListReplicas \* n_pub \+ b), tag, 1u\)")])
def test_number_read_by_all_before_the_workgroup_says_so(name, number, said):
    with open(os.path.join(CSRC, name)) as f:
        assert _said_behind_a_barrier(f.read(), number, said)


def test_the_check_sees_what_it_looks_for():
    good = 'n = ctrl[k]; { asm volatile("" : : "v"(rtag)); __syncthreads(); if (x) put(b); }'
    assert _said_behind_a_barrier(good, r"ctrl\[k\]", r"put\(b\)")
    for bad in (good.replace("__syncthreads(); ", ""), good.replace("__syncthreads();", "if (y) { __syncthreads(); }"),
                good.replace('asm volatile("" : : "v"(rtag)); ', ""), good.replace('"v"', '"s"'), "n = ctrl[k]; put(b); __syncthreads();"):
        assert not _said_behind_a_barrier(bad, r"ctrl\[k\]", r"put\(b\)")
