"""Order of statements in the kernels that no run shows: the compiler may hide a
missing one today.  Read from the sources, on the CPU."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_16074_amd", "csrc")


def source(name):
    return re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, name)).read())


def bodies(text, head):
    """Text of every brace block that starts at a match of `head`."""
    out = []
    for m in re.finditer(head, text):
        at = text.index("{", m.end() - 1)
        end, depth = at, 0
        while True:
            depth += {"{": 1, "}": -1}.get(text[end], 0)
            if depth == 0:
                break
            end += 1
        out.append(text[at:end])
    return out


@pytest.mark.parametrize("walk", ["tile_of", "flex_walk"])
def test_ring_walks_check_the_range_first(walk):
    """The walks divide by a group size that is zero or negative past the last tile."""
    found = [b for b in bodies(source("k_gemm.hip"), r"auto next = \[&\]") if walk + "(" in b]
    assert found
    for b in found:
        assert "return false" in b[: b.index(walk + "(")], b


def test_ring_reads_the_next_tile_only_where_there_is_one():
    ring = bodies(source("k_gemm.hip"), r"void ring_run\(")[0]
    assert ring.count("gn.K") == 1 and "more ? (gn.K" in ring


def test_ring_counts_the_stores_of_its_own_epilogue():
    """The counted wait behind a 16-bit epilogue takes the store count from the
    sizes the epilogue itself is written with."""
    text = source("k_gemm.hip")
    ring, epi = (bodies(text, r"void %s\(" % f)[0] for f in ("ring_run", "epilogue_bf16"))
    assert "using E16 = Epi16<EPI, TN, TM>" in ring and "wait_vmcnt<NI + E16::STORES>" in ring
    assert not re.search(r"STORES\s*=", ring)
    assert "using E = Epi16<EPI, TN, TM>" in epi and "NB = E::NB, NI = E::NI" in epi


@pytest.mark.parametrize("name", ["k_expert.hip", "k_attn.hip"])
def test_barriers_that_publish_fetched_tiles_follow_a_wait(name):
    """A barrier does not wait for LDS DMA: in a kernel that fetches tiles by it,
    the barrier at the top of the tile loop stands behind an explicit wait."""
    found = 0
    for body in bodies(source(name), r"__global__ [^;{]*"):
        if not re.search(r"\bissue(_kv)?\(|global_load_lds", body):
            continue
        loop = re.search(r"for \((?:int32_t|int) j\w* = ", body)
        assert loop, body[:200]
        top = re.search(r"__syncthreads\(\)|s_barrier\(\)", body[loop.start():])
        before = body[loop.start(): loop.start() + top.start()]
        assert re.search(r"s_waitcnt\(0\)|attn_wait_vmcnt<0>\(\)", before), body[:300]
        found += 1
    assert found >= 2
