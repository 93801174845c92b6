"""The clustering rounds of the BVH build as the host drives them, on the
CPU: csrc/ploc.h (the host's reading of what a group of rounds left) compiled
by itself, the rounds and the one-block tail as a model that keeps the device
code's buffers: the tail merges in LDS and writes back only the counts.
Boxes whose merged areas are not finite leave clusters that no round merges;
that has to end as a refusal, whether rounds before it made progress or not."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_04981_amd", "csrc")
DONE, MORE, STALLED = 0, 1, 2
R = 16  # the search window on either side


@pytest.fixture(scope="module")
def step(tmp_path_factory):
    d = tmp_path_factory.mktemp("ploc")
    src, lib = d / "ploc.cc", d / "libploc.so"
    src.write_text('#include "ploc.h"\nextern "C" int step(int b, int c, int n) { return ploc_step(b, c, n); }\n'
                   'extern "C" int tail() { return PLOC_TAIL; }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


def one_round(ids, lo, hi):
    """(survivors' ids, boxes, the merged pairs) of one round."""
    m = len(ids)
    best, nn = np.full(m, np.inf, np.float32), np.full(m, -1)
    with np.errstate(all="ignore"):
        for d in [*range(-R, 0), *range(1, R + 1)]:
            a, b = max(0, -d), m - max(0, d)
            if a >= b:
                continue
            e = np.fmax(hi[a:b], hi[a + d:b + d]) - np.fmin(lo[a:b], lo[a + d:b + d])
            area = e[:, 0] * e[:, 1] + e[:, 1] * e[:, 2] + e[:, 2] * e[:, 0]
            on = area < best[a:b]
            best[a:b][on], nn[a:b][on] = area[on], (np.arange(a, b) + d)[on]
    i = np.arange(m)
    mate = np.where((nn >= 0) & (nn[nn] == i), nn, -1)
    lead, keep = mate > i, ~((mate >= 0) & (mate < i))
    lo, hi = lo.copy(), hi.copy()
    lo[lead], hi[lead] = np.fmin(lo[lead], lo[mate[lead]]), np.fmax(hi[lead], hi[mate[lead]])
    pairs = [(ids[a], ids[mate[a]]) for a in np.nonzero(lead)[0]]
    return keep, lo, hi, lead, pairs


def cluster(step, lo, hi):
    """The host's loop; returns its outcome and the internal nodes' children."""
    n, tail = len(lo), step.tail()
    node = {}
    mem = [~i for i in range(n)], lo.astype(np.float32), hi.astype(np.float32)
    state = n, n - 2

    def merge(ids, lo, hi, nxt):
        keep, lo, hi, lead, pairs = one_round(ids, lo, hi)
        ids = list(ids)
        for k, (a, pair) in enumerate(zip(np.nonzero(lead)[0], pairs)):
            ids[a] = nxt - k
            node[nxt - k] = pair
        return [v for v, on in zip(ids, keep) if on], lo[keep], hi[keep], nxt - len(pairs)

    for _ in range(8 * n):
        m0 = state[0]
        if m0 > tail:
            for _ in range(math.ceil(math.log(m0 / tail) / math.log(1.2))):
                c = state[0]
                ids, l, h, nxt = merge(mem[0][:c], mem[1][:c], mem[2][:c], state[1])
                mem, state = (ids, l, h), (len(ids), nxt)
        if state[0] <= tail:  # the tail block: from memory, its merges not written back
            c = state[0]
            ids, l, h, nxt = mem[0][:c], mem[1][:c], mem[2][:c], state[1]
            while len(ids) > 1:
                before = nxt
                ids, l, h, nxt = merge(ids, l, h, nxt)
                if nxt == before:
                    break
            state = len(ids), nxt
        r = step.step(m0, *state)
        if r != MORE:
            return r, node
    raise AssertionError("the host's loop does not end")


def boxes(n, seed):
    rng = np.random.default_rng(seed)
    c = rng.uniform(-1, 1, (n, 3))
    c = c[np.lexsort((c[:, 2] // 0.2, c[:, 1] // 0.2, c[:, 0] // 0.2))]
    s = rng.uniform(0.001, 0.1, (n, 3))
    return c - s, c + s


@pytest.mark.parametrize("n", [2, 3, 300, 1024, 1025, 3000])
def test_finite_boxes_end_as_one_tree(step, n):
    r, node = cluster(step, *boxes(n, n))
    assert r == DONE and sorted(node) == list(range(n - 1))
    seen, todo = set(), [0]
    while todo:
        for c in node[todo.pop()]:
            assert c not in seen
            seen.add(c)
            if c >= 0:
                todo.append(c)
    assert {c for c in seen if c < 0} == {~i for i in range(n)} and len(seen) == 2 * n - 2


@pytest.mark.parametrize("n", [2, 300, 1024, 1025, 3000])
def test_an_infinite_box_is_refused(step, n):
    lo, hi = boxes(n, n)
    hi[n // 3, 1] = np.inf
    assert cluster(step, lo, hi)[0] == STALLED


@pytest.mark.parametrize("n", [300, 1500, 3000])
def test_areas_beyond_float_are_refused(step, n):
    """Two groups 1e20 apart on two axes: each merges by itself, their union's area is infinite."""
    lo, hi = boxes(n, n)
    lo, hi = lo * 1e13, hi * 1e13
    lo[n // 2:, :2] += 1e20
    hi[n // 2:, :2] += 1e20
    assert cluster(step, lo, hi)[0] == STALLED
