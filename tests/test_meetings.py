"""The meetings of the one-launch kernel's workgroups, every order of their
steps: nobody misses a word that another has overwritten.  Which words a meeting
uses comes from the kernel's own header, built for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2403_01261_amd", "csrc")
MEETINGS = 5

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "meeting.h"
using namespace gsl;
int main() {
  for (unsigned m = 0; m < 256; ++m) {
    printf("%u\n", meeting_copy(m));
    for (unsigned o = 0; o < 256; ++o)  // a word says its own meeting and launch, whatever its payload
      for (unsigned e : {1u, 7u, (1u << 24) - 1})
        if (meeting_posted(meeting_word(e, o, 0xffffffffu), e, m) != (o == m) || meeting_posted(meeting_word(e, o, 0), e ^ 2u, m))
          return 1;
  }
}
"""


@pytest.fixture(scope="module")
def copies(tmp_path_factory):
    """The word (of each workgroup) that every meeting uses."""
    d = tmp_path_factory.mktemp("host")
    src, out = str(d / "meeting.cpp"), str(d / "meeting")
    open(src, "w").write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", out], check=True)
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    return [int(x) for x in r.stdout.split()]


def explore(start, steps):
    """Every state reached from `start`; those without a step."""
    seen, todo, ends = {start}, [start], []
    while todo:
        s = todo.pop()
        nxt = steps(s)
        if not nxt:
            ends.append(s)
        for t in nxt:
            if t not in seen:
                seen.add(t)
                todo.append(t)
    return seen, ends


def meeting_steps(kinds, copies, groups):
    """State: the words of every workgroup by copy, the release word, and per
    workgroup (meeting, words still to be seen, or None before it posts).  A
    meeting is direct (True: everyone reads every word) or led by workgroup 0,
    which alone reads them and then releases the others."""
    n_copies = max(copies) + 1
    everyone = (1 << groups) - 1

    def steps(state):
        words, release, at = state
        out = []
        for w in range(groups):
            m, left = at[w]
            if m == len(kinds):
                continue
            base = copies[m] * groups
            reads = kinds[m] or w == 0
            if left is None:  # post
                new = list(words)
                new[base + w] = m
                out.append((tuple(new), release, at[:w] + ((m, everyone if reads else 0),) + at[w + 1:]))
            elif reads and left:  # look at one more word
                for j in range(groups):
                    if left >> j & 1 and words[base + j] == m:
                        out.append((words, release, at[:w] + ((m, left & ~(1 << j)),) + at[w + 1:]))
            elif reads:  # all seen
                rel = release if kinds[m] else m
                out.append((words, rel, at[:w] + ((m + 1, None),) + at[w + 1:]))
            elif release == m:
                out.append((words, release, at[:w] + ((m + 1, None),) + at[w + 1:]))
        return out

    return (tuple([-1] * (n_copies * groups)), -1, tuple([(0, None)] * groups)), steps


@pytest.mark.parametrize("groups", [2, 3])
@pytest.mark.parametrize("kinds", [[True] * MEETINGS, [False] * MEETINGS, [False, False, True, True, True],
                                   [True, False, True, False, True]])
def test_every_order_of_the_meetings_ends(copies, groups, kinds):
    seen, ends = explore(*meeting_steps(kinds, copies, groups))
    assert ends, "the meetings end at all"
    for words, _, at in ends:
        assert all(m == len(kinds) for m, _ in at), "a workgroup waits for ever: %s, words %s" % (at, words)


def sum_steps(meetings, copies, threads):
    """State: the sums by copy, the threads that wait at the barrier, and per
    thread (meeting, step, whether it has seen every sum whole).  The steps of a
    meeting: thread 0 clears the sums, a barrier, everyone adds one, a barrier,
    everyone reads the sum."""
    n_copies = max(copies) + 1

    def steps(state):
        sums, waiting, at = state
        out = []

        def put(w, m, step, whole, sums=sums, waiting=waiting):
            out.append((sums, waiting, at[:w] + ((m, step, whole),) + at[w + 1:]))

        if all(waiting):
            return [(sums, (False,) * threads, tuple((m, step + 1, whole) for m, step, whole in at))]
        for w in range(threads):
            m, step, whole = at[w]
            if m == meetings or waiting[w]:
                continue
            c = copies[m]
            if step == 0:
                put(w, m, 1, whole, sums=sums[:c] + (0,) + sums[c + 1:] if w == 0 else sums)
            elif step in (1, 3):
                put(w, m, step, whole, waiting=waiting[:w] + (True,) + waiting[w + 1:])
            elif step == 2:
                put(w, m, 3, whole, sums=sums[:c] + (sums[c] + 1,) + sums[c + 1:])
            else:
                put(w, m + 1, 0, whole and sums[c] == threads)
        return out

    return (tuple([0] * n_copies), (False,) * threads, tuple([(0, 0, True)] * threads)), steps


@pytest.mark.parametrize("threads", [2, 3])
def test_every_thread_reads_a_meetings_whole_sum(copies, threads):
    seen, ends = explore(*sum_steps(4, copies, threads))
    assert ends and all(m == 4 for _, _, at in ends for m, _, _ in at)
    assert all(whole for _, _, at in seen for _, _, whole in at), "a sum was cleared before its last reader"
