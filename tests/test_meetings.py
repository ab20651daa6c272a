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
