"""A wave's lanes hand data to each other through LDS without a workgroup barrier.  A
fence orders the memory accesses, but is no convergent operation: without a wave barrier
next to it the compiler may move it, and what it orders, into one side of a branch.
Every wavefront fence in the sources has its wave barrier."""
import os
import re

import paper_2601_00822_amd as pkg

CSRC = os.path.join(os.path.dirname(os.path.abspath(pkg.__file__)), "csrc")


def test_every_wavefront_fence_has_a_wave_barrier():
    fences, bare = 0, []
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".hpp", ".cpp")):
            continue
        with open(os.path.join(CSRC, name)) as fh:
            text = fh.read()
        for m in re.finditer(r'__builtin_amdgcn_fence\([^;]*"wavefront"\);', text):
            fences += 1
            if not re.match(r"\s*__builtin_amdgcn_wave_barrier\(\);", text[m.end():]):
                bare.append(f"{name}:{text.count(chr(10), 0, m.start()) + 1}")
    assert fences >= 3
    assert not bare, bare
