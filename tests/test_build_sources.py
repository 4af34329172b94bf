"""The package's source folder holds what the build compiles, or what those
sources include, and nothing else: a stray copy of a source would look like
part of the library and never be built."""
import os
import re

from paper_2306_10652_amd import build


def test_csrc_holds_only_what_is_built():
    reached, todo = set(), list(build.SOURCES)
    while todo:
        name = todo.pop()
        if name in reached:
            continue
        reached.add(name)
        text = open(os.path.join(build.CSRC, name)).read()
        for inc in re.findall(r'^\s*#include "([^"/]+)"', text, flags=re.M):
            todo.append(inc)
    assert sorted(os.listdir(build.CSRC)) == sorted(reached)
