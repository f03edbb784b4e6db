"""build_library(force=False) keeps a library only while it is newer than everything it was made of."""
import os
import re

from paper_2506_04642_amd import build


def test_every_included_file_is_a_source():
    known = {os.path.realpath(s) for s in build.sources()}
    todo, seen = list(known), set()
    while todo:
        path = todo.pop()
        if path in seen:
            continue
        seen.add(path)
        for name in re.findall(r'^\s*#include\s+"([^"]+)"', open(path).read(), re.M):
            found = [p for p in (os.path.join(os.path.dirname(path), name), os.path.join(build.CSRC, name)) if os.path.exists(p)]
            assert found, "%s includes %s, which is not there" % (path, name)
            todo.append(os.path.realpath(found[0]))
    assert seen <= known, sorted(seen - known)
