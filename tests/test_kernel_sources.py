"""Properties of the device code that no run on a GPU shows: read from the sources and from the code generated for them."""
import os
import re

import pytest

from paper_2605_28657_amd import build as b

KERNELS = [s for s in b.SOURCES if s.startswith("kernels_")]


def _calls(text, name):
    """(position, arguments) of every call of `name` in the text."""
    for m in re.finditer(re.escape(name) + r"\w*\(", text):
        depth, args, cur = 1, [], ""
        for ch in text[m.end():]:
            depth += (ch in "([{") - (ch in ")]}")
            if depth == 0:
                break
            if ch == "," and depth == 1:
                args.append(cur.strip())
                cur = ""
            else:
                cur += ch
        yield m.start(), args + [cur.strip()]


@pytest.mark.parametrize("src", KERNELS)
def test_scalar_offsets_stay_inside_the_descriptor(src):
    """A buffer load's range check covers the per-lane offset only: it is compared with (size - scalar offset), which means
    nothing once the scalar offset is past the size.  Prefetches run past a layer's last weight block, so wherever a
    load has a scalar offset, the block it is computed from must be held inside the layer (block_in)."""
    text = open(os.path.join(b.CSRC, src)).read()
    for pos, args in _calls(text, "__builtin_amdgcn_raw_buffer_load"):
        assert len(args) == 4, (src, args)
        if args[2] == "0":
            continue
        body = text[text.rfind("auto ", 0, pos):pos] + args[2]        # the lambda that issues the load
        assert "block_in(" in body, f"{src}: scalar offset {args[2]!r} is not held inside the layer"
