"""Behind a 16-byte buffer store whose offset has a scalar-register part the compiler may write the store's data registers
again at once; gfx950 has not read them all by then, and some lanes store what came next.  With a constant in that place the
compiler leaves the wait state.  Read from the source: whether a run shows it depends on what the scheduler puts there."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2001_07710_amd", "csrc")


def _arguments(text, at):
    """The arguments of the call whose opening bracket is at text[at]."""
    args, depth, start = [], 0, at + 1
    for i in range(at, len(text)):
        if text[i] in "([{":
            depth += 1
        elif text[i] in ")]}":
            depth -= 1
            if depth == 0:
                return args + [text[start:i].strip()]
        elif text[i] == "," and depth == 1:
            args.append(text[start:i].strip())
            start = i + 1
    raise AssertionError("no end of the call")


def test_wide_buffer_stores_have_no_scalar_offset():
    stores = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for call in re.finditer(r"raw(?:_ptr)?_buffer_store_b(?:96|128)\s*\(", text):
            args = _arguments(text, call.end() - 1)
            assert len(args) == 5 and args[3] == "0", (os.path.basename(path), args)
            stores += 1
        assert "buffer_store_dwordx" not in text and "buffer_store_format" not in text, path     # (none written by hand)
    assert stores >= 9
