"""Inline assembly of the kernels names what it writes: the compiler keeps values of its own in scalar registers across it."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_14838_amd", "csrc")
STRING = re.compile(r'"((?:[^"\\]|\\.)*)"')
WRITES = re.compile(r"\bs_\w+\s+(m0|vcc|exec)\b")                         # as the first operand
WRITES_SCC = re.compile(r"\bs_(?:add|sub|and|or|xor|lsh|ashr|cmp|min|max|not|bfe)")


def _statements():
    """(place, instructions, names in the clobber list) of every asm statement."""
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"\basm(?:\s+volatile)?\s*\(", text):
            end = text.index(";", m.end())
            parts = [[]]                                                  # strings between the colons outside of them
            for token in re.finditer(STRING.pattern + "|:", text[m.end():end]):
                if token.group(0) == ":":
                    parts.append([])
                else:
                    parts[-1].append(token.group(1))
            code = re.sub(r"\\[nt]", " ", "".join(parts[0]))
            yield "%s, asm %d" % (os.path.basename(path), text.count("asm", 0, m.end())), code, set(parts[3]) if len(parts) > 3 else set()


def test_every_scalar_register_written_is_named():
    found = list(_statements())
    assert sum("global_load_lds" in code for _, code, _ in found) == 3    # the statements are read as they are written
    for where, code, named in found:
        written = set(WRITES.findall(code)) | ({"scc"} if WRITES_SCC.search(code) else set())
        assert written <= named, (where, written, named)
