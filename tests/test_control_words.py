"""What one workgroup of the finalize kernel writes while others of its grid may
only just start: none of it may be a word they decide by."""
import os
import re

SOURCE = os.path.join(os.path.dirname(__file__), "..", "paper_2005_10761_amd", "csrc", "rtopk_encode.hip")


def _function(text, name):
    """The definition of ``name``, comments removed."""
    text = re.sub(r"//[^\n]*", "", text)
    start = text.index("{", re.search(r"\b%s\([^;{]*\)\s*\{" % name, text).end() - 1)
    depth = 0
    for i in range(start, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[start:i + 1]
    raise AssertionError(name)


def test_finalize_reads_no_control_word_that_it_writes():
    """A workgroup that starts late must come to the decision the others came to: to leave,
    or to stay for the selection over all candidates. With a word that workgroup 0 sets
    meanwhile it would stay alone and poll at check-in until its limit."""
    with open(SOURCE) as f:
        body = _function(f.read(), "finalize_body")
    fields = re.findall(r"ctl->(\w+)(\s*=(?!=))?", body)
    written = {name for name, assigned in fields if assigned}
    read = {name for name, assigned in fields if not assigned}
    assert {"mode", "overflow", "bd_lo", "c_def"} <= read and {"T", "K_star", "err"} <= written
    assert not read & written, read & written
