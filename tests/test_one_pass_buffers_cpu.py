"""Order of LDS accesses and barriers in the block loop of the one-pass profile, from its source.

The waves meet once per block of 64 rows (twice more where the block is done again). The next block's loads
go straight into the LDS buffers that this block's rows came in, as soon as a wave is past the last of
these barriers, so whatever a wave reads from them it has to read in front of it."""
import os
import re

SOURCE = os.path.join(os.path.dirname(__file__), "..", "paper_2310_01801_amd", "csrc", "profile_once.hip")


def _block(text, start):
    """The text between the brace that opens at or behind `start` and the one that closes it."""
    begin = text.index("{", start)
    depth = 0
    for i in range(begin, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[begin + 1:i]
    raise AssertionError("unbalanced braces")


def _lambdas(text):
    return {m.group(1): _block(text, m.end() - 1) for m in re.finditer(r"auto (\w+) = \[&\]\([^)]*\)[^{;]*\{", text)}


def _last_paths(body):
    """Per path through the block (done once; done again) the text in execution order, without the lambdas' own text."""
    for inner in _lambdas(body).values():
        body = body.replace(inner, "", 1)
    first = _block(body, body.index("if (!again)"))
    again = _block(body, body.index("if (again) {"))
    rest = body[body.index(again) + len(again):]
    return [first + rest, again + rest]


def test_rows_of_a_block_are_read_in_front_of_its_last_barrier():
    text = re.sub(r"//[^\n]*", "", open(SOURCE).read())
    loop = "for (int i = mine - 1; i >= 0; --i, buf ^= 1)"
    body = _block(text, text.index(loop) + len(loop))
    lambdas = _lambdas(body)
    for path in _last_paths(body):
        path = path.replace("if (again) fg_barrier();", "")   # (of the path that goes on to a later one)
        assert path.count("fg_barrier()") == 1
        behind = path[path.index("fg_barrier()"):]
        for name, inner in lambdas.items():
            if re.search(r"\b" + name + r"\(", behind):
                behind += inner
        reached = set(re.findall(r"\bs_[qx]\b", behind))
        assert not reached, "read behind the block's last barrier: %s" % sorted(reached)
