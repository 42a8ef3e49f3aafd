"""Launches that give a kernel one array twice, read from the sources: where one
of the two parameters is written through, neither may be __restrict__ (a load
through the other could then legally be moved past the store, for instance a
sort's reads past the barrier that its writes follow)."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2410_22697_amd", "csrc")


def _read(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def _split(s):
    """Top-level comma-separated parts of s."""
    parts, depth, cur = [], 0, ""
    for ch in s:
        depth += ch in "([{"
        depth -= ch in ")]}"
        if ch == "," and depth == 0:
            parts.append(cur)
            cur = ""
        else:
            cur += ch
    return [" ".join(p.split()) for p in parts + [cur]]


def _balanced(text, at):
    """The text between the parenthesis at `at` and its partner."""
    depth = 0
    for i in range(at, len(text)):
        depth += text[i] == "("
        depth -= text[i] == ")"
        if depth == 0:
            return text[at + 1:i]
    raise AssertionError("unbalanced")


def _kernels():
    out = {}
    for name in ("buffer_kernels.hpp", "sample_kernels.hpp"):
        text = _read(name)
        for m in re.finditer(r"__global__[^;{]*?void\s+(k_\w+)\s*(\()", text):
            out[m.group(1)] = _split(_balanced(text, m.start(2)))
    return out


def _launches():
    text = _read("massive.hip")
    for m in re.finditer(r"ms::(k_\w+)(?:<[^<>;]*>)?<<<[^;]*?>>>\s*(\()", text, re.S):
        if "__VA_ARGS__" not in _balanced(text, m.start(2)):
            yield m.group(1), _split(_balanced(text, m.start(2)))
    for m in re.finditer(r"\bMS_SCAN(\()(?=k_)", text):  # kernel, which scan, tiles, stream, its arguments
        kernel, _, _, _, *args = _split(_balanced(text, m.start(1)))
        yield kernel, args


def _clash(params, args):
    """Parameter pairs that get the same array, one of them written, one __restrict__."""
    bad = []
    for i in range(len(args)):
        for j in range(i + 1, len(args)):
            if args[i] != args[j] or "*" not in params[i] or "*" not in params[j]:
                continue
            written = [p for p in (params[i], params[j]) if not p.startswith("const")]
            if written and ("__restrict__" in params[i] or "__restrict__" in params[j]):
                bad.append((params[i], params[j]))
    return bad


def test_no_restrict_on_an_array_passed_twice():
    kernels, seen = _kernels(), 0
    for name, args in _launches():
        assert len(args) <= len(kernels[name]), (name, args)
        assert not _clash(kernels[name], args), (name, _clash(kernels[name], args))
        seen += 1
    assert seen > 25, "the launches were not found"


def test_one_block_sort_sorts_in_place():
    # keys always end where they began, and the values do unless a caller asks
    # for another array: none of the four may be __restrict__
    arrays = [p for p in _kernels()["k_sort_one"] if re.search(r"\b(keys|vals|keys_out|vals_out)$", p)]
    assert len(arrays) == 4
    assert not [p for p in arrays if "__restrict__" in p]
