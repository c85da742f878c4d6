"""LDS arrays of 4-byte or smaller elements that a kernel also takes as 64-bit
words: 64-bit LDS accesses and atomics need 8-byte alignment, which only the
declaration can give."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2207_04350_amd", "csrc")
DECL = re.compile(r"__shared__\s+(alignas\((\d+)\)\s+)?(u?int(?:8|16|32)_t|int|float)\s+([^;]+);")
CAST = re.compile(r"reinterpret_cast<\s*(?:const\s+)?(?:unsigned long long|uint64_t|int64_t)\s*\*>"
                  r"\(\s*(\w+)")


def _narrow_arrays_cast_wide(text):
    wide = set(CAST.findall(text))
    bad = []
    for _, align, _, names in DECL.findall(text):
        for name in re.findall(r"(\w+)\s*\[", names):
            if name in wide and int(align or 0) < 8:
                bad.append(name)
    return bad


def test_the_rule_sees_a_narrow_array():
    src = "__shared__ int32_t a[4];\nauto *w = reinterpret_cast<unsigned long long *>(a);"
    assert _narrow_arrays_cast_wide(src) == ["a"]
    assert _narrow_arrays_cast_wide(src.replace("__shared__", "__shared__ alignas(8)")) == []


def test_lds_arrays_taken_as_64_bit_words_are_aligned():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            assert _narrow_arrays_cast_wide(f.read()) == [], os.path.basename(path)
