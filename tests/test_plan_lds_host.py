"""The LDS that the counting kernel hands to the plan of a round (CPU only).

k_supertile_counts gives plan_round three arrays of LDS: sigma words each for the block
counts and the element starts, and NT / 64 words for the scan's wave totals.  Each must lie
inside the array it points into, also at the widest digits (11 bits).  The expressions are
taken from the source and evaluated.
"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_05302_amd", "csrc")


def kernel_source():
    text = open(os.path.join(CSRC, "kernels_prefix.hpp")).read()
    text = re.sub(r"//[^\n]*", "", text)
    start = text.index("void k_supertile_counts(")
    return text, text[start:text.index("\ntemplate", start)]


def evaluate(expr, env):
    return eval(re.sub(r"(?<![/])/(?![/])", "//", expr), {"__builtins__": {}}, env)


@pytest.mark.parametrize("nt", [512, 1024])
@pytest.mark.parametrize("bits", [1, 8, 10, 11])
def test_plan_arrays_lie_inside_their_lds(bits, nt):
    text, body = kernel_source()
    env = {"NT": nt, "sigma": 1 << bits}
    for name, value in re.findall(r"constexpr \w+ (k\w+) = ([^;]+);", text):
        if re.fullmatch(r"[\w\s<+*/-]+", value):
            env[name] = evaluate(value, env)
    arrays = {}  # the kernel's LDS arrays and their words
    for decl in re.findall(r"__shared__ uint32_t ([^;]+);", body):
        for name, size in re.findall(r"(\w+)\[([^\]?]+)\]", decl):
            arrays[name] = evaluate(size, env)
    call = re.search(r"plan_round<NT>\(([^;]+)\);", body).group(1)
    args = [a.strip() for a in call.split(",")]
    # plan_round(cnt, sigma, log2b, C, E, tmp, ...)
    for pointer, words in ((args[3], 1 << bits), (args[4], 1 << bits), (args[5], nt // 64)):
        array, _, offset = (s.strip() for s in pointer.partition("+"))
        at = evaluate(offset, env) if offset else 0
        assert at + words <= arrays[array], (pointer, at, words, arrays[array])
