"""Every kernel launch of the library is followed, in its function, by a check of the
launch's status: without one a launch that fails returns success with the output
untouched, and the error turns up in a later, unrelated call.  A helper named
launch_... or dispatch_... may leave the check to its callers."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2104_04609_amd", "csrc")
SOURCES = sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


CHECK = re.compile(r"BEM_LAUNCH_CHECK\(\)|hipGetLastError\(\)")


def unchecked(text):
    """Lines of launches with no check before the end of their function (a closing
    brace in the first column)."""
    text = re.sub(r"//[^\n]*", "", text)
    ends = [m.start() for m in re.finditer(r"^\}", text, re.M)] + [len(text)]
    helpers, bodies = [], []
    for begin, end in zip([0] + ends, ends):
        body = text[begin:end]
        name = re.search(r"^\S.*\b((?:launch|dispatch)_\w+)\(", body, re.M)
        if name and not CHECK.search(body):
            helpers.append(name[1])
        else:
            bodies.append((begin, body))
    launch = re.compile("|".join([r"hipLaunchKernelGGL\(|<<<"] + [rf"\b{h}[<(]" for h in helpers]))
    lines = []
    for begin, body in bodies:
        last = max([m.start() for m in CHECK.finditer(body)], default=-1)
        lines += [text.count("\n", 0, begin + m.start()) + 1 for m in launch.finditer(body)
                  if m.start() > last]
    return lines


@pytest.mark.parametrize("source", SOURCES)
def test_launches_are_checked(source):
    with open(os.path.join(CSRC, source)) as f:
        assert unchecked(f.read()) == []
