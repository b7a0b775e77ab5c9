"""The captured frame step is replayed only while every argument of its launches
is unchanged: its key holds each field of the structures that they take by
value (read from the sources; runs without a GPU)."""

import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_03989_amd", "csrc")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*|/\*.*?\*/", "", f.read(), flags=re.S)


def _fields(struct):
    body = re.search(r"struct %s \{(.*?)\n\};" % struct, _source("gbp_device.hpp"), flags=re.S).group(1)
    names = []
    for decl in body.split(";"):
        m = re.match(r"\s*(?:const\s+)?\w+\s*\*?\s*(\w.*)", decl.strip(), flags=re.S)
        if m:
            names += [re.match(r"\s*\*?(\w+)", n).group(1) for n in m.group(1).split(",")]
    return names


@pytest.mark.parametrize("struct,var,n", [("Geo", "g", 10), ("Strengths", "s", 14), ("Inputs", "in", 8)])
def test_every_field_is_in_the_key(struct, var, n):
    key = re.search(r"track_graph_key\(.*?\n\}", _source("pixvod_runtime.hip"), flags=re.S).group(0)
    fields = _fields(struct)
    assert len(fields) >= n, fields
    missing = [f for f in fields if not re.search(r"\b%s\.%s\b" % (var, f), key)]
    assert not missing, missing
