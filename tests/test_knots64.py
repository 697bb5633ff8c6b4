"""kep_knots64.h on the CPU: exactly the generator's output, each entry the
correctly rounded sine and cosine of n/64."""
import importlib.util
import math
import os
import re

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_0812_2976_amd", "csrc")
HEADER = os.path.join(CSRC, "kep_knots64.h")


def test_knots_header_is_what_the_generator_writes(tmp_path):
    spec = importlib.util.spec_from_file_location("gen_tables", os.path.join(CSRC, "gen_tables.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    out = tmp_path / "k.h"
    gen.write_knots(str(out))
    assert out.read_text() == open(HEADER).read()


def test_knots_are_sines_and_cosines():
    rows = re.findall(r"\{(\S+p\S+), (\S+p\S+)\},", open(HEADER).read())
    assert len(rows) == 209
    for n, (s, c) in enumerate(rows):
        s, c = float.fromhex(s), float.fromhex(c)
        # the host's sin and cos are within one ulp; the entry is the nearest binary64 value
        assert abs(s - math.sin(n / 64)) <= math.ulp(s) and abs(c - math.cos(n / 64)) <= math.ulp(c)
