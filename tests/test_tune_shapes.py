"""The launch shapes that the tuner times are fields of the context's tuning
that a kernel launch reads: not tracklet_form, whose values all run the one
tracklet kernel (the tuner would keep the one that noise favours)."""
import os
import re

from paper_1905_05515_amd import api

CSRC = os.path.join(os.path.dirname(os.path.abspath(api.__file__)), "csrc")


def read_fields():
    src = "".join(open(os.path.join(CSRC, f)).read() for f in ("neighbours.hip", "persistent.hip"))
    return set(re.findall(r"tune\.(\w+)|tune->(\w+)", src))


def test_every_tuned_field_is_read_by_a_launch():
    read = {a or b for a, b in read_fields()}
    tuned = {f for shapes in api.TUNE_SHAPES.values() for f, _ in shapes}
    assert tuned <= read, tuned - read
    assert tuned == set(api.TUNING_FIELDS) - {"tracklet_form"}
