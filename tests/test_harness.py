"""The byte counts behind the rates that the measurement harness reports."""
import os
import re

from paper_2604_18348_amd import harness

CSRC = os.path.join(os.path.dirname(os.path.abspath(harness.__file__)), "csrc")


def test_label_sort_bytes_are_those_of_the_sort_in_the_library():
    head = open(os.path.join(CSRC, "small_head.h")).read()
    number = lambda name, text: int(re.search(r"\b%s(?: =)? (\d+)" % name, text).group(1))  # noqa: E731
    assert harness.SORT_ONE_WORKGROUP == number("SMALL_SEGS", head) * number("SEG", head)
    assert number("RBITS", head) == 7
    assert harness.label_sort_bytes(75600, 65) == 12 * 75600       # labels read twice, the permutation written once
    # one pass of labels read, labels and values written; a second that reads both
    assert harness.label_sort_bytes(4096, 65) == 12 * 4096
    assert harness.label_sort_bytes(4096, 127) == 12 * 4096
    assert harness.label_sort_bytes(4096, 128) == 28 * 4096
