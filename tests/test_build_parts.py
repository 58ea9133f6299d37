"""The implicit-GEMM family is one source compiled into several objects: every part the build asks for exists, and what is
kept per object (the address of the developer build's time stamps) is set in each."""
import os
import re

from paper_1910_00078_amd import build


def test_every_object_of_the_family_is_instantiated_and_traced():
    parts = set(range(1, build.PARTS["kernels_igemm.hip"] + 1))
    text = open(os.path.join(build.CSRC, "kernels_igemm.hip")).read()
    numbers = lambda pattern: {int(n) for n in re.findall(pattern, text)}  # noqa: E731
    assert numbers(r"#define IGEMM_PART_(\d+)\(X\)") == parts
    assert numbers(r"#(?:el)?if CVX_PART == (\d+)") == parts
    assert numbers(r"IGEMM_PART_(\d+)\(IGEMM_INSTANTIATE\)") == parts
    everywhere = re.search(r"#define IGEMM_ALL\(X\) (.*)", text).group(1)
    assert {int(n) for n in re.findall(r"IGEMM_PART_(\d+)\(X\)", everywhere)} == parts
    traced = re.search(r"#define IGEMM_TRACE_PARTS\(X\) (.*)", text)
    assert traced and {int(n) for n in re.findall(r"X\((\d+)\)", traced.group(1))} == parts
