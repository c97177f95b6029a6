"""Which form the index half of a batch takes (csrc/fs_dedup_rule.h), at the lines that the header gives its measurements
for: compiled by itself and asked.  The parity of the forms is tested on the GPU (test_gpu_bucket_dedup.py,
test_gpu_small_index.py)."""
import os
import subprocess

import pytest

import paper_2604_24073_amd as fs

CSRC = os.path.join(os.path.dirname(fs.LIB_PATH), "csrc")
LINES = [                                                    # IDs, rows of the table, an operation of its own, by ranges
    (8193, 512, True, False), (786_432, 512, False, False), (60_000, 500, False, False),           # one pass: never
    (8193, 513, True, True), (393_216, 1 << 18, True, True), (393_217, 1 << 18, True, False),      # two: alone
    (786_432, 20_000, True, False), (393_217, 1 << 18, False, True), (1 << 20, 20_000, False, True),   # two: index half
    (393_217, (1 << 18) + 1, True, True), (1 << 20, 4_000_000, True, True), (1 << 20, 1 << 31, False, True),   # more
    ((1 << 20) + 1, 4_000_000, True, False), (9000, (1 << 31) + 1, False, False), (9000, 0, True, False)]      # do not fit

ONE_WORKGROUP = [(True, 500, 8192), (True, 1 << 40, 8192), (False, 65_536, 12_288), (False, 65_537, 10_240)]   # rows, IDs


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, exe = d / "rule.cpp", d / "rule"
    src.write_text('#include <stdio.h>\n#include <stdlib.h>\n#include "fs_dedup_rule.h"\n'
                   "int main(int argc, char **argv) {\n"
                   "    for (int i = 1; i + 2 < argc; i += 3)\n"
                   "        printf(\"%d\\n\", (int)fs::dedup_by_ranges(atoll(argv[i]), fs::key_bits_of(atoll(argv[i + 1])), atoi(argv[i + 2]) != 0));\n"
                   "    printf(\"one workgroup\\n\");\n" +
                   "".join("    printf(\"%%d\\n\", (int)fs::small_index_ids(%s, fs::key_bits_of(%dll)));\n" % (str(c).lower(), r)
                           for c, r, _ in ONE_WORKGROUP) + "}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    args = [str(int(x)) for line in LINES for x in line[:3]]
    return subprocess.run([str(exe), *args], check=True, capture_output=True, text=True).stdout.split()


@pytest.mark.parametrize("i", range(len(LINES)), ids=["%d IDs of %d rows%s" % (n, r, ", alone" if a else "") for n, r, a, _ in LINES])
def test_the_form_on_both_sides_of_every_line(rule, i):
    assert rule[i] == str(int(LINES[i][3]))


def test_most_ids_of_the_one_workgroup(rule):
    assert rule[len(LINES):] == ["one", "workgroup"] + [str(n) for _, _, n in ONE_WORKGROUP]
