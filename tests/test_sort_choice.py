"""When a build tries the short sort (csrc/sort_choice.h, compiled for the host): a
system that it does not suit pays for few tries however its number of particles
changes, and one that it suits again comes back to it."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1506_04553_amd", "csrc")
MAIN = """
#include <stdio.h>
#include "sort_choice.h"
// one line of 0 (the short sort suits) and 1 in; per build w (whole), f (short, failed), s out
int main() {
    p3t::SortChoice c;
    for (int ch; (ch = getchar()) == '0' || ch == '1';) {
        if (c.whole()) { putchar('w'); continue; }
        c.tried(ch == '1');
        putchar(ch == '1' ? 'f' : 's');
    }
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("sort_choice")
    (d / "main.cc").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "main.cc"),
                           "-o", str(d / "main")])
    return lambda dense: subprocess.run([str(d / "main")], input=dense, capture_output=True,
                                        text=True, check=True).stdout


def test_dense_systems_rarely_try(choose):
    out = choose("1" * 20000)
    assert out.startswith("f" + "w" * 16 + "f" + "w" * 32 + "f") and out.count("s") == 0
    assert out.count("f") <= 7 + 20000 // 1024
    assert max(len(r) for r in out.split("f")) == 1024


def test_others_return_to_the_short_sort(choose):
    assert choose("0" * 100) == "s" * 100
    assert choose("1" + "0" * 100) == "f" + "w" * 16 + "s" * 84
    # after a success the next failure costs as little as the first
    assert choose("1" * 60 + "0" * 300 + "1" + "0" * 20)[-21:] == "f" + "w" * 16 + "s" * 4
