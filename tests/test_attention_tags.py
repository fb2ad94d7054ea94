"""The tags of the long-context attention's partial words, compiled for the
host: never 0 (what a new handle's words hold), and different for all launches
in a row, also where the pass count starts over."""
import os
import subprocess

import pytest

from paper_2608_10362_amd import build

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "attention_tag.h"
using namespace specdec;
int main(int argc, char** argv) {
  const uint32_t layers = (uint32_t)strtoul(argv[1], 0, 10);
  uint32_t pass = (uint32_t)strtoul(argv[2], 0, 10);
  for (int i = 3; i < argc; ++i) {  // step by argv[i] passes, then print the pass and its first and last tag
    pass = attention_pass_after(pass, (uint32_t)strtoul(argv[i], 0, 10), layers);
    printf("%u %u %u\n", pass, attention_tag(pass, layers, 0u), attention_tag(pass, layers, layers - 1u));
  }
}
"""


@pytest.fixture(scope="module")
def tags(tmp_path_factory):
    d = tmp_path_factory.mktemp("tags")
    src, exe = d / "tags.cpp", str(d / "tags")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(src), "-o", exe], check=True, timeout=120)

    def run(layers, start, steps):
        out = subprocess.run([exe, str(layers), str(start)] + [str(s) for s in steps], check=True, timeout=60,
                             stdout=subprocess.PIPE, text=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


@pytest.mark.parametrize("layers", [1, 2, 3, 4, 22, 32, 80, 1 << 20])
def test_tags_around_the_start_over(tags, layers):
    P = (2 ** 32 - 1) // layers
    assert tags(layers, 0, [1]) == [(1, layers + 1, 2 * layers)]  # a new handle's first pass
    got = tags(layers, P - 4, [1] * 8)
    assert [g[0] for g in got] == [P - 3, P - 2, P - 1, 0, 1, 2, 3, 4]
    seen = set()
    for _, lo, hi in got:
        assert 0 < lo <= hi < 2 ** 32 and hi - lo == layers - 1
        assert not seen & {lo, hi}
        seen |= {lo, hi}
    # several passes at once (repeats outside a pass) land where single steps do
    assert tags(layers, P - 4, [3, 5])[-1] == got[7]


def test_header_is_part_of_the_kernels():
    csrc = build.CSRC
    for fn, call in (("attention.hip", "attention_tag("), ("sampling.hip", "attention_pass_after(")):
        assert call in open(os.path.join(csrc, fn)).read()
