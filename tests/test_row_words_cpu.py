"""Where eight 16-bit elements are read in whole 32-bit words: always inside the tensor, and the wanted elements among what
is read.  The address arithmetic of csrc/ss_device.h, compiled for the host."""
import os
import subprocess

from paper_2312_00752_amd import build

PROGRAM = r"""
#include <cstdio>
#include "ss_device.h"
int main()
{
    for (uintptr_t first = 4096; first < 4096 + 16; first += 2)         // a tensor's first element, at any element
        for (uintptr_t p = first; p < first + 64; p += 2) {             // eight elements of it
            const uintptr_t w = ss::row16_words(p, first);
            const bool inside = w >= first && w + 16 <= p + 16, holds = w == p || (w + 2 == p && w % 4 == 0);
            const bool words = p % 4 == 0 || p == first ? w == p : w % 4 == 0;
            if (!inside || !holds || !words) { std::printf("first %lu, elements at %lu: words from %lu\n", first, p, w); return 1; }
        }
    return 0;
}
"""


def test_words_lie_in_the_tensor(tmp_path):
    source, program = tmp_path / "row_words.hip", tmp_path / "row_words"
    source.write_text(PROGRAM)
    obj = str(program) + ".o"
    subprocess.run([build._hipcc(), "--offload-arch=gfx950", "-std=c++17", "-fPIC", "--offload-host-only", "-I", build.CSRC, "-I",
                    os.path.join(build.ROOT, "include"), "-c", str(source), "-o", obj], check=True, capture_output=True)
    subprocess.run(["g++", obj, "-o", str(program)], check=True, capture_output=True)
    out = subprocess.run([str(program)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
