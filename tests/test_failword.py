"""The failure word of the blocked Cholesky factorization (host code): every
wavefront leaves after the barrier of the panel that broke down, whether it
reads the word at once or only after a faster wavefront is through the next
panel."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_03754_amd", "csrc")

PROGRAM = r"""
#include "btc_failword.h"
// Panel at which a wavefront leaves (panels: none), bad[q] telling which panels
// have a bad pivot; late: it reads the word after a faster one has been through
// panel q + 1.
int leaves(int panels, const bool* bad, bool late) {
    int word = 0;
    for (int q = 0; q < panels; ++q) {
        if (bad[q] && !word) word = btc::panel_mark(q);
        int seen = word;
        // the faster wavefront is past this barrier only if it saw no failure
        if (late && !btc::panel_failed(word, q) && q + 1 < panels && bad[q + 1]) seen = btc::panel_mark(q + 1);
        if (btc::panel_failed(seen, q)) return q;
    }
    return panels;
}
int main() {
    for (int panels = 1; panels <= 8; ++panels)
        for (int mask = 0; mask < 1 << panels; ++mask) {
            bool bad[8];
            int want = panels;
            for (int q = panels - 1; q >= 0; --q)
                if ((bad[q] = (mask >> q) & 1)) want = q;
            if (leaves(panels, bad, false) != want || leaves(panels, bad, true) != want) return 1;
        }
    return 0;
}
"""


def test_every_wavefront_leaves_after_the_same_barrier(tmp_path):
    src, exe = tmp_path / "failword.cpp", tmp_path / "failword"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
