"""Roles of the waves of a sliding-histogram work-group, compiled for the host:
whatever SIMDs and LDS bases the waves have read, no role is taken twice."""
import os
import subprocess

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19926_amd", "csrc")

_MAIN = r"""
#include "mf_hist_role.h"
int main()
{
    for (int s = 0; s < 256; ++s)            // a SIMD for each wave
        for (int b = 0; b < 16; ++b) {       // an LDS base for each wave, zero or not
            uint32_t words[4];
            for (int i = 0; i < 4; ++i) words[i] = hist_role_word((s >> 2 * i) & 3, (b >> i & 1) ? 640 : 0);
            int seen = 0;
            for (int i = 0; i < 4; ++i) seen |= 1 << hist_role(words, i);
            if (seen != 15) return 1;
        }
    // four SIMDs: search on SIMDs 0 and 1 in the lower half of the LDS, on 2 and 3 in the upper
    for (uint32_t up = 0; up < 2; ++up) {
        const uint32_t words[4] = {hist_role_word(2, up), hist_role_word(0, up), hist_role_word(3, up), hist_role_word(1, up)};
        for (int i = 0; i < 4; ++i)
            if ((hist_role(words, i) < 2) != ((words[i] & 3) / 2 == up)) return 2;
    }
    return 0;
}
"""


def test_roles_are_a_permutation(tmp_path):
    src, exe = tmp_path / "roles.cpp", tmp_path / "roles"
    src.write_text(_MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", _CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
