"""Where the direct forward kernel keeps a lane's partial sums, checked on the host from the header the kernel uses."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# For every tile shape the launcher has and every width: each lane's sums go to slots of its own tile, and the slot read
# for an output is the one where that output was written.
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "kan_direct_slot.hpp"
int main()
{
    const int shapes[][2] = {{4, 4}, {8, 4}, {16, 4}, {16, 1}, {32, 1}, {64, 1}};
    for (auto &sh : shapes)
        for (int n_out = sh[1]; n_out <= 600; ++n_out) {
            const int lps = sh[0], T = sh[1], tj = lps * T;
            for (int tile0 = 0; tile0 < n_out; tile0 += tj) {
                std::vector<int> held(tj, -1);
                for (int l = 0; l < lps; ++l) {
                    const int first = direct_first_output(tile0 + l * T, T, n_out);
                    if (first < 0 || first + T > n_out) { std::printf("row %d %d %d\n", n_out, tile0, l); return 1; }
                    for (int r = 0; r < T; ++r) held[l * T + r] = first + r;
                }
                for (int j = tile0; j < n_out && j < tile0 + tj; ++j) {
                    const int s = direct_slot(j, tile0, T, n_out);
                    if (s < 0 || s >= tj || held[s] != j) { std::printf("slot %d %d %d: %d\n", n_out, tile0, j, s); return 1; }
                }
            }
        }
    return 0;
}
"""


def test_sums_stay_in_their_tile(tmp_path):
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_2408_11200_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout


def test_kernel_writes_only_its_own_slots():
    """The kernel's one store to the sums is at the lane's place in the tile, not at its moved-back output."""
    text = open(os.path.join(ROOT, "paper_2408_11200_amd", "csrc", "kan_direct.hip")).read()
    stores = [l.strip() for l in text.splitlines() if "sums[" in l and "] = " in l]
    assert len(stores) == 1 and "sums[(grp * NS + s) * TJ + lj * T + r] = " in stores[0]
