"""The staging loads of the prepared bf16 router, on the host: every load of every stage stays inside x and the router
matrix, and brings each chunk of each row to its place.  route_stage.h is plain C++; the check is a program around it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "route_stage.h"

// a load of 16 bytes per lane: out of the descriptor's range by its per-lane offset it reads zeros, else at both offsets
template <int NB, int KSP>
int check(int d, int E, int rows) {
    using S = RouteStage<NB, KSP>;
    const int n_chunks = d / 64, n_stages = (n_chunks + KSP - 1) / KSP, ring = 3;
    std::vector<int> at(S::BYTES / 16);
    for (int st = 0; st < n_stages + ring - 1; ++st) {
        for (auto& v : at) v = -1;
        for (int wave = 0; wave < S::NWV; ++wave)
            for (int i = 0; i < S::LPW; ++i) {
                if (S::spare(wave, i)) continue;
                const unsigned range = (unsigned)((S::is_x(i) ? rows : E) * d * 2);
                const unsigned soff = S::offset(st, S::last_offset(wave, i, n_chunks));
                for (int lane = 0; lane < 64; ++lane) {
                    const unsigned voff = S::lane_offset(wave, i, lane, d);
                    const unsigned slot = S::lds(wave, i) / 16 + lane;
                    if (slot >= at.size() || at[slot] >= 0) return std::printf("LDS NB=%d KSP=%d wave=%d i=%d\n", NB, KSP, wave, i), 1;
                    at[slot] = 1 << 30;
                    if (voff >= range) continue;
                    if (voff + soff + 16 > range)
                        return std::printf("%u bytes past NB=%d KSP=%d d=%d E=%d rows=%d stage=%d\n", voff + soff + 16 - range, NB, KSP, d, E, rows, st), 1;
                    at[slot] = (int)(voff + soff);
                }
            }
        if (st >= n_stages) continue;
        for (int sub = 0; sub < KSP && st * KSP + sub < n_chunks; ++sub)
            for (int r = 0; r < S::TB + S::EPT; ++r) {
                const int row = r < S::TB ? r : r - S::TB;
                if (row >= (r < S::TB ? rows : E)) continue;
                for (int p = 0; p < 8; ++p) {
                    const int got = at[(sub * (S::TB + S::EPT) + r) * 8 + (p ^ (r >> 1 & 7))];
                    if (got != row * d * 2 + (st * KSP + sub) * 128 + p * 16)
                        return std::printf("place NB=%d KSP=%d d=%d stage=%d row=%d piece=%d\n", NB, KSP, d, st, r, p), 1;
                }
            }
    }
    return 0;
}

int main() {
    for (int chunks = 1; chunks <= 40; ++chunks)
        for (int rows : {1, 7, 8, 31, 32}) {
            const int d = chunks * 64;
            for (int E : {1, 8, 9, 32}) if (check<1, 4>(d, E, rows)) return 1;
            for (int E : {33, 40, 60, 64}) if (check<2, 2>(d, E, rows)) return 1;
            for (int E : {65, 100, 128}) if (check<4, 1>(d, E, rows)) return 1;
            for (int E : {129, 250, 256}) if (check<8, 1>(d, E, rows)) return 1;
        }
    return 0;
}
"""


def test_staging_loads_stay_inside_their_matrices(tmp_path):
    src, exe = tmp_path / "stage.cpp", tmp_path / "stage"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2506_12417_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
