"""The pieces of 16 bytes in which a block of groups reads its input (csrc/input_piece.hpp) on the CPU: every piece of every block of many layers at the
tensor's last pixels, against the bytes one by one, zeros past the end."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <string.h>
#include "input_piece.hpp"

typedef unsigned __int128 u128;

int main()
{
    static unsigned char x[64 * 200];
    for (unsigned i = 0; i < sizeof(x); i++) x[i] = (unsigned char)(1 + i % 255);
    long n = 0, past = 0;
    for (int Cg = 1; Cg <= 40; Cg++)
        for (int groups = 2; groups <= 12 && Cg * groups <= 200; groups++)
            for (int per = 1; per <= groups; per++) {
                const int C = Cg * groups, pixels = 16 / C + 2, np = (per * Cg + 15) / 16;
                const uint32_t total = (uint32_t)(pixels * C), last = total - 16;
                for (int g0 = 0; g0 < groups; g0 += per)
                    for (int px = 0; px < pixels; px++)
                        for (int j = 0; j < np; j++, n++) {
                            const uint32_t b = (uint32_t)(px * C + g0 * Cg + 16 * j), from = b < last ? b : last;
                            u128 v;
                            memcpy(&v, x + from, 16);
                            const int d = dfq::piece_move(true, b, from);
                            if (d > 15) return 2;
                            if (d < 0) { v = 0; past++; }
                            else v >>= 8 * d;
                            for (int e = 0; e < 16; e++)
                                if ((unsigned char)(v >> (8 * e)) != (b + e < total ? x[b + e] : 0)) { printf("%d x %d, %d: byte %u\n", groups, Cg, per, b + e); return 1; }
                            if (dfq::piece_move(false, b, from) >= 0) return 3;
                        }
            }
    printf("%ld %ld\n", n, past);
    return 0;
}
"""


def test_pieces_past_the_end(tmp_path):
    src, exe = tmp_path / "pieces.cpp", tmp_path / "pieces"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__host__=", "-D__device__=", "-I", os.path.join(ROOT, "paper_1805_07941_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)
    pieces, past = map(int, r.stdout.split())
    assert pieces > 10000 and past > 100
