"""The wide weight reads of the first-layer kernels (csrc/weight_reads.hpp) on the CPU: tensors that begin and end at pages without
access, so that a byte read outside ends the program, over every run length and position, against the bytes one by one."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <string.h>
#include <sys/mman.h>
#include <unistd.h>
#include "weight_reads.hpp"

static int8_t *pages;         // one readable page between two that are not
static long page;

static int8_t *place(int bytes, bool at_end)
{
    int8_t *w = at_end ? pages + 2 * page - bytes : pages + page;
    for (int i = 0; i < bytes; i++) w[i] = (int8_t)(i * 37 + 11 + (i >> 8));
    return w;
}

static int check(const int8_t *w, int total, int o, int count, const unsigned char *got, int width)
{
    for (int i = 0; i < width; i++) {
        const unsigned char want = i < count && o + i < total ? (unsigned char)w[o + i] : 0;
        if (got[i] != want) { printf("total %d, from %d, %d wanted: byte %d\n", total, o, count, i); return 1; }
    }
    return 0;
}

int main()
{
    page = sysconf(_SC_PAGESIZE);
    pages = (int8_t *)mmap(nullptr, 3 * page, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (pages == (int8_t *)MAP_FAILED || mprotect(pages + page, page, PROT_READ | PROT_WRITE)) return 2;
    long n = 0;
    for (int at_end = 0; at_end < 2; at_end++) {
        // pieces as conv_smallc.hip asks for them: K x R runs of S * C <= 32 bytes, each in two pieces of 16
        for (int K = 1; K <= 5; K++)
            for (int R = 1; R <= 5; R++)
                for (int run = 1; run <= 32; run++) {
                    const int total = K * R * run;
                    const int8_t *w = place(total, at_end);
                    for (int k = 0; k < K + 2; k++)          // channels past the last read the last one's run and keep nothing
                        for (int r = 0; r < R; r++)
                            for (int h = 0; h < 2; h++, n++) {
                                const long long o = ((long long)(k < K ? k : K - 1) * R + r) * run + 16 * h;
                                const int left = run - 16 * h, count = k < K ? (left < 16 ? left : 16) : 0;
                                const unsigned __int128 v = dfq::weight_piece(w, total, o, count);
                                unsigned char got[16];
                                memcpy(got, &v, 16);
                                if (check(w, total, (int)o, count, got, 16)) return 1;
                            }
                }
        // runs as conv_stem.hip asks for them: from every byte of tensors of 24 bytes and more
        for (int total = 24; total <= 400; total += total < 60 ? 1 : 17) {
            const int8_t *w = place(total, at_end);
            for (int o = 0; o < total; o++, n++) {
                unsigned long long q[3];
                dfq::weight_run24(w, total, o, q);
                if (check(w, total, o, 24, (const unsigned char *)q, 24)) return 1;
            }
        }
    }
    printf("%ld reads\n", n);
    return 0;
}
"""


def test_reads_stay_inside_the_tensor(tmp_path):
    src, exe = tmp_path / "reads.cpp", tmp_path / "reads"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__host__=", "-D__device__=", "-I", os.path.join(ROOT, "paper_1805_07941_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)
    assert int(r.stdout.split()[0]) > 10000
