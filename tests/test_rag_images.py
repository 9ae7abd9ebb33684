"""What a launch of the ragged kernels counts in 31 bits (csrc/rag_images.hpp), over layers of every shape and the largest batches, on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <initializer_list>
#include "rag_images.hpp"

int main()
{
    const long long top = 1LL << 31;
    long n = 0, by_rows = 0;
    for (int H : {1, 2, 7, 56, 1000, 30000})
        for (int W : {1, 3, 56, 500})
            for (int C : {1, 3, 16, 83, 700})
                for (int R : {1, 3, 5, 17, 35, 200})
                    for (int S : {1, 3, 17})
                        for (int stride : {1, 2, 5, 40})
                            for (int pad : {0, 1, R / 2, R - 1})
                                for (int K : {1, 33}) {
                                    if ((long long)W * C < 16 || (H + 2LL * pad + R) * W * C >= top) continue;
                                    const long long h = (long long)H + 2 * pad - R, w = (long long)W + 2 * pad - S;
                                    if (h < 0 || w < 0) continue;
                                    const long long P = h / stride + 1, Q = w / stride + 1;
                                    if (P * Q >= top - 256) continue;
                                    const long long images = dfq::rag_images(H, W, C, K, R, stride, pad, 1, (int)P, (int)Q);
                                    // LDS rows of image i begin at i * slots, those of its output row p at p * min(stride, R) behind
                                    const long long slots = (P - 1) * (stride < R ? stride : R) + R;
                                    if (images < 1 || images * slots + 4096 >= top || images * P * Q + 256 >= top || images * H * W * C >= top) {
                                        printf("%d x %d x %d, %d x %d / %d, %d: %lld images\n", H, W, C, R, S, stride, pad, images);
                                        return 1;
                                    }
                                    n++;
                                    by_rows += slots > (long long)H * W * C && slots > P * Q;
                                }
    printf("%ld %ld\n", n, by_rows);
    return 0;
}
"""


def test_launches_stay_within_31_bits(tmp_path):
    src, exe = tmp_path / "images.cpp", tmp_path / "images"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_1805_07941_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)
    layers, by_rows = map(int, r.stdout.split())
    assert layers > 1000 and by_rows > 10
