// How many images a launch of the ragged kernels takes (conv_rag.hip, conv_rag_groups.hip): everything they count in 31 bits.
#pragma once

namespace dfq {

// Byte offsets into the input with the padding's reach, output pixels, tiles, and - where the input's rows are staged in LDS - the rows of all
// images one after the other: (P - 1) * min(stride, R) + R of an image, more than H where the kernel is higher than the image
// (17 x 3 over images of one pixel: 2^27 images of 16 bytes have 2^31 such rows).  A tile's last loads look a little past its rows.
inline long long rag_images(int H, int W, int C, int K, int R, int stride, int pad, int groups, int P, int Q)
{
    const long long image = (long long)H * W * C, pixels = (long long)P * Q, margin = ((long long)pad + R) * W * C;
    const long long tiles = (pixels / 64 + 1) * groups * ((K / groups + 31) / 32);
    const long long slots = (long long)(P - 1) * (stride < R ? stride : R) + R;
    const long long most[4] = {((1LL << 31) - 1 - margin) / image, ((1LL << 31) - 257) / pixels, ((1LL << 31) - 1) / tiles, ((1LL << 31) - 65536) / slots};
    long long n = most[0];
    for (int i = 1; i < 4; i++) n = most[i] < n ? most[i] : n;
    return n < 1 ? 1 : n;
}

}  // namespace dfq
