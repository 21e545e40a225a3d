// What the matrix-core convolution kernels (chela_kernels_convmx.hip) share with the call that makes the kernel's spectrum
// (chela_kernels_conv.hip): sizes and tables.
#pragma once
#include "chela_internal.h"

namespace chela {

typedef _Float16 f16;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;

constexpr int MX_N = 16384;                  // points of the transform = steps of a sequence at most

// The 32-point matrix is held times a number for which cos(k pi / 16), k < 8, lie as close to half precision as they get: a
// third of the rounding error of the entries themselves (2.6e-5 against 8.3e-5 root mean square).  MX_GAIN: what the rounded
// entries come to (least squares), taken out at the stores, once per product.
constexpr float MX_ENTRY = 1.11529f, MX_GAIN = 1.11520299f;
constexpr float MX_GAIN2 = MX_GAIN * MX_GAIN, MX_GAIN4 = MX_GAIN2 * MX_GAIN2;

// Tables, the same for every call: written behind the spectra by the call that makes those (worked out by every workgroup they
// were a sixth of the forward kernel's vector instructions), read from the L2.
//   T: the first matrix, [j][re, im][k1][n1] fp16: e((k1 + 1/4) (n1 / 16 + j / N))
//   R: e(sigma r / 1024), [sigma - 1][r] fp32 pairs, sigma = 1 .. 31 (row 0 would be ones)
//   M: the 32-point matrix e(r sigma / 32) = c - i s as an operand (first or second: it is symmetric), [c0, c1, s0, s1][lane]: lane
//      (r, h), element e of c_t, s_t stands for sigma = 16 t + 8 (e / 4) + 4 h + e % 4, the order in which a lane holds the rows
//      of a result
struct MxTables {
    f16 T[8 * 2 * 16 * 16];
    float2 R[31 * 32];
    f16x8 M[4 * 64];
};
static_assert((8 * 2 * 16 * 16 * 2 + 31 * 32 * 8) % 16 == 0, "copied in 16-byte pieces");
__device__ __forceinline__ float2 mx_e(int num, float unit)       // e(num * unit), num * unit exact
{
    float sn, cs;
    sincospif((float)num * (2.0f * unit), &sn, &cs);
    return make_float2(cs, -sn);
}
// entries i of each, i < MX_TABLE_STEPS
constexpr int MX_TABLE_STEPS = 8 * 256;
__device__ __forceinline__ void mx_write_tables(MxTables* __restrict__ tb, int i)
{
    const int j = i >> 8, k1 = (i >> 4) & 15, n1 = i & 15;
    // (4 k1 + 1) (1024 n1 + j) / (4 N) of a turn, the whole turns taken off
    const float2 e = mx_e(((4 * k1 + 1) * (1024 * n1 + j)) & (4 * MX_N - 1), 1.0f / (4.0f * MX_N));
    tb->T[(2 * j) * 256 + (i & 255)] = (f16)e.x;
    tb->T[(2 * j + 1) * 256 + (i & 255)] = (f16)e.y;
    if (i < 31 * 32) tb->R[i] = mx_e(((i >> 5) + 1) * (i & 31), 1.0f / 1024.0f);
    if (i < 4 * 64) {
        const int r = i & 31, h = (i >> 5) & 1, t = (i >> 6) & 1;
        f16x8 v;
#pragma unroll
        for (int e8 = 0; e8 < 8; ++e8) {
            const float2 p = mx_e((r * (16 * t + 8 * (e8 >> 2) + 4 * h + (e8 & 3))) & 31, 1.0f / 32.0f);
            v[e8] = (f16)(MX_ENTRY * (i < 128 ? p.x : -p.y));
        }
        tb->M[i] = v;
    }
}

// Behind the pairs of the spectrum buffer: the half-precision spectra [d][MX_N] words, the scales [d], the tables.
inline MxTables* mx_tables(void* extra, int d)
{
    return (MxTables*)((char*)extra + (((size_t)d * (MX_N + 1) * sizeof(unsigned) + 255) & ~(size_t)255));
}

}  // namespace chela
