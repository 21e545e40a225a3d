// Long convolution of Eq. 7-8 (Sec. 4.2) with the transforms on the matrix cores, for bf16 I/O and sequences of
// 4097 .. 16384 steps.
//
// A real sequence x of N = 16384 steps (zero beyond L) is evaluated at the N points exp(-2 pi i (k + 1/4) / N), the roots
// of z^N = -i: there the product of two real sequences is (low half) - i (high half) of their causal sum, so the real part
// of the way back is the causal result with no zero-padding, no pair of sequences to share a transform and nothing to
// untangle, and the quarter step costs nothing, because every twiddle below sits in a matrix or in a rotation anyway.
// With n = 1024 n1 + 32 n2 + n3 and k = k1 + 16 k2 + 512 k3 (n1, k1 < 16, the others < 32):
//     X1[k1,n2,n3] = e((k1 + 1/4) (32 n2 + n3) / N) sum_n1 e((k1 + 1/4) n1 / 16) x[n1,n2,n3]         e(t) = exp(-2 pi i t)
//     X2[k1,k2,n3] = e(k2 n3 / 1024)                sum_n2 e(k2 n2 / 32) X1[k1,n2,n3]
//     X [k1,k2,k3] =                                sum_n3 e(k3 n3 / 32) X2[k1,k2,n3]
// The way back is the conjugate of the same sums over the conjugate bins in the opposite order (the real part does not
// care about the last conjugation).  All sums are matrix products (fp16 operands, fp32 sums); rotations are applied in
// fp32, the part of the first one that differs from step to step of a lane's eight (e((k1 + 1/4) (n3 & 7) / N)) is worked
// into eight versions of the first matrix.
//
// Bound by vector instructions (issuing three quarters of the time in the forward kernel), so the layout is chosen to
// spend none on moving data:
//   - First pass: a lane loads eight consecutive steps of four rows n1, which is its operand of
//     v_mfma_f32_16x16x16_f16 (contraction over n1), and gets four k1 of the same eight columns.
//   - Tile k1 (32 x 32 columns) then belongs to one wave, which takes it through both other passes, the product with the
//     kernel's spectrum and both passes back without leaving its registers: a product of 32x32x16 with the data as first
//     operand leaves a lane the rows it has to supply as second operand of the next, and the other way round.
//   - Last pass: LDS transposing reads hand a lane its operand for the eight columns it loaded, the results leave as 16-byte
//     stores.
// So a sequence crosses LDS twice (64 KB of fp16, re and im planes), with three barriers.
// Ranges: the input is scaled by a power of two to max|v| < 1 and the kernel's spectrum is stored divided by 4 |k|_1, so that the
// result of a pass is at most 16384 on the way forward and N / 4 = 4096 on the way back (every pass there is a transform of the
// result), but for what the 32-point matrix is stored times, MX_ENTRY per pass: 20380 and 6337; half precision ends at 65504.
// All factors are put back on the way out.  Error against the fp64 definition on the workload's recipe: 4.2e-4 relative
// before the rounding of the output to bf16 (1.7e-3 on its own).
#include "chela_convmx.h"
#include <cfloat>
#include <cstdlib>
#include <type_traits>

namespace chela {

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int MX_T = 512;                    // threads: each owns eight columns of four rows n1 (32 steps)
constexpr int MX_W = MX_T / 64;              // waves; wave w owns columns 128 w .. 128 w + 127 and tiles w, w + 8
constexpr int MX_NT = 16 / MX_W;             // tiles per wave
constexpr int MX_PLANE = 16 * 2048;          // bytes of the re (or im) plane of a cube: [k1][n2][n3] fp16
constexpr int MX_CUBE = 2 * MX_PLANE;
static_assert(32768 * MX_ENTRY * MX_ENTRY < 65504, "the largest packed value: the sums of dk on their way back");

// One word of two halves, round to nearest even.
__device__ __forceinline__ unsigned mx_pack(float lo, float hi)
{
    f16x2 v;
    v[0] = (f16)lo;
    v[1] = (f16)hi;
    return __builtin_bit_cast(unsigned, v);
}
__device__ __forceinline__ f16x8 mx_h8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// Within a group of 16 lanes the transposing read hands lane p element p % 4 of the 8-byte pieces that lanes p / 4,
// p / 4 + 4, p / 4 + 8, p / 4 + 12 address.
__device__ __forceinline__ u32x2 mx_tr(const unsigned char* p)
{
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
}

// What depends on the lane only (LDS addresses, table entries) is worked out afresh by every stage behind an opaque copy of
// the lane index: kept from stage to stage it would fill the register file.
__device__ __forceinline__ int mx_fresh(int lane) { asm volatile("" : "+v"(lane)); return lane; }

__device__ __forceinline__ f32x16 mx_zero()
{
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}

__device__ __forceinline__ float2 mx_cmul(float2 a, float2 b) { return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

// T and R as they lie in LDS, and room to exchange maxima.
struct MxLds {
    f16 T[8 * 2 * 16 * 16];
    float2 R[31 * 32];
    float red[2 * MX_W];
};
struct MxMat { f16x8 c[2], s[2], ns[2]; };
__device__ __forceinline__ void mx_fetch_tables(MxLds& tb, const MxTables* __restrict__ src, int tid)
{
    constexpr int n16 = (int)((sizeof(src->T) + sizeof(src->R)) / 16);
    const u32x4* s = reinterpret_cast<const u32x4*>(src);
    u32x4* d = reinterpret_cast<u32x4*>(&tb);
#pragma unroll
    for (int k = 0; k < (n16 + MX_T - 1) / MX_T; ++k)
        if (tid + MX_T * k < n16) d[tid + MX_T * k] = s[tid + MX_T * k];
}
__device__ __forceinline__ void mx_fetch_matrix(MxMat& m, const MxTables* __restrict__ src, int lane)
{
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        m.c[t] = src->M[64 * t + lane];
        m.s[t] = src->M[64 * (2 + t) + lane];
        m.ns[t] = -m.s[t];
    }
}

// What a lane needs besides: rho = e((4 q + 1/4) (128 w + 8 c) / N) and g = e((128 w + 8 c) / N) for the first pass
// (lane = 16 q + c), u = e(r / 2048) for the way back (lane = 32 h + r).  By the hardware's sine and cosine of turns: what they
// are off by (1e-6) is nothing beside the fp16 that every rotated value is rounded to.
struct MxLane { float2 rho, g, u; };
__device__ __forceinline__ float2 mx_e_fast(int num, float unit)
{
    const float t = (float)num * unit;
    return make_float2(__builtin_amdgcn_cosf(t), -__builtin_amdgcn_sinf(t));
}
__device__ __forceinline__ void mx_build_lane(MxLane& c, int lane, int w)
{
    const int col = 128 * w + 8 * (lane & 15);
    c.rho = mx_e_fast((16 * (lane >> 4) + 1) * col, 1.0f / (4.0f * MX_N));
    c.g = mx_e_fast(col, 1.0f / MX_N);
    c.u = mx_e_fast(lane & 31, 1.0f / 2048.0f);
}
// e((k1 + 1/4) 8 / N), the same in all lanes
__device__ __forceinline__ float2 mx_step(int k1)
{
    const float2 st = mx_e_fast((4 * k1 + 1) * 8, 1.0f / (4.0f * MX_N));
    return make_float2(__builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, st.x))),
                       __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, st.y))));
}

// ---- first pass: v[i][j] = step 1024 (4 q + i) + 128 w + 8 c + j, times s, into the cube.  EXACT: v are bf16 numbers, which
// times a power of two are half-precision ones; else what they lose in rounding goes through the same product (the rounding of
// the input weighs as much as any two others: it is not averaged over a pass).
template <bool EXACT>
__device__ __forceinline__ void mx_first(unsigned char* cube, const MxLds& tb, const MxLane& lc, const float (&v)[4][8],
                                         float s, int w, int lane)
{
    lane = mx_fresh(lane);
    const int c = lane & 15, q = lane >> 4;
    float2 rho[4];
    rho[0] = lc.rho;
#pragma unroll
    for (int k = 1; k < 4; ++k) rho[k] = mx_cmul(rho[k - 1], lc.g);
    // rows of 64 bytes (n3) in natural order
    unsigned char* p = cube + 4 * q * 2048 + (4 * w + (c >> 2)) * 64 + (c & 3) * 16;
    u32x2 out[2][4];
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        __builtin_amdgcn_sched_barrier(0);
        float re[2][4], im[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const f16* t = tb.T + (2 * (j + u)) * 256 + c * 16 + 4 * q;
            const f16x4 ar = *reinterpret_cast<const f16x4*>(t), ai = *reinterpret_cast<const f16x4*>(t + 256);
            u32x2 bw;
            bw[0] = mx_pack(v[0][j + u] * s, v[1][j + u] * s);
            bw[1] = mx_pack(v[2][j + u] * s, v[3][j + u] * s);
            const f16x4 b = __builtin_bit_cast(f16x4, bw);
            const f32x4 z = {0.f, 0.f, 0.f, 0.f};
            f32x4 xr = __builtin_amdgcn_mfma_f32_16x16x16f16(ar, b, z, 0, 0, 0);
            f32x4 xi = __builtin_amdgcn_mfma_f32_16x16x16f16(ai, b, z, 0, 0, 0);
            if constexpr (!EXACT) {
                u32x2 lw;
                lw[0] = mx_pack(fmaf(v[0][j + u], s, -(float)b[0]), fmaf(v[1][j + u], s, -(float)b[1]));
                lw[1] = mx_pack(fmaf(v[2][j + u], s, -(float)b[2]), fmaf(v[3][j + u], s, -(float)b[3]));
                const f16x4 lo = __builtin_bit_cast(f16x4, lw);
                xr = __builtin_amdgcn_mfma_f32_16x16x16f16(ar, lo, xr, 0, 0, 0);
                xi = __builtin_amdgcn_mfma_f32_16x16x16f16(ai, lo, xi, 0, 0, 0);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                re[u][k] = xr[k] * rho[k].x - xi[k] * rho[k].y;
                im[u][k] = xr[k] * rho[k].y + xi[k] * rho[k].x;
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            out[0][k][(j >> 1) & 1] = mx_pack(re[0][k], re[1][k]);
            out[1][k][(j >> 1) & 1] = mx_pack(im[0][k], im[1][k]);
            if (j & 2) {
                *reinterpret_cast<u32x2*>(p + k * 2048 + (j >> 2) * 8) = out[0][k];
                *reinterpret_cast<u32x2*>(p + MX_PLANE + k * 2048 + (j >> 2) * 8) = out[1][k];
            }
        }
    }
}

// (re, im) = data times the 32-point matrix; DATA_FIRST: the data's lanes are the rows of the result.
template <bool DATA_FIRST>
__device__ __forceinline__ void mx_mul(const MxMat& m, const u32x4 (&re)[2], const u32x4 (&im)[2], f32x16& xr, f32x16& xi)
{
    auto mul = [](f16x8 d, f16x8 k, f32x16 acc) __attribute__((always_inline)) {
        return DATA_FIRST ? __builtin_amdgcn_mfma_f32_32x32x16_f16(d, k, acc, 0, 0, 0)
                          : __builtin_amdgcn_mfma_f32_32x32x16_f16(k, d, acc, 0, 0, 0);
    };
    xr = mul(mx_h8(re[0]), m.c[0], mx_zero());
    xi = mul(mx_h8(im[0]), m.c[0], mx_zero());
    xr = mul(mx_h8(re[1]), m.c[1], xr);
    xi = mul(mx_h8(im[1]), m.c[1], xi);
    xr = mul(mx_h8(im[0]), m.s[0], xr);
    xi = mul(mx_h8(re[0]), m.ns[0], xi);
    xr = mul(mx_h8(im[1]), m.s[1], xr);
    xi = mul(mx_h8(re[1]), m.ns[1], xi);
}

// Register 4 a + b of lane (r, h) is row sigma = 8 a + 4 h + b, column r: turn by e(sigma r / 1024) and pack as operand.
__device__ __forceinline__ void mx_rotate(const f32x16& xr, const f32x16& xi, const float2* R, int lane, u32x4 (&re)[2],
                                          u32x4 (&im)[2])
{
    lane = mx_fresh(lane);
    const int r = lane & 31, h = lane >> 5;
    const float2* Rl = R + h * (4 * 32) + r;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; b += 2) {
            float x[2], y[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int i = 4 * a + b + u;
                float2 p = a > 0 || b + u > 0 ? Rl[(8 * a + b + u - 1) * 32] : R[3 * 32 + r];
                if (a == 0 && b + u == 0) {
                    p.x = h == 0 ? 1.f : p.x;
                    p.y = h == 0 ? 0.f : p.y;
                }
                x[u] = xr[i] * p.x - xi[i] * p.y;
                y[u] = xr[i] * p.y + xi[i] * p.x;
            }
            re[a >> 1][2 * (a & 1) + (b >> 1)] = mx_pack(x[0], x[1]);
            im[a >> 1][2 * (a & 1) + (b >> 1)] = mx_pack(y[0], y[1]);
        }
}

// ---- tile k1 through the second and third pass: register 4 a + b of lane (r, h) ends as bin k2 = r, k3 = 8 a + 4 h + b
__device__ __forceinline__ void mx_tile_in(const unsigned char* cube, const MxLds& tb, const MxMat& m, int k1, int lane,
                                           f32x16& xr, f32x16& xi)
{
    lane = mx_fresh(lane);
    const int h = lane >> 5, p = lane & 15, g = (lane >> 4) & 1;
    u32x4 re[2], im[2];
    const unsigned char* t = cube + k1 * 2048 + (4 * h + (p >> 2)) * 64 + (4 * g + (p & 3)) * 8;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const u32x2 a = mx_tr(t + s * 1024), b = mx_tr(t + s * 1024 + 512);
        re[s] = u32x4{a[0], a[1], b[0], b[1]};
        const u32x2 c = mx_tr(t + MX_PLANE + s * 1024), d = mx_tr(t + MX_PLANE + s * 1024 + 512);
        im[s] = u32x4{c[0], c[1], d[0], d[1]};
    }
    mx_mul<true>(m, re, im, xr, xi);              // rows n3, columns k2
    mx_rotate(xr, xi, tb.R, lane, re, im);
    mx_mul<false>(m, re, im, xr, xi);             // rows k3, columns k2
}

// ---- the way back of tile k1 from its (conjugate) bins, packed along k3, into the cube: row n2 of 64 bytes holds n3 = 8 a + j at
// place 4 j + a, its 8-byte pieces (one j each) exchanged by k1 and n2 so that neither the writers here (32 rows) nor the
// readers of the last pass (4 rows of 8 tiles) share banks.
__device__ __forceinline__ int mx_swizzle(int k1, int n2) { return ((k1 & 3) | (k1 >> 3) << 2) ^ (n2 >> 2); }
__device__ __forceinline__ void mx_tile_out(unsigned char* cube, const MxLds& tb, const MxMat& m, float2 u, float2 st,
                                            int k1, int lane, u32x4 (&re)[2], u32x4 (&im)[2])
{
    lane = mx_fresh(lane);
    const int r = lane & 31, h = lane >> 5;
    f32x16 xr, xi;
    mx_mul<true>(m, re, im, xr, xi);              // rows k2, columns n3
    mx_rotate(xr, xi, tb.R, lane, re, im);
    mx_mul<true>(m, re, im, xr, xi);              // rows n3, columns n2
    // e((k1 + 1/4) (32 n2 + 8 a) / N), the first factor being e(2 k1 n2 / 1024) e(n2 / 2048)
    float2 e[4];
    e[0] = tb.R[(k1 > 0 ? 2 * k1 - 1 : 0) * 32 + r];
    if (k1 == 0) e[0] = make_float2(1.f, 0.f);
    e[0] = mx_cmul(e[0], u);
#pragma unroll
    for (int a = 1; a < 4; ++a) e[a] = mx_cmul(e[a - 1], st);
    unsigned char* row = cube + k1 * 2048 + r * 64;
    const int sw = mx_swizzle(k1, r);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        float x[4], y[4];                         // Re, -Im
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float ur = xr[4 * a + b], ui = xi[4 * a + b];
            x[a] = ur * e[a].x - ui * e[a].y;
            y[a] = -ur * e[a].y - ui * e[a].x;
        }
        u32x2 vx, vy;
        vx[0] = mx_pack(x[0], x[1]); vx[1] = mx_pack(x[2], x[3]);
        vy[0] = mx_pack(y[0], y[1]); vy[1] = mx_pack(y[2], y[3]);
        unsigned char* d = row + ((4 * h + b) ^ sw) * 8;
        *reinterpret_cast<u32x2*>(d) = vx;
        *reinterpret_cast<u32x2*>(d + MX_PLANE) = vy;
    }
}

// ---- last pass: y[i][j] = N times step 1024 (4 q + i) + 128 w + 8 c + j, up to the scales
__device__ __forceinline__ void mx_last(const unsigned char* cube, const MxLds& tb, int w, int lane, float (&y)[4][8])
{
    lane = mx_fresh(lane);
    const int p = lane & 15, q = lane >> 4;
    const int k0 = 8 * (q & 1) + (p >> 2);                                  // k1 of this lane's first piece; + 4: the second
    const unsigned char* pl = cube + (q >> 1) * MX_PLANE + k0 * 2048 + (4 * w + (p & 3)) * 64;
    const int sw = mx_swizzle(k0, 4 * w);                                   // (the same for k0 + 4, and for the four rows)
    const f16* t = tb.T + (q >> 1) * 256 + k0 * 16 + 4 * (p & 3);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const unsigned char* tj = reinterpret_cast<const unsigned char*>(t + 2 * j * 256);
        const u32x2 a0 = mx_tr(tj), a1 = mx_tr(tj + 4 * 16 * 2);
        const unsigned char* d = pl + ((j ^ sw) & 7) * 8;
        const u32x2 b0 = mx_tr(d), b1 = mx_tr(d + 4 * 2048);
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        const f32x4 r = __builtin_amdgcn_mfma_f32_16x16x32_f16(mx_h8(u32x4{a0[0], a0[1], a1[0], a1[1]}),
                                                               mx_h8(u32x4{b0[0], b0[1], b1[0], b1[1]}), z, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i][j] = r[i];
    }
}

// A lane's steps are t0 + 1024 i + j, i < 4, j < 8.
__device__ __forceinline__ int mx_first_step(int w, int lane) { return 4096 * (lane >> 4) + 128 * w + 8 * (lane & 15); }

// The short kernel's taps as operands of v_mfma_f32_16x16x32_bf16, whose other operand is x as it lies in memory: lane 16 q + c
// supplies eight steps of row 4 q + i (contraction index 8 q + e), result 4 q + b of column c is step 4 blk + b of row 4 q + i, so the
// matrix is block-diagonal in q: row (q, b), index (q, e): w[8 D + 4 blk + b - e] for the piece D pieces in front.  The taps
// go in as three bf16 parts each, cut off, not rounded: all 24 bits (products with bf16 x are exact, sums fp32).  A quarter of the
// matrix is of use, and still: 48 of these instructions replace 288 multiply-adds and some 60 unpackings per wave (9 taps:
// forward of 768 x 4 x 16384 steps 125 -> 118 us, long-stage gradients 243 -> 225; 32 taps: forward 165 -> 134).
//   [part][D][blk][b][e], then eight zeros for the lanes off the diagonal
#define MX_TAP_WORDS(nh) (3 * ((nh) + 1) * 2 * 4 * 8)
template <int HALO>
__device__ __forceinline__ void mx_write_taps(unsigned short* taps, const float* __restrict__ wc, int m, int tid)
{
    constexpr int NH = HALO / 8, WORDS = MX_TAP_WORDS(NH);
#pragma unroll
    for (int k = 0; k < (WORDS + 8 + MX_T - 1) / MX_T; ++k) {
        const int x = tid + MX_T * k, e = x & 7, b = (x >> 3) & 3, blk = (x >> 5) & 1, pd = x >> 6;
        if (x >= WORDS + 8) break;
        const int part = pd / (NH + 1), j = 8 * (pd - part * (NH + 1)) + 4 * blk + b - e;
        const float w = x < WORDS && j >= 0 && j < m ? wc[j] : 0.f;
        auto cut = [](float v) __attribute__((always_inline)) {
            return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v) & 0xffff0000u);
        };
        const float hi = cut(w), mid = cut(w - hi), lo = w - hi - mid;
        taps[x] = (unsigned short)(__builtin_bit_cast(unsigned, part == 0 ? hi : part == 1 ? mid : lo) >> 16);
    }
}

// ---- a sequence in registers: 16-byte pieces of rows n1 = 4 q + i, steps t0 + 1024 i .. + 7, and the HALO steps in front of
// each (the taps' history).  Buffer loads: what lies before the row's start or beyond its end reads as zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t mx_rsrc(const void* row, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), 0, bytes, 0x00020000);
}
// History comes from the registers of the lanes in front; the first lanes of a row's 16 get theirs from the lanes that have
// fetched it for them: lane 16 (D - 1) + 4 q + i the piece 8 D steps in front of this wave's part of row 4 q + i.
template <int HALO>
struct MxSeq {
    static_assert(HALO % 8 == 0 && HALO <= 32, "");
    static constexpr int NH = HALO / 8;
    u32x4 r[4], front;
    __device__ __forceinline__ void load(const bf16* row, int L, int w, int lane)
    {
        lane = mx_fresh(lane);
        const int t0 = mx_first_step(w, lane);
        const __amdgpu_buffer_rsrc_t rs = mx_rsrc(row, 2 * L);
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, 2 * (t0 + 1024 * i), 0, 0));
        if (HALO > 0)
            front = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rs, 2 * (1024 * (lane & 15) + 128 * w - 8 - 8 * (lane >> 4)), 0, 0));
    }
    // the piece 8 D steps in front of row i's
    template <int D>
    __device__ __forceinline__ u32x4 piece(int lane, int i) const
    {
        const int from = 16 * (D - 1 - (lane & 15)) + 4 * (lane >> 4);         // (of use to the first D lanes only)
        u32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            x[e] = (unsigned)__builtin_amdgcn_update_dpp(__builtin_amdgcn_ds_bpermute(4 * (from + i), (int)front[e]),
                                                         (int)r[i][e], 0x110 + D, 0xf, 0xf, false);      // row_shr:D
        return x;
    }
    template <int D>
    __device__ __forceinline__ void pieces(int lane, u32x4 (&x)[4]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = piece<D>(lane, i);
    }
    // The wave's largest magnitude (of the steps themselves).
    __device__ __forceinline__ float wave_max() const
    {
        typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
        u16x2 mx = {0, 0};
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, r[i][e] & 0x7fff7fffu));
        float v = __builtin_bit_cast(float, (unsigned)(mx[0] > mx[1] ? mx[0] : mx[1]) << 16);
        v = v > FLT_MAX ? FLT_MAX : v == v ? v : 0.f;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
        return v;
    }
    // the steps themselves
    __device__ __forceinline__ void values(float (&v)[4][8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[i][2 * e] = __builtin_bit_cast(float, r[i][e] << 16);
                v[i][2 * e + 1] = __builtin_bit_cast(float, r[i][e] & 0xffff0000u);
            }
    }
    // u = K_s x.  (Steps beyond the sequence's end come out as whatever their history gives.)
    __device__ __forceinline__ void short_conv(const unsigned short* taps, int lane, float (&v)[4][8]) const
    {
        lane = mx_fresh(lane);
        f32x4 acc[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        const bool mine = (lane >> 4) == ((lane & 15) >> 2);
        const unsigned short* t = taps + (mine ? 8 * (lane & 3) : MX_TAP_WORDS(NH));
        auto add = [&](const u32x4 (&x)[4], int D) __attribute__((always_inline)) {
#pragma unroll
            for (int part = 0; part < 3; ++part)
#pragma unroll
                for (int blk = 0; blk < 2; ++blk) {
                    const int at = ((part * (NH + 1) + D) * 2 + blk) * 32;
                    const bf16x8 a = *reinterpret_cast<const bf16x8*>(t + (mine ? at : 0));
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[i][blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, x[i]), acc[i][blk], 0, 0, 0);
                }
        };
        add(r, 0);
        u32x4 x[4];
        if constexpr (NH >= 1) { pieces<1>(lane, x); add(x, 1); }
        if constexpr (NH >= 2) { pieces<2>(lane, x); add(x, 2); }
        if constexpr (NH >= 4) { pieces<3>(lane, x); add(x, 3); pieces<4>(lane, x); add(x, 4); }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[i][e] = acc[i][e >> 2][e & 3];
    }
    // v = silu(K_s x), zero from the sequence's end on; HALO = 0: v = x.  (In exact arithmetic what the taps make of the history
    // there would do no harm, it is behind every step that is wanted.  But it would have a say in the scale, and its rounding
    // errors spread over all steps: difference taps on a constant of -50, 5000 steps: Z off by 6.8e-3 where it now is by 1.7e-3,
    // d_k_long by 9.8e-3 and 3e-4.)
    __device__ __forceinline__ void activated(const unsigned short* taps, int L, int w, int lane, float (&v)[4][8]) const
    {
        if constexpr (HALO == 0) {
            values(v);
        } else {
            short_conv(taps, lane, v);
            const int t0 = mx_first_step(w, mx_fresh(lane));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool in = t0 + 1024 * i < L;         // (L is a multiple of 8)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float a = v[i][e] * __builtin_amdgcn_rcpf(1.f + __expf(-v[i][e]));
                    asm("" : "+v"(a));               // (a select, not a branch around each exponential)
                    v[i][e] = in ? a : 0.f;
                }
            }
        }
    }
};

__device__ __forceinline__ float mx_wave_max(const float (&v)[4][8], float mx = 0.f)
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(v[i][e]));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    return mx;
}
// The power of two that takes bm into [1/2, 1) (1 for zero).
__device__ __forceinline__ float mx_scale(float bm)
{
    const int e = 253 - (__builtin_bit_cast(int, bm) >> 23);
    return bm > 0.f ? __builtin_bit_cast(float, e > 0 ? e << 23 : 0x00400000) : 1.0f;
}

// Bins times the kernel's, conjugate, packed along k3.  CORR: with the conjugate kernel.
template <bool CORR>
__device__ __forceinline__ void mx_product(const f32x16& xr, const f32x16& xi, const u32x4 (&kq)[4], u32x4 (&re)[2], u32x4 (&im)[2])
{
    float none = 0.f;
    asm("" : "+s"(none));
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; b += 2) {
            float x[2], y[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const unsigned kw = kq[a][b + u];
                const f16x2 k = __builtin_bit_cast(f16x2, kw);
                const float zr = xr[4 * a + b + u], zi = xi[4 * a + b + u];
                // (multiply-adds all: the mixed-precision ones take the half-precision factor as it is)
                const float p = fmaf(zi, (float)k[1], none), q = fmaf(zi, (float)k[0], none);
                x[u] = CORR ? fmaf(zr, (float)k[0], p) : fmaf(zr, (float)k[0], -p);
                y[u] = CORR ? fmaf(zr, (float)k[1], -q) : -fmaf(zr, (float)k[1], q);
            }
            re[a >> 1][2 * (a & 1) + (b >> 1)] = mx_pack(x[0], x[1]);
            im[a >> 1][2 * (a & 1) + (b >> 1)] = mx_pack(y[0], y[1]);
        }
}

// One sequence per workgroup, id = c B + b, ids first .. end - 1.  HALO: steps of history the short kernel needs (m - 1 <= HALO;
// v = silu(K_s x)); 0: no short kernel, v = x.  L is a multiple of 8.
// Two workgroups per compute unit (80 KB of LDS, 128 registers): one's activation runs beside the other's matrix products.
// Workgroups that walk several sequences with the next
// one's input on its way took 122 us (three each) and 128 us (six, all resident at once) where these take 117: of two that
// start together on a unit the older one gets ahead, and the other finishes alone.
// 768 channels x 4 sequences of 16384 steps, 9 taps: 117 us (198 with two sequences per transform of 2 x 16384 points, whose
// six passes each went through LDS, one workgroup per unit).
template <int HALO>
__global__ __launch_bounds__(MX_T, 4) void convmx_fwd_kernel(const bf16* __restrict__ X, const float* __restrict__ w_short,
                                                             int m, const unsigned* __restrict__ Ks,
                                                             const float* __restrict__ kscale, const MxTables* __restrict__ tables,
                                                             bf16* __restrict__ Y, int B,
                                                             int d, int L, int first, int end)
{
    __shared__ __attribute__((aligned(16))) unsigned char cube[MX_CUBE];
    __shared__ __attribute__((aligned(16))) MxLds tb;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive workgroups run on the eight XCDs in turn: those of one XCD take neighbouring ids, which share spectra in its L2
    const int id = first + (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (id >= end) return;
    const int c = id / B, b = id - c * B;
    const long row = ((long)b * d + c) * L;
    MxSeq<HALO> xs;
    xs.load(X + row, L, w, lane);
    unsigned short* taps = reinterpret_cast<unsigned short*>(cube);       // (until the first pass)
    if (HALO > 0) mx_write_taps<HALO>(taps, w_short + (long)c * m, m, tid);
    mx_fetch_tables(tb, tables, tid);
    __syncthreads();
    MxLane lc;
    mx_build_lane(lc, lane, w);
    float s;
    {
        float v[4][8];
        xs.activated(taps, L, w, lane, v);
        const float mx = mx_wave_max(v);
        if (lane == 0) tb.red[w] = mx;
        __syncthreads();
        float bm = 0.f;
#pragma unroll
        for (int i = 0; i < MX_W; ++i) bm = fmaxf(bm, tb.red[i]);
        s = mx_scale(bm);
        mx_first<HALO == 0>(cube, tb, lc, v, s, w, lane);
    }
    const u32x4* kc = reinterpret_cast<const u32x4*>(Ks + (long)c * MX_N);
    MxMat m32;
    mx_fetch_matrix(m32, tables, lane);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < MX_NT; ++n) {
        const int k1 = w + MX_W * n;
        u32x4 kq[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) kq[a] = kc[(k1 * 4 + a) * 64 + mx_fresh(lane)];
        f32x16 xr, xi;
        mx_tile_in(cube, tb, m32, k1, lane, xr, xi);
        u32x4 re[2], im[2];
        mx_product<false>(xr, xi, kq, re, im);
        mx_tile_out(cube, tb, m32, lc.u, mx_step(k1), k1, lane, re, im);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    const float osc = kscale[c] / (s * ((float)MX_N * MX_GAIN4));
    float y[4][8];
    mx_last(cube, tb, w, lane, y);
    const __amdgpu_buffer_rsrc_t rs = mx_rsrc(Y + row, 2 * L);        // (stores beyond the row's end are dropped)
    const int t0 = mx_first_step(w, mx_fresh(lane));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (bf16)(y[i][e] * osc);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rs, 2 * (t0 + 1024 * i), 0, 0);
    }
}

// ---- the short stage's gradient of one sequence, dV = osc y still in registers (y as mx_last leaves it):
//   du = dV silu'(u), u = K_s x worked out again;  dX[t] = sum_j w[j] du[t + j];  dw[j] += sum_t du[t] x[t - j], all fp32.
// A lane's look-ahead comes from the lanes behind it in its row of 16, for the last of them by way of LDS: `edge` holds the first
// HALO steps of each wave's 128 of each row n1, in the order of the steps, and zeros behind the last.
// As a kernel of its own this stage read dV (fp32, written by this one) and x again: 768 channels x 4 sequences of 16384 steps, both
// stages' gradients, 9 taps: 329 -> 290 us (1 tap 323 -> 261, 12 taps 353 -> 315, 17, which that kernel stages, 675 -> 345; one
// card, in turn).
// TAPS: the number of taps, so that the tap loops are as long as it takes (branches around single taps' products spilled 36 values).
// Below zero: dV leaves for a kernel of its own, and -TAPS is the history that v needs.
constexpr int MX_SHORT_TAPS = 17;
constexpr bool mx_bwd_short(int taps) { return taps > 0 && taps <= MX_SHORT_TAPS; }
constexpr int mx_halo(int taps) { return taps <= 0 ? -taps : taps <= 9 ? 8 : taps <= 17 ? 16 : 32; }
template <int TAPS> using mx_dv_t = std::conditional_t<(TAPS >= 0), bf16, float>;
__device__ __forceinline__ float mx_quad_sum(float v)
{
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xb1, 0xf, 0xf, true));     // lanes 1 0 3 2
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4e, 0xf, 0xf, true));   // 2 3 0 1
}
// dv silu'(u)
__device__ __forceinline__ float mx_du(float dv, float u)
{
    const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-u));
    return dv * sg * (1.f + u * (1.f - sg));
}
template <int TAPS>
__device__ __forceinline__ void mx_short_bwd(const MxSeq<mx_halo(TAPS)>& xs, const unsigned short* taps, const float* __restrict__ wc,
                                             float (&y)[4][8], float osc, float* edge, float* tsum, bf16* out, int L, int w,
                                             int tid)
{
    constexpr int HALO = mx_halo(TAPS), NH = HALO / 8;
    static_assert(NH == 1 || NH == 2, "");
    const int lane = mx_fresh(tid & 63), c = lane & 15, q = lane >> 4;
    const int t0 = mx_first_step(w, lane);
    {
        float u[4][8];
        xs.short_conv(taps, lane, u);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = t0 + 1024 * i < L;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float du = mx_du(y[i][e] * osc, u[i][e]);
                asm("" : "+v"(du));                  // (a select, not a branch around each exponential)
                y[i][e] = in ? du : 0.f;
            }
        }
    }
    if (c < NH) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float4* p = reinterpret_cast<float4*>(edge + (((4 * q + i) * MX_W + w) * NH + c) * 8);
            p[0] = make_float4(y[i][0], y[i][1], y[i][2], y[i][3]);
            p[1] = make_float4(y[i][4], y[i][5], y[i][6], y[i][7]);
        }
    }
    if (tid < 8 * NH) edge[16 * MX_W * HALO + tid] = 0.f;
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rs = mx_rsrc(out, 2 * L);        // (stores beyond the row's end are dropped)
    float acc[TAPS], wj[TAPS];
#pragma unroll
    for (int j = 0; j < TAPS; ++j) { acc[j] = 0.f; wj[j] = wc[j]; }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        float x[8 * (NH + 1)], du[8 * (NH + 1)], dx[8];
        auto unpack = [&](u32x4 p, int at) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[at + 2 * e] = __builtin_bit_cast(float, p[e] << 16);
                x[at + 2 * e + 1] = __builtin_bit_cast(float, p[e] & 0xffff0000u);
            }
        };
        unpack(xs.r[i], HALO);
        unpack(xs.template piece<1>(lane, i), HALO - 8);
        if constexpr (NH == 2) unpack(xs.template piece<2>(lane, i), 0);
        const float* next = edge + ((4 * q + i) * MX_W + w + 1) * HALO;
#pragma unroll
        for (int e = 0; e < 8; ++e) { du[e] = y[i][e]; dx[e] = 0.f; }
        auto ahead = [&](auto D) __attribute__((always_inline)) {
            constexpr int dd = decltype(D)::value;
            const float4* p = reinterpret_cast<const float4*>(next + (c + dd >= 16 ? c + dd - 16 : 0) * 8);
            const float4 a = p[0], b = p[1];
            const float o[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                du[8 * dd + e] = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, o[e]),
                                                    __builtin_bit_cast(int, y[i][e]), 0x100 + dd, 0xf, 0xf, false));   // row_shl
        };
        ahead(std::integral_constant<int, 1>());
        if constexpr (NH == 2) ahead(std::integral_constant<int, 2>());
#pragma unroll
        for (int j = 0; j < TAPS; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                dx[e] = fmaf(wj[j], du[e + j], dx[e]);
                acc[j] = fmaf(du[e], x[HALO + e - j], acc[j]);
            }
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (bf16)dx[e];
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rs, 2 * (t0 + 1024 * i), 0, 0);
    }
#pragma unroll
    for (int j = 0; j < TAPS; ++j) {
        asm volatile("" : "+v"(acc[j]));          // (summed up by now, all of them side by side, not one after the other below)
        acc[j] = mx_quad_sum(acc[j]);
    }
    if ((lane & 3) == 0) {
        float* slot = tsum + (tid >> 2);
        float t[TAPS];
#pragma unroll
        for (int j = 0; j < TAPS; ++j) t[j] = slot[j * (MX_T / 4)];
#pragma unroll
        for (int j = 0; j < TAPS; ++j) slot[j * (MX_T / 4)] = t[j] + acc[j];
    }
}

// The same for a sequence with an infinity or a NaN in x.  Those meet the zeros of the taps' matrix, which spoils u in eight columns of
// three other rows of 1024 steps; here, on the vector ALU, only the steps of dX that x has a part in are lost (dw is lost anyway).
// It comes second and writes dX again, because a branch in front of it, or one in the middle to another way to u, cost all
// sequences 2 % of the kernel with 9 taps and up to 7 % with more.  dv: 64 KB, cube: where mx_last() took y from.
template <int TAPS>
__device__ __forceinline__ void mx_short_bwd_alone(const bf16* x, const float* __restrict__ wc, const unsigned char* cube,
                                                   const MxLds& tb, float osc, float* dv, bf16* out, int L, int w, int tid)
{
    const int lane = tid & 63, t0 = mx_first_step(w, lane);
    __syncthreads();            // (all have read what lay in dv)
    {
        float y[4][8];
        mx_last(cube, tb, w, lane, y);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float4* p = reinterpret_cast<float4*>(dv + t0 + 1024 * i);
            p[0] = make_float4(y[i][0] * osc, y[i][1] * osc, y[i][2] * osc, y[i][3] * osc);
            p[1] = make_float4(y[i][4] * osc, y[i][5] * osc, y[i][6] * osc, y[i][7] * osc);
        }
    }
#pragma unroll 1
    for (int k = 0; k < 32; ++k) {
        const int t = t0 + 1024 * (k >> 3) + (k & 7);
        float u = 0.f;
#pragma unroll
        for (int j = 0; j < TAPS; ++j)
            if (t >= j && t < L) u = fmaf(wc[j], (float)x[t - j], u);
        dv[t] = t < L ? mx_du(dv[t], u) : 0.f;
    }
    __syncthreads();
#pragma unroll 1
    for (int k = 0; k < 32; ++k) {      // (the lane that has written these steps before)
        const int t = t0 + 1024 * (k >> 3) + (k & 7);
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < TAPS; ++j)
            if (t + j < L) s = fmaf(wc[j], dv[t + j], s);
        if (t < L) out[t] = (bf16)s;
    }
}

// The two long-stage gradients of the convolution (they share the spectrum of dZ); a workgroup walks the sequences of a
// channel, every gridDim.y-th one where a channel is shared, and then those of the next channel blockIdx.x + gridDim.x, ...
//   dv = corr(dZ, k_long): bins of dZ times the conjugate of the kernel's, back;
//   dk[c][s] = sum_b sum_t dZ_b[t] v_b[t - s]: bins of dZ_b times the conjugate of those of v_b = silu(K_s x_b) (recomputed),
//   added up over the sequences in fp32 registers, back once per channel.  At the points used a negative lag is imaginary,
//   as is the second half of a causal sum.
// Both sequences' cubes lie in LDS side by side, so that a wave meets the same tile of both.  Sums of dk: all sequences'
// shares are kept in one unit, a power of two: the largest 1 / (scale of dZ_b x scale of v_b) so far, for a quieter sequence's time
// 16 times that of its own.  (A factor of 1/16 goes with v's scale, half precision has the exponents.  All of it in v's scale, a
// sequence entered with fewer and fewer bits: 2^23 below the loudest its share of dk came out 0.3 times what it is, now right to
// the loud one's rounding.  Below 2^-60 the way back's half precision has nothing left of it.)
// The finished sums H are packed times 32768 / (sqrt N |H|_2), which bounds every sum on the way back by 32768 (Cauchy-Schwarz),
// times MX_ENTRY^2 = 40760, and leaves a typical bin at order one.
// One workgroup per compute unit (144 KB of LDS, with the taps and their sums up to 153; 256 registers, up to 3 values spilled
// without the short stage, 7 .. 16 with it, most of them used at a channel's end only), issuing vector instructions 69 % of the
// time with the short stage.  768 channels x 4 sequences of 16384 steps, 9 taps: 417 -> 240 us (the spectrum of dZ waited in memory
// for that of v, and the sums went back once per pair of sequences).
// mx_bwd_short(TAPS): the short stage's gradient too (dV is dX then, and the taps' sums go to dw): see mx_short_bwd.  Else dV is fp32
// [B][d][L] for the short-stage kernel, or dX itself when there is no short stage (TAPS = 0, v = x).
template <int TAPS>
__global__ __launch_bounds__(MX_T, 2) void convmx_longbwd_kernel(const bf16* __restrict__ X, const float* __restrict__ w_short,
                                                              int m, const unsigned* __restrict__ Ks,
                                                              const float* __restrict__ kscale,
                                                              const MxTables* __restrict__ tables,
                                                              const bf16* __restrict__ dZ, mx_dv_t<TAPS>* __restrict__ dV,
                                                              float* __restrict__ dw, int dw_stride,
                                                              float* __restrict__ dk, int B, int d, int L)
{
    typedef mx_dv_t<TAPS> DVT;
    constexpr int HALO = mx_halo(TAPS);
    constexpr bool SHORT = mx_bwd_short(TAPS);
    if (SHORT) m = TAPS;
    __shared__ __attribute__((aligned(16))) unsigned char cube[2][MX_CUBE];       // of dZ, of v
    __shared__ __attribute__((aligned(16))) MxLds tb;
    __shared__ __attribute__((aligned(16))) unsigned short taps[HALO > 0 ? MX_TAP_WORDS(HALO / 8) + 8 : 8];
    __shared__ float tsum[SHORT ? TAPS * (MX_T / 4) : 1];                   // the taps' sums, a slot per tap and four lanes
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if constexpr (SHORT)
        for (int x = tid; x < TAPS * (MX_T / 4); x += MX_T) tsum[x] = 0.f;
    mx_fetch_tables(tb, tables, tid);
    MxMat m32;
    mx_fetch_matrix(m32, tables, lane);
    if (HALO > 0) mx_write_taps<HALO>(taps, w_short + (long)blockIdx.x * m, m, tid);
    __syncthreads();
    MxLane lc;
    mx_build_lane(lc, lane, w);
    float2 st[MX_NT];
#pragma unroll
    for (int n = 0; n < MX_NT; ++n) st[n] = mx_step(w + MX_W * n);

    MxSeq<0> zs;
    MxSeq<HALO> xs;
    const int b0 = blockIdx.y;          // (< B)
    zs.load(dZ + ((long)b0 * d + blockIdx.x) * L, L, w, lane);
    xs.load(X + ((long)b0 * d + blockIdx.x) * L, L, w, lane);
    float hr[MX_NT][16], hi[MX_NT][16], unit = 0.f, top = 0.f;       // the sums, their unit, the largest it was
#pragma unroll
    for (int n = 0; n < MX_NT; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) hr[n][i] = hi[n][i] = 0.f;
    for (int c = blockIdx.x, b = b0; c < d;) {
        const long row = ((long)b * d + c) * L;
        bool lost;
        float s_d, f;           // f: from the sums' unit so far to the present one
        {
            float v[4][8];
            xs.activated(taps, L, w, lane, v);
            // (an infinity or a NaN in x leaves neither of the results of its column finite: mx_short_bwd_alone)
            const float any = (v[0][0] + v[1][0]) + (v[2][0] + v[3][0]);
            const float mv = mx_wave_max(v, SHORT && any - any != 0.f ? INFINITY : 0.f), md = zs.wave_max();
            if (lane == 0) { tb.red[w] = md; tb.red[MX_W + w] = mv; }
            __syncthreads();
            float bd = 0.f, bv = 0.f;
#pragma unroll
            for (int i = 0; i < MX_W; ++i) { bd = fmaxf(bd, tb.red[i]); bv = fmaxf(bv, tb.red[MX_W + i]); }
            lost = SHORT && __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, bv)) == 0x7f800000;
            s_d = mx_scale(bd);
            const float sv = mx_scale(bv), here = bd > 0.f && bv > 0.f ? 1.0f / (s_d * sv) : 0.f;
            const float next = here >= unit || here == 0.f ? fmaxf(here, unit) : fmaxf(fminf(unit, here * 0x1p4f), top * 0x1p-60f);
            f = next > 0.f ? unit / next : 1.f;
            const float s_v = next > 0.f ? sv * (here / next) : 0.f;
            unit = next;
            top = fmaxf(top, unit);
            mx_first<HALO == 0>(cube[1], tb, lc, v, s_v, w, lane);
            __builtin_amdgcn_sched_barrier(0);
            zs.values(v);
            mx_first<true>(cube[0], tb, lc, v, s_d, w, lane);
        }
        __syncthreads();
        const u32x4* kc = reinterpret_cast<const u32x4*>(Ks + (long)c * MX_N);
#pragma unroll
        for (int n = 0; n < MX_NT; ++n) {
            const int k1 = w + MX_W * n;
            f32x16 zr, zi, vr, vi;
            mx_tile_in(cube[1], tb, m32, k1, lane, vr, vi);
            u32x4 kq[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) kq[a] = kc[(k1 * 4 + a) * 64 + mx_fresh(lane)];
            mx_tile_in(cube[0], tb, m32, k1, lane, zr, zi);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                hr[n][i] = fmaf(zr[i], vr[i], fmaf(zi[i], vi[i], hr[n][i] * f));
                hi[n][i] = fmaf(zi[i], vr[i], fmaf(-zr[i], vi[i], hi[n][i] * f));
                // (here and not where the sums are used: with the products of both tiles kept that long, 80 values were spilled)
                asm volatile("" : "+v"(hr[n][i]), "+v"(hi[n][i]));
            }
            u32x4 re[2], im[2];
            mx_product<true>(zr, zi, kq, re, im);
            mx_tile_out(cube[0], tb, m32, lc.u, st[n], k1, lane, re, im);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        const float osc = kscale[c] / (s_d * ((float)MX_N * MX_GAIN4));
        const int cc = c;
        const bool done = (b += gridDim.y) >= B;
        if (done) { b = b0; c += gridDim.x; }
        MxSeq<HALO> xc;         // the sequence once more: kept in registers past the tiles it would push others out
        if constexpr (SHORT) xc.load(X + row, L, w, lane);
        // the next sequence (after the last one: that one again)
        const long next = c < d ? ((long)b * d + c) * L : row;
        xs.load(X + next, L, w, lane);
        if constexpr (!SHORT) zs.load(dZ + next, L, w, lane);
        float y[4][8];
        mx_last(cube[0], tb, w, lane, y);
        DVT* out = dV + row;
        const int t0 = mx_first_step(w, mx_fresh(lane));
        if constexpr (SHORT) {
            // (cube[1] is free from the tiles' barrier on)
            mx_short_bwd<TAPS>(xc, taps, w_short + (long)cc * TAPS, y, osc, reinterpret_cast<float*>(cube[1]), tsum, out, L, w, tid);
            zs.load(dZ + next, L, w, lane);     // (not before: there are no registers for it, and v comes first)
            if (__builtin_expect(lost, 0))
                mx_short_bwd_alone<TAPS>(X + row, w_short + (long)cc * TAPS, cube[0], tb, osc, reinterpret_cast<float*>(cube[1]), out,
                                         L, w, tid);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                typedef __attribute__((ext_vector_type(8))) DVT out8;
                out8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (DVT)(y[i][e] * osc);
                if (t0 + 1024 * i < L) *reinterpret_cast<out8*>(out + t0 + 1024 * i) = o;
            }
        }
        if (done) {         // ---- the sums' way back
            if (HALO > 0 && c < d) mx_write_taps<HALO>(taps, w_short + (long)c * m, m, tid);      // (barriers before and behind)
            float ss = 0.f;
            const float back = top > 0.f ? unit / top : 0.f;
#pragma unroll
            for (int n = 0; n < MX_NT; ++n)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    hr[n][i] *= back;
                    hi[n][i] *= back;
                    ss = fmaf(hr[n][i], hr[n][i], fmaf(hi[n][i], hi[n][i], ss));
                }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
            if (lane == 0) tb.red[w] = ss;
            __syncthreads();
            ss = 0.f;
#pragma unroll
            for (int i = 0; i < MX_W; ++i) ss += tb.red[i];
            if constexpr (SHORT) {
                for (int j = w; j < m; j += MX_W) {
                    float* slot = tsum + j * (MX_T / 4) + lane;
                    float v = slot[0] + slot[64];
                    slot[0] = slot[64] = 0.f;
#pragma unroll
                    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
                    if (lane == 0) dw[((long)cc * gridDim.y + blockIdx.y) * dw_stride + j] = v;
                }
            }
            const float g = ss > 0.f ? 256.f * rsqrtf(ss) : 0.f;             // 32768 / (sqrt(16384) |H|_2)
#pragma unroll
            for (int n = 0; n < MX_NT; ++n) {
                u32x4 re[2], im[2];
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int q = 0; q < 4; q += 2) {
                        re[a >> 1][2 * (a & 1) + (q >> 1)] = mx_pack(hr[n][4 * a + q] * g, hr[n][4 * a + q + 1] * g);
                        im[a >> 1][2 * (a & 1) + (q >> 1)] = mx_pack(-hi[n][4 * a + q] * g, -hi[n][4 * a + q + 1] * g);
                    }
                mx_tile_out(cube[1], tb, m32, lc.u, st[n], w + MX_W * n, lane, re, im);
#pragma unroll
                for (int i = 0; i < 16; ++i) hr[n][i] = hi[n][i] = 0.f;
            }
            __syncthreads();
            mx_last(cube[1], tb, w, lane, y);
            const float kosc = g > 0.f ? top / (g * ((float)MX_N * MX_GAIN4 * MX_GAIN2)) : 0.f;
            unit = top = 0.f;
            float* o = dk + ((long)b0 * d + cc) * L;         // (a shared channel: its slices are added up by mx_dk_kernel)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (t0 + 1024 * i < L) {
                    float4* p = reinterpret_cast<float4*>(o + t0 + 1024 * i);
                    p[0] = make_float4(y[i][0] * kosc, y[i][1] * kosc, y[i][2] * kosc, y[i][3] * kosc);
                    p[1] = make_float4(y[i][4] * kosc, y[i][5] * kosc, y[i][6] * kosc, y[i][7] * kosc);
                }
            }
        }
    }
}

// dk = the sum of the slices part[g][n], in a fixed order; n a multiple of 4.  dw (may be null): likewise, of part_w[c][g][kConvMaxTaps].
__global__ __launch_bounds__(256) void mx_dk_kernel(const float4* __restrict__ part, float4* __restrict__ dk, int G, long n4,
                                                    const float* __restrict__ part_w, float* __restrict__ dw, int d, int m)
{
    if (dw != nullptr && threadIdx.x < m)
        for (long c = blockIdx.x; c < d; c += gridDim.x) {
            float t = 0.f;
            for (int g = 0; g < G; ++g) t += part_w[(c * G + g) * kConvMaxTaps + threadIdx.x];
            dw[c * m + threadIdx.x] = t;
        }
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n4; i += (long)gridDim.x * 256) {
        float4 t = part[i];
        for (int g = 1; g < G; ++g) {
            const float4 o = part[g * n4 + i];
            t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
        }
        dk[i] = t;
    }
}

// ------------------------------------------------------------------------------------------------ host side
bool convmx_applies(int L, int dtype)
{
    // (rows of a multiple of 8 steps start on 16-byte boundaries: the kernel moves 16-byte pieces only)
    if (dtype != 0 || L <= 4096 || L > MX_N || (L & 7) != 0) return false;
    const char* e = getenv("CHELA_CONV_MATRIX");      // tuning aid: 0 keeps the vector-ALU kernels for every size
    return !(e && atoi(e) == 0);
}

// (twice the words that are used: the size that callers of the query know)
size_t convmx_spectrum_bytes(int d, int L)
{
    if (d <= 0 || L <= 4096 || L > MX_N) return 0;
    return (size_t)d * (2 * MX_N) * sizeof(unsigned) + (((size_t)d * sizeof(float) + 255) & ~(size_t)255);
}

static int mx_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    (void)hipGetLastError();
    return cus;
}

hipError_t launch_convmx_fwd(const void* X, const float* w_short, int m, const void* extra, void* Y, int B, int d, int L,
                             hipStream_t st)
{
    const unsigned* Ks = (const unsigned*)extra;
    const float* scale = (const float*)(Ks + (size_t)d * MX_N);
    const MxTables* tables = mx_tables((void*)extra, d);
    const long total = (long)d * B;
    if (total > 0x7ffffff0L) return hipErrorInvalidValue;
    ProfScope prof(KID_CONV_FWD, st);
    // (a launch has less than 2^32 threads: 2^23 sequences are one too many)
    constexpr long most = 1L << 22;
    for (long first = 0; first < total; first += most) {
        const long end = total - first < most ? total : first + most;
        const dim3 grid((unsigned)((end - first + 7) / 8 * 8));
#define CHELA_MX_FWD(H_)                                                                                                \
    hipLaunchKernelGGL((convmx_fwd_kernel<H_>), grid, dim3(MX_T), 0, st, (const bf16*)X, w_short, m, Ks, scale, tables,    \
                       (bf16*)Y, B, d, L, (int)first, (int)end)
        if (!w_short) CHELA_MX_FWD(0);
        else if (m <= 9) CHELA_MX_FWD(8);
        else if (m <= 17) CHELA_MX_FWD(16);
        else CHELA_MX_FWD(32);
#undef CHELA_MX_FWD
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The gradient kernel's workgroups, one per compute unit.  A channel's sequences are shared out where that shortens the longest
// workgroup's work: its rounds x (its sequences + 0.4, the sums' way back; + 0.2 with the slices to be added up).  128 channels
// x 3 sequences of 8192 steps, both stages' gradients: 64 us, in three shares 54.
static int mx_bwd_shares(int B, int d, int L)
{
    const int cus = mx_cus(), max_share = conv_mx_share(B, d, L);
    int G = 1;
    float best = 0.f;
    for (int g = 1; g <= max_share; ++g) {
        const float t = (float)(((long)d * g + cus - 1) / cus) * ((B + g - 1) / g + (g > 1 ? 0.6f : 0.4f));
        if (g == 1 || t < best) { best = t; G = g; }
    }
    return G;
}

// The short stage inside that kernel costs the same whatever L is (the layout's lanes are there for 16384 steps), the kernel of its
// own and dV on its way through memory go with L and cost two launches.  Both stages' gradients, apart and in one, us:
//   taps                    1            4            9           10           12           16
//   512 x 4 x  8192    165  160     160  153     161  160     167  171     172  178     179  187
//   512 x 4 x  9216    160  149     166  151     169  162     179  172     185  178     190  187
//   512 x 4 x 11264    176  151     181  154     182  164     191  174     194  180     205  191
//   512 x 4 x 13312    188  154     190  159     194  168     206  178     212  187     226  201
// one sequence per workgroup (256 x 1 x 4104): 33 and 27 us with one tap, 40 and 36 with 16; 17 taps (512 x 4 x 4104): 243 and 213.
// So: where every workgroup has one sequence, and from a length on that goes with the taps.
bool convmx_bwd_short(int m, int B, int d, int L, int* shares)
{
    if (!mx_bwd_short(m)) return false;
    const int G = mx_bwd_shares(B, d, L);
    if (shares) *shares = G;
    if ((long)d * G <= mx_cus() && G >= B) return true;
    return L >= (m <= 9 ? 8192 : m <= 16 ? 9216 : 0);
}

hipError_t launch_convmx_longbwd(const void* X, const float* w_short, int m, const void* extra, const void* dZ, void* dV,
                                 float* dw, float* dk, float* part, float* tap_part, int B, int d, int L, hipStream_t st)
{
    const unsigned* Ks = (const unsigned*)extra;
    const float* scale = (const float*)(Ks + (size_t)d * MX_N);
    const MxTables* tables = mx_tables((void*)extra, d);
    int G;
    const bool fused = w_short && convmx_bwd_short(m, B, d, L, &G);
    if (!fused) G = mx_bwd_shares(B, d, L);
    const int cus = mx_cus();
    const long rounds = ((long)d * G + cus - 1) / cus;
    const dim3 grid((unsigned)((d + rounds - 1) / rounds), (unsigned)G);
    float* const sums = G > 1 ? part : dk;
    ProfScope prof(KID_CONV_LONG_BWD, st);
    float* const taps = G > 1 ? tap_part : dw;
    const int tap_stride = G > 1 ? kConvMaxTaps : m;
#define CHELA_MX_BWD(T_)                                                                                                \
    case T_:                                                                                                            \
        hipLaunchKernelGGL((convmx_longbwd_kernel<T_>), grid, dim3(MX_T), 0, st, (const bf16*)X, w_short, m, Ks, scale, \
                           tables, (const bf16*)dZ, (mx_dv_t<T_>*)dV, taps, tap_stride, sums, B, d, L);                 \
        break;
    switch (!w_short ? 0 : fused ? m : -mx_halo(m)) {
        CHELA_MX_BWD(-32) CHELA_MX_BWD(-16) CHELA_MX_BWD(-8) CHELA_MX_BWD(0)
        CHELA_MX_BWD(1) CHELA_MX_BWD(2) CHELA_MX_BWD(3) CHELA_MX_BWD(4) CHELA_MX_BWD(5) CHELA_MX_BWD(6)
        CHELA_MX_BWD(7) CHELA_MX_BWD(8) CHELA_MX_BWD(9) CHELA_MX_BWD(10) CHELA_MX_BWD(11) CHELA_MX_BWD(12)
        CHELA_MX_BWD(13) CHELA_MX_BWD(14) CHELA_MX_BWD(15) CHELA_MX_BWD(16) CHELA_MX_BWD(17)
    }
#undef CHELA_MX_BWD
    if (G > 1) {
        const long n4 = (long)d * L / 4;
        const long wgs = (n4 + 255) / 256;
        hipLaunchKernelGGL(mx_dk_kernel, dim3((unsigned)(wgs < 2048 ? wgs : 2048)), dim3(256), 0, st, (const float4*)part,
                           (float4*)dk, G, n4, tap_part, fused ? dw : nullptr, d, m);
    }
    return hipGetLastError();
}

}  // namespace chela
