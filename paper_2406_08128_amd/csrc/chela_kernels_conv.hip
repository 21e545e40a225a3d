// Short-long convolutions (Sec. 4.2, Eq. 8): Z = K_l( silu( K_s(X) ) ), depthwise and causal, tensors [B][d][L].
//
// The long kernel is as long as the sequence, so K_l goes through the Fourier domain (Eq. 7).  One workgroup
// owns one (batch, channel) sequence and never leaves the chip between load and store:
//   load x, short kernel + silu  ->  real sequence v, zero-padded to N = 2M >= 2L (so that the circular product of
//   Eq. 7 equals the causal sum), packed as M complex numbers z[n] = v[2n] + i v[2n+1]  ->  complex FFT of length M
//   in LDS  ->  product with the kernel's spectrum, linear in the pair of packed bins (k, M - k)  ->  inverse FFT
//   ->  y[2n], y[2n+1] = Re, Im.
// FFT: in place, decimation in frequency forward (natural order in, digit-reversed out) and the exact inverse of
// every pass in reverse order (digit-reversed in, natural out), so no reordering pass exists; the point-wise
// stage addresses the spectrum through the digit reversal.  M = 2^a 16^b, a < 4: an optional leading pass of radix 2, 4 or 8, then
// radix-16 passes with one 16-point transform per thread held in registers (four layers of radix 2, the twiddles worked
// into the butterflies); the first pass forward and the last one back need no LDS on their outer side.  The LDS
// array carries one complex of padding per 16, which makes the stride-1 and stride-16 passes conflict-free.
// Arithmetic is fp32 on the vector ALU: with one kernel per channel there is no operand shared across channels
// except the DFT matrix itself, and fp32 matrix instructions are no faster than the ALU on this chip.
#include "chela_convmx.h"
#include <algorithm>
#include <cfloat>
#include <cstdlib>

namespace chela {

typedef __bf16 bf16;

struct cplx { float x, y; };
__device__ __forceinline__ cplx mk(float x, float y) { cplx c; c.x = x; c.y = y; return c; }
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return mk(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return mk(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ cplx cmul(cplx a, cplx b) { return mk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
// s + a b
__device__ __forceinline__ cplx cfma(cplx a, cplx b, cplx s)
{
    return mk(fmaf(-a.y, b.y, fmaf(a.x, b.x, s.x)), fmaf(a.y, b.x, fmaf(a.x, b.y, s.y)));
}
__device__ __forceinline__ cplx conj(cplx a) { return mk(a.x, -a.y); }
__device__ __forceinline__ cplx mul_neg_i(cplx a) { return mk(a.y, -a.x); }   // a * (-i)
__device__ __forceinline__ cplx mul_pos_i(cplx a) { return mk(-a.y, a.x); }   // a * (+i)

// a + t b and a - t b in place (a, b), t = tx + i ty: four fused multiply-adds for the sum and 2a - (a + t b) for the
// difference, six instructions where a product and two additions take eight.
__device__ __forceinline__ void bfly(cplx& a, cplx& b, float tx, float ty)
{
    const cplx m = mk(fmaf(-ty, b.y, fmaf(tx, b.x, a.x)), fmaf(ty, b.x, fmaf(tx, b.y, a.y)));
    b = mk(fmaf(2.f, a.x, -m.x), fmaf(2.f, a.y, -m.y));
    a = m;
}
__device__ __forceinline__ void bfly1(cplx& a, cplx& b) { const cplx m = cadd(a, b); b = csub(a, b); a = m; }
// the same with t turned by a quarter (forward: -i t, inverse: +i t); QT: t = 1
template <bool INV> __device__ __forceinline__ void bfly_q(cplx& a, cplx& b, float tx, float ty)
{
    if (INV) bfly(a, b, -ty, tx); else bfly(a, b, ty, -tx);
}
template <bool INV> __device__ __forceinline__ void bfly1_q(cplx& a, cplx& b)
{
    const cplx r = INV ? mul_pos_i(b) : mul_neg_i(b);
    b = csub(a, r);
    a = cadd(a, r);
}

// Sixteenth and eighth roots of unity: cos and sin of pi / 8, sqrt(1/2).  As fp32 numbers all three are too small, so that every root shrinks
// what it multiplies, and a transform and back lose 1e-7 of a sequence of one sign; at 4096 and 16384 points the rounding of the
// table of powers happens to make up for a half and for nearly all of it.  At the sizes in between (conv_fine) the first, and the
// second part of the eighth root in w^2 w8, are the next numbers above.  64 channels, fp32, inputs of one sign, 5003 steps: Z
// 2.3e-7 -> 1.2e-7 from 64 bits (in 16384 points 1.5e-7), dX 2.1e-7 -> 0.8e-7 (0.9e-7); of either sign: 2.7e-7 -> 2.2e-7 (2.9e-7).
constexpr float kC1 = 0.92387953251128674f, kS1 = 0.38268343236508977f, kR2 = 0.70710678118654752f;
constexpr float kC1Above = 0x1.d906bep-1f, kR2Above = 0x1.6a09e8p-1f;

// w^2 of a w on the unit circle and not far from 1
__device__ __forceinline__ cplx unit_square(cplx w) { const float y2 = 2.f * w.y; return mk(fmaf(-y2, w.y, 1.f), y2 * w.x); }

// 16-point DFT in registers with the twiddles of its INPUTS taken along:  X_p = sum_q x_q (w w16^p)^q, w16 =
// exp(-2 pi i / 16) (INV: conjugate).  In: v[q] = x_q.  Out: X_p sits in slot rev4(p) (the four bits of p reversed).
// w2 = w^2, w4 = w^4, w8 = w^8.  Radix 2 over q: 16 values of a polynomial, and level by level only the powers w^8, w^4, w^2 and w of the base are met,
// times eighth and sixteenth roots: eight distinct complex twiddles (21 instructions from those) for 32 butterflies of six
// instructions, 220 in all, where a plain 16-point transform with fifteen twiddles in front of or behind it takes 290
// (its chain of powers 56, its products 60).  UNIT: w = 1 (148 instructions).  HALF_IN: x_8 .. x_15 are zero (not read).
// HALF_OUT: only X_0 .. X_7 are wanted.  FINE: conv_fine(M).
__host__ __device__ constexpr int rev4(int p) { return ((p & 1) << 3) | ((p & 2) << 1) | ((p & 4) >> 1) | ((p & 8) >> 3); }
template <bool INV, bool UNIT, bool FINE, bool HALF_IN = false, bool HALF_OUT = false>
__device__ __forceinline__ void dft16(cplx (&v)[16], cplx w, cplx w2, cplx w4, cplx w8)
{
    constexpr float SG = INV ? 1.f : -1.f, C1 = FINE ? kC1Above : kC1, R2b = FINE ? kR2Above : kR2;
    if (HALF_IN) {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q + 8] = v[q];
    } else if (UNIT) {
#pragma unroll
        for (int q = 0; q < 8; ++q) bfly1(v[q], v[q + 8]);
    }
    if (UNIT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) { bfly1(v[q], v[q + 4]); bfly1_q<INV>(v[q + 8], v[q + 12]); }
    } else {
        if (!HALF_IN) {
#pragma unroll
            for (int q = 0; q < 8; ++q) bfly(v[q], v[q + 8], w8.x, w8.y);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) { bfly(v[q], v[q + 4], w4.x, w4.y); bfly_q<INV>(v[q + 8], v[q + 12], w4.x, w4.y); }
    }
    // slots now: x_q sums with the bits of p seen so far (lowest first) in the top bits of the slot
    const cplx w2b = UNIT ? mk(kR2, SG * R2b) : cmul(w2, mk(kR2, SG * R2b));             // w^2 w8
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (UNIT) { bfly1(v[q], v[q + 2]); bfly1_q<INV>(v[q + 4], v[q + 6]); }
        else { bfly(v[q], v[q + 2], w2.x, w2.y); bfly_q<INV>(v[q + 4], v[q + 6], w2.x, w2.y); }
        bfly(v[q + 8], v[q + 10], w2b.x, w2b.y);
        bfly_q<INV>(v[q + 12], v[q + 14], w2b.x, w2b.y);
    }
    const cplx d1 = UNIT ? mk(C1, SG * kS1) : cmul(w, mk(C1, SG * kS1));
    const cplx d2 = UNIT ? mk(kR2, SG * kR2) : cmul(w, mk(kR2, SG * kR2));
    const cplx d3 = UNIT ? mk(kS1, SG * C1) : cmul(w, mk(kS1, SG * C1));
    // (HALF_OUT: the differences, X_(p+8), are dead and the compiler drops them)
    if (UNIT) { bfly1(v[0], v[1]); bfly1_q<INV>(v[2], v[3]); }
    else { bfly(v[0], v[1], w.x, w.y); bfly_q<INV>(v[2], v[3], w.x, w.y); }
    bfly(v[8], v[9], d1.x, d1.y);
    bfly_q<INV>(v[10], v[11], d1.x, d1.y);
    bfly(v[4], v[5], d2.x, d2.y);
    bfly_q<INV>(v[6], v[7], d2.x, d2.y);
    bfly(v[12], v[13], d3.x, d3.y);
    bfly_q<INV>(v[14], v[15], d3.x, d3.y);
}

__host__ __device__ constexpr int conv_threads(int M) { return M / 16 < 64 ? 64 : M / 16; }
// radix of the pass that leads where M is no power of 16 (1: none)
__host__ __device__ constexpr int conv_lead(int M) { return M == 1024 || M == 16384 ? 4 : M == 2048 ? 8 : M == 8192 ? 2 : 1; }
__host__ __device__ constexpr int conv_pad(int i) { return i + (i >> 4); }

// 2048 and 8192 points: twiddles that cost no more and are nearer what they should be (see twiddle, PairTwiddle).  A sequence fills
// more of a smaller transform, so more of its rounding errors lies on the steps that are wanted; this makes up for it.  The
// others stay as they were: the gradient kernel of 4096 points then spilled more, 420 -> 480 us at 32 x 512 x 4096.
__host__ __device__ constexpr bool conv_fine(int M) { return M == 2048 || M == 8192; }

// Place of W^e in the table of powers: the passes walk it by 1, by 4, by 8, by 16, (M = 8192) by 32 or (M = 16384) by 64, and
// sixteen neighbours of any such walk lie in sixteen different places of the 256 bytes that the banks span.  (M = 2048: with no
// room in between, see ConvLds.)
template <int M>
__host__ __device__ constexpr int power_pos(int e)
{
    return M == 2048 ? e ^ (e >> 4) : e + (e >> 4) + (M == 16384 ? e >> 6 : M == 8192 ? e >> 5 : 0);
}

template <int M>
struct ConvLds {
    // complex slots; at the smallest size 16 more than the transform needs, so that two real sequences with 32 steps of margin
    // each fit (others have that room in their padding; it is not used only where the 128 bytes count)
    static constexpr int DATA = conv_pad(M) + (M == 2048 ? 0 : 16);
    // + twiddles: the powers W^e that the passes ask for (e < M / 16), each with its square or fourth power
    // (M = 2048: 20 KB with the eighth powers, see twiddle: just so much that the forward kernel's eight workgroups fit a unit; with
    // seven, 32 x 512 x 2048 took 119 us, so 103)
    static constexpr int POWERS = M == 2048 ? M / 16 : power_pos<M>(M / 16 - 1) + 1;
    static constexpr int BYTES = DATA * 8 + POWERS * (M == 2048 ? 24 : 16);
};

// w = exp(-2 pi i e / M) (INV: its conjugate), w2 = w^2 and w4 = w^4, e < M / 16.  One of the powers comes from the table as well:
// dft16 squares on to w^8, and every squaring doubles the error it is handed.  Where w was multiplied up from two tables of 128
// and squared here (M = 16384), the gradient of 128 channels x 16384 steps, fp32, was 6.3 .. 7.7e-7 from 64 bits; with the
// square from the table 4.0 .. 4.7e-7, and 4 x 256 channels take 209 us instead of 250.  With the fourth power from it, and the
// square by a formula that holds on the unit circle only (conv_fine), the last square is one step from the table and not two:
// 64 channels x 6001 steps 4.2e-7 -> 3.4e-7.  M = 2048: the eighth power, too (64 x 2048 steps 3.3e-7 -> 3.1e-7).  (Both before kC1Above and
// kR2Above; with them 2.7e-7 and 2.6e-7.)
template <int M, bool INV>
__device__ __forceinline__ void twiddle(const float4* tw, int e, cplx& w, cplx& w2, cplx& w4, cplx& w8)
{
    const float4 t = tw[power_pos<M>(e)];
    w = mk(t.x, INV ? -t.y : t.y);
    const cplx p = mk(t.z, INV ? -t.w : t.w);
    w2 = conv_fine(M) ? unit_square(w) : p;
    w4 = conv_fine(M) ? p : mk(fmaf(p.x, p.x, -p.y * p.y), 2.f * p.x * p.y);
    if (M == 2048) {
        const float2 q = reinterpret_cast<const float2*>(tw + ConvLds<M>::POWERS)[power_pos<M>(e)];
        w8 = mk(q.x, INV ? -q.y : q.y);
    } else w8 = mk(fmaf(w4.x, w4.x, -w4.y * w4.y), 2.f * w4.x * w4.y);
}

// Storage position of spectrum bin k (0 <= k < M) after the forward passes.
template <int M>
__device__ __forceinline__ int spectrum_pos(int k)
{
    int pos = 0, span = M;
    constexpr int R = conv_lead(M);
    if (R > 1) { span /= R; pos += (k & (R - 1)) * span; k >>= R == 2 ? 1 : R == 4 ? 2 : 3; }
#pragma unroll
    for (int s = span; s > 1; s /= 16) { pos += (k & 15) * (s / 16); k >>= 4; }
    return pos;
}

// The number of the bins (their low digits) that the blocks of length N16 hold after the forward passes before: block
// index in storage order -> digits reversed.
template <int M, int N16>
__device__ __forceinline__ int block_bin(int block)
{
    constexpr int NB = M / N16, R = conv_lead(M) > 1 ? conv_lead(M) : 16;      // blocks; what the first digit counts to
    if (NB <= 16) return block;                                                // one digit
    if (NB == 16 * R) return (block >> 4) + (block & 15) * R;
    static_assert(NB <= 16 || NB == 16 * R || NB == 256 * R, "");
    return (block >> 8) + ((block >> 4) & 15) * R + (block & 15) * (16 * R);
}

// One radix-16 pass over sub-transforms of length N16 (stride N16 / 16), forward or inverse, 16-point transforms
// in registers, T threads.  With the length fixed at compile time the 16 LDS addresses are one base plus constants
// (the padding of a multiple of 16 is itself a constant).  Both directions take their twiddles at the inputs, as the
// powers of ONE number per transform that dft16 works into its butterflies:
//   forward, digits of k found so far = K:   sum_q x_q W_(16 NB)^(q K) w16^(p q),  NB = M / N16 blocks
//   inverse, point j of the sub-transform:   sum_q X_q conj(W_N16^(q j)) conj(w16^(p q))
// so the first pass either way has none.  HALF: forward, inputs 8 .. 15 are zero; inverse, outputs 8 .. 15 are not wanted.
template <int M, int T, int N16, bool INV, bool HALF>
__device__ __forceinline__ void pass16(cplx* a, const float4* tw, int tid)
{
    constexpr int S = N16 / 16;
    constexpr int STEP = S >= 16 ? S + S / 16 : 1;                 // padded distance between the transform's points
    constexpr bool UNIT = INV ? S == 1 : N16 == M;
    for (int g = tid; g < M / 16; g += T) {
        const int block = g / S, j = g - block * S;
        cplx* p0 = a + (S >= 16 ? conv_pad(block * N16 + j) : 17 * g);
        cplx v[16];
        cplx w = mk(1.f, 0.f), w2 = w, w4 = w, w8 = w;
        if (!UNIT) twiddle<M, INV>(tw, INV ? j * (M / N16) : block_bin<M, N16>(block) * S, w, w2, w4, w8);
#pragma unroll
        for (int q = 0; q < (HALF && !INV ? 8 : 16); ++q) v[q] = p0[q * STEP];
        dft16<INV, UNIT, conv_fine(M), HALF && !INV, HALF && INV>(v, w, w2, w4, w8);
#pragma unroll
        for (int p = 0; p < (HALF && INV ? 8 : 16); ++p) p0[p * STEP] = v[rev4(p)];
    }
}

// The forward transform of the packed sequence z[n], n = tid + T i < M/2 (its upper half is zero: L <= M real steps), from
// registers into a[], and the way back, of which only the first M/2 results are wanted, into registers again: the first
// pass forward and the last one back never go through LDS.  A __syncthreads() separates the passes; the caller
// synchronises before and after.
// FULL (M = 16384): z[n] is given for all n = tid + T i < M.
template <int M, int T, bool FULL = false>
__device__ __forceinline__ void fft_forward(const cplx (&z)[FULL ? M / T : M / T / 2], cplx* a, const float4* tw, int tid)
{
    static_assert(!FULL || conv_lead(M) == 4, "the leading radix-4 pass only");
    if constexpr (M == 256) {               // (16 of a wave's threads work in a pass: the input is dealt out again)
#pragma unroll
        for (int i = 0; i < M / T / 2; ++i) a[conv_pad(tid + T * i)] = z[i];
        __syncthreads();
        pass16<M, T, 256, false, true>(a, tw, tid);
    } else {
        static_assert(M / T == 16, "sixteen points per thread");
        if constexpr (conv_lead(M) == 2) {
            // (with its partner zero a point goes into both halves as it is)
            constexpr int sp = M / 2 + M / 32;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                cplx* p0 = a + conv_pad(tid + T * j);
                p0[0] = z[j];
                p0[sp] = z[j];
            }
            __syncthreads();
            pass16<M, T, 4096, false, false>(a, tw, tid);
            __syncthreads();
        } else if constexpr (conv_lead(M) == 8) {
            // x_0 .. x_3 of two columns, x_4 .. x_7 being zero: even bins from x_q, odd ones from x_q w8^q
            constexpr int s = M / 8, sp = s + s / 16;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                cplx* p0 = a + conv_pad(tid + T * j);
                cplx v[4], u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = z[2 * q + j];
                u[0] = v[0];
                u[1] = cmul(v[1], mk(kR2, -kR2));
                u[2] = mul_neg_i(v[2]);
                u[3] = cmul(v[3], mk(-kR2, -kR2));
                bfly1(v[0], v[2]);
                bfly1(v[1], v[3]);
                bfly1(u[0], u[2]);
                bfly1(u[1], u[3]);
                const cplx r = mul_neg_i(v[3]), t = mul_neg_i(u[3]);
                p0[0] = cadd(v[0], v[1]);
                p0[sp] = cadd(u[0], u[1]);
                p0[2 * sp] = cadd(v[2], r);
                p0[3 * sp] = cadd(u[2], t);
                p0[4 * sp] = csub(v[0], v[1]);
                p0[5 * sp] = csub(u[0], u[1]);
                p0[6 * sp] = csub(v[2], r);
                p0[7 * sp] = csub(u[2], t);
            }
            __syncthreads();
        } else if constexpr (conv_lead(M) == 4) {
            constexpr int s = M / 4, sp = s + s / 16;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                cplx* p0 = a + conv_pad(tid + T * j);
                cplx v0 = z[j], v1 = z[j + 4], r = mul_neg_i(v1);
                if constexpr (FULL) {
                    const cplx v2 = z[j + 8], v3 = z[j + 12];
                    r = mul_neg_i(csub(v1, v3));
                    v1 = cadd(v1, v3);
                    const cplx e = csub(v0, v2);
                    v0 = cadd(v0, v2);
                    p0[sp] = cadd(e, r);
                    p0[3 * sp] = csub(e, r);
                    p0[0] = cadd(v0, v1);
                    p0[2 * sp] = csub(v0, v1);
                    continue;
                }
                p0[0] = cadd(v0, v1);
                p0[sp] = cadd(v0, r);
                p0[2 * sp] = csub(v0, v1);
                p0[3 * sp] = csub(v0, r);
            }
            __syncthreads();
            if constexpr (M == 16384) { pass16<M, T, 4096, false, false>(a, tw, tid); __syncthreads(); }
        } else {
            constexpr int S = M / 16, STEP = S + S / 16;
            cplx v[16];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = z[q];
            dft16<false, true, conv_fine(M), true>(v, mk(1.f, 0.f), mk(1.f, 0.f), mk(1.f, 0.f), mk(1.f, 0.f));
            cplx* p0 = a + conv_pad(tid);
#pragma unroll
            for (int p = 0; p < 16; ++p) p0[p * STEP] = v[rev4(p)];
            __syncthreads();
        }
        pass16<M, T, 256, false, false>(a, tw, tid);
    }
    __syncthreads();
    pass16<M, T, 16, false, false>(a, tw, tid);
}

template <int M, int T>
__device__ __forceinline__ void fft_inverse(cplx* a, cplx (&y)[M / T / 2], const float4* tw, int tid)
{
    pass16<M, T, 16, true, false>(a, tw, tid);
    __syncthreads();
    if constexpr (M == 256) {
        pass16<M, T, 256, true, true>(a, tw, tid);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < M / T / 2; ++i) y[i] = a[conv_pad(tid + T * i)];
    } else {
        pass16<M, T, 256, true, false>(a, tw, tid);
        __syncthreads();
        if constexpr (conv_lead(M) == 2) {
            pass16<M, T, 4096, true, false>(a, tw, tid);
            __syncthreads();
            // y = x_0 + conj(W^(tid + T j)) x_1: W^T is a sixteenth root
            constexpr int sp = M / 2 + M / 32;
            constexpr float CX[8] = {1.f, kC1Above, kR2, kS1, 0.f, -kS1, -kR2, -kC1Above}, CY[8] = {0.f, kS1, kR2, kC1Above, 1.f, kC1Above, kR2, kS1};
            cplx t, t2, t4, t8;
            twiddle<M, true>(tw, tid, t, t2, t4, t8);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const cplx* p0 = a + conv_pad(tid + T * j);
                const cplx c = j == 0 ? t : j == 4 ? mul_pos_i(t) : cmul(t, mk(CX[j], CY[j]));
                y[j] = cfma(c, p0[sp], p0[0]);
            }
        } else if constexpr (conv_lead(M) == 8) {
            // y_p = sum_q x_q t^q conj(w8)^(p q), p < 4, t = conj(W^(tid + T j)), W^T a sixteenth root: even and odd q apart
            constexpr int s = M / 8, sp = s + s / 16;
            cplx t, t2, t4, t8;
            twiddle<M, true>(tw, tid, t, t2, t4, t8);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const cplx* p0 = a + conv_pad(tid + T * j);
                if (j == 1) { t = cmul(t, mk(kC1Above, kS1)); t2 = cmul(t2, mk(kR2, kR2)); t4 = mul_pos_i(t4); }
                cplx v[4], u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) { v[q] = p0[2 * q * sp]; u[q] = p0[(2 * q + 1) * sp]; }
                bfly(v[0], v[2], t4.x, t4.y);
                bfly(v[1], v[3], t4.x, t4.y);
                bfly(u[0], u[2], t4.x, t4.y);
                bfly(u[1], u[3], t4.x, t4.y);
                bfly(v[0], v[1], t2.x, t2.y);
                bfly_q<true>(v[2], v[3], t2.x, t2.y);
                bfly(u[0], u[1], t2.x, t2.y);
                bfly_q<true>(u[2], u[3], t2.x, t2.y);
                // (slots 0, 2, 1, 3 now hold p = 0, 1, 2, 3)
                y[j] = cfma(t, u[0], v[0]);
                y[j + 2] = cfma(cmul(t, mk(kR2, kR2)), u[2], v[2]);
                y[j + 4] = cfma(mul_pos_i(t), u[1], v[1]);
                y[j + 6] = cfma(cmul(t, mk(-kR2, kR2)), u[3], v[3]);
            }
        } else if constexpr (conv_lead(M) == 4) {
            if constexpr (M == 16384) { pass16<M, T, 4096, true, false>(a, tw, tid); __syncthreads(); }
            constexpr int s = M / 4, sp = s + s / 16;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const cplx* p0 = a + conv_pad(tid + T * j);
                cplx t1, t2, t4, t8;
                // W^(tid + j M/16): W^tid times sixteenth roots
                twiddle<M, true>(tw, tid, t1, t2, t4, t8);
                t1 = j == 0 ? t1 : cmul(t1, j == 1 ? mk(kC1, kS1) : j == 2 ? mk(kR2, kR2) : mk(kS1, kC1));
                t2 = j == 0 ? t2 : j == 2 ? mul_pos_i(t2) : cmul(t2, j == 1 ? mk(kR2, kR2) : mk(-kR2, kR2));
                const cplx t3 = cmul(t2, t1);
                cplx v0 = p0[0], v1 = cmul(p0[sp], t1), v2 = p0[2 * sp], v3 = p0[3 * sp];
                bfly(v0, v2, t2.x, t2.y);
                bfly(v1, v3, t3.x, t3.y);
                y[j] = cadd(v0, v1);
                y[j + 4] = cadd(v2, mul_pos_i(v3));
            }
        } else {
            constexpr int S = M / 16, STEP = S + S / 16;
            const cplx* p0 = a + conv_pad(tid);
            cplx v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = p0[q * STEP];
            cplx w, w2, w4, w8;
            twiddle<M, true>(tw, tid, w, w2, w4, w8);
            dft16<true, false, conv_fine(M), false, true>(v, w, w2, w4, w8);
#pragma unroll
            for (int p = 0; p < 8; ++p) y[p] = v[rev4(p)];
        }
    }
}

// A row for buffer loads and stores: what lies at or beyond its end reads as zero and is not written, which takes the
// branches around single accesses out of the kernels.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* row, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), 0, bytes, 0x00020000);     // (untyped, raw offsets)
}

// raw_t: the pair (x[t], x[t+1]) as it sits in memory, so that a sequence fetched ahead costs as few registers as it
// costs bytes; load_pair() reads an aligned pair, load_single() builds one from single reads (odd row lengths), `off` and
// `imm` being byte offsets of x[t] in the row; unpack() converts.
template <typename T> struct IoPair;
template <> struct IoPair<float> {
    typedef float2 raw_t;
    static __device__ __forceinline__ raw_t load_pair(__amdgpu_buffer_rsrc_t r, int off)
    {
        return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    }
    static __device__ __forceinline__ raw_t load_single(__amdgpu_buffer_rsrc_t r, int off)
    {
        return make_float2(__builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0)),
                           __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off + 4, 0, 0)));
    }
    static __device__ __forceinline__ void unpack(raw_t r, float& a, float& b) { a = r.x; b = r.y; }
    static __device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, int off, float a, float b)
    {
        typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
        u32x2 v;
        v[0] = __builtin_bit_cast(unsigned, a);
        v[1] = __builtin_bit_cast(unsigned, b);
        __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
    }
    static __device__ __forceinline__ void store_single(__amdgpu_buffer_rsrc_t r, int off, float a, float b)
    {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, a), r, off, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, b), r, off + 4, 0, 0);
    }
};
template <> struct IoPair<bf16> {
    typedef unsigned raw_t;
    static __device__ __forceinline__ raw_t load_pair(__amdgpu_buffer_rsrc_t r, int off)
    {
        return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    }
    static __device__ __forceinline__ raw_t load_single(__amdgpu_buffer_rsrc_t r, int off)
    {
        return (unsigned)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0) |
               (unsigned)__builtin_amdgcn_raw_buffer_load_b16(r, off + 2, 0, 0) << 16;
    }
    static __device__ __forceinline__ void unpack(raw_t u, float& a, float& b)
    {
        a = __builtin_bit_cast(float, u << 16);
        b = __builtin_bit_cast(float, u & 0xffff0000u);
    }
    static __device__ __forceinline__ unsigned pack(float a, float b)
    {
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        bf16x2 v;
        v[0] = (bf16)a;
        v[1] = (bf16)b;
        return __builtin_bit_cast(unsigned, v);
    }
    static __device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, int off, float a, float b)
    {
        __builtin_amdgcn_raw_buffer_store_b32(pack(a, b), r, off, 0, 0);
    }
    static __device__ __forceinline__ void store_single(__amdgpu_buffer_rsrc_t r, int off, float a, float b)
    {
        const unsigned v = pack(a, b);
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v, r, off, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(v >> 16), r, off + 2, 0, 0);
    }
};

// Eight consecutive elements at a 16-byte aligned position.
__device__ __forceinline__ void load8(const float* p, float (&v)[8])
{
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16* p, float (&v)[8])
{
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    const unsigned w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[2 * e] = __builtin_bit_cast(float, w[e] << 16);
        v[2 * e + 1] = __builtin_bit_cast(float, w[e] & 0xffff0000u);
    }
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8])
{
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16* p, const float (&v)[8])
{
    typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16)v[e];
    *reinterpret_cast<bf16x8*>(p) = o;
}

template <int M, int T>
__device__ __forceinline__ void build_tables(float4* tw, int tid)
{
    float s, c, s2, c2;
    for (int e = tid; e < M / 16; e += T) {
        sincospif(-2.0f * (float)e / (float)M, &s, &c);
        sincospif((conv_fine(M) ? -8.0f : -4.0f) * (float)e / (float)M, &s2, &c2);
        tw[power_pos<M>(e)] = make_float4(c, s, c2, s2);
        if (M == 2048) {
            sincospif(-16.0f * (float)e / (float)M, &s, &c);
            reinterpret_cast<float2*>(tw + ConvLds<M>::POWERS)[power_pos<M>(e)] = make_float2(c, s);
        }
    }
}

// Order in which the point-wise stages walk the bin pairs (k, M - k), 0 <= k < M/2.  The forward passes leave
// bin k at a digit-reversed position, so lanes that took consecutive k would all hit the same LDS banks (strides of
// M/4 and M/64 complex).  Pair l takes k = ((l & 63) << HB) | (l >> 6) instead: the 64 lanes of a wave then differ
// in the HIGH bits of k, i.e. in the low digits of the storage position.  Pair 0 stands for the two self-paired bins 0
// and M/2.  The kernel spectrum is stored in the same order, one float4 per pair, so its loads coalesce.
template <int M>
__device__ __forceinline__ int pair_bin(int l)
{
    int hb = 0;
#pragma unroll
    for (int x = M / 128; x > 1; x >>= 1) ++hb;
    return ((l & 63) << hb) | (l >> 6);
}

// Positions in a[] of the pairs l = tid + T i of a thread.  With sixteen points per thread the eight pairs of a thread
// differ in two digits of k only, k = k(0) + (T/64) i: bins k lie at constant distances from the first one, bins M - k at
// the same distances backwards, except where no lower digit borrows (the first wave's i = 0 and 4).  Four registers and
// constant offsets, where working each position out took some 40 instructions per pair and sequence.
template <int M, int T>
struct PairPos {
    static constexpr int NP = M / 2 / T;                  // pairs per thread: 8 (2 at M = 256)
    static constexpr bool LIN = NP == 8;
    static constexpr int SA = M == 1024 ? 272 : M == 2048 ? 544 : 1088;     // padded distance of i and i + 1; 17 of i and i + 4
    int a1[LIN ? 1 : NP], a2[LIN ? 3 : NP];
    static __device__ __forceinline__ int bin_pos(int k) { return conv_pad(spectrum_pos<M>(k & (M - 1))); }
    __device__ __forceinline__ PairPos(int tid)
    {
        if constexpr (LIN) {
            a1[0] = bin_pos(pair_bin<M>(tid));
            a2[0] = bin_pos(tid == 0 ? M / 2 : M - pair_bin<M>(tid));
            a2[1] = bin_pos(M - pair_bin<M>(tid + 4 * T));
            a2[2] = bin_pos(M - pair_bin<M>(tid + T)) + SA;
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int k = pair_bin<M>(tid + T * i);
                a1[i] = bin_pos(k);
                a2[i] = bin_pos(k == 0 ? M / 2 : M - k);
            }
        }
    }
    __device__ __forceinline__ int first(int i) const { return LIN ? a1[0] + (i & 3) * SA + (i >> 2) * 17 : a1[LIN ? 0 : i]; }
    __device__ __forceinline__ int second(int i) const
    {
        if (!LIN) return a2[LIN ? 0 : i];
        return i == 0 ? a2[0] : i == 4 ? a2[1] : a2[2] - (i & 3) * SA - (i >> 2) * 17;
    }
};

// W_2M^k = exp(-i pi k / M) for the bins a thread meets when it walks its pairs: k = k(0) + (T/64) i, one sincospi per
// thread and one rotation per pair, by exp(-i pi / 1024) (M = 256: exp(-i pi / 256)); conv_fine: from the first each time.
template <int M, int T>
struct PairTwiddle {
    static_assert(M / T == 16 || (M == 256 && T == 64), "the rotation below");
    cplx first;
    static constexpr cplx step = M == 256 ? cplx{0.99992470183914454f, -0.012271538285719925f}
                                          : cplx{0.99999529380957617f, -0.0030679567629659763f};
    // of pair i + 1, w being that of pair i
    __device__ __forceinline__ cplx after(int i, cplx w) const
    {
        constexpr float CX[8] = {0.99999529380957619f, 0.99998117528260111f, 0.99995764455196390f, 0.99992470183914450f,
                                 0.99988234745421256f, 0.99983058179582340f, 0.99976940535121528f, 0.99969881869620425f};
        constexpr float CY[8] = {-0.00306795676296598f, -0.00613588464915448f, -0.00920375478205982f, -0.01227153828571993f,
                                 -0.01533920628498810f, -0.01840672990580482f, -0.02147408027546951f, -0.02454122852291229f};
        return conv_fine(M) ? cmul(first, mk(CX[i & 7], CY[i & 7])) : cmul(w, step);
    }
    __device__ __forceinline__ PairTwiddle(int tid)
    {
        float s, c;
        sincospif(-(float)pair_bin<M>(tid) / (float)M, &s, &c);
        first = mk(c, s);
    }
};

// A real sequence v of length 2M packed as z[n] = v[2n] + i v[2n+1] has the spectrum
//     V[k] = E + w O,  conj V[M-k] = E - w O,   E = (A + B)/2,  O = (A - B)/(2i),   A = Z[k], B = conj Z[M-k], w = W_2M^k.
// The product with a kernel's spectrum K, packed again, is linear in (A, B).  With P = (K[k] + conj K[M-k])/2, D =
// (K[k] - conj K[M-k])/2 and w = c - i s it comes to
//     A' = P A + D r,  r = -s A + i c B;      B' = P B + D q,  q = s B - i c A
// -- 24 multiply-adds per pair; untangling to V, multiplying and packing again took over 50.  (P, D) of a kernel are E and
// w O of its own packed transform.  Correlation: conj P, conj D.
// Gradient of the kernel, sums over sequences of G conj(V) for two packed spectra (A, B) and (a, b), r and q of (a, b):
//     2 al = A conj(a) + B conj(b),  2 be = A conj(r) + B conj(q);   packed: A' = al + i be conj(w), B' = al - i be conj(w).
// Pair 0 holds the self-paired bins 0 and M/2 (A = Z[0] = x + i y, B = conj Z[M/2]): kernel entries (P, D) of bin 0, both
// real, then K[M/2];  A' = (P x + D y) + i (P y + D x), B' = K[M/2] B;  sums (x x' + y y') + i (x y' + y x') and B conj(b).
__device__ __forceinline__ void pair_rot(cplx A, cplx B, cplx w, cplx& r, cplx& q)
{
    r = mk(fmaf(w.y, A.x, -w.x * B.y), fmaf(w.y, A.y, w.x * B.x));
    q = mk(fmaf(-w.y, B.x, w.x * A.y), fmaf(-w.y, B.y, -w.x * A.x));
}
// s + a conj(b)
__device__ __forceinline__ cplx cfmac(cplx a, cplx b, cplx s)
{
    return mk(fmaf(a.y, b.y, fmaf(a.x, b.x, s.x)), fmaf(a.y, b.x, fmaf(-a.x, b.y, s.y)));
}

// (A, B) times the kernel entry K; self: pair 0.
template <bool CORR>
__device__ __forceinline__ void pair_mul(cplx& A, cplx& B, cplx w, float4 K, bool self)
{
    const cplx P = mk(K.x, CORR ? -K.y : K.y), D = mk(K.z, CORR ? -K.w : K.w);
    if (self) {
        A = mk(fmaf(K.x, A.x, K.y * A.y), fmaf(K.x, A.y, K.y * A.x));
        B = cmul(D, B);
        return;
    }
    cplx r, q;
    pair_rot(A, B, w, r, q);
    A = cfma(D, r, cmul(P, A));
    B = cfma(D, q, cmul(P, B));
}

// Adds the share of (A, B) conj (a, b) to a pair's sums (twice al and be; pair 0: the two self-paired bins' own).
__device__ __forceinline__ void pair_acc(float4& S, cplx A, cplx B, cplx a, cplx b, cplx w, bool self)
{
    cplx al = mk(S.x, S.y), be = mk(S.z, S.w);
    if (self) {
        al = mk(fmaf(A.x, a.x, fmaf(A.y, a.y, al.x)), fmaf(A.x, a.y, fmaf(A.y, a.x, al.y)));
        be = cfmac(B, b, be);
    } else {
        cplx r, q;
        pair_rot(a, b, w, r, q);
        al = cfmac(A, a, cfmac(B, b, al));
        be = cfmac(A, r, cfmac(B, q, be));
    }
    S = make_float4(al.x, al.y, be.x, be.y);
}

// A pair's sums, packed for the transform back.
__device__ __forceinline__ void pair_pack(float4 S, cplx w, bool self, cplx& A, cplx& B)
{
    if (self) { A = mk(S.x, S.y); B = mk(S.z, S.w); return; }
    const cplx al = mk(0.5f * S.x, 0.5f * S.y), be = mul_pos_i(cmul(mk(0.5f * S.z, 0.5f * S.w), conj(w)));
    A = cadd(al, be);
    B = csub(al, be);
}

// The kernel's entry from its own packed transform.  (1/M, which closes the way back, is not in the entries but in the
// stores behind it: a kernel of 1e-36, an ordinary fp32 number, would leave subnormal entries, with fewer bits the
// larger the transform: 8e-6 instead of 3e-7 of error in Z at 5000 steps, 1.5e-5 at 16384.)
__device__ __forceinline__ float4 pair_kernel(cplx A, cplx B, cplx w, bool self)
{
    if (self) return make_float4(A.x, A.y, B.x, B.y);
    const cplx D = cmul(w, mul_neg_i(mk(0.5f * (A.x - B.x), 0.5f * (A.y - B.y))));
    return make_float4(0.5f * (A.x + B.x), 0.5f * (A.y + B.y), D.x, D.y);
}

// One sequence of L <= M steps in registers: the pairs (x[2n], x[2n+1]) for n = tid + T i.  Only n < M/2 can lie
// inside the sequence, so half of a thread's M/T slots are enough.  A kernel that walks several sequences fetches the
// next one into these registers while the transforms of the current one run.
template <int M, int T, typename IO>
struct SeqRegs {
    static constexpr int HELD = M / T / 2;
    typename IoPair<IO>::raw_t r[HELD];
    // vec_ok: x sits on a pair boundary (rows of an even number of steps; a block of a longer row may hold an even
    // number of steps and still start on an odd element, so the blocked kernels pass the parity of the whole row)
    __device__ __forceinline__ void load(const IO* __restrict__ x, int L, int tid) { load(x, L, tid, (L & 1) == 0); }
    __device__ __forceinline__ void load(const IO* __restrict__ x, int L, int tid, bool vec_ok)
    {
        const __amdgpu_buffer_rsrc_t row = row_rsrc(x, L * (int)sizeof(IO));
        if (vec_ok && (L & 1) == 0) {
#pragma unroll
            for (int i = 0; i < HELD; ++i) r[i] = IoPair<IO>::load_pair(row, 2 * (tid + T * i) * (int)sizeof(IO));
        } else {
#pragma unroll
            for (int i = 0; i < HELD; ++i) r[i] = IoPair<IO>::load_single(row, 2 * (tid + T * i) * (int)sizeof(IO));
        }
    }
};

// x (one sequence of L <= M steps, in registers) as M floats, zeros beyond L, behind 32 steps of history, zeros at a
// sequence's start, so that no tap needs a bounds check.
// hist: null for a sequence's first step, else a pointer at the first of these L steps inside a longer row, whose 32
// predecessors are then the history.
constexpr int kHist = 32;
template <int M, int T, typename IO>
__device__ __forceinline__ void stage_raw(const SeqRegs<M, T, IO>& x, float* sx, int tid, const IO* __restrict__ hist)
{
    if (tid < kHist) sx[tid] = hist != nullptr ? (float)hist[tid - kHist] : 0.f;
#pragma unroll
    for (int i = 0; i < M / T / 2; ++i) {
        float v0, v1;
        IoPair<IO>::unpack(x.r[i], v0, v1);
        *reinterpret_cast<float2*>(sx + kHist + 2 * (tid + T * i)) = make_float2(v0, v1);
    }
}

// u = K_s x at a thread's steps.  Outputs t and t+1 share all but one of their inputs; x is read in aligned pairs
// (x[t-2p], x[t-2p+1]): x[t-2p+1] meets taps 2p (for t+1) and 2p-1 (for t), x[t-2p] meets taps 2p+1 (for t+1) and 2p (t).
// (steps beyond the sequence's end are worked out too, for the caller to drop: a branch around each read would keep the
// reads from being issued together)
template <int M, int T>
__device__ __forceinline__ void short_conv(const float* sx, const float* __restrict__ wc, int m, int tid,
                                           cplx (&z)[M / T / 2])
{
#pragma unroll
    for (int i = 0; i < M / T / 2; ++i) z[i] = mk(0.f, 0.f);
    for (int p = 0; 2 * p <= m; ++p) {
        const float w2p = 2 * p < m ? wc[2 * p] : 0.f, w2pm1 = p > 0 ? wc[2 * p - 1] : 0.f;
        const float w2pp1 = 2 * p + 1 < m ? wc[2 * p + 1] : 0.f;
#pragma unroll
        for (int i = 0; i < M / T / 2; ++i) {
            const float2 xv = *reinterpret_cast<const float2*>(sx + kHist + 2 * (tid + T * i) - 2 * p);
            z[i].y = fmaf(w2p, xv.y, fmaf(w2pp1, xv.x, z[i].y));
            z[i].x = fmaf(w2pm1, xv.y, fmaf(w2p, xv.x, z[i].x));
        }
    }
}

// x -> optional short kernel and activation (wc) -> packed complex z[n] = v[2n] + i v[2n+1] in registers, zero beyond L.
// With a short kernel a[] serves as staging room; it is free again (synchronised) at the end.
template <int M, int T, typename IO>
__device__ __forceinline__ void stage_input(const SeqRegs<M, T, IO>& x, const float* __restrict__ wc, int m, int L,
                                            cplx* a, int tid, cplx (&z)[M / T / 2], const IO* __restrict__ hist = nullptr)
{
    constexpr int HELD = M / T / 2;
    if (wc != nullptr) {
        float* sx = reinterpret_cast<float*>(a);
        stage_raw<M, T, IO>(x, sx, tid, hist);
        __syncthreads();
        short_conv<M, T>(sx, wc, m, tid, z);
#pragma unroll
        for (int i = 0; i < HELD; ++i) {
            const int t = 2 * (tid + T * i);
            z[i].x = t < L ? z[i].x * __builtin_amdgcn_rcpf(1.f + __expf(-z[i].x)) : 0.f;
            z[i].y = (t + 1 < L) ? z[i].y * __builtin_amdgcn_rcpf(1.f + __expf(-z[i].y)) : 0.f;
        }
        __syncthreads();
    } else {
#pragma unroll
        for (int i = 0; i < HELD; ++i) IoPair<IO>::unpack(x.r[i], z[i].x, z[i].y);
    }
}

// A thread's results out to y[t], t = 2 (tid + T i) < L.
template <int M, int T, typename OUT>
__device__ __forceinline__ void store_steps(const cplx (&v)[M / T / 2], OUT* __restrict__ y, int L, bool vec_ok, float scale,
                                            int tid)
{
    const __amdgpu_buffer_rsrc_t row = row_rsrc(y, L * (int)sizeof(OUT));
    const bool pairs = vec_ok && (L & 1) == 0;
#pragma unroll
    for (int i = 0; i < M / T / 2; ++i) {
        const int off = 2 * (tid + T * i) * (int)sizeof(OUT);
        if (pairs) IoPair<OUT>::store_pair(row, off, v[i].x * scale, v[i].y * scale);
        else IoPair<OUT>::store_single(row, off, v[i].x * scale, v[i].y * scale);
    }
}

// Sum over the four lanes of a quad, in all of them.
__device__ __forceinline__ float quad_sum(float v)
{
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xb1, 0xf, 0xf, true));   // [1,0,3,2]
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4e, 0xf, 0xf, true));   // [2,3,0,1]
    return v;
}

// What depends on the thread but not on the sequence (LDS addresses, bin positions, twiddles) is recomputed per sequence
// behind an opaque copy of the thread index: hoisted out of the loop over sequences it would fill the register file.
// Every stage takes a fresh copy, so that values shared between stages do not stay live in between.
__device__ __forceinline__ int fresh(int tid) { asm volatile("" : "+v"(tid)); return tid; }

// Kernel spectrum of one channel: the entries of the M/2 pairs in pair order (the buffer has room for one more).
// PAIRS: not the entries where they have fewer points than the copy (a launch of their own then, see conv_points).
// MX (M = 16384): also the copy that the matrix-core kernels read, the bins at exp(-2 pi i (k + 1/4) / M) (a transform of its
// own, of the sequence turned by exp(-2 pi i n / (4 M))), divided by 4 |k|_1, as half-precision (re, im) words, stored where
// the lane that holds bin k = k1 + 16 k2 + 512 k3 will look: word ((k1 * 4 + a) * 64 + lane) * 4 + b with lane = k2 + 32 h and
// k3 = 8 a + 4 h + b; scale[c] = 4 |k|_1 (both zero where 0.25 / |k|_1 is no finite number, below 7.4e-40); those kernels'
// tables are written by one workgroup more than there are channels where that has a compute unit to itself, else by the first
// channels' on the side (as one more it starts last: 768 channels 69 us, 63 without it and with the loads of the second transform in
// front of the first one's stores; a single channel 16, with the tables on its side 17).  Without the copy 768 channels take 42 us;
// fp32 I/O, which does not read it, pays for it all the same, because this call does not know what the spectrum is for (4 % of a
// fp32 training step of 2 x 768 x 16384).
template <int M, bool MX, bool PAIRS = true>
__global__ __launch_bounds__(conv_threads(M)) void longconv_spectrum_kernel(const float* __restrict__ k,
                                                                           float4* __restrict__ Kf,
                                                                           uint4* __restrict__ Ks,
                                                                           float* __restrict__ scale,
                                                                           MxTables* __restrict__ tables, int d, int L)
{
    static_assert(!MX || M == 16384, "the matrix-core kernels' transform has 2 x 16384 points");
    constexpr int T = conv_threads(M), NP = PairPos<M, T>::NP;
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    __shared__ float red[MX ? T / 64 : 1];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    const long c = blockIdx.x;
    if constexpr (MX) {
        if (c >= d) {
            for (int i = tid; i < MX_TABLE_STEPS; i += T) mx_write_tables(tables, i);
            return;
        }
    }
    SeqRegs<M, T, float> kr;
    kr.load(k + c * (long)L, L, tid);
    if constexpr (MX) {
        if ((int)gridDim.x == d)
            for (long i = c * T + tid; i < MX_TABLE_STEPS; i += (long)d * T) mx_write_tables(tables, (int)i);
    }
    build_tables<M, T>(tw, tid);
    cplx z[M / T / 2];
    stage_input<M, T, float>(kr, nullptr, 0, L, a, tid, z);
    if constexpr (MX) {
        float n1 = 0.f;
#pragma unroll
        for (int i = 0; i < M / T / 2; ++i) n1 += fabsf(z[i].x) + fabsf(z[i].y);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) n1 += __shfl_xor(n1, o);
        if ((tid & 63) == 0) red[tid >> 6] = n1;
    }
    __syncthreads();
    if constexpr (PAIRS) {
        fft_forward<M, T>(z, a, tw, tid);
        __syncthreads();
    }
    float inv = 0.f;
    if constexpr (MX) {
        float n1 = 0.f;
        for (int i = 0; i < T / 64; ++i) n1 += red[i];
        inv = n1 > 0.f ? 0.25f / n1 : 0.f;
        const bool nothing = inv > FLT_MAX;
        if (nothing) inv = 0.f;
        if (tid == 0) scale[c] = n1 > 0.f && !nothing ? 4.f * n1 : 0.f;
    }
    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
    auto half2 = [&](float re, float im) __attribute__((always_inline)) {
        f16x2 v;
        v[0] = (_Float16)(re * inv);
        v[1] = (_Float16)(im * inv);
        return __builtin_bit_cast(unsigned, v);
    };
    // the second transform's input: asked for in front of the stores (a load behind them comes back when they are done)
    float x2[MX ? M / T : 1];
    if constexpr (MX) {
        const __amdgpu_buffer_rsrc_t row = row_rsrc(k + c * (long)L, L * 4);
#pragma unroll
        for (int i = 0; i < M / T; ++i)
            x2[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(row, 4 * (tid + T * i), 0, 0));
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (PAIRS) {
        float4* out = Kf + c * (long)(M / 2 + 1);
        const PairPos<M, T> pos(tid);
        const PairTwiddle<M, T> pw(tid);
        cplx w = pw.first;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            out[tid + T * i] = pair_kernel(a[pos.first(i)], conj(a[pos.second(i)]), w, i == 0 && tid == 0);
            w = pw.after(i, w);
        }
    }
    if constexpr (MX) {
        // steps tid + T i this time, turned by exp(-2 pi i (tid + T i) / (4 M)), T i / (4 M) = i / 64
        cplx z2[M / T];
        float s, co;
        sincospif(-(float)tid / (float)(2 * M), &s, &co);
        cplx t = mk(co, s);
#pragma unroll
        for (int i = 0; i < M / T; ++i) {
            z2[i] = mk(x2[i] * t.x, x2[i] * t.y);
            t = cmul(t, mk(0.99518472667219693f, -0.098017140329560602f));
        }
        __syncthreads();                                            // a[] has been read out
        fft_forward<M, T, true>(z2, a, tw, tid);
        __syncthreads();
        uint4* dst = Ks + c * (long)(M / 4);
#pragma unroll
        for (int j = 0; j < M / 4 / T; ++j) {
            const int o = tid + T * j, ln = o & 63, k0 = (o >> 8) + 16 * (ln & 31) + 512 * (8 * ((o >> 6) & 3) + 4 * (ln >> 5));
            unsigned v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const cplx x = a[conv_pad(spectrum_pos<M>(k0 + 512 * i))];
                v[i] = half2(x.x, x.y);
            }
            dst[o] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    }
}

// Bound by vector instruction issue: 1785 instructions per wave and sequence of 4096 steps (2900 before the pairs became
// linear in the packed bins, their places constant offsets, the outer passes stayed in registers and the rows' ends were
// left to buffer loads and stores), issuing 92 .. 95 % of the time: 512 channels x 32 sequences, bf16, 320 -> 207 us.
// Workgroup g takes the sequences (b, c) = g, g + gridDim.x, ... of the B d in turn (w_short == nullptr: no short
// kernel and no activation, the plain long convolution).  The launch holds no more workgroups than are resident
// at once, so that the tables are built once per workgroup, a sequence's input is fetched while the inverse transform
// of the one before runs, and its kernel spectrum while the forward transform runs: with one workgroup per sequence
// each of those latencies was exposed once per sequence, since at the larger sizes a compute unit holds one
// workgroup only.
template <int M, typename IN, typename OUT>
__global__ __launch_bounds__(conv_threads(M)) __attribute__((amdgpu_waves_per_eu(4)))
void shortlong_conv_kernel(const IN* __restrict__ X,
                                                                        const float* __restrict__ w_short, int m,
                                                                        const float4* __restrict__ Kf,
                                                                        OUT* __restrict__ Y, int d, int L, long total)
{
    constexpr int T = conv_threads(M), NP = PairPos<M, T>::NP;
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    build_tables<M, T>(tw, tid);
    const PairPos<M, T> pos(tid);
    const PairTwiddle<M, T> pw(tid);
    SeqRegs<M, T, IN> xr;
    long bc = blockIdx.x;
    if (bc < total) xr.load(X + bc * (long)L, L, tid);
    for (; bc < total; bc += gridDim.x) {
        const int c = (int)(bc % d);
        int tp = fresh(tid);
        __syncthreads();        // the tables are built / the previous sequence has been read out of a[]
        cplx z[M / T / 2];
        stage_input<M, T, IN>(xr, w_short ? w_short + (long)c * m : nullptr, m, L, a, tp, z);
        const float4* Kc = Kf + (long)c * (M / 2 + 1);
        float4 kq[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) kq[i] = Kc[tp + T * i];
        tp = fresh(tid);
        fft_forward<M, T>(z, a, tw, tp);
        __syncthreads();
        cplx w = pw.first;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            cplx &p1 = a[pos.first(i)], &p2 = a[pos.second(i)];
            cplx A = p1, B = conj(p2);
            pair_mul<false>(A, B, w, kq[i], i == 0 && tid == 0);
            p1 = A;
            p2 = conj(B);
            w = pw.after(i, w);
        }
        if (bc + gridDim.x < total) xr.load(X + (bc + gridDim.x) * (long)L, L, tp);     // the next sequence, in flight
        __syncthreads();
        tp = fresh(tid);
        fft_inverse<M, T>(a, z, tw, tp);
        store_steps<M, T, OUT>(z, Y + bc * (long)L, L, (L & 1) == 0, 1.0f / (float)M, tp);
    }
}

// The long-stage gradients in one kernel: they share the spectrum of dZ.  One workgroup per channel walks the
// batch; per sequence it transforms dZ once, keeps the packed bins of its own bin pairs in registers, multiplies
// by the CONJUGATE kernel spectrum (correlation instead of convolution: dV[t] = sum_{s >= t} k[s - t] dZ[s]) and
// transforms back (out as DVT: dX itself when there is no short stage, fp32 scratch for the short-stage kernel, or on into
// the short stage below), then transforms v = silu(K_s x) (recomputed from x) and adds DZ conj(V) to the running sums of
// its bin pairs (in registers, at the two largest sizes in memory); after the last sequence the sums are transformed back once
// (dk).  Three transforms per sequence, where a correlation kernel and a kernel-gradient kernel of their own would need
// four.
// SPLIT: grid.y workgroups share a channel, each takes every grid.y-th sequence and leaves its sums in its own slice
// of the scratch array ([grid.y][d][M/2 + 1] pairs); longconv_dk_finish_kernel adds the slices up and transforms back.
// Used when there are too few channels to fill the GPU.
// SHORT: the short stage's gradient as well (m <= kFuseTaps): dV stays in registers, u = K_s x is there already for v,
// dU = dV silu'(u) meets its neighbours through LDS: dX out (dV is DVT = IO dX here), the taps' sums into `part`
// (dw itself; SPLIT: [d][grid.y][kShortMaxTaps], added up by longconv_dk_finish_kernel).  As a kernel of its own that stage reads
// x again, and dV, 4 bytes a step written here and read there, and works u out once more: 512 channels x 32 sequences of 4096 steps, bf16, the two kernels 527 + 150 us,
// in one 475, and 407 .. 416 with what came after (3080 instructions per wave and sequence, issuing 82 % of the time).
// bf16 I/O asks for three workgroups per compute unit (168 registers; values spilled: 30 with shared channels, 45 with one
// workgroup per channel, at M = 1024 31 and 48; training step 645 us against 707 with two and nothing spilled), fp32 I/O,
// which holds twice the fetched words, for two (234 against 262 us at 512 x 8 x 4000).
constexpr int kFuseTaps = kConvFuseTaps, kShortMaxTaps = kConvMaxTaps;

template <int M, typename IO, typename DVT, bool SPLIT, bool SHORT>
__global__ __launch_bounds__(conv_threads(M)) __attribute__((amdgpu_waves_per_eu(M == 256 || M >= 8192 ? 4 : sizeof(IO) == 2 ? 3 : 2)))
void longconv_bwd_kernel(const IO* __restrict__ X,
                                                                      const float* __restrict__ w_short, int m,
                                                                      const float4* __restrict__ Kf,
                                                                      const IO* __restrict__ dZ,
                                                                      DVT* __restrict__ dV, float* __restrict__ dk,
                                                                      float4* __restrict__ acc_ws, float* __restrict__ part,
                                                                      int B, int d, int L)
{
    constexpr int T = conv_threads(M), NP = PairPos<M, T>::NP, HELD = M / T / 2;
    // At the two largest sizes sixteen waves share the register file: the running sums then live in a scratch array in
    // memory ([d][M/2 + 1] pairs; every thread only ever touches its own pairs, between uses they sit in the caches).
    constexpr bool ACC_MEM = M >= 8192;
    float4* accm = (ACC_MEM || SPLIT) ? acc_ws + ((long)blockIdx.y * d + blockIdx.x) * (M / 2 + 1) : nullptr;
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    const int c = blockIdx.x;
    build_tables<M, T>(tw, tid);
    // the pairs' places and twiddles: worked out once, at the two largest sizes, where the six registers would be spilled ones,
    // wherever they are used
    auto stage_tid = [&]() __attribute__((always_inline)) { return ACC_MEM ? fresh(tid) : tid; };
    const float4* Kc = Kf + (long)c * (M / 2 + 1);
    const float* wc = w_short ? w_short + (long)c * m : nullptr;
    const bool vec_ok = (L & 1) == 0;
    const float scale = 1.0f / (float)M;
    float4 sums[ACC_MEM ? 1 : NP];
    cplx GA[NP], GB[NP], z[HELD];
    // the taps' sums: one slot per tap and four lanes, so that they take no registers
    __shared__ float taps[SHORT ? (kFuseTaps + 1) * (T / 4) : 1];
    if constexpr (!ACC_MEM) {
#pragma unroll
        for (int i = 0; i < NP; ++i) sums[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if constexpr (SHORT) {
        for (int x = tid; x < (kFuseTaps + 1) * (T / 4); x += T) taps[x] = 0.f;
    }

    // Inputs are fetched one stage ahead, into registers: dZ of the next sequence while v is transformed, x while the
    // correlation is transformed back.
    SeqRegs<M, T, IO> zr, xr;
    if ((int)blockIdx.y < B) zr.load(dZ + ((long)blockIdx.y * d + c) * L, L, tid);
    for (int b = blockIdx.y; b < B; b += gridDim.y) {
        const long row = ((long)b * d + c) * L;
        int tp = fresh(tid);
        // ---- spectrum of dZ; correlation with the kernel: DZ conj(K)
        stage_input<M, T, IO>(zr, nullptr, 0, L, a, tp, z);
        // the kernel's entries: in flight during the transform, at the two largest sizes, where they would spill, a few at a
        // time behind it
        constexpr int KU = ACC_MEM ? 4 : NP;
        float4 kq[KU];
        if constexpr (!ACC_MEM) {
#pragma unroll
            for (int i = 0; i < NP; ++i) kq[i] = Kc[tp + T * i];
        }
        __syncthreads();        // the tables are built / a[] has been read out
        fft_forward<M, T>(z, a, tw, tp);
        __syncthreads();
        tp = fresh(tid);
        xr.load(X + row, L, tp);
        {
            const int ts = stage_tid();
            const PairPos<M, T> pos(ts);
            const PairTwiddle<M, T> pw(ts);
#pragma unroll
            for (int i = 0; i < NP; ++i) { GA[i] = a[pos.first(i)]; GB[i] = conj(a[pos.second(i)]); }
            cplx w = pw.first;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if (ACC_MEM && i % KU == 0) {
#pragma unroll
                    for (int u = 0; u < KU; ++u) kq[u] = Kc[tp + T * (i + u)];
                }
                cplx A = GA[i], B = GB[i];
                pair_mul<true>(A, B, w, kq[i % KU], i == 0 && tid == 0);
                a[pos.first(i)] = A;
                a[pos.second(i)] = conj(B);
                w = pw.after(i, w);
                __builtin_amdgcn_sched_barrier(0);   // one pair at a time: the unrolled pairs must not pile up in registers
            }
        }
        __syncthreads();
        tp = fresh(tid);
        fft_inverse<M, T>(a, z, tw, tp);
        tp = fresh(tid);
        if constexpr (SHORT) {
            float* sx = reinterpret_cast<float*>(a);
            float* su = sx + kHist + M;              // dU, zeros beyond L
            cplx u[HELD];
            __syncthreads();                         // a[] has been read out
            stage_raw<M, T, IO>(xr, sx, tp, nullptr);
            if (tp < kHist) su[M + tp] = 0.f;
            __syncthreads();
            short_conv<M, T>(sx, wc, m, tp, u);
#pragma unroll
            for (int i = 0; i < HELD; ++i) {
                const int t = 2 * (tp + T * i);
                const float s0 = __builtin_amdgcn_rcpf(1.f + __expf(-u[i].x)), s1 = __builtin_amdgcn_rcpf(1.f + __expf(-u[i].y));
                const bool two = t + 1 < L;
                // (silu'(u) times 1/M, which is a power of two, at the cost of silu'(u))
                z[i].x = t < L ? z[i].x * s0 * fmaf(u[i].x, fmaf(-scale, s0, scale), scale) : 0.f;
                z[i].y = two ? z[i].y * s1 * fmaf(u[i].y, fmaf(-scale, s1, scale), scale) : 0.f;
                *reinterpret_cast<float2*>(su + t) = make_float2(z[i].x, z[i].y);
                u[i].x = t < L ? u[i].x * s0 : 0.f;
                u[i].y = two ? u[i].y * s1 : 0.f;
            }
            __syncthreads();
            // dX[t] = sum_j w[j] dU[t + j], shares of dw[j] = sum_t dU[t] x[t - j], in aligned pairs as in short_conv
            cplx dx[HELD];
#pragma unroll
            for (int i = 0; i < HELD; ++i) dx[i] = mk(0.f, 0.f);
            for (int p = 0; 2 * p <= m; ++p) {
                const bool ev = 2 * p < m, above = 2 * p + 1 < m;
                const float w2p = ev ? wc[2 * p] : 0.f, w2pm1 = p > 0 ? wc[2 * p - 1] : 0.f;
                const float w2pp1 = above ? wc[2 * p + 1] : 0.f;
                float ta = 0.f, tb = 0.f, tc = 0.f;          // taps 2p - 1, 2p, 2p + 1
                constexpr int U = HELD < 4 ? HELD : 4;       // steps read together
#pragma unroll
                for (int i0 = 0; i0 < HELD; i0 += U) {
                    float2 dv[U], xv[U];
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        const int t = 2 * (tp + T * (i0 + q));
                        dv[q] = *reinterpret_cast<const float2*>(su + t + 2 * p);
                        xv[q] = *reinterpret_cast<const float2*>(sx + kHist + t - 2 * p);
                    }
                    if (p > 0) {
#pragma unroll
                        for (int q = 0; q < U; ++q) {
                            dx[i0 + q].y = fmaf(w2pm1, dv[q].x, dx[i0 + q].y);
                            ta = fmaf(z[i0 + q].x, xv[q].y, ta);
                        }
                    }
                    if (ev) {
#pragma unroll
                        for (int q = 0; q < U; ++q) {
                            cplx& o = dx[i0 + q];
                            o = mk(fmaf(w2p, dv[q].x, o.x), fmaf(w2p, dv[q].y, o.y));
                            tb = fmaf(z[i0 + q].x, xv[q].x, fmaf(z[i0 + q].y, xv[q].y, tb));
                        }
                    }
                    if (above) {
#pragma unroll
                        for (int q = 0; q < U; ++q) {
                            dx[i0 + q].x = fmaf(w2pp1, dv[q].y, dx[i0 + q].x);
                            tc = fmaf(z[i0 + q].y, xv[q].x, tc);
                        }
                    }
                }
                ta = quad_sum(ta);
                tb = quad_sum(tb);
                tc = quad_sum(tc);
                if ((tp & 3) == 0) {
                    float* o = taps + tp / 4;
                    if (p > 0) o[(2 * p - 1) * (T / 4)] += ta;
                    o[2 * p * (T / 4)] += tb;
                    if (above) o[(2 * p + 1) * (T / 4)] += tc;
                }
            }
            store_steps<M, T, DVT>(dx, dV + row, L, vec_ok, 1.0f, tp);
#pragma unroll
            for (int i = 0; i < HELD; ++i) z[i] = u[i];
        } else {
            store_steps<M, T, DVT>(z, dV + row, L, vec_ok, scale, tp);
            if (wc != nullptr) __syncthreads();      // a[] has been read out
            // ---- v = silu(K_s x) (x itself without a short stage)
            stage_input<M, T, IO>(xr, wc, m, L, a, tp, z);
        }
        if (b + (int)gridDim.y < B) zr.load(dZ + ((long)(b + gridDim.y) * d + c) * L, L, tp);
        __syncthreads();
        tp = fresh(tid);
        // ---- its spectrum; running sums of DZ conj(V)
        fft_forward<M, T>(z, a, tw, tp);
        __syncthreads();
        {
            const int ts = stage_tid();
            const PairPos<M, T> pos(ts);
            const PairTwiddle<M, T> pw(ts);
            cplx w = pw.first;
            constexpr int U = NP < 4 ? NP : 4;       // pairs read together
#pragma unroll
            for (int i0 = 0; i0 < NP; i0 += U) {
                cplx A[U], Bc[U];
#pragma unroll
                for (int u = 0; u < U; ++u) { A[u] = a[pos.first(i0 + u)]; Bc[u] = conj(a[pos.second(i0 + u)]); }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = i0 + u;
                    const bool self = i == 0 && tid == 0;
                    if constexpr (ACC_MEM) {
                        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (b != (int)blockIdx.y) t = accm[tid + T * i];
                        pair_acc(t, GA[i], GB[i], A[u], Bc[u], w, self);
                        accm[tid + T * i] = t;
                    } else {
                        pair_acc(sums[i], GA[i], GB[i], A[u], Bc[u], w, self);
                    }
                    w = pw.after(i, w);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
    }
    if constexpr (SHORT) {
        // this workgroup's tap sums (a barrier has passed since the last was added)
        for (int j = tid / 64; j < m; j += T / 64) {
            float v = 0.f;
            for (int x = tid & 63; x < T / 4; x += 64) v += taps[j * (T / 4) + x];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if ((tid & 63) == 0) part[((long)c * gridDim.y + blockIdx.y) * (SPLIT ? kShortMaxTaps : m) + j] = v;
        }
    }
    if constexpr (SPLIT) {
        // this workgroup's share of the sums stays in its slice of the scratch array (it is there already when the
        // sums were kept in memory)
        if constexpr (!ACC_MEM) {
#pragma unroll
            for (int i = 0; i < NP; ++i) accm[tid + T * i] = sums[i];
        }
        return;
    }
    {
        const int ts = stage_tid();
        const PairPos<M, T> pos(ts);
        const PairTwiddle<M, T> pw(ts);
        cplx w = pw.first;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            float4 t;
            if constexpr (ACC_MEM) t = B > 0 ? accm[tid + T * i] : make_float4(0.f, 0.f, 0.f, 0.f);
            else t = sums[i];
            cplx A, Bc;
            pair_pack(t, w, i == 0 && tid == 0, A, Bc);
            a[pos.first(i)] = A;
            a[pos.second(i)] = conj(Bc);
            w = pw.after(i, w);
        }
    }
    __syncthreads();
    fft_inverse<M, T>(a, z, tw, tid);
    store_steps<M, T, float>(z, dk + (long)c * L, L, vec_ok, scale, tid);
}

// Gradient through the activation and the short kernel, where the transform kernel does not work it out itself.  dV is the
// gradient with respect to v = silu(u), u = K_s x:
//   dU = dV silu'(u),  dX[t] = sum_j w[j] dU[t+j],  dw[c][j] = sum_b sum_t dU[b,c,t] x[b,c,t-j].
// Up to 16 taps (the paper's sizes, 3 and 2 log10 L + 1, stay below that for any L up to 10^7): every wave for itself, no
// LDS and no barrier.  A lane holds 8 consecutive steps; x's history it reads along (a line its neighbour reads too), dU
// ahead it gets from the next lanes' registers, so that the last one or two lanes of a strip only supply: 63 (62) x 8 steps
// per strip.  A wave walks kStripsPerWave strips of a channel, the next strip's loads in flight.  Each workgroup leaves its
// share of the tap sums in `part` ([d][n_share][kShortMaxTaps]); shortconv_dw_kernel adds the shares of a channel in a fixed
// order.  TAPS: the number of taps, the tap loops are as long as the kernel needs.
// 4 x 768 sequences of 16384 steps, bf16, 9 taps (403 MB): 86 us; staged through LDS by 2048 steps, x twice and dU once
// with two-way bank conflicts and three barriers, 117; with branches around plain loads 97.
constexpr int kStripsPerWave = 8;
__host__ __device__ constexpr int strip_steps(int taps) { return (64 - (taps + 6) / 8) * 8; }

// Eight consecutive elements as they sit in memory.
template <typename IO> struct Raw8 {
    static constexpr int NR = sizeof(IO) / 2;
    uint4 r[NR];
    // Steps t .. t + 7 of a row of L (a multiple of 8, as t is: whole or empty), zero outside it.  Buffer loads: the bounds
    // check is theirs, where branches around plain loads cost a third of the kernel's instructions in selects and copies.
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t row, int t)
    {
#pragma unroll
        for (int k = 0; k < NR; ++k)
            r[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(row, t * (int)sizeof(IO) + 16 * k, 0, 0));
    }
    // Any L >= 8, t a multiple of 8: one access, aligned to an element only, from within the row, which stands for steps t .. t + 7 where
    // all of them lie in it; the piece with the row's end in it step by step (one lane of a row's last strip).  Pieces
    // outside are whatever the row holds: valid() says which to drop, where they are used, so that nothing waits for the loads here.
    __device__ __forceinline__ void load(const IO* __restrict__ x, int t, int L)
    {
        __builtin_memcpy(r, x + max(0, min(t, L - 8)), sizeof(r));
        if (t < L && t + 8 > L) {
            IO v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = t + e < L ? x[t + e] : (IO)0.f;
            __builtin_memcpy(r, v, sizeof(v));
        }
    }
    static __device__ __forceinline__ bool valid(int t, int L) { return t >= 0 && t < L; }
    __device__ __forceinline__ void unpack(float* v) const
    {
        if constexpr (sizeof(IO) == 2) {
            const unsigned w[4] = {r[0].x, r[0].y, r[0].z, r[0].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[2 * e] = __builtin_bit_cast(float, w[e] << 16);
                v[2 * e + 1] = __builtin_bit_cast(float, w[e] & 0xffff0000u);
            }
        } else {
            __builtin_memcpy(v, r, 32);
        }
    }
};

__device__ __forceinline__ float from_next_lane(float v)        // lane i: the value of lane i + 1 (lane 63: anything)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, false));
}

// VEC: L is a multiple of 8 (every row starts on a 16-byte boundary).  Other rows (longer than 4096 steps, like all that come here) move
// in 16-byte pieces just the same, aligned to their elements only: step by step they took three times as long as whole ones, 10 x 512 x 4591,
// fp32, 173 us, now 72; 4 x 768 x 8190, bf16, 121, now 57.
template <typename IO, int TAPS, bool VEC>
__global__ __launch_bounds__(256) void shortconv_bwd_kernel(const IO* __restrict__ X, const float* __restrict__ w_short,
                                                           const float* __restrict__ dV, IO* __restrict__ dX,
                                                           float* __restrict__ part, int B, int d, int L, int n_share)
{
    constexpr int AHEAD = (TAPS + 6) / 8, STEPS = strip_steps(TAPS);      // lanes that supply; steps of a strip
    constexpr int NH = AHEAD;                                             // pieces of 8 steps of history
    __shared__ float red[TAPS][4];
    const int tid = threadIdx.x, lane = tid & 63, c = blockIdx.x % d, share = blockIdx.x / d;      // channels fastest
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per_row = (L + STEPS - 1) / STEPS, n_items = B * per_row;
    float acc[TAPS];
#pragma unroll
    for (int j = 0; j < TAPS; ++j) acc[j] = 0.f;
    Raw8<IO> xr[NH + 1];
    Raw8<float> gr;
    auto fetch = [&](int item) __attribute__((always_inline)) {
        const int b = item / per_row, t = (item - b * per_row) * STEPS + 8 * lane;
        const long row = ((long)b * d + c) * L;
        if constexpr (VEC) {
            const __amdgpu_buffer_rsrc_t rx = row_rsrc(X + row, L * (int)sizeof(IO)), rg = row_rsrc(dV + row, L * 4);
#pragma unroll
            for (int k = 0; k <= NH; ++k) xr[k].load(rx, t - 8 * (NH - k));
            gr.load(rg, t);
        } else {
#pragma unroll
            for (int k = 0; k <= NH; ++k) xr[k].load(X + row, t - 8 * (NH - k), L);
            gr.load(dV + row, t, L);
        }
    };
    const int first = (share * 4 + w) * kStripsPerWave, last = min(first + kStripsPerWave, n_items);
    if (first < last) fetch(first);
    for (int item = first; item < last; ++item) {
        const int b = item / per_row, t = (item - b * per_row) * STEPS + 8 * lane;
        float x[8 * (NH + 1)], g[8], du[8 * (AHEAD + 1)];
#pragma unroll
        for (int k = 0; k <= NH; ++k) {
            xr[k].unpack(x + 8 * k);
            if constexpr (!VEC) {
                const bool in = Raw8<IO>::valid(t - 8 * (NH - k), L);
#pragma unroll
                for (int e = 0; e < 8; ++e) x[8 * k + e] = in ? x[8 * k + e] : 0.f;
            }
        }
        gr.unpack(g);
        if (item + 1 < last) fetch(item + 1);
        float wj[TAPS];
#pragma unroll
        for (int j = 0; j < TAPS; ++j) wj[j] = w_short[(long)c * TAPS + j];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float u = 0.f;
#pragma unroll
            for (int j = 0; j < TAPS; ++j) u = fmaf(wj[j], x[8 * NH + e - j], u);
            const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-u));
            du[e] = t + (VEC ? 0 : e) < L ? g[e] * sg * (1.f + u * (1.f - sg)) : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8 * AHEAD; ++e) du[8 + e] = from_next_lane(du[e]);
        if (lane < 64 - AHEAD) {
            float dx[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v = 0.f;
#pragma unroll
                for (int j = 0; j < TAPS; ++j) {
                    v = fmaf(wj[j], du[e + j], v);
                    acc[j] = fmaf(du[e], x[8 * NH + e - j], acc[j]);
                }
                dx[e] = v;
            }
            IO* y = dX + ((long)b * d + c) * L + t;
            if constexpr (VEC) { if (t < L) store8(y, dx); }
            else if (t + 8 <= L) {
                IO v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (IO)dx[e];
                __builtin_memcpy(y, v, sizeof(v));
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) if (t + e < L) y[e] = (IO)dx[e];
            }
        }
    }
    // this workgroup's tap sums: wave reduction, then across the four waves
#pragma unroll
    for (int j = 0; j < TAPS; ++j) {
        float v = acc[j];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) red[j][w] = v;
    }
    __syncthreads();
    if (tid < TAPS)
        part[((long)c * n_share + share) * kShortMaxTaps + tid] = red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
}

// More taps (m <= 32): the (batch entry, tile of TL steps) pairs of a channel are dealt out to workgroups in runs of
// kShortTilesPerWg (a run may cross from one sequence into the next); x is staged with MT steps of history and dU with MT
// steps of look-ahead.
constexpr int kShortTile = 2048, kShortTilesPerWg = 4;

template <typename IO>
__global__ __launch_bounds__(256) void shortconv_bwd_staged_kernel(const IO* __restrict__ X, const float* __restrict__ w_short,
                                                           int m, const float* __restrict__ dV, IO* __restrict__ dX,
                                                           float* __restrict__ part, int B, int d, int L, int n_share)
{
    constexpr int TL = kShortTile, TAPS = kShortMaxTaps, MT = TAPS, H = MT;  // H: halo on either side
    constexpr int NX = MT + 8;                                        // inputs behind eight consecutive outputs
    __shared__ __attribute__((aligned(16))) float sx[TL + 2 * H];      // x[t0 - H .. t0 + TL + H)
    __shared__ __attribute__((aligned(16))) float su[TL + H + 8];      // dU[t0 .. t0 + TL + H) (+ slack for 16-byte reads)
    __shared__ float red[MT][4];
    const int tid = threadIdx.x, c = blockIdx.x % d, share = blockIdx.x / d;      // channels fastest
    const int tiles_per_row = (L + TL - 1) / TL, n_items = B * tiles_per_row;
    float wreg[TAPS], acc[TAPS];
#pragma unroll
    for (int j = 0; j < TAPS; ++j) { wreg[j] = j < m ? w_short[(long)c * m + j] : 0.f; acc[j] = 0.f; }
    const bool vec8 = (L & 7) == 0;       // every row starts 16-byte aligned
    for (int item = share * kShortTilesPerWg; item < (share + 1) * kShortTilesPerWg && item < n_items; ++item) {
    const int b = item / tiles_per_row, t0 = (item - b * tiles_per_row) * TL;
    const long row = ((long)b * d + c) * L;
    __syncthreads();
    for (int i8 = tid; i8 < (TL + 2 * H) / 8; i8 += 256) {      // eight steps per thread: one 16-byte load where whole
        const int t = t0 - H + 8 * i8;
        float xv[8];
        if (vec8 && t >= 0 && t + 8 <= L) load8(X + row + t, xv);
        else {
#pragma unroll
            for (int e = 0; e < 8; ++e) xv[e] = (t + e >= 0 && t + e < L) ? (float)X[row + t + e] : 0.f;
        }
        *reinterpret_cast<float4*>(sx + 8 * i8) = make_float4(xv[0], xv[1], xv[2], xv[3]);
        *reinterpret_cast<float4*>(sx + 8 * i8 + 4) = make_float4(xv[4], xv[5], xv[6], xv[7]);
    }
    __syncthreads();
    // each thread takes 8 consecutive steps: the MT + 8 inputs they need are read once, as 16-byte LDS reads
    {
        const int i0 = 8 * tid;                         // TL = 8 * 256
        float xs[NX];                                   // x[t0 + i0 - MT .. t0 + i0 + 8)
#pragma unroll
        for (int r = 0; r < NX / 4; ++r) {
            const float4 v = *reinterpret_cast<const float4*>(sx + i0 + 4 * r);      // sx index of x[t0 + i] is H + i
            xs[4 * r] = v.x; xs[4 * r + 1] = v.y; xs[4 * r + 2] = v.z; xs[4 * r + 3] = v.w;
        }
        float du8[8], g8[8];
        const int tc = t0 + i0;
        const bool whole = vec8 && tc + 8 <= L;         // eight steps in range at a 16-byte aligned address
        if (whole) {
            const float4 a0 = *reinterpret_cast<const float4*>(dV + row + tc), a1 = *reinterpret_cast<const float4*>(dV + row + tc + 4);
            g8[0] = a0.x; g8[1] = a0.y; g8[2] = a0.z; g8[3] = a0.w; g8[4] = a1.x; g8[5] = a1.y; g8[6] = a1.z; g8[7] = a1.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) g8[e] = tc + e < L ? dV[row + tc + e] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float u = 0.f;
#pragma unroll
            for (int j = 0; j < TAPS; ++j) u = fmaf(wreg[j], xs[MT + e - j], u);
            const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-u));
            du8[e] = tc + e < L ? g8[e] * sg * (1.f + u * (1.f - sg)) : 0.f;
        }
        *reinterpret_cast<float4*>(su + i0) = make_float4(du8[0], du8[1], du8[2], du8[3]);
        *reinterpret_cast<float4*>(su + i0 + 4) = make_float4(du8[4], du8[5], du8[6], du8[7]);
    }
    if (tid < H) {
        // the H steps of look-ahead beyond the tile, one per thread (as two more 8-step pieces they would double the
        // first wave's share of this phase)
        const int i = TL + tid, t = t0 + i;
        float u = 0.f;
#pragma unroll
        for (int j = 0; j < TAPS; ++j) u = fmaf(wreg[j], sx[H + i - j], u);
        const float sg = __builtin_amdgcn_rcpf(1.f + __expf(-u));
        su[i] = t < L ? dV[row + t] * sg * (1.f + u * (1.f - sg)) : 0.f;
    }
    __syncthreads();
    {
        const int i0 = 8 * tid;                         // TL = 8 * 256
        float xs[NX], ds[NX];                           // x as above; dU[t0 + i0 .. t0 + i0 + MT + 8)
#pragma unroll
        for (int r = 0; r < NX / 4; ++r) {
            const float4 v = *reinterpret_cast<const float4*>(sx + i0 + 4 * r);
            xs[4 * r] = v.x; xs[4 * r + 1] = v.y; xs[4 * r + 2] = v.z; xs[4 * r + 3] = v.w;
            const float4 g = *reinterpret_cast<const float4*>(su + i0 + 4 * r);
            ds[4 * r] = g.x; ds[4 * r + 1] = g.y; ds[4 * r + 2] = g.z; ds[4 * r + 3] = g.w;
        }
        float dx8[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float dx = 0.f;
#pragma unroll
            for (int j = 0; j < TAPS; ++j) {
                dx = fmaf(wreg[j], ds[e + j], dx);
                acc[j] = fmaf(ds[e], xs[MT + e - j], acc[j]);
            }
            dx8[e] = dx;
        }
        const int tc = t0 + i0;
        if (vec8 && tc + 8 <= L) store8(dX + row + tc, dx8);
        else {
#pragma unroll
            for (int e = 0; e < 8; ++e) if (tc + e < L) dX[row + tc + e] = (IO)dx8[e];
        }
    }
    }
    // this workgroup's tap sums: wave reduction, then across the four waves
#pragma unroll
    for (int j = 0; j < TAPS; ++j) {
        float v = acc[j];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if ((tid & 63) == 0) red[j][tid >> 6] = v;
    }
    __syncthreads();
    if (tid < TAPS)
        part[((long)c * n_share + share) * kShortMaxTaps + tid] = red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
}

__global__ __launch_bounds__(64) void shortconv_dw_kernel(const float* __restrict__ part, float* __restrict__ dw, int m,
                                                         int n_share)
{
    const int c = blockIdx.x, j = threadIdx.x;
    if (j >= m) return;
    float t = 0.f;
    for (int s = 0; s < n_share; ++s) t += part[((long)c * n_share + s) * kShortMaxTaps + j];
    dw[(long)c * m + j] = t;
}


// =============================================================================================== sequences beyond one transform
// L > 16384: the sequence and the long kernel are cut into blocks of BK = 16384 steps, x_0 .. x_{nb-1} and
// k_0 .. k_{nb-1}.  Output block j of the causal sum is
//     y_j = sum_{i <= j}  low half of  circ_{2 BK}( [x_i ; 0] , [k_{j-i} ; k_{j-i-1}] )          (k_{-1} = 0)
// (the taps that reach from block i into block j are the 2 BK - 1 taps around lag (j - i) BK: the upper half of the
// second operand holds the ones below that lag, which a circular product of length 2 BK wraps onto the low outputs
// exactly where they belong).  So every block is transformed by the same length-M machinery as a short sequence
// (zero upper half in, low half out), the sum over i is taken on the spectra, in registers, and one inverse
// transform per output block follows.  The spectrum of [k_m ; k_{m-1}] is A_m + (-1)^bin A_{m-1} with A_m the
// spectrum of [k_m ; 0] (a shift by half the period), which is what longconv_spectrum_blocked_kernel stores:
// [d][nb][M/2 + 1] pairs in pair order.  The two long-stage gradients have the same shape:
//     dv_i = sum_{j >= i} low half of the circular CORRELATION of [dz_j ; 0] with [k_{j-i} ; k_{j-i-1}]   (conjugate spectra),
//     dk_m = low half of the inverse of  D_m + (-1)^bin D_{m+1},   D_m = sum_b sum_i DZ_{i+m} conj(V_i).
// The work per sequence grows with nb (nb + 1) / 2 block pairs, against nb log nb for one long transform held in
// memory: this path is here so that no length is refused, not to be the fastest way to convolve a million steps.
constexpr int kBlkM = 16384;                 // transform length and block length (steps)
// Threads per workgroup of the blocked kernels.  1024 leave each thread 128 registers, which hold the accumulators since
// the bin pairs' places are no longer kept across the transforms (up to 3 values spilled).  When they did not (40 to 70
// spilled), 512 threads with 256 registers each were slower all the same (2.39 against 1.94 ms at B1 d2048 L65536; now
// 1.15): sixteen waves hide the transforms' LDS latencies better than eight.
constexpr int kBlkT = conv_threads(kBlkM);

// Spectra G_m of the blocks of the long kernel; one workgroup per (channel, block).
__global__ __launch_bounds__(kBlkT) void longconv_spectrum_blocked_kernel(const float* __restrict__ k,
                                                                                       float4* __restrict__ Gf, int L,
                                                                                       int nb)
{
    constexpr int M = kBlkM, T = kBlkT, NP = PairPos<M, T>::NP;
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    const long c = blockIdx.x;
    const int mb = blockIdx.y;
    const bool row_vec = (L & 1) == 0;
    build_tables<M, T>(tw, tid);
    const PairPos<M, T> pos(tid);
    const PairTwiddle<M, T> pw(tid);
    // the block before sits in the upper half of the period: (-1)^bin (a thread's bins, k and M - k, all have one parity)
    const float odd = (pair_bin<M>(tid) & 1) ? -1.f : 1.f;
    float4 sum[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) sum[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int which = (mb > 0 ? mb - 1 : mb); which <= mb; ++which) {
        const int len = min(M, L - which * M);
        SeqRegs<M, T, float> kr;
        kr.load(k + c * (long)L + (long)which * M, len, tid, row_vec);
        cplx z[M / T / 2];
        stage_input<M, T, float>(kr, nullptr, 0, len, a, tid, z);
        __syncthreads();                  // tables built / the block before has been read out of a[]
        fft_forward<M, T>(z, a, tw, tid);
        __syncthreads();
        const float sg = which < mb ? odd : 1.f;
        cplx w = pw.first;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float4 v = pair_kernel(a[pos.first(i)], conj(a[pos.second(i)]), w, i == 0 && tid == 0);
            sum[i].x += sg * v.x; sum[i].y += sg * v.y; sum[i].z += sg * v.z; sum[i].w += sg * v.w;
            w = pw.after(i, w);
        }
    }
    float4* out = Gf + (c * nb + mb) * (long)(M / 2 + 1);
#pragma unroll
    for (int i = 0; i < NP; ++i) out[tid + T * i] = sum[i];
}

// Forward (CORR = false: X -> optional short kernel and activation -> causal sum with the long kernel, block `blk` of
// the output from the blocks 0 .. blk of the input) and correlation (CORR = true: dZ -> dV, block blk from the blocks
// blk .. nb-1, conjugate spectra; no short stage).  Work items (sequence, output block), the costliest blocks first,
// dealt to a launch of no more workgroups than are resident at once.
template <typename IN, typename OUT, bool CORR>
__global__ __launch_bounds__(kBlkT) void longconv_blocked_kernel(const IN* __restrict__ X,
                                                                              const float* __restrict__ w_short, int m,
                                                                              const float4* __restrict__ Gf,
                                                                              OUT* __restrict__ Y, int d, int L, int nb,
                                                                              long BD)
{
    constexpr int M = kBlkM, T = kBlkT, NP = PairPos<M, T>::NP;
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    const bool row_vec = (L & 1) == 0;
    build_tables<M, T>(tw, tid);
    const PairPos<M, T> pos(tid);
    const PairTwiddle<M, T> pw(tid);
    const long items = BD * nb;
    for (long id = blockIdx.x; id < items; id += gridDim.x) {
        const int r = (int)(id / BD);
        const long bc = id - (long)r * BD;
        const int blk = CORR ? r : nb - 1 - r;            // costliest first: nb - blk (CORR) or blk + 1 input blocks
        const int c = (int)(bc % d);
        const int o0 = CORR ? blk : 0, o1 = CORR ? nb - 1 : blk;
        const IN* xrow = X + bc * (long)L;
        const float* wc = (!CORR && w_short) ? w_short + (long)c * m : nullptr;
        cplx accA[NP], accB[NP];                            // sums over the input blocks of X_o G_|o - blk|, packed
#pragma unroll
        for (int i = 0; i < NP; ++i) { accA[i] = mk(0.f, 0.f); accB[i] = mk(0.f, 0.f); }
        SeqRegs<M, T, IN> xr;
        cplx z[M / T / 2];
        xr.load(xrow + (long)o0 * M, min(M, L - o0 * M), tid, row_vec);
        for (int o = o0; o <= o1; ++o) {
            int tp = fresh(tid);
            __syncthreads();    // tables built / a[] has been read out
            stage_input<M, T, IN>(xr, wc, m, min(M, L - o * M), a, tp, z, (wc && o > 0) ? xrow + (long)o * M : nullptr);
            if (o < o1) xr.load(xrow + (long)(o + 1) * M, min(M, L - (o + 1) * M), tp, row_vec);   // the next block, in flight
            tp = fresh(tid);
            fft_forward<M, T>(z, a, tw, tp);
            __syncthreads();
            tp = fresh(tid);
            const float4* Gc = Gf + ((long)c * nb + (CORR ? o - blk : blk - o)) * (long)(M / 2 + 1);
            float4 kq[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) kq[i] = Gc[tp + T * i];
            cplx w = pw.first;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                cplx A = a[pos.first(i)], B = conj(a[pos.second(i)]);
                pair_mul<CORR>(A, B, w, kq[i], i == 0 && tid == 0);
                accA[i] = cadd(accA[i], A);
                accB[i] = cadd(accB[i], B);
                w = pw.after(i, w);
                __builtin_amdgcn_sched_barrier(0);   // one pair at a time: the unrolled pairs must not pile up in registers
            }
        }
        __syncthreads();        // every thread has read its bins of the last input block
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            a[pos.first(i)] = accA[i];
            a[pos.second(i)] = conj(accB[i]);
        }
        __syncthreads();
        const int tp = fresh(tid);
        fft_inverse<M, T>(a, z, tw, tp);
        store_steps<M, T, OUT>(z, Y + bc * (long)L + (long)blk * M, min(M, L - blk * M), row_vec, 1.0f / (float)M, tp);
    }
}

// Sums D_mb = sum_b sum_i DZ_{i+mb} conj(V_i) of one channel and one block distance, kept in memory ([d][nb][M/2 + 1]
// pairs; every thread only ever touches its own pairs).  One workgroup per (channel, distance), the distances with
// the most block pairs first.
template <typename IO>
__global__ __launch_bounds__(kBlkT) void longconv_dk_blocked_kernel(const IO* __restrict__ X,
                                                                                 const float* __restrict__ w_short, int m,
                                                                                 const IO* __restrict__ dZ,
                                                                                 float4* __restrict__ acc_ws, int B, int d,
                                                                                 int L, int nb)
{
    constexpr int M = kBlkM, T = kBlkT, NP = PairPos<M, T>::NP;
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    const int c = blockIdx.x, mb = blockIdx.y;
    const bool row_vec = (L & 1) == 0;
    build_tables<M, T>(tw, tid);
    float4* accm = acc_ws + ((long)c * nb + mb) * (long)(M / 2 + 1);
    const float* wc = w_short ? w_short + (long)c * m : nullptr;
    const int n_i = nb - mb;                     // block pairs (i, i + mb) per sequence
    const long n_pairs = (long)B * n_i;
    cplx GA[NP], GB[NP], z[M / T / 2];
    SeqRegs<M, T, IO> zr, xr;
    zr.load(dZ + (long)c * L + (long)mb * M, min(M, L - mb * M), tid, row_vec);      // pair 0: b = 0, i = 0
    for (long pr = 0; pr < n_pairs; ++pr) {
        const int b = (int)(pr / n_i), i = (int)(pr - (long)b * n_i), j = i + mb;
        const long row = ((long)b * d + c) * (long)L;
        int tp = fresh(tid);
        stage_input<M, T, IO>(zr, nullptr, 0, min(M, L - j * M), a, tp, z);
        xr.load(X + row + (long)i * M, min(M, L - i * M), tp, row_vec);
        __syncthreads();        // tables built / a[] has been read out
        fft_forward<M, T>(z, a, tw, tp);
        __syncthreads();
        {
            const PairPos<M, T> pos(fresh(tid));
#pragma unroll
            for (int q = 0; q < NP; ++q) { GA[q] = a[pos.first(q)]; GB[q] = conj(a[pos.second(q)]); }
        }
        __syncthreads();
        tp = fresh(tid);
        stage_input<M, T, IO>(xr, wc, m, min(M, L - i * M), a, tp, z, (wc && i > 0) ? X + row + (long)i * M : nullptr);
        if (pr + 1 < n_pairs) {
            const int b2 = (int)((pr + 1) / n_i), i2 = (int)(pr + 1 - (long)b2 * n_i);
            zr.load(dZ + ((long)b2 * d + c) * (long)L + (long)(i2 + mb) * M, min(M, L - (i2 + mb) * M), tp, row_vec);
        }
        tp = fresh(tid);
        fft_forward<M, T>(z, a, tw, tp);
        __syncthreads();
        tp = fresh(tid);
        const PairPos<M, T> pos(tp);
        const PairTwiddle<M, T> pw(tp);
        cplx w = pw.first;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
            if (pr > 0) t = accm[tid + T * q];
            pair_acc(t, GA[q], GB[q], a[pos.first(q)], conj(a[pos.second(q)]), w, q == 0 && tid == 0);
            accm[tid + T * q] = t;
            w = pw.after(i, w);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// dk block mb of a channel from the sums above: inverse of D_mb + (-1)^bin D_{mb+1}, low half.
__global__ __launch_bounds__(kBlkT) void longconv_dk_blocked_finish_kernel(const float4* __restrict__ acc_ws,
                                                                                        float* __restrict__ dk, int d,
                                                                                        int L, int nb)
{
    constexpr int M = kBlkM, T = kBlkT;
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    const int c = blockIdx.x, mb = blockIdx.y;
    build_tables<M, T>(tw, tid);
    const float4* D0 = acc_ws + ((long)c * nb + mb) * (long)(M / 2 + 1);
    const float4* D1 = mb + 1 < nb ? D0 + (M / 2 + 1) : nullptr;
    const PairPos<M, T> pos(tid);
    const PairTwiddle<M, T> pw(tid);
    const float odd = (pair_bin<M>(tid) & 1) ? -1.f : 1.f;
    cplx w = pw.first;
#pragma unroll
    for (int i = 0; i < PairPos<M, T>::NP; ++i) {
        float4 t = D0[tid + T * i];
        if (D1 != nullptr) {
            const float4 o = D1[tid + T * i];
            t.x += odd * o.x; t.y += odd * o.y; t.z += odd * o.z; t.w += odd * o.w;
        }
        cplx A, B;
        pair_pack(t, w, i == 0 && tid == 0, A, B);
        a[pos.first(i)] = A;
        a[pos.second(i)] = conj(B);
        w = pw.after(i, w);
    }
    __syncthreads();
    cplx z[M / T / 2];
    fft_inverse<M, T>(a, z, tw, tid);
    store_steps<M, T, float>(z, dk + (long)c * L + (long)mb * M, min(M, L - mb * M), (L & 1) == 0, 1.0f / (float)M, tid);
}

// Between the powers of four from 1024 on the size in the middle as well: half the work for half of all lengths.  Training steps, us:
// 32 x 512 x 2048, bf16, in 4096 points 622, in 2048 312; 16 x 256 x 1874 195, 104; 8 x 768 x 1500, fp32, 291, 162; 10 x 512 x 4591,
// fp32, in 16384 points 1205, in 8192 715; 2 x 128 x 4652, bf16, 94, 68; 4 x 768 x 8192, fp32, 777, 470.  (512 points would have 32
// threads' worth of 16-point transforms, and cost a wave what 1024 do.)
int conv_points(int L)
{
    return L > 1024 && L <= 2048 ? 2048 : L > 4096 && L <= 8192 ? 8192 : conv_fft_size(L);
}

int conv_fft_size(int L)
{
    if (L <= 256) return 256;
    if (L <= 1024) return 1024;
    if (L <= 4096) return 4096;
    if (L <= 16384) return 16384;
    return 0;
}

hipError_t launch_longconv_spectrum(const float* k, void* Kf, int d, int L, hipStream_t st)
{
    const int M = conv_points(L);
    ProfScope prof(KID_CONV_SPECTRUM, st);
    float4* out = (float4*)Kf;
    if (const int nb = conv_blocks(L)) {
        hipLaunchKernelGGL(longconv_spectrum_blocked_kernel, dim3(d, nb), dim3(kBlkT), 0, st, k, out, L, nb);
        return hipGetLastError();
    }
    uint4* mx = (uint4*)((char*)Kf + conv_pairs_bytes(d, L));
    float* scale = (float*)(mx + (size_t)d * (MX_N / 4));
    MxTables* tables = mx_tables(mx, d);
    const bool copy = L > 4096 && (L & 7) == 0;       // (rows of other lengths never meet the matrix-core kernels)
#define CHELA_SPECTRUM(M_, ...)                                                                                         \
    hipLaunchKernelGGL((longconv_spectrum_kernel<M_, __VA_ARGS__>), grid, dim3(conv_threads(M_)), 0, st, k, out, mx, scale, tables, d, L)
    if (copy && M == 8192) {
        const dim3 grid(d + (d < 256 ? 1 : 0));
        CHELA_SPECTRUM(16384, true, false);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const dim3 grid(d + (copy && M == 16384 && d < 256 ? 1 : 0));
    switch (M) {
        case 256: CHELA_SPECTRUM(256, false); break;
        case 1024: CHELA_SPECTRUM(1024, false); break;
        case 2048: CHELA_SPECTRUM(2048, false); break;
        case 4096: CHELA_SPECTRUM(4096, false); break;
        case 8192: CHELA_SPECTRUM(8192, false); break;
        case 16384:
            if (copy) CHELA_SPECTRUM(16384, true);
            else CHELA_SPECTRUM(16384, false);
            break;
        default: return hipErrorInvalidValue;
    }
#undef CHELA_SPECTRUM
    return hipGetLastError();
}

// Workgroups of `kernel` that the GPU holds at once (what its LDS and registers allow per compute unit x the units).
template <typename K>
static long resident_workgroups(K kernel, int threads)
{
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    (void)hipGetLastError();
    return (long)cus * per_cu;
}

// The blocked kernel for L > 16384: work items (sequence, output block) over no more workgroups than are resident.
template <typename IN, typename OUT, bool CORR>
static hipError_t conv_blocked_launch(const IN* X, const float* w, int m, const float4* Gf, OUT* Y, long BD, int d, int L,
                                      hipStream_t st)
{
    const int nb = conv_blocks(L);
    static const long slots = resident_workgroups(longconv_blocked_kernel<IN, OUT, CORR>, kBlkT);
    const long items = BD * nb;
    const dim3 grid((unsigned)(items < slots ? items : slots));
    hipLaunchKernelGGL((longconv_blocked_kernel<IN, OUT, CORR>), grid, dim3(kBlkT), 0, st, X, w, m, Gf, Y, d,
                       L, nb, BD);
    return hipGetLastError();
}

template <typename IN, typename OUT>
static hipError_t conv_dispatch(const IN* X, const float* w, int m, const float4* Kf, OUT* Y, long BD, int d, int L,
                                hipStream_t st)
{
    const int M = conv_points(L);
    ProfScope prof(KID_CONV_FWD, st);
    if (conv_blocks(L)) return conv_blocked_launch<IN, OUT, false>(X, w, m, Kf, Y, BD, d, L, st);
    // no more workgroups than are resident at once, each with an equal share of the sequences
#define CHELA_CONV_FWD(M_)                                                                                              \
    case M_: {                                                                                                          \
        static const long slots = resident_workgroups(shortlong_conv_kernel<M_, IN, OUT>, conv_threads(M_));            \
        const long rounds = (BD + slots - 1) / slots;                                                                   \
        const dim3 grid((unsigned)((BD + rounds - 1) / rounds));                                                        \
        hipLaunchKernelGGL((shortlong_conv_kernel<M_, IN, OUT>), grid, dim3(conv_threads(M_)), 0, st, X, w, m, Kf, Y, d, \
                           L, BD);                                                                                      \
    } break;
    switch (M) {
        CHELA_CONV_FWD(256) CHELA_CONV_FWD(1024) CHELA_CONV_FWD(2048) CHELA_CONV_FWD(4096) CHELA_CONV_FWD(8192) CHELA_CONV_FWD(16384)
        default: return hipErrorInvalidValue;
    }
#undef CHELA_CONV_FWD
    return hipGetLastError();
}

hipError_t launch_shortlong_conv(const void* X, const float* w_short, int m, const void* Kf, void* Y, long BD, int d,
                                 int L, int dtype, hipStream_t st)
{
    if (dtype == 0)
        return conv_dispatch<bf16, bf16>((const bf16*)X, w_short, m, (const float4*)Kf, (bf16*)Y, BD, d, L, st);
    return conv_dispatch<float, float>((const float*)X, w_short, m, (const float4*)Kf, (float*)Y, BD, d, L, st);
}

// Second step of the split long-stage gradient: add up the G slices of a channel's sums, transform back, store dk.  dw (may be
// null): the tap sums' shares part_w[d][G][kShortMaxTaps] as well; with a launch of its own for them 128 channels x 3 sequences
// of 1000 steps took 25.3 us, so 23.7 (512 x 1 x 4096, whose kernel writes dw itself: 28.4, 26.1; 32 x 512 x 4096: 423.5, 422.3).
template <int M>
__global__ __launch_bounds__(conv_threads(M)) void longconv_dk_finish_kernel(const float4* __restrict__ part,
                                                                            float* __restrict__ dk, int G, int d, int L,
                                                                            const float* __restrict__ part_w,
                                                                            float* __restrict__ dw, int m)
{
    constexpr int T = conv_threads(M);
    __shared__ __attribute__((aligned(16))) unsigned char lds[ConvLds<M>::BYTES];
    cplx* a = reinterpret_cast<cplx*>(lds);
    float4* tw = reinterpret_cast<float4*>(a + ConvLds<M>::DATA);
    const int tid = threadIdx.x;
    const int c = blockIdx.x;
    if (M <= 4096 && dw != nullptr && tid < m) {        // (beyond, the short stage is not part of the kernel in front)
        float t = 0.f;
        for (int g = 0; g < G; ++g) t += part_w[((long)c * G + g) * kShortMaxTaps + tid];
        dw[(long)c * m + tid] = t;
    }
    build_tables<M, T>(tw, tid);
    constexpr int NP = PairPos<M, T>::NP;
    // (slice by slice, all of a thread's pairs of U slices in flight together; pair by pair, every read waited for the one before:
    // 17 x 256 channels x 448 steps, fp32, 44 us of a training step of 108, now 14; the call of 32 x 512 x 4096, bf16, 421 -> 416)
    constexpr int U = 2;
    float4 sum[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) sum[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    const float4* slice = part + (long)c * (M / 2 + 1) + tid;
    for (int g = 0; g < G; g += U) {       // fixed order: deterministic
        float4 o[U][NP];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < NP; ++i)
                o[u][i] = g + u < G ? slice[(long)(g + u) * d * (M / 2 + 1) + T * i] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < NP; ++i) { sum[i].x += o[u][i].x; sum[i].y += o[u][i].y; sum[i].z += o[u][i].z; sum[i].w += o[u][i].w; }
    }
    const PairPos<M, T> pos(tid);
    const PairTwiddle<M, T> pw(tid);
    cplx w = pw.first;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const float4 t = sum[i];
        cplx A, B;
        pair_pack(t, w, i == 0 && tid == 0, A, B);
        a[pos.first(i)] = A;
        a[pos.second(i)] = conj(B);
        w = pw.after(i, w);
    }
    __syncthreads();
    cplx z[M / T / 2];
    fft_inverse<M, T>(a, z, tw, tid);
    store_steps<M, T, float>(z, dk + (long)c * L, L, (L & 1) == 0, 1.0f / (float)M, tid);
}

// SHORT: the short stage's gradient in the same kernel (dV is dX then, `part` is scratch for the tap sums of shared channels).
template <typename IO, typename DVT, bool SHORT>
static hipError_t conv_longbwd_dispatch(const IO* X, const float* w, int m, const float4* Kf, const IO* dZ, DVT* dV,
                                        float* dk, float* dw, float4* acc_ws, float* part, int B, int d, int L, hipStream_t st)
{
    const int M = conv_points(L), G = conv_bwd_groups(B, d, L);
    ProfScope prof(KID_CONV_LONG_BWD, st);
    if (const int nb = conv_blocks(L)) {
        // dV block by block (correlation with the kernel's blocks), then the sums of the kernel gradient per block
        // distance and their way back
        hipError_t e = conv_blocked_launch<IO, DVT, true>(dZ, nullptr, 0, Kf, dV, (long)B * d, d, L, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((longconv_dk_blocked_kernel<IO>), dim3(d, nb), dim3(kBlkT), 0, st, X, w, m, dZ,
                           acc_ws, B, d, L, nb);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(longconv_dk_blocked_finish_kernel, dim3(d, nb), dim3(kBlkT), 0, st, acc_ws, dk, d,
                           L, nb);
        return hipGetLastError();
    }
    const dim3 grid(d, G);
#define CHELA_LONGBWD(M_, SHORT_)                                                                                       \
    case M_:                                                                                                            \
        if (G > 1) {                                                                                                    \
            hipLaunchKernelGGL((longconv_bwd_kernel<M_, IO, DVT, true, SHORT_>), grid, dim3(conv_threads(M_)), 0, st, X, w, \
                               m, Kf, dZ, dV, dk, acc_ws, part, B, d, L);                                               \
            hipLaunchKernelGGL((longconv_dk_finish_kernel<M_>), dim3(d), dim3(conv_threads(M_)), 0, st, acc_ws, dk, G, d, L, \
                               part, SHORT_ ? dw : nullptr, m);                                                         \
        } else                                                                                                          \
            hipLaunchKernelGGL((longconv_bwd_kernel<M_, IO, DVT, false, SHORT_>), grid, dim3(conv_threads(M_)), 0, st, X, w, \
                               m, Kf, dZ, dV, dk, acc_ws, dw, B, d, L);                                                 \
        break;
    switch (M) {
        CHELA_LONGBWD(256, SHORT) CHELA_LONGBWD(1024, SHORT) CHELA_LONGBWD(2048, SHORT) CHELA_LONGBWD(4096, SHORT)
        CHELA_LONGBWD(8192, false) CHELA_LONGBWD(16384, false)
        default: return hipErrorInvalidValue;
    }
#undef CHELA_LONGBWD
    return hipGetLastError();
}

// ws: conv_bwd_ws_floats() floats, laid out as said there.
template <typename IO>
static hipError_t conv_bwd_impl(const IO* X, const float* w_short, int m, const float4* Kf, const IO* dZ, IO* dX,
                                float* dw, float* dk, float* ws, int B, int d, int L, hipStream_t st)
{
    hipError_t e;
    const long BD = (long)B * d;
    float4* acc_ws = reinterpret_cast<float4*>(ws);
    ws += conv_bwd_acc_floats(B, d, L, sizeof(IO) == 2);
    // bf16 I/O at the lengths the matrix-core kernels serve: its own copy of the spectrum lies behind the pairs
    const bool mx = sizeof(IO) == 2 && convmx_applies(L, 0);
    const void* mx_spec = (const char*)Kf + conv_pairs_bytes(d, L);
    if (w_short == nullptr) { // no short stage: v = x and dX is the correlation of dZ with the long kernel itself
        if (mx) return launch_convmx_longbwd(X, nullptr, 0, mx_spec, dZ, dX, nullptr, dk, (float*)acc_ws, nullptr, B, d, L, st);
        return conv_longbwd_dispatch<IO, IO, false>(X, nullptr, 0, Kf, dZ, dX, dk, nullptr, acc_ws, nullptr, B, d, L, st);
    }
    if (conv_bwd_fused(m, L))
        return conv_longbwd_dispatch<IO, IO, true>(X, w_short, m, Kf, dZ, dX, dk, dw, acc_ws, ws, B, d, L, st);
    if (mx && convmx_bwd_short(m, B, d, L))
        return launch_convmx_longbwd(X, w_short, m, mx_spec, dZ, dX, dw, dk, (float*)acc_ws, ws, B, d, L, st);
    float* ws_dV = ws;
    float* ws_part = ws + (size_t)BD * L;                                   // [d][n_share][32] (room for [d][B * tiles][32])
    // workgroups per channel: (batch entry, strip) or (batch entry, tile) pairs over what one takes
    const bool strips = m <= 16;
    const long n_items = (long)B * (strips ? (L + strip_steps(m) - 1) / strip_steps(m) : (L + kShortTile - 1) / kShortTile);
    const long per_wg = strips ? 4 * kStripsPerWave : kShortTilesPerWg;
    const int n_share = (int)((n_items + per_wg - 1) / per_wg);
    if ((long)d * n_share > 0x7fffffffL || n_items > 0x7ffffff0L) return hipErrorInvalidValue;
    e = mx ? launch_convmx_longbwd(X, w_short, m, mx_spec, dZ, ws_dV, nullptr, dk, (float*)acc_ws, nullptr, B, d, L, st)
           : conv_longbwd_dispatch<IO, float, false>(X, w_short, m, Kf, dZ, ws_dV, dk, nullptr, acc_ws, nullptr, B, d, L, st);
    if (e != hipSuccess) return e;
    {
        ProfScope prof(KID_CONV_SHORT_BWD, st);
        const dim3 grid((unsigned)((long)d * n_share));
        // one instantiation per tap count: the tap loops are most of this kernel's instructions
#define CHELA_SHORT_BWD(T_)                                                                                             \
    case T_:                                                                                                            \
        if ((L & 7) == 0)                                                                                               \
            hipLaunchKernelGGL((shortconv_bwd_kernel<IO, T_, true>), grid, dim3(256), 0, st, X, w_short, ws_dV, dX, ws_part, \
                               B, d, L, n_share);                                                                       \
        else                                                                                                            \
            hipLaunchKernelGGL((shortconv_bwd_kernel<IO, T_, false>), grid, dim3(256), 0, st, X, w_short, ws_dV, dX, ws_part, \
                               B, d, L, n_share);                                                                       \
        break;
        switch (m) {
            CHELA_SHORT_BWD(1) CHELA_SHORT_BWD(2) CHELA_SHORT_BWD(3) CHELA_SHORT_BWD(4) CHELA_SHORT_BWD(5) CHELA_SHORT_BWD(6)
            CHELA_SHORT_BWD(7) CHELA_SHORT_BWD(8) CHELA_SHORT_BWD(9) CHELA_SHORT_BWD(10) CHELA_SHORT_BWD(11)
            CHELA_SHORT_BWD(12) CHELA_SHORT_BWD(13) CHELA_SHORT_BWD(14) CHELA_SHORT_BWD(15) CHELA_SHORT_BWD(16)
            default:
                if (m < 17 || m > kShortMaxTaps) return hipErrorInvalidValue;
                hipLaunchKernelGGL((shortconv_bwd_staged_kernel<IO>), grid, dim3(256), 0, st, X, w_short, m, ws_dV, dX, ws_part,
                                   B, d, L, n_share);
        }
#undef CHELA_SHORT_BWD
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(shortconv_dw_kernel, dim3(d), dim3(64), 0, st, ws_part, dw, m, n_share);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// Backward of Z = K_l(silu(K_s X)): dX (I/O dtype), dw [d][m] (with a short kernel, m <= 32), dk [d][L] fp32.
hipError_t launch_shortlong_conv_bwd(const void* X, const float* w_short, int m, const void* Kf, const void* dZ,
                                     void* dX, float* dw, float* dk, float* ws, int B, int d, int L, int dtype,
                                     hipStream_t st)
{
    const float4* K = (const float4*)Kf;
    if (dtype == 0)
        return conv_bwd_impl<bf16>((const bf16*)X, w_short, m, K, (const bf16*)dZ, (bf16*)dX, dw, dk, ws, B, d, L, st);
    return conv_bwd_impl<float>((const float*)X, w_short, m, K, (const float*)dZ, (float*)dX, dw, dk, ws, B, d, L, st);
}

}  // namespace chela
