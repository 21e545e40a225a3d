// fp32 kernels: causal linear attention with fp32 I/O and fp32 accuracy on the bf16 matrix instruction
// v_mfma_f32_32x32x16_bf16 (the path exists for accuracy, the bf16 path for speed).  Also the state scan and the copy probe
// shared by both paths.
//
// Structure (Sec. 4.1): a (b,h) sequence is cut into segments; within a segment one workgroup walks the
// chunks in order with the d_k x d_v state S in accumulator registers.  Per chunk: masked left product
// P = (Q K^T) o M, O = P V + Q S (both parts summed in the same accumulators), then S += K^T V.  Segment start
// states come from a pre-pass (segment totals of K^T V), added up by the sweeps or by a scan.
//
// Arithmetic.  Every operand (tiles, scores, published state) is three bf16 parts that together hold all of its 24 bits, and
// a product is the six products of parts that matter, each exact, summed in fp32: 6 x 32 cycles of the matrix pipe for 16
// steps of a 32 x 32 tile where the fp32 instruction takes 512.  Values that three parts do not hold are met with the fp32
// instruction itself (Hard).  Errors against 64 bits, 24 x 3001 tokens, 64 x 64: O 4.95e-7 with the fp32 instruction, now
// 1.1e-7, gradients 2.6e-7, now 1.1e-7; lower over 9 shapes of 64 to 262000 tokens x 4 state sizes x 9 distributions (of
// either sign, positive, constant), by a sixth where the difference is smallest.  What bounds it: instruction issue --
// splitting a value takes 5.5 vector instructions, looking at it 1.5 -- and, with the GPU full, power (1.5 .. 2.1
// GHz).  Measured, us, fp32 instruction -> three parts: 24 x 3001, 64 x 64: forward 51.8 -> 40.3, backward 94 -> 77; 64 x
// 4096, 64 x 64: 109 -> 91, 284 -> 239; 24 x 3001, 128 x 128: 127 -> 108, 343 -> 277; 16 x 400, 64 x 64: 39 -> 11.2, 41 ->
// 19.0 (of these two 25 are the plan's).
// Two halves in fp16 would be half the instructions, but 22 bits, and a token 2^30 louder than its chunk would cost the
// others theirs.
#include "chela_internal.h"

namespace chela {

// ------------------------------------------------------------------------------------------------ scan
// states[z][bh][seg][e] (z = 0 .. n_arrays-1, arrays `array_stride` floats apart), one thread per (z, bh, 4 e's),
// serial over the (few) segments, coalesced over e.  The loads of U segments are issued before the first add so that
// one memory round trip serves U segments.
// An optional carried-in state seeds the running sum of array z: init[z] is [rows][cols] fp32 per head; if
// init_cols > 0 the array itself is stored transposed ([cols][rows], cols = init_cols... see below) and the seed is
// read transposed: element e = a * init_cols + b of the array takes init[b * (elems / init_cols) + a].
struct ScanModes { int mode[2]; const float* init[2]; };

__global__ __launch_bounds__(256) void scan_states_kernel(float* __restrict__ st, size_t array_stride, int n_seg,
                                                         int elems, ScanModes modes, int init_cols)
{
    const long bh = blockIdx.x;     // heads on grid.x: its limit is 2^31-1, the others' 65535
    const int z = blockIdx.z;
    const int mode = modes.mode[z];
    const int e = (blockIdx.y * 256 + threadIdx.x) * 4;
    if (e >= elems) return;
    float* p = st + (size_t)z * array_stride + (size_t)bh * n_seg * elems + e;
    float4 run = make_float4(0.f, 0.f, 0.f, 0.f);
    if (modes.init[z] != nullptr) {
        const float* in = modes.init[z] + (size_t)bh * elems;
        if (init_cols > 0) {
            const int a = e / init_cols, b = e % init_cols, rows = elems / init_cols;   // 4 consecutive b, one a
            run = make_float4(in[(size_t)b * rows + a], in[(size_t)(b + 1) * rows + a], in[(size_t)(b + 2) * rows + a],
                              in[(size_t)(b + 3) * rows + a]);
        } else {
            run = *reinterpret_cast<const float4*>(in + e);
        }
    }
    constexpr int U = 16;                      // segments in flight per thread
    const bool suffix = (mode == SCAN_EXCL_SUFFIX);
    for (int s0 = 0; s0 < n_seg; s0 += U) {
        float4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u;
            const int idx = suffix ? (n_seg - 1 - s) : s;
            v[u] = s < n_seg ? *reinterpret_cast<const float4*>(p + (size_t)idx * elems) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u;
            if (s < n_seg) {
                const int idx = suffix ? (n_seg - 1 - s) : s;
                float4* dst = reinterpret_cast<float4*>(p + (size_t)idx * elems);
                if (mode == SCAN_INCL_PREFIX) {
                    run.x += v[u].x; run.y += v[u].y; run.z += v[u].z; run.w += v[u].w;
                    *dst = run;
                } else {
                    *dst = run;
                    run.x += v[u].x; run.y += v[u].y; run.z += v[u].z; run.w += v[u].w;
                }
            }
        }
    }
}

hipError_t scan_states(float* states, size_t array_stride, int n_arrays, const int* modes, const float* const* init,
                       int init_cols, long BH, int n_seg, int elems, hipStream_t st)
{
    ScanModes m{};
    for (int z = 0; z < n_arrays && z < 2; ++z) { m.mode[z] = modes[z]; m.init[z] = init ? init[z] : nullptr; }
    dim3 grid((unsigned)BH, (elems / 4 + 255) / 256, n_arrays);
    ProfScope prof(KID_SCAN, st);
    hipLaunchKernelGGL(scan_states_kernel, grid, dim3(256), 0, st, states, array_stride, n_seg, elems, m, init_cols);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ copy probe
// Grid-stride 16-byte copy: the plain streaming kernel that byte counters are calibrated against.
__global__ __launch_bounds__(256) void copy_probe_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n)
{
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t st)
{
    const size_t n = bytes / 16;
    size_t blocks = (n + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    ProfScope prof(KID_COPY, st);
    hipLaunchKernelGGL(copy_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const uint4*)src, (uint4*)dst, n);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------ stream probe
// NI arrays read and NO arrays written, element i of every array by the same thread, grid-stride, 16 bytes per
// access: the friendliest kernel there is for a given mix of read and write streams.  What it reaches is the
// bandwidth this GPU actually delivers for that mix, the yardstick for kernels that move the same mix.
struct StreamArgs {
    const uint4* in[4];
    uint4* out[4];
};

template <int NI, int NO>
__global__ __launch_bounds__(256) void stream_probe_kernel(StreamArgs a, size_t n)
{
    // Array k is walked from a different starting point (wrapping round): arrays allocated at equal distances would
    // otherwise put all streams of a thread on the same memory channel at the same time.
    const size_t stride = (size_t)gridDim.x * 256;
    const size_t rot = n > 65536 ? 4099 : 0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
        uint4 v[NI];
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            size_t j = i + k * rot;
            if (j >= n) j -= n;
            v[k] = a.in[k][j];
        }
        uint4 x = v[0];
#pragma unroll
        for (int k = 1; k < NI; ++k) { x.x ^= v[k].x; x.y ^= v[k].y; x.z ^= v[k].z; x.w ^= v[k].w; }
#pragma unroll
        for (int k = 0; k < NO; ++k) {
            size_t j = i + (NI + k) * rot;
            if (j >= n) j -= n;
            a.out[k][j] = x;
            x.x += 1u;
        }
        // nothing to write (a read-only mix): a store the compiler cannot rule out keeps the loads alive; the probe's
        // inputs never hold the pattern, so nothing is ever stored (the address is the thread's own element of input 0)
        if (NO == 0 && (x.x ^ x.y) == 0x9e3779b9u && x.z == 0x7f4a7c15u) const_cast<uint4*>(a.in[0])[i] = x;
    }
}

template <int NI>
static hipError_t stream_dispatch(const StreamArgs& a, int n_out, size_t n, dim3 grid, hipStream_t st)
{
    switch (n_out) {
    case 0: hipLaunchKernelGGL((stream_probe_kernel<NI, 0>), grid, dim3(256), 0, st, a, n); break;
    case 1: hipLaunchKernelGGL((stream_probe_kernel<NI, 1>), grid, dim3(256), 0, st, a, n); break;
    case 2: hipLaunchKernelGGL((stream_probe_kernel<NI, 2>), grid, dim3(256), 0, st, a, n); break;
    case 3: hipLaunchKernelGGL((stream_probe_kernel<NI, 3>), grid, dim3(256), 0, st, a, n); break;
    case 4: hipLaunchKernelGGL((stream_probe_kernel<NI, 4>), grid, dim3(256), 0, st, a, n); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Zero `n` floats.  Used instead of hipMemsetAsync so that every call of the library can be captured into a HIP graph
// (memset nodes have replayed wrongly on this platform).
__global__ __launch_bounds__(256) void zero_fill_kernel(float* __restrict__ p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = 0.f;
}

hipError_t launch_zero_fill(float* p, size_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_stream_probe(const void* const* in, int n_in, void* const* out, int n_out, size_t bytes, hipStream_t st)
{
    StreamArgs a{};
    for (int k = 0; k < n_in; ++k) a.in[k] = (const uint4*)in[k];
    for (int k = 0; k < n_out; ++k) a.out[k] = (uint4*)out[k];
    const size_t n = bytes / 16;
    size_t blocks = (n + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    const dim3 grid((unsigned)blocks);
    ProfScope prof(KID_STREAM_PROBE, st);
    switch (n_in) {
    case 1: return stream_dispatch<1>(a, n_out, n, grid, st);
    case 2: return stream_dispatch<2>(a, n_out, n, grid, st);
    case 3: return stream_dispatch<3>(a, n_out, n, grid, st);
    case 4: return stream_dispatch<4>(a, n_out, n, grid, st);
    default: return hipErrorInvalidValue;
    }
}

typedef __attribute__((ext_vector_type(16))) float f32x16;

// ------------------------------------------------------------------------------------------------ matrix-core probe
// Nothing but v_mfma_f32_32x32x16_bf16 on registers: every wave keeps four independent accumulator tiles going, so
// that an instruction never waits for the one before it, `iters` rounds of four.  What this reaches is the matrix
// rate the GPU actually delivers (clock included), the yardstick next to the published 2.5 PFLOP/s.
typedef __attribute__((ext_vector_type(8))) __bf16 probe_bf16x8;

__global__ __launch_bounds__(256) void mfma_probe_kernel(float* __restrict__ out, int iters)
{
    const int lane = threadIdx.x & 63;
    probe_bf16x8 a, b;
#pragma unroll
    for (int e = 0; e < 8; ++e) { a[e] = (__bf16)(1.0f / (1 + ((lane + e) & 7))); b[e] = (__bf16)(0.25f * ((lane ^ e) & 3)); }
    f32x16 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[q], 0, 0, 0);
    }
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) t += acc[q][e];
    out[(size_t)blockIdx.x * 256 + threadIdx.x] = t;          // keeps the arithmetic alive
}

// `out` holds blocks * 256 floats; each of the blocks * 4 waves issues iters * 16 matrix instructions of 32768 FLOP.
hipError_t launch_mfma_probe(float* out, int blocks, int iters, hipStream_t st)
{
    ProfScope prof(KID_MFMA_PROBE, st);
    hipLaunchKernelGGL(mfma_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, st, out, iters);
    return hipGetLastError();
}

__device__ __forceinline__ f32x16 zero16f()
{
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}

// ------------------------------------------------------------------------------------------------ three bf16 parts
typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

// Two fp32 values as the sums of three bf16 ones, packed in pairs (first value in the low half), each part the remainder before it
// rounded to nearest: |m| <= 2^-8 |x|, |l| <= 2^-17 |x|, and what is behind l is nothing, because the remainders are exact and 15 and 6
// bits wide: h + m + l is the value, where it is none of those that Hard looks out for.
struct Pair3 { unsigned h, m, l; };
template <bool NEG = false>
__device__ __forceinline__ unsigned cvt_pk_bf16(float lo, float hi)      // round to nearest even
{
    // (written out: the compiler would convert the low half a second time where its value is wanted as a float again)
    unsigned d;
    if (NEG) asm("v_cvt_pk_bf16_f32 %0, -%1, -%2" : "=v"(d) : "v"(lo), "v"(hi));
    else asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(d) : "v"(lo), "v"(hi));
    return d;
}
// NEG: of -x0 and -x1, in no more instructions.
template <bool NEG = false>
__device__ __forceinline__ Pair3 split_pair(float x0, float x1)
{
    const unsigned h = cvt_pk_bf16<NEG>(x0, x1);
    if (NEG) { x0 = -x0; x1 = -x1; }
    const float r0 = x0 - __builtin_bit_cast(float, h << 16), r1 = x1 - __builtin_bit_cast(float, h & 0xffff0000u);
    const unsigned m = cvt_pk_bf16(r0, r1);
    const unsigned l = cvt_pk_bf16(r0 - __builtin_bit_cast(float, m << 16), r1 - __builtin_bit_cast(float, m & 0xffff0000u));
    return {h, m, l};
}

// What three parts cannot hold: values that are not zero and below 2^-110 (their last bits lie below the smallest bf16 value,
// 2^-133), infinities, and values that round to one as bf16.  The first are looked for among all operands (three vector
// instructions on two values: twice the bits, less those of 2^-110, wrap round to more than a zero's); the others leave
// a NaN or an infinity in every result they reach, so it is enough to look at the results.  A workgroup that met
// any of them does its segment over with the fp32 instruction, which takes every value as it is: 24 x 3001 tokens with a small
// query in every row, 64 x 64, forward and backward, 292 us instead of 118.  Looking costs 3 to 4 % of a call (two instructions fewer per
// pair, where no zero is near, and a branch: no gain).
struct Hard {
    static constexpr unsigned kLeast = 2u * 0x08800000u;
    enum { kBad = 1, kTiny = 2 };
    unsigned tiny = 0u;
    float bad = 0.f;
    __device__ __forceinline__ void operands(float x, float y)
    {
        tiny = max(tiny, max((__builtin_bit_cast(unsigned, x) << 1) - kLeast, (__builtin_bit_cast(unsigned, y) << 1) - kLeast));
        asm("" : "+v"(tiny));       // (opaque: as one maximum over all of a tile the terms would all be worked out before the first is used)
    }
    __device__ __forceinline__ void result(float x) { bad = fmaf(x, 0.f, bad); }
    // What any of the workgroup's lanes met.  votes: four words of LDS that nothing else uses.
    __device__ __forceinline__ int anywhere(int* votes, int w, int lane) const
    {
        const int mine = (__any(tiny > 0u - kLeast) ? kTiny : 0) | (__any(!(bad == 0.f)) ? kBad : 0);
        if (lane == 0) votes[w] = mine;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(votes[0] | votes[1] | votes[2] | votes[3]);
    }
    // Of a result and what it was at first: without small operands a finite one was right, and keeps its bits.
    static __device__ __forceinline__ float choose(int met, float again, float first) { return met & kTiny || !(first - first == 0.f) ? again : first; }
};

// An operand of the 32x32x16 instruction in its three parts.
struct Op3 { bf16x8 h, m, l; };

// A B with six products of parts, the leading ones and the others in sums of their own: those, below 2^-8 of them, then round 2^-8
// finer.  A product of two parts is exact in fp32.  What is left out (m l, l m, l l) is at most 2^-24 of a product, what rounding it
// once could cost; with a leading part cut off instead of rounded it was up to 2^-22.
__device__ __forceinline__ void mul3(const Op3& a, const Op3& b, f32x16& hi, f32x16& lo)
{
    lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, lo, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, lo, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, lo, 0, 0, 0);
    hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, hi, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, lo, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, lo, 0, 0, 0);
}

// acc + the five small ones.
__device__ __forceinline__ f32x16 mul_small(const Op3& a, const Op3& b, f32x16 acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, acc, 0, 0, 0);
}

// Eight consecutive values as an operand.
__device__ __forceinline__ Op3 split8(const float (&x)[8])
{
    u32x4 h, m, l;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const Pair3 p = split_pair(x[2 * q], x[2 * q + 1]);
        h[q] = p.h; m[q] = p.m; l[q] = p.l;
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// A tile in LDS: three planes of ROWS x D bf16, one per part.  The 16-byte pieces of a row are permuted by an XOR with bits of the
// row number, chosen so that neither a read along rows (16 lanes, 16 rows, one piece) nor a transposing read (4 rows, four
// pieces side by side) meets a bank twice: neighbouring 128-byte rows already lie in different halves of the banks.
template <int D>
__device__ __forceinline__ int piece_xor(int row)
{
    if (D == 64) return ((row >> 3) & 1) | ((row >> 1) & 2) | ((row << 1) & 4);
    return ((row >> 2) & 3) | ((row << 2) & 12);
}
template <int D>
__device__ __forceinline__ int tile_at(int row, int piece) { return row * D + ((piece ^ piece_xor<D>(row)) << 3); }

// Lane (r = lane%32, h = lane/32) gets X[row0 + r][k0 + 8h .. +7]; row0 is a multiple of 32, k0 of 16.
template <int ROWS, int D>
__device__ __forceinline__ Op3 ld3_nat(const bf16* X, int row0, int k0, int lane)
{
    const bf16* p = X + row0 * D + tile_at<D>(lane & 31, (k0 >> 3) + (lane >> 5));
    return {*reinterpret_cast<const bf16x8*>(p), *reinterpret_cast<const bf16x8*>(p + ROWS * D),
            *reinterpret_cast<const bf16x8*>(p + 2 * ROWS * D)};
}

__device__ __forceinline__ bf16x8 tr_pair(const bf16* lo, const bf16* hi)
{
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)lo);
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)hi);
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// The operand whose contraction index is the ROW: slot e of lane (r, h) is T[k0 + 8h + e][m0 + r], or with PERM, the order
// in which an accumulator tile re-used as an operand holds its rows, T[k0 + 8 (e/4) + 4h + e%4][m0 + r].  Within 16 lanes the
// transposing read hands lane p the column p of a 4 x 16 block whose rows the lanes address as p / 4, 8-byte pieces as p % 4.
template <int D, bool PERM>
__device__ __forceinline__ bf16x8 ldh_tr(const bf16* T, int k0, int m0, int lane)
{
    const int p = lane & 15, g = (lane >> 4) & 1, h = lane >> 5;
    const int row = (PERM ? 4 : 8) * h + (p >> 2), row2 = row + (PERM ? 8 : 4);
    const int piece = (m0 >> 3) + 2 * g + ((p >> 1) & 1);
    return tr_pair(T + k0 * D + tile_at<D>(row, piece) + 4 * (p & 1), T + k0 * D + tile_at<D>(row2, piece) + 4 * (p & 1));
}
template <int ROWS, int D, bool PERM>
__device__ __forceinline__ Op3 ld3_tr(const bf16* T, int k0, int m0, int lane)
{
    return {ldh_tr<D, PERM>(T, k0, m0, lane), ldh_tr<D, PERM>(T + ROWS * D, k0, m0, lane), ldh_tr<D, PERM>(T + 2 * ROWS * D, k0, m0, lane)};
}

// The rows of one chunk: logical positions c0 .. c0 + C of a row-major [N][D] matrix (in reverse where rev), as a buffer that ends
// with the chunk's last row below p_end.  What lies beyond reads as zero and is not written, without a branch, so that
// the compiler can count what is outstanding (s_waitcnt vmcnt(n)) across loads and stores; a chunk at or behind p_end is empty.
template <int C, int D>
struct ChunkRows {
    __amdgpu_buffer_rsrc_t rs;
    int last;                    // -1: ascending; else the row number of logical row 0
    __device__ __forceinline__ ChunkRows(const float* base, int c0, int p_end, int N, bool rev)
    {
        const int rows = __builtin_amdgcn_readfirstlane(max(0, min(C, p_end - c0)));
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base) + (size_t)(rev ? N - c0 - rows : c0) * D, 0, rows * D * 4, 0x00020000);
        last = rev ? rows - 1 : -1;
    }
    // byte offset of a row: negative, that is beyond every end, for rows that a reversed chunk does not have
    __device__ __forceinline__ int at(int row) const { return (last >= 0 ? last - row : row) * (D * 4); }
    __device__ __forceinline__ float4 load4(int off) const
    {
        return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    }
};

// One chunk's tile -> three planes in LDS, in two steps so that the loads of the next chunk can be in flight while the current one
// is worked on: fetch() brings a thread's share of the tile into registers, stash() splits it and puts it into LDS.
template <int C, int D>
struct TileRegsF32 {
    static constexpr int V4 = D / 4, NV = C * V4 / 256;
    float4 v[NV];
    __device__ __forceinline__ void fetch(const ChunkRows<C, D>& rows, unsigned tid)
    {
#pragma unroll
        for (int n = 0; n < NV; ++n) v[n] = rows.load4(rows.at(tid / V4 + 256 / V4 * n) + (int)(tid % V4) * 16);
    }
    template <bool NEG = false>
    __device__ __forceinline__ void stash(bf16* lds, unsigned tid, Hard& hard) const
    {
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const int row = tid / V4 + 256 / V4 * n, c4 = tid % V4;
            hard.operands(v[n].x, v[n].y);
            hard.operands(v[n].z, v[n].w);
            const Pair3 p0 = split_pair<NEG>(v[n].x, v[n].y), p1 = split_pair<NEG>(v[n].z, v[n].w);
            bf16* d = lds + tile_at<D>(row, c4 >> 1) + 4 * (c4 & 1);
            *reinterpret_cast<u32x2*>(d) = u32x2{p0.h, p1.h};
            *reinterpret_cast<u32x2*>(d + C * D) = u32x2{p0.m, p1.m};
            *reinterpret_cast<u32x2*>(d + 2 * C * D) = u32x2{p0.l, p1.l};
        }
    }
};

// acc[n] + sign K^T V over K2 tokens for NT 32 x 32 tiles (i0(n), j0(n)).  The tokens are summed up by themselves and added to the running
// sum in one go: as operands of one chain of matrix instructions each would be rounded to the last place of the running
// sum.  The operands of the next step are read while the current one's instructions run.  The small products do not go into the
// sum of the leading ones: the instruction aligns what it adds to the largest term, and drops, always downwards, what lies far
// below.  With all six in one sum 2 x 65000 tokens of positive keys were 2.5e-7 from 64 bits, with the fp32 instruction 2.1e-7, so 1.0e-7.
// A sum of their own costs a tile of registers; where there is none (SMALL_FIRST, the pre-pass: 21 to 54 would be spilled) they go first,
// over all tokens, and the leading ones on top.
template <int K2, int DK, int DV, int NT, bool SMALL_FIRST, class I0, class J0>
__device__ __forceinline__ void state_tiles(f32x16* acc, const bf16* k, const bf16* v, float sign, int lane, I0 i0, J0 j0)
{
    constexpr int STEPS = K2 / 16 * NT, ALL = SMALL_FIRST ? 2 * STEPS : STEPS;
    f32x16 t[NT], lo[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) { t[n] = zero16f(); lo[n] = zero16f(); }
    Op3 a[2], b[2];
    a[0] = ld3_tr<K2, DK, false>(k, 0, i0(0), lane);
    b[0] = ld3_tr<K2, DV, false>(v, 0, j0(0), lane);
    int cur = 0;                 // (which b is in use: a step whose tile shares the step before's columns of V reads none)
#pragma unroll
    for (int s = 0; s < ALL; ++s) {
        int nxt = cur;
        if (s + 1 < ALL) {
            const int s0 = (s + 1) % STEPS / NT * 16, n = (s + 1) % NT;
            const bool lead = s + 1 >= STEPS;            // (the leading parts only)
            if (lead) a[(s + 1) & 1].h = ldh_tr<DK, false>(k, s0, i0(n), lane);
            else a[(s + 1) & 1] = ld3_tr<K2, DK, false>(k, s0, i0(n), lane);
            if (n == 0 || j0(n) != j0(n - 1)) {
                nxt = cur ^ 1;
                if (lead) b[nxt].h = ldh_tr<DV, false>(v, s0, j0(n), lane);
                else b[nxt] = ld3_tr<K2, DV, false>(v, s0, j0(n), lane);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x16& sum = t[s % NT];
        if (!SMALL_FIRST) mul3(a[s & 1], b[cur], sum, lo[s % NT]);
        else if (s < STEPS) sum = mul_small(a[s & 1], b[cur], sum);
        else sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s & 1].h, b[cur].h, sum, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        cur = nxt;
    }
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[n][e] = fmaf(sign, SMALL_FIRST ? t[n][e] : t[n][e] + lo[n][e], acc[n][e]);
}

// ------------------------------------------------------------------------------------------------ the same on fp32 instructions
// For the segments with values that three bf16 parts do not hold (Hard), which no ordinary input has: v_mfma_f32_32x32x2_f32, one
// float of A and one of B per lane, 4-byte reads from row-major tiles in LDS with odd leading dimensions.  Nothing is prefetched.
__device__ __forceinline__ f32x16 gemm_tile_exact(int k_steps, f32x16 acc, const float* a, int a_rs, int a_ks, const float* b, int b_ks,
                                                  int b_ns, int lane)
{
    const int r = lane & 31, h = lane >> 5;
    const float *pa = a + r * a_rs + h * a_ks, *pb = b + h * b_ks + r * b_ns;
#pragma unroll 8
    for (int k = 0; k < k_steps; k += 2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[k * a_ks], pb[k * b_ks], acc, 0, 0, 0);
    return acc;
}

template <int C, int D>
__device__ __forceinline__ void stage_exact(float* lds, const ChunkRows<C, D>& rows, int tid)
{
#pragma unroll 4
    for (int x = tid; x < C * (D / 4); x += 256) {
        const int row = x / (D / 4), c4 = x % (D / 4);
        const float4 v = rows.load4(rows.at(row) + c4 * 16);
        float* d = lds + row * (D + 1) + c4 * 4;
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    }
}

// acc[n] += K^T V over the R tokens in LDS, tiles w, w + 4, ...; the tokens summed up by themselves first.
template <int R, int DK, int DV, int NT>
__device__ __forceinline__ void state_tiles_exact(f32x16 (&acc)[NT], const float* k, const float* v, int w, int lane)
{
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int id = w + 4 * n, ib = id / (DV / 32), jb = id % (DV / 32);
        const f32x16 t = gemm_tile_exact(R, zero16f(), k + ib * 32, 1, DK + 1, v + jb * 32, DV + 1, 1, lane);
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[n][e] += t[e];
    }
}

template <int R, int DK, int DV>
__device__ __forceinline__ void f32_seg_state_exact(const float* Kb, const float* Vb, float* o, int p0, int p1, int N, bool rev, float* lds,
                                                    int tid, int w, int met)
{
    constexpr int JB = DV / 32, NT = (DK / 32) * JB / 4;
    float *sK = lds, *sV = lds + R * (DK + 1);
    const int lane = tid & 63, r = lane & 31, h = lane >> 5;
    f32x16 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] = zero16f();
    for (int c0 = p0; c0 < p1; c0 += R) {
        __syncthreads();
        stage_exact<R, DK>(sK, ChunkRows<R, DK>(Kb, c0, p1, N, rev), tid);
        stage_exact<R, DV>(sV, ChunkRows<R, DV>(Vb, c0, p1, N, rev), tid);
        __syncthreads();
        state_tiles_exact<R, DK, DV, NT>(acc, sK, sV, w, lane);
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int id = w + 4 * n, ib = id / JB, jb = id % JB;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            float* at = o + (ib * 32 + 8 * (e >> 2) + 4 * h + (e & 3)) * DV + jb * 32 + r;
            *at = Hard::choose(met, acc[n][e], *at);
        }
    }
}

// LDS: Q, K [C][DK+1]; V [C][DV+1]; S [DK][DV+1]; the scores [C][C+1] in K's place once it has been read.  s0, n_s0: as in f32_sweep_body.
constexpr int f32_exact_kp(int c, int dk) { return c * (dk + 1) > c * (c + 1) ? c * (dk + 1) : c * (c + 1); }
constexpr int f32_exact_lds(int c, int dk, int dv) { return c * (dk + 1) + f32_exact_kp(c, dk) + (c + dk) * (dv + 1); }     // floats

template <int C, int DK, int DV>
__device__ __forceinline__ void f32_sweep_exact(const float* Qb, const float* Kb, const float* Vb, float* Ob, const float* s0, int n_s0,
                                                bool s0_transposed, int p0, int p1, int N, bool rev, float* lds, int tid, int w,
                                                int met)
{
    constexpr int LDK = DK + 1, LDV = DV + 1, LDP = C + 1;
    constexpr int TB = C / 32, JB = DV / 32, IB = DK / 32, WJ = 4 / TB, NJ = JB / WJ, NS = IB * JB / 4;
    float *sQ = lds, *sK = sQ + C * LDK, *sV = sK + f32_exact_kp(C, DK), *sS = sV + C * LDV, *sP = sK;
    const int tb = w % TB, jg = w / TB;
    f32x16 accS[NS];
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const int id = w + 4 * n, i0 = id / JB * 32 + 4 * ((tid & 63) >> 5), j = id % JB * 32 + (tid & 31);
        accS[n] = zero16f();
        const float* p = s0 + (s0_transposed ? j * DK + i0 : i0 * DV + j);
        const int step = s0_transposed ? 1 : DV;
#pragma unroll 1
        for (int k = 0; k < n_s0; ++k, p += DK * DV)
#pragma unroll
            for (int e = 0; e < 16; ++e) accS[n][e] += p[(8 * (e >> 2) + (e & 3)) * step];
    }
#pragma unroll 1
    for (int c0 = p0; c0 < p1; c0 += C) {
        asm volatile("" : "+v"(tid));       // (opaque: nothing that depends on the lane alone is kept in registers across the loop)
        const int lane = tid & 63, r = lane & 31, h = lane >> 5;
        __syncthreads();
        stage_exact<C, DK>(sQ, ChunkRows<C, DK>(Qb, c0, p1, N, rev), tid);
        stage_exact<C, DK>(sK, ChunkRows<C, DK>(Kb, c0, p1, N, rev), tid);
        stage_exact<C, DV>(sV, ChunkRows<C, DV>(Vb, c0, p1, N, rev), tid);
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            const int id = w + 4 * n, ib = id / JB, jb = id % JB;
#pragma unroll
            for (int e = 0; e < 16; ++e) sS[(ib * 32 + 8 * (e >> 2) + 4 * h + (e & 3)) * LDV + jb * 32 + r] = accS[n][e];
        }
        __syncthreads();
        // scores of the tiles on and below the diagonal (the WJ waves of a row block share them out), then the state
        constexpr int NP = (TB + WJ - 1) / WJ;
        f32x16 pt[NP];
#pragma unroll
        for (int sb = 0; sb < TB; ++sb)
            if (sb <= tb && sb % WJ == jg)
                pt[sb / WJ] = gemm_tile_exact(DK, zero16f(), sQ + tb * 32 * LDK, LDK, 1, sK + sb * 32 * LDK, 1, LDK, lane);
        if (c0 + C < p1) state_tiles_exact<C, DK, DV, NS>(accS, sK, sV, w, lane);
        __syncthreads();
#pragma unroll
        for (int sb = 0; sb < TB; ++sb)
            if (sb <= tb && sb % WJ == jg)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = 8 * (e >> 2) + 4 * h + (e & 3);
                    sP[(tb * 32 + row) * LDP + sb * 32 + r] = sb == tb && r > row ? 0.f : pt[sb / WJ][e];
                }
        __syncthreads();
        const ChunkRows<C, DV> out(Ob, c0, p1, N, rev);
#pragma unroll
        for (int n = 0; n < NJ; ++n) {
            const int j0 = (jg * NJ + n) * 32;
            f32x16 acc = gemm_tile_exact(DK, zero16f(), sQ + tb * 32 * LDK, LDK, 1, sS + j0, LDV, 1, lane);
            acc = gemm_tile_exact(32 * (tb + 1), acc, sP + tb * 32 * LDP, LDP, 1, sV + j0, LDV, 1, lane);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int off = out.at(tb * 32 + 8 * (e >> 2) + 4 * h + (e & 3)) + (j0 + r) * 4;
                const float first = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(out.rs, off, 0, 0));
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, Hard::choose(met, acc[e], first)), out.rs, off, 0, 0);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------ segment totals
// out[bh][seg][i*DV + j] = sum over the segment's tokens of K[t][i] * V[t][j].  The last segment's total is never
// used by an exclusive prefix, so its workgroups leave at once.  Wave w owns output tiles w, w+4, ...
constexpr int kF32SegRows = 64;                 // tokens staged per step
constexpr int f32_seg_lds(int dk, int dv) { return kF32SegRows * (dk + dv) * 3; }     // bf16 elements

template <int DK, int DV>
__device__ __forceinline__ void f32_seg_state_body(const float* __restrict__ K, const float* __restrict__ V,
                                                   float* __restrict__ out, int N, int seg_len, int n_seg, bool rev,
                                                   bf16* lds, int* votes)
{
    constexpr int R = kF32SegRows;
    bf16* sK = lds;
    bf16* sV = lds + 3 * R * DK;
    const int seg = blockIdx.y;
    const long bh = blockIdx.x;
    if (seg == n_seg - 1) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* Kb = K + (size_t)bh * N * DK;
    const float* Vb = V + (size_t)bh * N * DV;
    const int p0 = seg * seg_len, p1 = min(N, p0 + seg_len);
    constexpr int JB = DV / 32, NT = (DK / 32) * JB / 4;
    static_assert(R * (DK + DV + 2) * 4 <= f32_seg_lds(DK, DV) * 2, "the fp32 tiles of a segment done over");
    Hard hard;
    f32x16 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] = zero16f();
    // two steps' rows in flight: a step's products are over before one round trip to memory is
    TileRegsF32<R, DK> rk[2];
    TileRegsF32<R, DV> rv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        rk[u].fetch(ChunkRows<R, DK>(Kb, p0 + u * R, p1, N, rev), tid);
        rv[u].fetch(ChunkRows<R, DV>(Vb, p0 + u * R, p1, N, rev), tid);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (int cc = p0; cc < p1; cc += 2 * R) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c0 = cc + u * R;
            if (c0 >= p1) break;
            __syncthreads();
            rk[u].stash(sK, tid, hard);
            // (every other step with -V: what the instruction drops downwards is then as often too much as too little.  S after 262144 tokens,
            // in 2^-24 of its size: 5.9 too small, now 0.0)
            const bool odd = (c0 / R) & 1;
            if (odd) rv[u].template stash<true>(sV, tid, hard);
            else rv[u].stash(sV, tid, hard);
            __syncthreads();
            rk[u].fetch(ChunkRows<R, DK>(Kb, c0 + 2 * R, p1, N, rev), tid);
            rv[u].fetch(ChunkRows<R, DV>(Vb, c0 + 2 * R, p1, N, rev), tid);
            state_tiles<R, DK, DV, NT, true>(acc, sK, sV, odd ? -1.f : 1.f, lane, [&](int n) { return ((w + 4 * n) / JB) * 32; },
                                       [&](int n) { return ((w + 4 * n) % JB) * 32; });
        }
    }
    float* o = out + ((size_t)bh * n_seg + seg) * DK * DV;
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) hard.result(acc[n][e]);
    const int met = hard.anywhere(votes, w, lane), r = lane & 31, h = lane >> 5;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int id = w + 4 * n, ib = id / JB, jb = id % JB;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) o[(ib * 32 + 8 * a + 4 * h + b) * DV + jb * 32 + r] = acc[n][4 * a + b];
    }
    if (met) {
        __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0): each lane reads again what it has written
        f32_seg_state_exact<R, DK, DV>(Kb, Vb, o, p0, p1, N, rev, reinterpret_cast<float*>(lds), tid, w, met);
    }
}

// (64 x 128: as many waves per SIMD as the LDS has room for workgroups)
template <int DK, int DV>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DK + DV == 128 ? 3 : DK + DV == 192 ? 2 : 1)))
void f32_seg_state_kernel(const float* __restrict__ K, const float* __restrict__ V,
                                                           float* __restrict__ out, int N, int seg_len, int n_seg)
{
    __shared__ __attribute__((aligned(16))) bf16 lds[f32_seg_lds(DK, DV)];
    __shared__ int votes[4];
    f32_seg_state_body<DK, DV>(K, V, out, N, seg_len, n_seg, false, lds, votes);
}

// The backward's two sets of totals, V^T K in reading order and Q^T dO from the end, side by side on grid.z.
template <int DK, int DV>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DK + DV == 128 ? 3 : DK + DV == 192 ? 2 : 1)))
void f32_bwd_seg_state_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                                                               const float* __restrict__ V, const float* __restrict__ dO,
                                                               float* __restrict__ out, size_t array_stride, int N,
                                                               int seg_len, int n_seg)
{
    __shared__ __attribute__((aligned(16))) bf16 lds[f32_seg_lds(DK, DV)];
    __shared__ int votes[4];
    if (blockIdx.z == 0) f32_seg_state_body<DV, DK>(V, K, out, N, seg_len, n_seg, false, lds, votes);
    else f32_seg_state_body<DK, DV>(Q, dO, out + array_stride, N, seg_len, n_seg, true, lds, votes);
}

// ------------------------------------------------------------------------------------------------ main sweep
// One workgroup (4 waves) per (segment, bh).  Wave w owns output rows [32*tb, +32) with tb = w % TB and NJ column
// tiles.  LDS: K [C][DK], V [C][DV] and S^T [DV][DK], each as three planes.  Queries come straight from memory in
// operand order; the scores of a row block stay in the registers of the waves that need them.
constexpr int f32_sweep_chunk(int dk, int dv) { return dk == 128 && dv == 128 ? 32 : 64; }   // what fits 160 KB of LDS
constexpr int f32_sweep_lds(int dk, int dv)                                                  // bf16 elements
{
    const int c = f32_sweep_chunk(dk, dv);
    return 3 * (c * dk + c * dv + dk * dv);
}

template <int C, int DK, int DV>
__device__ __forceinline__ void f32_sweep_body(const float* __restrict__ Q, const float* __restrict__ K,
                                               const float* __restrict__ V, float* __restrict__ O,
                                               const float* __restrict__ S0, int N, int seg_len, int n_seg, bool rev,
                                               bool s0_transposed, bool folded, bf16* lds, int* votes)
{
    constexpr int TB = C / 32, JB = DV / 32, IB = DK / 32, KK = DK / 16;
    constexpr int WJ = 4 / TB, NJ = JB / WJ;
    // State tiles: column tiles jg*NJ .. of S belong to the TB waves that share jg, in equal parts.
    constexpr int NS = IB * NJ / TB;
    static_assert(JB % WJ == 0 && (TB == 1 || TB == 2), "unsupported tile shape");
    static_assert(f32_exact_lds(C, DK, DV) * 4 <= f32_sweep_lds(DK, DV) * 2, "the fp32 tiles of a segment done over");
    bf16* sK = lds;
    bf16* sV = sK + 3 * C * DK;
    bf16* sS = sV + 3 * C * DV;
    const int seg = blockIdx.y;
    const long bh = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tb = w % TB, jg = w / TB;
    const int r = lane & 31, h = lane >> 5;
    const float* Qb = Q + (size_t)bh * N * DK;
    const float* Kb = K + (size_t)bh * N * DK;
    const float* Vb = V + (size_t)bh * N * DV;
    float* Ob = O + (size_t)bh * N * DV;
    const int p0 = seg * seg_len, p1 = min(N, p0 + seg_len);
    const int q_own = tb * NS;
    Hard hard;

    // (the first chunk's tiles are asked for first: they are what the loop waits for)
    TileRegsF32<C, DK> rk;
    TileRegsF32<C, DV> rv;
    float4 rq[DK / 8];
    auto fetch_q = [&](int c0) __attribute__((always_inline)) {      // row r of the wave's 32, features 16 kk + 8 h ..
        const ChunkRows<C, DK> rows(Qb, c0, p1, N, rev);
        const int off = rows.at(tb * 32 + r) + 32 * h;
#pragma unroll
        for (int x = 0; x < DK / 8; ++x) rq[x] = rows.load4(off + (x >> 1) * 64 + (x & 1) * 16);
    };
    rk.fetch(ChunkRows<C, DK>(Kb, p0, p1, N, rev), tid);
    rv.fetch(ChunkRows<C, DV>(Vb, p0, p1, N, rev), tid);
    __builtin_amdgcn_sched_barrier(0);
    fetch_q(p0);
    // start state of this segment, as accumulator tiles: the sum of the n_s0 states that lie one behind the other at s0, in their order
    // (the one a scan has left, or the totals of the segments in front; none for the first segment).  s0_transposed: they
    // are stored as [DV][DK] (left there by a call with keys and values exchanged).  Four states' loads are in flight.
    f32x16 accS[NS];
    const int n_s0 = S0 == nullptr || seg == 0 ? 0 : folded ? seg : 1;
    const float* s0 = S0 + ((size_t)bh * n_seg + (folded ? 0 : seg)) * DK * DV;
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const int q = q_own + n, ib = q % IB, jb = jg * NJ + q / IB;
        accS[n] = zero16f();
        constexpr int U = 4;
        for (int k = 0; k < n_s0; k += U) {
            f32x16 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float* p = s0 + (size_t)min(k + u, n_s0 - 1) * (DK * DV);
                // (one uniform branch around each unrolled set of loads, so that the loads of a tile are issued together)
                if (s0_transposed) {
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        const float4 v = *reinterpret_cast<const float4*>(p + (jb * 32 + r) * DK + ib * 32 + 8 * a + 4 * h);
                        x[u][4 * a] = v.x; x[u][4 * a + 1] = v.y; x[u][4 * a + 2] = v.z; x[u][4 * a + 3] = v.w;
                    }
                } else {
#pragma unroll
                    for (int a = 0; a < 4; ++a)
#pragma unroll
                        for (int b = 0; b < 4; ++b) x[u][4 * a + b] = p[(ib * 32 + 8 * a + 4 * h + b) * DV + jb * 32 + r];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u < n_s0) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) accS[n][e] += x[u][e];
                }
        }
    }
    // One chunk's products as a list of steps: the operand of the next step is read from LDS while the current one's instructions
    // run, and the splitting of queries and scores goes in between those.  Keys of the wave's own row block (the masked
    // tile), the state before the chunk, then, for the second row block, the keys of the first.
    auto products = [&](int c0, int more) __attribute__((always_inline)) {
        constexpr int NA = KK, NB = NJ * KK, NC = 2 * NJ;
        int ln = lane;      // (opaque: what depends on the lane alone would otherwise be kept in registers across the loop)
        asm volatile("" : "+v"(ln));
        Op3 aQ[KK], aP[2], op[2];
        f32x16 pT, pL, hi[NJ], lo[NJ];
        auto split_q = [&](int kk) __attribute__((always_inline)) {
            const float4 x = rq[2 * kk], y = rq[2 * kk + 1];
            const float e[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
            for (int q = 0; q < 8; q += 2) hard.operands(e[q], e[q + 1]);
            aQ[kk] = split8(e);
        };
        // scores of keys 16 x .. 16 x + 15 of the block as first operand: the accumulator tile holds them as it wants them
        auto split_p = [&](int x, bool mask) __attribute__((always_inline)) {
            float e[8], v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int row = 16 * x + 8 * (q >> 2) + 4 * (ln >> 5) + (q & 3);        // key within the block; ln & 31 = query
                v[q] = pT[8 * x + q] + pL[8 * x + q];
                if (q & 1) hard.operands(v[q - 1], v[q]);
                e[q] = !mask || row <= (ln & 31) ? v[q] : 0.f;
            }
            aP[x] = split8(e);
        };
        auto keys = [&](int sb, int kk) __attribute__((always_inline)) { return ld3_nat<C, DK>(sK + sb * 32 * DK, 0, kk * 16, ln); };
        auto state = [&](int s) __attribute__((always_inline)) { return ld3_nat<DV, DK>(sS, (jg * NJ + s / KK) * 32, s % KK * 16, ln); };
        auto vals = [&](int sb, int s) __attribute__((always_inline)) {
            return ld3_tr<C, DV, true>(sV + sb * 32 * DV, s / NJ * 16, (jg * NJ + s % NJ) * 32, ln);
        };
        split_q(0);
        op[0] = keys(tb, 0);
        pT = zero16f();
        pL = zero16f();
#pragma unroll
        for (int n = 0; n < NJ; ++n) { hi[n] = zero16f(); lo[n] = zero16f(); }
#pragma unroll
        for (int s = 0; s < NA + NB + NC; ++s) {
            if (s + 1 < NA) op[(s + 1) & 1] = keys(tb, s + 1);
            else if (s + 1 < NA + NB) op[(s + 1) & 1] = state(s + 1 - NA);
            else if (s + 1 < NA + NB + NC) op[(s + 1) & 1] = vals(tb, s + 1 - NA - NB);
            __builtin_amdgcn_sched_barrier(0);
            if (s < NA) {                    // P^T[s][t] = k_s . q_t (each of the WJ waves of a row block for itself)
                if (s + 1 < KK) split_q(s + 1);
                mul3(op[s & 1], aQ[s], pT, pL);
            } else if (s < NA + NB) {        // inter-chunk part Q S_prev
                const int n = (s - NA) / KK;
                mul3(aQ[(s - NA) % KK], op[s & 1], hi[n], lo[n]);
                if (s == NA) split_p(0, true);
                if (s == NA + 1) split_p(1, true);
            } else {                         // intra-chunk part P V
                const int x = (s - NA - NB) / NJ, n = (s - NA - NB) % NJ;
                mul3(aP[x], op[s & 1], hi[n], lo[n]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 == NA) fetch_q(c0 + C);
        }
        if (TB > 1 && tb > 0) {
            op[0] = keys(0, 0);
            pT = zero16f();
        pL = zero16f();
#pragma unroll
            for (int s = 0; s < NA + NC; ++s) {
                if (s + 1 < NA) op[(s + 1) & 1] = keys(0, s + 1);
                else if (s + 1 < NA + NC) op[(s + 1) & 1] = vals(0, s + 1 - NA);
                __builtin_amdgcn_sched_barrier(0);
                if (s < NA) {
                    mul3(op[s & 1], aQ[s], pT, pL);
                } else {
                    const int x = (s - NA) / NJ, n = (s - NA) % NJ;
                    if (s == NA) split_p(0, false);
                    mul3(aP[x], op[s & 1], hi[n], lo[n]);
                    if (s == NA) split_p(1, false);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const ChunkRows<C, DV> rows(Ob, c0, p1, N, rev);
        int off = rows.at(tb * 32 + 4 * (ln >> 5)) + (jg * NJ * 32 + (ln & 31)) * 4;
        const int step = rev ? -DV * 4 : DV * 4;
#pragma unroll
        for (int n = 0; n < NJ; ++n)
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    // (a streaming store: 32 lanes write one whole 128-byte line, and nothing here reads it again)
                    const float v = hi[n][4 * a + b] + lo[n][4 * a + b];
                    hard.result(v);
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rows.rs, off + (8 * a + b) * step + n * 128, 0, 2);
                }
        // state update S += K^T V (not needed after the segment's last chunk)
        if (more)
            state_tiles<C, DK, DV, NS, false>(accS, sK, sV, 1.f, ln, [&](int n) { return (q_own + n) % IB * 32; },
                                        [&](int n) { return (jg * NJ + (q_own + n) / IB) * 32; });
    };
    // (nothing outstanding on the way into the loop: what a chunk waits for at its start is then counted from the chunk before,
    // whose output stores, younger than its loads, need not have arrived)
    __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0)
    int c0 = p0;
    do {
        unsigned tv = tid;       // (opaque, as in products())
        asm volatile("" : "+v"(tv));
        __syncthreads();   // previous chunk fully consumed
        rk.stash(sK, tv, hard);
        rv.stash(sV, tv, hard);
        // publish the state before this chunk, [j][i]: a lane holds four consecutive i of one j
#pragma unroll
        for (int n = 0; n < NS; ++n) {
            {
                const int q = q_own + n, ib = q % IB, jb = jg * NJ + q / IB;
#pragma unroll
                for (int e = 0; e < 16; e += 2) hard.operands(accS[n][e], accS[n][e + 1]);
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const Pair3 x = split_pair(accS[n][4 * a], accS[n][4 * a + 1]), y = split_pair(accS[n][4 * a + 2], accS[n][4 * a + 3]);
                    bf16* d = sS + jb * 32 * DK + tile_at<DK>(tv & 31, ib * 4 + a) + 4 * (tv >> 5 & 1);
                    *reinterpret_cast<u32x2*>(d) = u32x2{x.h, y.h};
                    *reinterpret_cast<u32x2*>(d + DK * DV) = u32x2{x.m, y.m};
                    *reinterpret_cast<u32x2*>(d + 2 * DK * DV) = u32x2{x.l, y.l};
                }
            }
        }
        __syncthreads();
        // the next chunk, in flight during the arithmetic
        rk.fetch(ChunkRows<C, DK>(Kb, c0 + C, p1, N, rev), tid);
        rv.fetch(ChunkRows<C, DV>(Vb, c0 + C, p1, N, rev), tid);
        __builtin_amdgcn_sched_barrier(0);
        // (opaque: known to be the loop's own condition, the loads above would be moved behind the branch on it)
        int more = c0 + C < p1;
        more = __builtin_amdgcn_readfirstlane(more);
        asm volatile("" : "+s"(more));
        products(c0, more);
        c0 += C;
    } while (c0 < p1);
    if (const int met = hard.anywhere(votes, w, lane)) {
        __builtin_amdgcn_s_waitcnt(0x0f70);     // vmcnt(0): each lane reads again what it has written
        f32_sweep_exact<C, DK, DV>(Qb, Kb, Vb, Ob, s0, n_s0, s0_transposed, p0, p1, N, rev, reinterpret_cast<float*>(lds), tid, w, met);
    }
}

// (64 x 64: two workgroups fit a compute unit's LDS, so the registers have to allow for two waves per SIMD)
template <int DK, int DV>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DK == 64 && DV == 64 ? 2 : 1)))
void f32_sweep_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, float* __restrict__ O,
                      const float* __restrict__ S0, int N, int seg_len, int n_seg, bool folded)
{
    __shared__ __attribute__((aligned(16))) bf16 lds[f32_sweep_lds(DK, DV)];
    __shared__ int votes[4];
    f32_sweep_body<f32_sweep_chunk(DK, DV), DK, DV>(Q, K, V, O, S0, N, seg_len, n_seg, false, false, folded, lds, votes);
}

// The gradient is three instances of the forward map (time-reversal duality), independent of one another, so they ride
// on grid.z of one launch:
//   dQ = LinAttn(query dO, key V, value K)             causal          states V^T K   (first array)
//   dK = LinAttn(query V,  key dO, value Q)            anti-causal     states dO^T Q  (the second array, transposed)
//   dV = LinAttn(query K,  key Q, value dO)            anti-causal     states Q^T dO  (second array)
template <int DK, int DV>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DK == 64 && DV == 64 ? 2 : 1)))
void f32_bwd_sweep_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                          const float* __restrict__ dO, float* __restrict__ dQ, float* __restrict__ dK, float* __restrict__ dV,
                          const float* __restrict__ S0, size_t array_stride, int N, int seg_len, int n_seg, bool folded)
{
    constexpr int C = f32_sweep_chunk(DK, DV);
    constexpr int LA = f32_sweep_lds(DK, DV), LB = f32_sweep_lds(DV, DK);
    __shared__ __attribute__((aligned(16))) bf16 lds[LA > LB ? LA : LB];
    __shared__ int votes[4];
    const int z = blockIdx.z;
    const float* S1 = S0 != nullptr ? S0 + array_stride : nullptr;
    if constexpr (DK == DV) {
        f32_sweep_body<C, DK, DV>(z == 0 ? dO : z == 1 ? V : K, z == 0 ? V : z == 1 ? dO : Q, z == 0 ? K : z == 1 ? Q : dO,
                                  z == 0 ? dQ : z == 1 ? dK : dV, z == 0 ? S0 : S1, N, seg_len, n_seg, z != 0, z == 1, folded, lds, votes);
    } else if (z < 2) {
        f32_sweep_body<C, DV, DK>(z == 0 ? dO : V, z == 0 ? V : dO, z == 0 ? K : Q, z == 0 ? dQ : dK, z == 0 ? S0 : S1, N,
                                  seg_len, n_seg, z != 0, z == 1, folded, lds, votes);
    } else {
        f32_sweep_body<C, DK, DV>(K, Q, dO, dV, S1, N, seg_len, n_seg, true, false, folded, lds, votes);
    }
}

template <int DK, int DV>
static hipError_t f32_fwd_impl(const float* Q, const float* K, const float* V, float* O, long BH, int N, const Plan& plan,
                               float* ws, hipStream_t st)
{
    hipError_t e;
    const dim3 grid((unsigned)BH, plan.n_seg);
    const bool folded = fold_scan(plan, false, false);
    if (plan.n_seg > 1) {
        {
            ProfScope prof(KID_SEG_STATE_F32, st);
            hipLaunchKernelGGL((f32_seg_state_kernel<DK, DV>), grid, dim3(256), 0, st, K, V, ws, N, plan.seg_len,
                               plan.n_seg);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const int mode = SCAN_EXCL_PREFIX;
        if (!folded && (e = scan_states(ws, 0, 1, &mode, nullptr, 0, BH, plan.n_seg, DK * DV, st)) != hipSuccess) return e;
    }
    ProfScope prof(KID_SWEEP_F32, st);
    hipLaunchKernelGGL((f32_sweep_kernel<DK, DV>), grid, dim3(256), 0, st, Q, K, V, O, plan.n_seg > 1 ? ws : nullptr, N,
                       plan.seg_len, plan.n_seg, folded);
    return hipGetLastError();
}

template <int DK, int DV>
static hipError_t f32_bwd_impl(const float* Q, const float* K, const float* V, const float* dO, float* dQ, float* dK,
                               float* dV, long BH, int N, const Plan& plan, float* ws, hipStream_t st)
{
    hipError_t e;
    const size_t stride = (size_t)BH * plan.n_seg * DK * DV;
    const bool folded = fold_scan(plan, false, true);
    if (plan.n_seg > 1) {
        {
            ProfScope prof(KID_SEG_STATE_F32, st);
            hipLaunchKernelGGL((f32_bwd_seg_state_kernel<DK, DV>), dim3((unsigned)BH, plan.n_seg, 2), dim3(256), 0, st, Q, K, V,
                               dO, ws, stride, N, plan.seg_len, plan.n_seg);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const int modes[2] = {SCAN_EXCL_PREFIX, SCAN_EXCL_PREFIX};
        if (!folded && (e = scan_states(ws, stride, 2, modes, nullptr, 0, BH, plan.n_seg, DK * DV, st)) != hipSuccess) return e;
    }
    ProfScope prof(KID_SWEEP_F32, st);
    hipLaunchKernelGGL((f32_bwd_sweep_kernel<DK, DV>), dim3((unsigned)BH, plan.n_seg, 3), dim3(256), 0, st, Q, K, V, dO, dQ, dK,
                       dV, plan.n_seg > 1 ? ws : nullptr, stride, N, plan.seg_len, plan.n_seg, folded);
    return hipGetLastError();
}

#define CHELA_F32_DIMS(F_, ...)                                                                                        \
    if (dk == 64 && dv == 64) return F_<64, 64>(__VA_ARGS__);                                                          \
    if (dk == 64 && dv == 128) return F_<64, 128>(__VA_ARGS__);                                                        \
    if (dk == 128 && dv == 64) return F_<128, 64>(__VA_ARGS__);                                                        \
    if (dk == 128 && dv == 128) return F_<128, 128>(__VA_ARGS__);                                                      \
    return hipErrorInvalidValue;

hipError_t launch_f32_fwd(const float* Q, const float* K, const float* V, float* O, long BH, int N, int dk, int dv,
                          const Plan& plan, float* ws, hipStream_t st)
{
    CHELA_F32_DIMS(f32_fwd_impl, Q, K, V, O, BH, N, plan, ws, st)
}

hipError_t launch_f32_bwd(const float* Q, const float* K, const float* V, const float* dO, float* dQ, float* dK, float* dV,
                          long BH, int N, int dk, int dv, const Plan& plan, float* ws, hipStream_t st)
{
    CHELA_F32_DIMS(f32_bwd_impl, Q, K, V, dO, dQ, dK, dV, BH, N, plan, ws, st)
}
#undef CHELA_F32_DIMS

}  // namespace chela
