// Learned correction network for the octree multigrid (gfx950).
//
// The network maps a leaf box's scaled residual (8^3 plus its one-cell ghost
// layer, 10^3) to a correction on the box's 8^3 cells:
//   conv 3^3 valid 1->16, ReLU, conv 3^3 same 16->16, ReLU, conv 3^3 same 16->1.
// Weights, the input and both hidden activations are BF16 (round to nearest
// even), accumulation is FP32.  Parameters are kept as FP32 masters in the
// order W1[16][27], b1[16], W2[16 out][16 in][27], b2[16], W3[16][27], b3,
// with tap t = (dk*3 + dj)*3 + di.
//
// Forward: a box's activations stay in LDS (one box at a time per workgroup).
//  * layer 1 is an implicit GEMM [16 cells x 32 taps (27 used)] x [32 x 16
//    channels]: one 16x16x32 BF16 MFMA per 16-cell tile;
//  * layer 2 is an implicit GEMM with K = 27 taps x 16 channels, taken as 18
//    16x16x32 MFMAs per tile (the kernel rows of one z offset paired, 16
//    channels each, per instruction) and blocked along z, so that each
//    loaded input slice serves the three output slices it reaches;
//    activations are stored [padded cell][channel];
//  * layer 3 first forms Q[dk, dj][cell] = sum over di and c of W3[c][dk, dj,
//    di] a2[c][cell + di - 1] (N = 9 kernel rows, K = 3 x 16), then y[cell] =
//    b3 + the 9 terms Q[dk, dj][cell + (dk - 1, dj - 1)], which turns the
//    16->1 convolution into a dense GEMM plus a 9-term sum.
// The backward pass (training only) keeps its FP32 gradients: each is split
// exactly into three BF16 parts for the matrix cores.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <vector>

#include "mg.h"
#include "nn.h"

namespace mg {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kW1 = 0, kB1 = 432, kW2 = 448, kB2 = 7360, kW3 = 7376, kB3 = 7808;
constexpr int kP1 = 0, kP2 = 512;  // offsets in the packed fragments

__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
// The same rounding (nearest even) by the hardware conversion; a NaN stays a
// NaN (its payload may differ from f2bf's).  Two values per instruction.
__device__ __forceinline__ uint16_t f2bf_hw(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
// max(z, 0) that propagates NaN (a non-finite weight must reach the output)
__device__ __forceinline__ float relu(float z) { return __builtin_elementwise_maximum(z, 0.0f); }

// offset of tap t in a 10^3 block (x fastest)
__host__ __device__ constexpr int tap_off(int t) { return (t / 9) * 100 + ((t / 3) % 3) * 10 + t % 3; }

// colour-split index -> natural cell index (k*8 + j)*8 + i
__device__ __forceinline__ int cs_to_nat(int e) {
    int c = e >> 8, r = e & 255, m = r & 3, j = (r >> 2) & 7, k = r >> 5;
    int i = 2 * m + ((j + k + c) & 1);
    return (k * 8 + j) * 8 + i;
}
__device__ __forceinline__ int cs_idx(int i, int j, int k) {
    return (((i + j + k) & 1) << 8) + ((k * 8 + j) << 2) + (i >> 1);
}

template <typename T>
__device__ __forceinline__ T block_sum256(T v, T *S) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    int t = threadIdx.x;
    __syncthreads();
    if ((t & 63) == 0) S[t >> 6] = v;
    __syncthreads();
    return (S[0] + S[1]) + (S[2] + S[3]);
}

// ------------------------------------------------------------ weight packing
// Fragments in the lane order of the MFMA B operand (lane l holds column
// l % 16, K rows 8 (l / 16) .. +7).  Layer 3's few are formed by the forward.
// One entry a thread: 2 us (one workgroup walking all entries: 12 us).
__global__ __launch_bounds__(256) void k_nn_pack(const float *__restrict__ prm, uint16_t *__restrict__ pk) {
    const int e = blockIdx.x * 256 + threadIdx.x;  // grid: kNnPacked / 256
    float v = 0.0f;
    if (e < kP2) {
        int lane = e >> 3, q = e & 7, o = lane & 15, g = lane >> 4, t = 8 * g + q;
        if (t < 27) v = prm[kW1 + o * 27 + t];
    } else {
        // fragment f = (2 dk + type) 3 + di: type 0 has kernel rows dj = 0
        // in K groups 0-1 and dj = 1 in groups 2-3, type 1 dj = 2 in
        // groups 0-1 and zeros in 2-3
        int e2 = e - kP2, f = e2 >> 9, r = e2 & 511, lane = r >> 3, q = r & 7;
        int dk = f / 6, type = (f / 3) & 1, di = f % 3, o = lane & 15, g = lane >> 4, ch = 8 * (g & 1) + q;
        int dj = type == 0 ? (g < 2 ? 0 : 1) : (g < 2 ? 2 : -1);
        if (dj >= 0) v = prm[kW2 + (o * 16 + ch) * 27 + (dk * 3 + dj) * 3 + di];
    }
    pk[e] = f2bf(v);
}
static_assert(kNnPacked % 256 == 0, "one thread per packed entry");

// ------------------------------------------------------------------ forward
// x [nbox][1000] FP32 (10^3, x fastest), y [nbox][512] FP32 (natural order).
// idx (optional) maps output position q to input box idx[q].  SAVE stores a1
// and a2 (BF16, [nbox][16][512]) for training.
//
// Persistent workgroups of 4 waves: the weight fragments stay in registers
// while a workgroup walks over boxes q = blockIdx.x, + gridDim.x, ..., and
// each thread prefetches its part of the next box's input during the current
// box.  Tiles are 16 consecutive cells (two x-rows of 8); wave w owns the
// tiles of y-rows (2w, 2w+1) at every z.  In layers 1 and 2 a tile's cells are
// the columns of the product, so that a lane ends with four channels of one
// cell and stores them at once.
//
// Layer 1 needs, per lane, four pairs of consecutive taps: (x, x + 1) within a
// kernel row, or the last of a row and the first of the next, 8 or 78 cells
// on.  The input is staged as arrays of such pairs, and an operand is four
// LDS reads at constant offsets (not eight of one value and their packing).
//
// Layer 2 pairs the kernel rows within one z offset dk (dj = 0 with 1, and
// dj = 2 alone: 18 MFMAs per 16-cell tile, 27 taps in 32-wide K groups) so
// that a loaded input slice serves the three output slices it reaches: each
// wave walks the z-slices of its y-rows and loads every input fragment once
// (6 per slice), instead of once per output tile (15 per tile).  The
// x-shifted operands are loaded from A1 one cell to either side (moving one
// fragment across lanes with DPP row shifts instead costs 16 vector
// instructions per pair for the shifts and row-end masks, which bounded an
// earlier version).  Activations are rounded to BF16 (nearest even) by the
// hardware conversion.
//
// Layer 3 takes the three di of a kernel row into K, so one pass of 9 columns
// replaces two of 16 and the sum over shifted cells has 9 terms, loaded
// without branches (with 27 columns it was 54 predicated reads a thread, each
// waited for by itself).
//
// Bound by the latencies between the barriers of a box: three workgroups a CU
// (168 registers, 45 KB of LDS) keep the matrix cores busy for half of the
// time.  9473 boxes: 137 us before the pairs, the 9 columns and the row layout
// below, now 91; LDS instructions 10.5M -> 6.3M, vector instructions 34.9M ->
// 18.0M.  The LDS matters first: at 54 KB only two workgroups fit, 132 us.
constexpr int kFwdThreads = 256;  // 4 waves; 3 workgroups per CU

template <bool SAVE>
__global__ __launch_bounds__(kFwdThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_nn_fwd(const float *__restrict__ x, float *__restrict__ y,
                                                        const int32_t *__restrict__ idx, int64_t nbox,
                                                        const uint16_t *__restrict__ pk,
                                                        const float *__restrict__ prm,
                                                        uint16_t *__restrict__ a1o,
                                                        uint16_t *__restrict__ a2o) {
    // A1 (u16): cell (x, y, z), y and z padded by one (zero), at (10 z + y) *
    // kRow + 16 x; A2 the same without padding.  A lane whose x-shifted cell is
    // outside reads a zero row instead.  Rows of 8 cells, 64 LDS banks, gave
    // the fewest bank conflicts: 12.4M cycles on 9473 boxes, against 19.0M with
    // 16 bytes more a row and 24.4M with the halves of the channels apart.
    constexpr int kRow = 8 * 16, kA1 = 100 * kRow, kA2 = 64 * kRow;
    // Q [9][kQs] FP32, in A1's space
    constexpr int kQs = 520, kQ = 9 * kQs;
    // the pairs of the input, in A2's space: (c, c + 1), (c, c + 8), (c, c + 78)
    constexpr int kPairs = 1000;
    static_assert(kQ * 4 <= kA1 * 2 && kQ % 4 == 0 && 3 * kPairs * 4 <= kA2 * 2, "overlays fit");
    // the weights of layers 1 and 3 and the biases: with the rest in registers
    // they spilled
    __shared__ uint4 RA[kA1 / 8], RB[kA2 / 8], W1[64], W3[2][64], Z[1];
    __shared__ f32x4 bias[8];
    uint16_t *A1 = reinterpret_cast<uint16_t *>(RA), *A2 = reinterpret_cast<uint16_t *>(RB);
    float *Q = reinterpret_cast<float *>(RA);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, row = lane & 15, g = lane >> 4;
    const int o = lane & 15;
    // the lane's cell of tile (w, z): (i, j, z)
    const int i = row & 7, j = 2 * w + (row >> 3);
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};

    // ---- weights, once per workgroup
    if (t < 64) W1[t] = *reinterpret_cast<const uint4 *>(pk + kP1 + t * 8);
    if (t < 32) reinterpret_cast<float *>(bias)[t] = prm[t < 16 ? kB1 + t : kB2 + t - 16];
    bf16x8 B2[18];
#pragma unroll
    for (int f = 0; f < 18; f++)
        B2[f] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pk + kP2 + (f * 64 + lane) * 8));
    // layer 3, column o = kernel row 3 dk + dj: di = 0 in K groups 0-1 and
    // di = 1 in 2-3, then di = 2 and nothing
    if (t < 128) {
        u32x4 f = {0u, 0u, 0u, 0u};
        const int di = t < 64 ? g >> 1 : 2;
        if (o < 9 && (t < 64 || g < 2)) {
            const float *p = prm + kW3 + 8 * (g & 1) * 27 + 3 * o + di;
#pragma unroll
            for (int q = 0; q < 4; q++) f[q] = f2bf(p[54 * q]) | ((uint32_t)f2bf(p[54 * q + 27]) << 16);
        }
        W3[t >> 6][lane] = __builtin_bit_cast(uint4, f);
    }
    if (t == 0) Z[0] = make_uint4(0, 0, 0, 0);
    const float b3 = prm[kB3];
    // layer 1: where the pairs of taps (8 g + 2 h, + 1) of the lane's cell at
    // z = 0 are; taps 27 to 31 are padding
    const uint32_t *pair[4];
#pragma unroll
    for (int h = 0; h < 4; h++) {
        const int tp = 8 * g + 2 * h, next = tp / 3 % 3 == 2 ? 2 : 1;
        const int at = tp < 27 ? tap_off(tp) : 0;
        pair[h] = reinterpret_cast<const uint32_t *>(RB) + (tp < 27 && tp % 3 == 2 ? next * kPairs : 0) + at + j * 10 + i;
    }
    const uint32_t last = g == 3 ? 0x0000ffffu : 0xffffffffu, none = g == 3 ? 0u : 0xffffffffu;
    const int put = i * 16 + 4 * g;  // where the lane's four channels of a cell go
    const uint32_t save = 4 * g * 512 + j * 8 + i;
    int64_t q = blockIdx.x;
    float xn[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (q < nbox) {
        const float *xb = x + (idx ? (int64_t)idx[q] : q) * 1000;
#pragma unroll
        for (int h = 0; h < 4; h++)
            if (t + 256 * h < 1000) xn[h] = xb[t + 256 * h];
    }
    // A1's padding is zero; a box overwrites the part that holds Q
    for (int e = t + kQ / 4; e < kA1 / 8; e += kFwdThreads) RA[e] = make_uint4(0, 0, 0, 0);
    for (; q < nbox; q += gridDim.x) {
        __syncthreads();  // the previous box is done with every LDS buffer
        for (int e = t; e < kQ / 4; e += kFwdThreads) RA[e] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int h = 0; h < 4; h++) {
            const int c = t + 256 * h;
            const uint16_t v = f2bf_hw(xn[h]);
            if (c < 1000) {
                A2[2 * c] = v;
                A2[2 * (kPairs + c)] = v;
                A2[2 * (2 * kPairs + c)] = v;
                if (h > 0 || c >= 1) *(volatile uint16_t *)(A2 + 2 * c - 1) = v;  // (not one misaligned store with A2[2 c])
                if (h > 0 || c >= 8) A2[2 * (kPairs + c - 8) + 1] = v;
                if (h > 0 || c >= 78) A2[2 * (2 * kPairs + c - 78) + 1] = v;
            }
        }
        const int64_t qn = q + gridDim.x;
        if (qn < nbox) {
            const float *xb = x + (idx ? (int64_t)idx[qn] : qn) * 1000;
#pragma unroll
            for (int h = 0; h < 4; h++)
                if (t + 256 * h < 1000) xn[h] = xb[t + 256 * h];
        }
        __syncthreads();
        // ---- layer 1: K = 27 taps (padded to 32) of the input
        const bf16x8 B1 = __builtin_bit_cast(bf16x8, W1[lane]);
        const f32x4 bias1 = bias[g];
#pragma unroll 4
        for (int k = 0; k < 8; k++) {
            u32x4 f;
#pragma unroll
            for (int h = 0; h < 4; h++) f[h] = pair[h][100 * k];
            f[1] &= last;
            f[2] &= none;
            f[3] &= none;
            const f32x4 D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B1, __builtin_bit_cast(bf16x8, f), zero, 0, 0, 0);
            u16x4 av;
#pragma unroll
            for (int r = 0; r < 4; r++) av[r] = f2bf_hw(relu(D[r] + bias1[r]));
            *reinterpret_cast<u16x4 *>(A1 + (10 * (k + 1) + j + 1) * kRow + put) = av;
            if (SAVE) {  // a1 for training, [box][channel][cell]
#pragma unroll
                for (int r = 0; r < 4; r++) (a1o + q * 8192)[save + r * 512 + k * 64] = av[r];
            }
        }
        __syncthreads();
        // ---- layer 2, blocked along z.  Each padded input slice zs is loaded
        // once (per x-shift di: the kernel rows dj = 0 | 1 in K groups 0-1 |
        // 2-3, and dj = 2 | nothing) and feeds the three output slices
        // k = zs - dk it reaches; an output slice is complete after its
        // input slice k + 2.  Cells outside and "nothing" are read from the
        // zero y-row 0.
        {
            const uint16_t *srcA[3], *srcB[3];
#pragma unroll
            for (int di = 0; di < 3; di++) {
                const int at = ((i + di - 1) & 7) * 16 + 8 * (g & 1);
                const bool in = (unsigned)(i + di - 1) < 8u;
                srcA[di] = A1 + (in ? (j + (g >> 1)) * kRow : 0) + at;
                srcB[di] = A1 + (in && g < 2 ? (j + 2) * kRow : 0) + at;
            }
            const f32x4 bias2 = bias[4 + g];
            f32x4 acc[3] = {zero, zero, zero};
#pragma unroll
            for (int zs = 0; zs < 10; zs++) {
                bf16x8 FA[3], FB[3];
#pragma unroll
                for (int di = 0; di < 3; di++) {
                    FA[di] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(srcA[di] + 10 * zs * kRow));
                    FB[di] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(srcB[di] + 10 * zs * kRow));
                }
#pragma unroll
                for (int e = 0; e < 6; e++) {  // in each sum: di, then its two fragments
#pragma unroll
                    for (int dk = 0; dk < 3; dk++) {
                        const int k = zs - dk, di = e >> 1;
                        if (k < 0 || k > 7) continue;
                        acc[k % 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B2[(dk * 2 + (e & 1)) * 3 + di],
                                                                             e & 1 ? FB[di] : FA[di], acc[k % 3], 0, 0, 0);
                    }
                }
                const int kd = zs - 2;  // the output slice completed by this input slice
                if (kd >= 0) {
                    u16x4 av;
#pragma unroll
                    for (int r = 0; r < 4; r++) av[r] = f2bf_hw(relu(acc[kd % 3][r] + bias2[r]));
                    *reinterpret_cast<u16x4 *>(A2 + (kd * 8 + j) * kRow + put) = av;
                    if (SAVE) {
#pragma unroll
                        for (int r = 0; r < 4; r++) (a2o + q * 8192)[save + r * 512 + kd * 64] = av[r];
                    }
                    acc[kd % 3] = zero;
                }
            }
        }
        __syncthreads();  // A1 is dead; its space holds Q from here on
        // ---- layer 3: Q[kernel row][cell], from the cells (x - 1 | x) and
        // (x + 1 | nothing) in K groups 0-1 | 2-3
        const bf16x8 B3a = __builtin_bit_cast(bf16x8, W3[0][lane]), B3b = __builtin_bit_cast(bf16x8, W3[1][lane]);
        const int xa = i + (g >> 1) - 1;
        const uint16_t *none3 = reinterpret_cast<const uint16_t *>(Z), *src3 = A2 + j * kRow + 8 * (g & 1);
#pragma unroll 4
        for (int k = 0; k < 8; k++) {
            const uint16_t *pa = xa >= 0 ? src3 + k * 8 * kRow + xa * 16 : none3;
            const uint16_t *pb = g < 2 && i < 7 ? src3 + k * 8 * kRow + (i + 1) * 16 : none3;
            const bf16x8 Fa = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa));
            const bf16x8 Fb = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pb));
            f32x4 D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Fa, B3a, zero, 0, 0, 0);
            D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Fb, B3b, D, 0, 0, 0);
            if (o < 9) *reinterpret_cast<f32x4 *>(Q + o * kQs + 16 * (w + 4 * k) + 4 * g) = D;
        }
        __syncthreads();
        // kernel rows outside the box read a zero
        const int oj = (t >> 2) & 7, ok = t >> 5;
        float2 s[9];
#pragma unroll
        for (int e = 0; e < 9; e++) {
            const int dk = e / 3 - 1, dj = e % 3 - 1;
            const bool in = (dk < 0 ? ok > 0 : dk > 0 ? ok < 7 : true) && (dj < 0 ? oj > 0 : dj > 0 ? oj < 7 : true);
            const float *p = in ? Q + e * kQs + 2 * t + dk * 64 + dj * 8 : reinterpret_cast<const float *>(Z);
            s[e] = *reinterpret_cast<const float2 *>(p);
        }
        float2 sum = make_float2(b3, b3);
#pragma unroll
        for (int e = 0; e < 9; e++) {
            sum.x += s[e].x;
            sum.y += s[e].y;
        }
        __builtin_memcpy(y + q * 512 + 2 * t, &sum, 8);  // y may be aligned to 4 bytes only
    }
}

// ----------------------------------------------------------------- backward
// Loss = mean over boxes and cells of (y - target)^2; gy = 2 (y - target) / N,
// gz2 = (transposed conv of gy with W3) * [a2 > 0], gz1 = (transposed conv of
// gz2 with W2) * [a1 > 0], and the weight gradients dW3 = <gy, a2>, dW2 =
// <gz2, a1>, dW1 = <gz1, x> over the cells, with the BF16-rounded weights the
// forward used.  Every product has one BF16 factor (a weight, an activation
// or the input) and one FP32 factor g.  The FP32 one is split exactly into
// three BF16 values g = hi + mid + lo (8 significand bits each, by
// truncation), so three BF16 MFMAs give the exact products with FP32
// accumulation: no gradient is rounded below 32 bits.
struct Split3 {
    uint32_t p[3];  // BF16 patterns in the high halves
};
__device__ __forceinline__ Split3 split3(float v) {
    Split3 s;
    s.p[0] = __float_as_uint(v) & 0xffff0000u;
    // a non-finite value is its own high part (inf - inf would turn it into a NaN)
    float r = v - __uint_as_float(s.p[0]);
    r = __builtin_isfinite(v) ? r : 0.0f;
    s.p[1] = __float_as_uint(r) & 0xffff0000u;
    s.p[2] = __float_as_uint(r - __uint_as_float(s.p[1]));
    return s;
}
// Eight values as three MFMA operands (a lane's eight K entries)
__device__ __forceinline__ void split_frag(const float v[8], bf16x8 f[3]) {
    u32x4 d[3];
#pragma unroll
    for (int h = 0; h < 4; h++) {
        const Split3 a = split3(v[2 * h]), b = split3(v[2 * h + 1]);
#pragma unroll
        for (int s = 0; s < 3; s++) d[s][h] = (a.p[s] >> 16) | (b.p[s] & 0xffff0000u);
    }
#pragma unroll
    for (int s = 0; s < 3; s++) f[s] = __builtin_bit_cast(bf16x8, d[s]);
}
__device__ __forceinline__ f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// Eight consecutive BF16 values from position e of an LDS array (a lane's
// eight x-neighbours; e may be odd): five dwords, shifted by a half.
__device__ __forceinline__ bf16x8 row8(const uint16_t *p, int e) {
    const uint32_t *d = reinterpret_cast<const uint32_t *>(p) + (e >> 1);
    const uint32_t sh = (e & 1) * 16;
    u32x4 o;
    uint32_t lo = d[0];
#pragma unroll
    for (int h = 0; h < 4; h++) {
        const uint32_t hi = d[h + 1];
        o[h] = __builtin_amdgcn_alignbit(hi, lo, sh);
        lo = hi;
    }
    return __builtin_bit_cast(bf16x8, o);
}

// Operand fragments of the transposed convolutions, in k_nn_pack's lane
// order: first W2 with input and output channels and the tap direction
// exchanged (18 fragments, rows paired as in the forward), then W3 [27 taps,
// padded to 32][16 channels].
constexpr int kPT3 = 18 * 512, kPackedT = kPT3 + 512;
static_assert(kPackedT % 256 == 0 && kPackedT * 2 <= kNnParams * 4, "one thread per entry; fits in one partial gradient");
__global__ __launch_bounds__(256) void k_nn_pack_t(const float *__restrict__ prm, uint16_t *__restrict__ pk) {
    const int e = blockIdx.x * 256 + threadIdx.x;  // grid: kPackedT / 256
    const int lane = (e & 511) >> 3, q = e & 7, n = lane & 15, g = lane >> 4;
    float v = 0.0f;
    if (e < kPT3) {
        const int f = e >> 9, dk = f / 6, type = (f / 3) & 1, di = f % 3, o = 8 * (g & 1) + q;
        const int dj = type == 0 ? (g < 2 ? 0 : 1) : (g < 2 ? 2 : -1);
        if (dj >= 0) v = prm[kW2 + (o * 16 + n) * 27 + ((2 - dk) * 3 + 2 - dj) * 3 + 2 - di];
    } else if (8 * g + q < 27) {
        v = prm[kW3 + n * 27 + 8 * g + q];
    }
    pk[e] = f2bf(v);
}

// gy of box q into three zero-padded 10^3 arrays of BF16 parts (positions
// kGyLen apart); the padding is cleared once, before the first box.
constexpr int kGyLen = 1016;
__device__ __forceinline__ void gy_store(uint16_t *gys, int c, float v) {
    const Split3 s = split3(v);
    const int at = (((c >> 6) + 1) * 10 + ((c >> 3) & 7) + 1) * 10 + (c & 7) + 1;
#pragma unroll
    for (int h = 0; h < 3; h++) gys[h * kGyLen + at] = (uint16_t)(s.p[h] >> 16);
}

// gz2, gz1 (FP32, [box][channel][cell]) and the box's sum of squared errors.
// Persistent workgroups of 4 waves, one box at a time; tiles of 16 cells as in
// the forward, wave w owning the tiles of y-rows (2w, 2w+1), so that gz2 stays
// in the registers of the wave that formed it.  gz2 is one MFMA per part and
// tile (K = 27 taps); gz1 is the forward's z-blocked layer 2 on the transposed
// weights, once per part of gz2, which goes through one padded LDS buffer
// [cell][channel] in turn while the eight output tiles accumulate in
// registers.  Bound by the LDS reads of the padded buffer (180 16-byte reads
// a lane and box) and the 432 MFMAs a wave and box: 40 us for 1024 boxes
// (FP32 multiply-adds, each reading one LDS operand, took 299 us).
constexpr int kNnActBlocks = 512;  // 2 per CU: at 3 (168 registers) the weights, gz2 and the eight sums spill
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_nn_bwd_act(
    const float *__restrict__ y, const float *__restrict__ tgt, const int32_t *__restrict__ idx, int64_t nbox,
    const uint16_t *__restrict__ a1o, const uint16_t *__restrict__ a2o, const uint16_t *__restrict__ pkt,
    float scale2, float *__restrict__ gz2o, float *__restrict__ gz1o, double *__restrict__ lossp) {
    constexpr int kGy = 168, kGz = 10 * kGy, kG = 10 * kGz;  // as A1 in the forward
    __shared__ __attribute__((aligned(16))) uint16_t G[kG];
    __shared__ __attribute__((aligned(16))) uint16_t gys[3 * kGyLen];
    __shared__ double S[4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, row = lane & 15, g = lane >> 4, n = lane & 15;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 B2[18];
#pragma unroll
    for (int f = 0; f < 18; f++)
        B2[f] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(pkt + (f * 64 + lane) * 8));
    const bf16x8 B3 = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(pkt + kPT3 + lane * 8));
    // this lane's eight taps of gy, from its cell of the wave's tile at k = 0
    // (taps 27-31 are masked to 0: their weights are, but 0 * inf is not)
    const uint16_t *gt[8];
    uint32_t tm[4];
#pragma unroll
    for (int h = 0; h < 8; h++) {
        const int tp = 8 * g + h < 27 ? 8 * g + h : 26;
        gt[h] = gys + 222 + (2 * w + (row >> 3)) * 10 + (row & 7) - tap_off(tp);
        if (!(h & 1)) tm[h >> 1] = (8 * g + h < 27 ? 0xffffu : 0u) | (8 * g + h + 1 < 27 ? 0xffff0000u : 0u);
    }
    // the padding of both buffers stays 0: only interior cells are written
    for (int e = t; e < kG / 8; e += 256) reinterpret_cast<uint4 *>(G)[e] = make_uint4(0, 0, 0, 0);
    for (int e = t; e < 3 * kGyLen / 8; e += 256) reinterpret_cast<uint4 *>(gys)[e] = make_uint4(0, 0, 0, 0);
    for (int64_t q = blockIdx.x; q < nbox; q += gridDim.x) {
        const int64_t src = idx ? (int64_t)idx[q] : q;
        __syncthreads();  // the buffers are cleared, or the previous box is done with them
        double ls = 0.0;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int c = t + 256 * h;
            const float d = y[q * 512 + c] - tgt[src * 512 + c];
            ls += (double)d * (double)d;
            gy_store(gys, c, scale2 * d);
        }
        const double tot = block_sum256(ls, S);  // also orders the writes of gys before the reads below
        if (t == 0) lossp[q] = tot;
        f32x4 gz2[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int m = 4 * k + w;
            const u16x4 mask = *reinterpret_cast<const u16x4 *>(a2o + (q * 16 + n) * 512 + 16 * m + 4 * g);
            f32x4 D = zero;
#pragma unroll
            for (int s = 0; s < 3; s++) {
                u32x4 A;
#pragma unroll
                for (int h = 0; h < 4; h++)
                    A[h] = tm[h] & (gt[2 * h][s * kGyLen + k * 100] |
                                    ((uint32_t)gt[2 * h + 1][s * kGyLen + k * 100] << 16));
                D = mfma32(__builtin_bit_cast(bf16x8, A), B3, D);
            }
#pragma unroll
            for (int r = 0; r < 4; r++) gz2[k][r] = (mask[r] & 0x7fff) ? D[r] : 0.0f;
            *reinterpret_cast<f32x4 *>(gz2o + (q * 16 + n) * 512 + 16 * m + 4 * g) = gz2[k];
            __builtin_amdgcn_sched_barrier(0);  // one tile's gathers at a time: hoisted, they spill
        }
        f32x4 acc[8];
#pragma unroll
        for (int k = 0; k < 8; k++) acc[k] = zero;
        const int i = row & 7, jj = 2 * w + (row >> 3);
        const int colA = (g < 2 ? 0 : 1) * kGy, colB = 2 * kGy;  // kernel row of each K group
#pragma unroll 1
        for (int s = 0; s < 3; s++) {
            if (s > 0) __syncthreads();  // the previous part has been read
#pragma unroll
            for (int k = 0; k < 8; k++) {
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int cr = 4 * g + r;  // cell within the tile: x, and which of the two y-rows
                    const uint32_t u = __float_as_uint(gz2[k][r]);
                    G[(k + 1) * kGz + (2 * w + (cr >> 3) + 1) * kGy + ((cr & 7) + 1) * 16 + n] = (uint16_t)(u >> 16);
                    // what is left for the next part
                    gz2[k][r] = __builtin_isfinite(gz2[k][r])
                                    ? gz2[k][r] - __uint_as_float(u & 0xffff0000u) : 0.0f;
                }
            }
            __syncthreads();
#pragma unroll
            for (int zs = 0; zs < 10; zs++) {
                const uint16_t *src2 = G + zs * kGz + jj * kGy + i * 16 + 8 * (g & 1);
                uint4 FA[3], FB[3];
#pragma unroll
                for (int di = 0; di < 3; di++) {
                    FA[di] = *reinterpret_cast<const uint4 *>(src2 + colA + di * 16);
                    FB[di] = g < 2 ? *reinterpret_cast<const uint4 *>(src2 + colB + di * 16) : make_uint4(0, 0, 0, 0);
                }
#pragma unroll
                for (int dk = 0; dk < 3; dk++) {
                    const int k = zs - dk;
                    if (k < 0 || k > 7) continue;
#pragma unroll
                    for (int di = 0; di < 3; di++) {
                        acc[k] = mfma32(__builtin_bit_cast(bf16x8, FA[di]), B2[(dk * 2 + 0) * 3 + di], acc[k]);
                        acc[k] = mfma32(__builtin_bit_cast(bf16x8, FB[di]), B2[(dk * 2 + 1) * 3 + di], acc[k]);
                    }
                }
                if (zs & 1) __builtin_amdgcn_sched_barrier(0);  // two slices' loads in flight
            }
        }
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int64_t at = (q * 16 + n) * 512 + 16 * (4 * k + w) + 4 * g;
            const u16x4 mask = *reinterpret_cast<const u16x4 *>(a1o + at);
            f32x4 o;
#pragma unroll
            for (int r = 0; r < 4; r++) o[r] = (mask[r] & 0x7fff) ? acc[k][r] : 0.0f;
            *reinterpret_cast<f32x4 *>(gz1o + at) = o;
        }
    }
}

// Weight gradients: workgroup r sums over boxes r, r + gridDim.x, ... in MFMA
// accumulators and writes its partial gradient (parameter order) to
// part[r][kNnParams].  Each product is a GEMM over the 512 cells, 32 (four
// x-rows) a step, the steps dealt to the four waves: a lane's eight K entries
// are one x-row.
//  dW2[o][c][tap]: rows o = gz2 (read once, straight from memory, and split),
//    columns c = a1 shifted by the tap: 27 accumulators; a1 sits zero-padded
//    and channel-major in LDS, and one read of a row of 10 serves the three
//    x-shifts.
//  dW1[o][tap]: rows o = gz1, columns the taps of x (27 of 32; column 27 is
//    ones and gives db1).
//  dW3[c][tap]: rows c = a2 (straight from memory), columns the taps of gy.
// 1024 boxes: 44 us, bound by the latency of the two workgroups a CU that the
// 27 accumulators allow (an FP32 vector version with one LDS read per
// multiply-add took 633 us).
constexpr int kUrow = 12, kUch = 1204;  // u16 per padded x-row (8-byte rows) and per channel
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_nn_wgrad(
    const float *__restrict__ x, const float *__restrict__ y, const float *__restrict__ tgt,
    const int32_t *__restrict__ idx, int64_t nbox, float scale2, const uint16_t *__restrict__ a1o,
    const uint16_t *__restrict__ a2o, const float *__restrict__ gz2o, const float *__restrict__ gz1o,
    float *__restrict__ part) {
    __shared__ __attribute__((aligned(16))) uint16_t U[16 * kUch];
    __shared__ __attribute__((aligned(16))) uint16_t xs[1016];
    __shared__ __attribute__((aligned(16))) uint16_t gys[3 * kGyLen];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, n = lane & 15, g = lane >> 4;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 acc2[27], acc1[2], acc3[2];
#pragma unroll
    for (int tp = 0; tp < 27; tp++) acc2[tp] = zero;
    acc1[0] = acc1[1] = acc3[0] = acc3[1] = zero;
    float db2 = 0.0f, db3 = 0.0f;
    // tap of this lane's column in the two column tiles (columns 27-31 are unused or ones)
    int xoff[2], goff[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int tp = 16 * h + n < 27 ? 16 * h + n : 0;
        xoff[h] = tap_off(tp);
        goff[h] = 222 - tap_off(tp);
    }
    const bool ones = n == 27 - 16;
    for (int e = t; e < 16 * kUch / 4; e += 256) reinterpret_cast<uint2 *>(U)[e] = make_uint2(0, 0);
    for (int e = t; e < 3 * kGyLen / 8; e += 256) reinterpret_cast<uint4 *>(gys)[e] = make_uint4(0, 0, 0, 0);
    if (t < 16) xs[1000 + t] = 0;
    for (int64_t q = blockIdx.x; q < nbox; q += gridDim.x) {
        const int64_t src = idx ? (int64_t)idx[q] : q;
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 4; h++) {  // row r of 64 of channel ch, written one cell to the right
            const int e = t + 256 * h, ch = e >> 6, r = e & 63;
            const uint4 v = *reinterpret_cast<const uint4 *>(a1o + (q * 16 + ch) * 512 + r * 8);
            uint32_t *d = reinterpret_cast<uint32_t *>(U + ch * kUch + (((r >> 3) + 1) * 10 + (r & 7) + 1) * kUrow);
            *reinterpret_cast<uint2 *>(d) = make_uint2(v.x << 16, __builtin_amdgcn_alignbit(v.y, v.x, 16));
            *reinterpret_cast<uint2 *>(d + 2) =
                make_uint2(__builtin_amdgcn_alignbit(v.z, v.y, 16), __builtin_amdgcn_alignbit(v.w, v.z, 16));
            d[4] = v.w >> 16;
        }
#pragma unroll
        for (int h = 0; h < 4; h++)
            if (t + 256 * h < 1000) xs[t + 256 * h] = f2bf(x[src * 1000 + t + 256 * h]);
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int c = t + 256 * h;
            const float v = scale2 * (y[q * 512 + c] - tgt[src * 512 + c]);
            db3 += v;
            gy_store(gys, c, v);
        }
        __syncthreads();
#pragma unroll 1
        for (int st = 0; st < 4; st++) {
            const int k = 2 * w + (st >> 1), j = 4 * (st & 1) + g;  // this lane's x-row
            const int64_t at = (q * 16 + n) * 512 + (k * 8 + j) * 8;
            float v2[8], v1[8];
            *reinterpret_cast<f32x4 *>(v2) = *reinterpret_cast<const f32x4 *>(gz2o + at);
            *reinterpret_cast<f32x4 *>(v2 + 4) = *reinterpret_cast<const f32x4 *>(gz2o + at + 4);
            *reinterpret_cast<f32x4 *>(v1) = *reinterpret_cast<const f32x4 *>(gz1o + at);
            *reinterpret_cast<f32x4 *>(v1 + 4) = *reinterpret_cast<const f32x4 *>(gz1o + at + 4);
            const bf16x8 a2 = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(a2o + at));
            db2 += ((v2[0] + v2[1]) + (v2[2] + v2[3])) + ((v2[4] + v2[5]) + (v2[6] + v2[7]));
            bf16x8 A[3];
            split_frag(v2, A);
#pragma unroll
            for (int r = 0; r < 9; r++) {  // kernel rows (dk, dj) = (r / 3, r % 3)
                const uint32_t *d = reinterpret_cast<const uint32_t *>(
                    U + n * kUch + ((k + r / 3) * 10 + j + r % 3) * kUrow);
                const uint2 d01 = *reinterpret_cast<const uint2 *>(d), d23 = *reinterpret_cast<const uint2 *>(d + 2);
                const uint32_t d4 = d[4];
                const u32x4 b[3] = {{d01.x, d01.y, d23.x, d23.y},
                                    {__builtin_amdgcn_alignbit(d01.y, d01.x, 16),
                                     __builtin_amdgcn_alignbit(d23.x, d01.y, 16),
                                     __builtin_amdgcn_alignbit(d23.y, d23.x, 16),
                                     __builtin_amdgcn_alignbit(d4, d23.y, 16)},
                                    {d01.y, d23.x, d23.y, d4}};
#pragma unroll
                for (int s = 0; s < 3; s++)
#pragma unroll
                    for (int di = 0; di < 3; di++)
                        acc2[3 * r + di] = mfma32(A[s], __builtin_bit_cast(bf16x8, b[di]), acc2[3 * r + di]);
            }
            split_frag(v1, A);
            const int rowx = (k * 10 + j) * 10;
            bf16x8 X[2] = {row8(xs, rowx + xoff[0]), row8(xs, rowx + xoff[1])};
            const u32x4 one = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
            if (ones) X[1] = __builtin_bit_cast(bf16x8, one);
#pragma unroll
            for (int s = 0; s < 3; s++)
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    acc1[h] = mfma32(A[s], X[h], acc1[h]);
                    acc3[h] = mfma32(a2, row8(gys + s * kGyLen, rowx + goff[h]), acc3[h]);
                }
        }
    }
    // the four waves' sums, added in wave order in LDS and written by all
    float *P = reinterpret_cast<float *>(U);  // dW2 [16][16][27], then dW1, db1 [16][28], dW3 [16][27], db2 [16], db3
    constexpr int oP1 = 6912, oP3 = oP1 + 448, oPb = oP3 + 432;
    static_assert((oPb + 17) * 4 <= 16 * kUch * 2, "the sums fit in the activations' space");
    db2 += __shfl_xor(db2, 16);
    db2 += __shfl_xor(db2, 32);
    for (int off = 32; off > 0; off >>= 1) db3 += __shfl_xor(db3, off);
    for (int v = 0; v < 4; v++) {
        __syncthreads();
        if (v != w) continue;
        auto add = [&](int at, float val) { P[at] = v ? P[at] + val : val; };
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int o = 4 * g + r;
#pragma unroll
            for (int tp = 0; tp < 27; tp++) add((o * 16 + n) * 27 + tp, acc2[tp][r]);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                if (16 * h + n < 28) add(oP1 + o * 28 + 16 * h + n, acc1[h][r]);
                if (16 * h + n < 27) add(oP3 + o * 27 + 16 * h + n, acc3[h][r]);
            }
        }
        if (lane < 16) add(oPb + n, db2);
        if (lane == 0) add(oPb + 16, db3);
    }
    __syncthreads();
    float *pr = part + (int64_t)blockIdx.x * kNnParams;
    for (int e = t; e < kNnParams; e += 256) {
        int at;
        if (e < kB1) at = oP1 + e / 27 * 28 + e % 27;
        else if (e < kW2) at = oP1 + (e - kB1) * 28 + 27;
        else if (e < kB2) at = e - kW2;
        else if (e < kW3) at = oPb + e - kB2;
        else if (e < kB3) at = oP3 + e - kW3;
        else at = oPb + 16;
        pr[e] = P[at];
    }
}

// grad[p] = sum over workgroups of part[r][p] (FP64, fixed order: 8 strided
// sums, then their sum); block 0 also writes the mean squared error.  32
// parameters x 8 rows a block: the rows of a parameter are summed by 8
// threads instead of one (512 rows: 7 us against 132, a chain of 512 loads).
__global__ __launch_bounds__(256) void k_nn_reduce(const float *__restrict__ part, int nblk,
                                                   const double *__restrict__ lossp, int64_t nbox,
                                                   float *__restrict__ grad, double *__restrict__ loss) {
    __shared__ double R[8][32];
    const int t = threadIdx.x, c = t & 31, rw = t >> 5, p = blockIdx.x * 32 + c;
    double s = 0.0;
    if (p < kNnParams) {
#pragma unroll 8
        for (int r = rw; r < nblk; r += 8) s += (double)part[(int64_t)r * kNnParams + p];
    }
    R[rw][c] = s;
    __syncthreads();
    if (rw == 0 && p < kNnParams)
        grad[p] = (float)(((R[0][c] + R[1][c]) + (R[2][c] + R[3][c])) + ((R[4][c] + R[5][c]) + (R[6][c] + R[7][c])));
    if (blockIdx.x == 0) {
        __shared__ double S[4];
        double v = 0.0;
        for (int64_t b = threadIdx.x; b < nbox; b += 256) v += lossp[b];
        double tot = block_sum256(v, S);
        if (threadIdx.x == 0) *loss = tot / (512.0 * (double)nbox);
    }
}

__global__ __launch_bounds__(256) void k_nn_adam(float *__restrict__ p, float *__restrict__ m,
                                                 float *__restrict__ v, const float *__restrict__ g,
                                                 float lr, float b1, float b2, float eps, float bc1,
                                                 float bc2) {
    int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= kNnParams) return;
    float gg = g[e];
    float mm = b1 * m[e] + (1.0f - b1) * gg;
    float vv = b2 * v[e] + (1.0f - b2) * gg * gg;
    m[e] = mm;
    v[e] = vv;
    p[e] -= lr * (mm / bc1) / (sqrtf(vv / bc2) + eps);
}

// ------------------------------------------------------- learned tree step
// Network input of leaf position q: h^2 r on the box and on the face-ghost
// layers taken from same-level leaf neighbours (0 elsewhere), divided by the
// box's RMS of h^2 r (1 when that is 0).  Each XCD takes a contiguous share of
// the boxes (neighbours' values from its own L2), wave d loads the ghosts of
// face d, waves 0-1 those of faces 4-5 too, and all loads go out before the
// first store: 16164 boxes 47 us before, now 33.
__global__ __launch_bounds__(256) void k_nn_gather(const float *__restrict__ r32,
                                                   const int32_t *__restrict__ leaf, int64_t nleaf,
                                                   const int32_t *__restrict__ nbr,
                                                   const int32_t *__restrict__ cfslot,
                                                   const int32_t *__restrict__ ijk4, double len,
                                                   float *__restrict__ x, float *__restrict__ scale) {
    __shared__ __attribute__((aligned(16))) float X[1000];
    __shared__ double S[4];
    const int64_t q = (int64_t)(blockIdx.x & 7) * ((nleaf + 7) >> 3) + (blockIdx.x >> 3);
    if (q >= nleaf) return;
    const int64_t b = leaf[q];
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), u = t & 7, v = (t >> 3) & 7;
    const float r0 = r32[b * 512 + t], r1 = r32[b * 512 + 256 + t];
    float gh[2] = {0.0f, 0.0f};
    int at[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        const int d = min(w + 4 * r, 5), a = d >> 1, side = d & 1;
        const int i = side ? 0 : 7, p = side ? 9 : 0;  // the layer in the neighbour and in X
        const int nb = nbr[b * 6 + d];
        if (nb >= 0 && cfslot[b * 6 + d] != -2 && w + 4 * r < 6)  // a leaf (-2: it has children)
            gh[r] = r32[(int64_t)nb * 512 + (a == 0 ? cs_idx(i, u, v) : a == 1 ? cs_idx(u, i, v) : cs_idx(u, v, i))];
        at[r] = a == 0 ? ((v + 1) * 10 + u + 1) * 10 + p : a == 1 ? ((v + 1) * 10 + p) * 10 + u + 1 : (p * 10 + v + 1) * 10 + u + 1;
    }
    const int l = ijk4[b * 4 + 3];
    const double h = len / (8.0 * (double)(1 << (l - 1)));
    const float h2 = (float)(h * h);
    for (int e = t; e < 1000; e += 256) X[e] = 0.0f;
    __syncthreads();
    double ss = 0.0;
#pragma unroll
    for (int c = 0; c < 2; c++) {
        const int n = cs_to_nat(t + 256 * c), i = n & 7, j = (n >> 3) & 7, k = n >> 6;
        const float z = h2 * (c ? r1 : r0);
        X[((k + 1) * 10 + j + 1) * 10 + i + 1] = z;
        ss += (double)z * (double)z;
    }
    X[at[0]] = h2 * gh[0];
    if (w < 2) X[at[1]] = h2 * gh[1];
    double tot = block_sum256(ss, S);  // also orders the X writes before the reads below
    float rms = (float)sqrt(tot / 512.0);
    float sc = rms > 0.0f ? rms : 1.0f;
    if (t < 250) {
        float4 z = reinterpret_cast<const float4 *>(X)[t];
        z.x /= sc;
        z.y /= sc;
        z.z /= sc;
        z.w /= sc;
        __builtin_memcpy(x + q * 1000 + 4 * t, &z, 16);  // x may be aligned to 4 bytes only
    }
    if (t == 0) scale[q] = sc;
}

// e32 on the listed leaf boxes <- scale * y.
__global__ __launch_bounds__(256) void k_nn_scatter(const float *__restrict__ y,
                                                    const float *__restrict__ scale,
                                                    const int32_t *__restrict__ leaf,
                                                    float *__restrict__ e32) {
    const int64_t q = blockIdx.x;
    const int64_t b = leaf[q];
    const float sc = scale[q];
    for (int e = threadIdx.x; e < 512; e += 256) e32[b * 512 + e] = sc * y[q * 512 + cs_to_nat(e)];
}

// Per listed box: the volume-weighted sums <r, q> and <q, q> of one column
// (the per-level learned step).
__global__ __launch_bounds__(256) void k_nn_dots1(const float *__restrict__ r32, const float *__restrict__ q,
                                                  const int32_t *__restrict__ list,
                                                  const int32_t *__restrict__ ijk4, double len,
                                                  double *__restrict__ partial) {
    __shared__ double S[4];
    const int64_t p = blockIdx.x;
    const int64_t b = list[p];
    const int t = threadIdx.x;
    const int l = ijk4[b * 4 + 3];
    const double h = len / (8.0 * (double)(1 << (l - 1)));
    double rq = 0.0, qq = 0.0;
    for (int e = t; e < 512; e += 256) {
        double r = r32[b * 512 + e], c = q[p * 512 + e];
        rq += r * c;
        qq += c * c;
    }
    const double vol = h * h * h;
    double a = block_sum256(rq, S);
    double c = block_sum256(qq, S);
    if (t == 0) {
        partial[2 * p] = a * vol;
        partial[2 * p + 1] = c * vol;
    }
}

// phi += steps[tree][level] * (scale * y) on the leaf boxes (boxes whose
// step is 0 are left untouched, also where the correction is not finite).
__global__ __launch_bounds__(256) void k_nn_update(double *__restrict__ phi,
                                                   const float *__restrict__ y,
                                                   const float *__restrict__ scale,
                                                   const int32_t *__restrict__ leaf,
                                                   const int32_t *__restrict__ ijk4,
                                                   const int32_t *__restrict__ tid,
                                                   const double *__restrict__ steps, int stride) {
    const int64_t q = blockIdx.x;
    const int64_t b = leaf[q];
    const int l = ijk4[b * 4 + 3];
    const double st = steps[(int64_t)tid[b] * stride + l];
    const float sc = scale[q];
    if (st == 0.0) return;
    for (int e = threadIdx.x; e < 512; e += 256) {
        float c = sc * y[q * 512 + cs_to_nat(e)];
        phi[b * 512 + e] += st * (double)c;
    }
}

// Training target of leaf position q: (ref - phi) / scale in natural order,
// ref in natural order [n][512].
__global__ __launch_bounds__(256) void k_nn_targets(const double *__restrict__ phi,
                                                    const double *__restrict__ ref,
                                                    const float *__restrict__ scale,
                                                    const int32_t *__restrict__ leaf,
                                                    float *__restrict__ target) {
    const int64_t q = blockIdx.x;
    const int64_t b = leaf[q];
    const double sc = scale[q];
    for (int e = threadIdx.x; e < 512; e += 256) {
        int n = cs_to_nat(e);
        target[q * 512 + n] = (float)((ref[b * 512 + n] - phi[b * 512 + e]) / sc);
    }
}

}  // namespace

int64_t nn_train_layout(int64_t nbox, char *base, NnTrainWs *w) {
    int64_t o = 0;
    auto take = [&](int64_t bytes) {
        int64_t at = o;
        o += nn_align256(bytes);
        return at;
    };
    int64_t oy = take(4 * 512 * nbox), oa1 = take(2 * 8192 * nbox), oa2 = take(2 * 8192 * nbox);
    int64_t og2 = take(4 * 8192 * nbox), og1 = take(4 * 8192 * nbox), olp = take(8 * nbox);
    int64_t opart = take(4 * nn_wgrad_blocks(nbox) * kNnParams), oloss = take(8);
    if (base && w) {
        w->y = (float *)(base + oy);
        w->a1 = (uint16_t *)(base + oa1);
        w->a2 = (uint16_t *)(base + oa2);
        w->gz2 = (float *)(base + og2);
        w->gz1 = (float *)(base + og1);
        w->lossp = (double *)(base + olp);
        w->part = (float *)(base + opart);
        w->loss = (double *)(base + oloss);
    }
    return o;
}

void launch_nn_pack(const float *prm, uint16_t *pk, hipStream_t s) {
    hipLaunchKernelGGL(k_nn_pack, dim3(kNnPacked / 256), dim3(256), 0, s, prm, pk);
}

void launch_nn_forward(const float *prm, const uint16_t *pk, int64_t nbox, const int32_t *idx,
                       const float *x, float *y, uint16_t *a1, uint16_t *a2, hipStream_t s) {
    if (nbox <= 0) return;
    unsigned grid = (unsigned)(nbox < kNnFwdBlocks ? nbox : kNnFwdBlocks);
    if (a1)
        hipLaunchKernelGGL(k_nn_fwd<true>, dim3(grid), dim3(kFwdThreads), 0, s, x, y, idx, nbox, pk, prm,
                           a1, a2);
    else
        hipLaunchKernelGGL(k_nn_fwd<false>, dim3(grid), dim3(kFwdThreads), 0, s, x, y, idx, nbox, pk, prm,
                           a1, a2);
}

void launch_nn_backward(const float *prm, int64_t nbox, const int32_t *idx, const float *x,
                        const float *target, const NnTrainWs &w, float *grad, hipStream_t s) {
    if (nbox <= 0) return;
    float scale2 = (float)(2.0 / (512.0 * (double)nbox));
    // the partial gradients' buffer holds the transposed weights until the
    // weight-gradient kernel writes it
    uint16_t *pkt = reinterpret_cast<uint16_t *>(w.part);
    hipLaunchKernelGGL(k_nn_pack_t, dim3(kPackedT / 256), dim3(256), 0, s, prm, pkt);
    unsigned grid = (unsigned)(nbox < kNnActBlocks ? nbox : kNnActBlocks);
    hipLaunchKernelGGL(k_nn_bwd_act, dim3(grid), dim3(256), 0, s, w.y, target, idx, nbox, w.a1, w.a2,
                       (const uint16_t *)pkt, scale2, w.gz2, w.gz1, w.lossp);
    int nblk = (int)nn_wgrad_blocks(nbox);
    hipLaunchKernelGGL(k_nn_wgrad, dim3((unsigned)nblk), dim3(256), 0, s, x, w.y, target, idx, nbox,
                       scale2, w.a1, w.a2, w.gz2, w.gz1, w.part);
    hipLaunchKernelGGL(k_nn_reduce, dim3((kNnParams + 31) / 32), dim3(256), 0, s, w.part, nblk,
                       w.lossp, nbox, grad, w.loss);
}

void launch_nn_adam(float *prm, float *m, float *v, const float *g, float lr, float b1, float b2,
                    float eps, float bc1, float bc2, hipStream_t s) {
    hipLaunchKernelGGL(k_nn_adam, dim3((kNnParams + 255) / 256), dim3(256), 0, s, prm, m, v, g, lr, b1,
                       b2, eps, bc1, bc2);
}

void launch_nn_gather(const float *r32, const int32_t *leaf, int64_t nleaf, const int32_t *nbr,
                      const int32_t *cfslot, const int32_t *ijk4, double len, float *x, float *scale, hipStream_t s) {
    if (nleaf <= 0) return;
    hipLaunchKernelGGL(k_nn_gather, dim3((unsigned)(8 * ((nleaf + 7) >> 3))), dim3(256), 0, s, r32, leaf, nleaf, nbr,
                       cfslot, ijk4, len, x, scale);
}

void launch_nn_scatter(const float *y, const float *scale, const int32_t *leaf, int64_t nleaf, float *e32,
                       hipStream_t s) {
    if (nleaf <= 0) return;
    hipLaunchKernelGGL(k_nn_scatter, dim3((unsigned)nleaf), dim3(256), 0, s, y, scale, leaf, e32);
}

void launch_nn_dots1(const float *r32, const float *q, const int32_t *list, int64_t n, const int32_t *ijk4,
                     double len, double *partial, hipStream_t s) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_nn_dots1, dim3((unsigned)n), dim3(256), 0, s, r32, q, list, ijk4, len, partial);
}

void launch_nn_update(double *phi, const float *y, const float *scale, const int32_t *leaf,
                      int64_t nleaf, const int32_t *ijk4, const int32_t *tid, const double *steps,
                      int stride, hipStream_t s) {
    if (nleaf <= 0) return;
    hipLaunchKernelGGL(k_nn_update, dim3((unsigned)nleaf), dim3(256), 0, s, phi, y, scale, leaf, ijk4, tid,
                       steps, stride);
}

void launch_nn_targets(const double *phi, const double *ref, const float *scale,
                       const int32_t *leaf, int64_t nleaf, float *target, hipStream_t s) {
    if (nleaf <= 0) return;
    hipLaunchKernelGGL(k_nn_targets, dim3((unsigned)nleaf), dim3(256), 0, s, phi, ref, scale, leaf,
                       target);
}

// ------------------------------------------------ allocation-free training
// The training buffers of mg_nn_gradient_static: one file-scope array, which
// every GPU the library runs on holds until the process ends.  In host code
// the name `scratch` is only a stand-in for the device address; the address
// on the current device comes from hipGetSymbolAddress, once per device.
__device__ __align__(256) char scratch[kNnStaticBytes];

namespace {
std::mutex g_scratch_mu;
std::vector<void *> g_scratch_ptr;  // device address of `scratch`, per device
}  // namespace

int nn_static_workspace(int device, void **out) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= device) g_scratch_ptr.resize(device + 1, nullptr);
    if (!g_scratch_ptr[device]) {
        int cur = 0;
        if (hipGetDevice(&cur) != hipSuccess) return MG_EHIP;
        if (cur != device && hipSetDevice(device) != hipSuccess) return MG_EHIP;
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess || !p) return MG_EHIP;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return MG_OK;
}

}  // namespace mg
