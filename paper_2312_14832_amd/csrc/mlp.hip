// Warm-start network for parametric LPs: forward, backward and Adam on the
// GPU with hand-written kernels.
//
// The network maps a sketch of an instance's perturbation (in_dim features,
// standardized) through `layers` ReLU layers of width `hidden` to `rank`
// coefficients alpha, and then through a linear layer of width out_dim (a
// rank-`rank` factor whose bias starts at the base solution) to a predicted
// primal-dual point z = (x, y) that seeds the solver.  Shapes are row-major
// with the batch as the leading dimension: Y[B x N] = X[B x K] W[K x N] + b.
//
// GEMMs: LDS-tiled kernels.
//   BF16 mode: operands rounded to bfloat16, products on MFMA
//     (v_mfma_f32_32x32x16_bf16, gfx950), FP32 accumulation over K in
//     ascending steps of 16 whatever the tile, so the tile size changes no
//     bit of a result: 256x256, 128x128 or 64x64 outputs per workgroup
//     (k_gemm_mfma), picked by how well they fill the GPU (mfma_tile).
//   FP32 mode: 64x64 or 128x128 tiles with FP32 FMA (every thread 4x4 blocks,
//     k_gemm_fp32); used to check gradients against the FP64 reference at FP32
//     accuracy.
// Long reductions (dL/dalpha contracts over out_dim) are split over
// workgroups and the partial tiles are summed in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "host_util.h"
#include "lp.h"

namespace pdlp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// float -> bfloat16, round to nearest even (NaN kept quiet)
__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// ----------------------------------------------------------------------------
// FP32 GEMM
// ----------------------------------------------------------------------------

constexpr int GT = 64;   // output tile that splits of K are counted by
constexpr int GK = 32;   // the unit of a split of K

// element (r, c) of op(X) where op(X) is R x C; stored [R x C] (ld) or, when
// transposed, [C x R]
template <bool TR>
__device__ __forceinline__ float load_op(const float *X, int ld, int r, int c, int R, int Cc)
{
    if (r >= R || c >= Cc) return 0.0f;
    return X[TR ? (size_t)c * ld + r : (size_t)r * ld + c];
}

// This thread's vectors of four of one staged operand: T rows of op(X)^T from
// r0 on, FK of k from k0 on.  KC: k contiguous in memory, otherwise the rows
// are.  Any alignment (a global load takes any address of a float); what lies
// past R or ke is zero.
constexpr int FK = 16;   // K per LDS stage
template <bool KC, int T>
__device__ __forceinline__ void fp32_load(float4 *out, const float *X, int ld, int R, int r0, int k0, int ke)
{
#pragma unroll
    for (int h = 0; h < T * FK / 1024; ++h) {
        const int v = (int)threadIdx.x + 256 * h;
        const int r = r0 + (KC ? v / (FK / 4) : v % (T / 4) * 4), k = k0 + (KC ? v % (FK / 4) * 4 : v / (T / 4));
        if (KC ? (r < R && k + 4 <= ke) : (r + 4 <= R && k < ke)) {
            __builtin_memcpy(&out[h], X + (KC ? (size_t)r * ld + k : (size_t)k * ld + r), 16);
        } else {
            float e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = KC ? load_op<false>(X, ld, r, k + i, R, ke) : load_op<true>(X, ld, r + i, k, R, ke);
            out[h] = make_float4(e[0], e[1], e[2], e[3]);
        }
    }
}

// to LDS as [k][row], rows padded by 4
template <bool KC, int T>
__device__ __forceinline__ void fp32_store(float (*S)[T + 4], const float4 *val)
{
#pragma unroll
    for (int h = 0; h < T * FK / 1024; ++h) {
        const int v = (int)threadIdx.x + 256 * h;
        const int r = KC ? v / (FK / 4) : v % (T / 4) * 4, k = KC ? v % (FK / 4) * 4 : v / (T / 4);
        if (KC) {
            S[k][r] = val[h].x;
            S[k + 1][r] = val[h].y;
            S[k + 2][r] = val[h].z;
            S[k + 3][r] = val[h].w;
        } else {
            *(float4 *)&S[k][r] = val[h];
        }
    }
}

// C (+ split offset) = op(A)[M x K] op(B)[K x N] over K range of this split;
// epilogue when splits == 1: + bias[N], ReLU.  A T x T tile per workgroup, a
// thread R x R of it (R = T / 16) in 4 x 4 blocks 64 apart, each element one
// chain of fmaf in the order of k.  Two LDS buffers, the next stage on its way
// in registers.  With one element to a load and none on its way 4096^3 took
// 3.38 ms, 1.77 now (78 TFLOP/s; 85 over longer runs); 1024^3 195 -> 82 us, 256 x
// 1024 x 1024 145 -> 74 us (host call included).
template <bool TA, bool TB, int T>
__global__ __launch_bounds__(256) void k_gemm_fp32(const float *A, int lda, const float *B, int ldb, float *C, int ldc,
                                                   int M, int N, int K, int kps, const float *bias, int relu)
{
    constexpr int Q = T / 64, V = T * FK / 1024;
    __shared__ __attribute__((aligned(16))) float As[2][FK][T + 4];
    __shared__ __attribute__((aligned(16))) float Bs[2][FK][T + 4];
    const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
    const int kb = blockIdx.z * kps, ke = min(K, kb + kps);
    float *Cout = C + (size_t)blockIdx.z * (size_t)M * ldc;
    const int t = threadIdx.x;
    const int tr = (t >> 4) * 4, tc = (t & 15) * 4;
    float acc[4 * Q][4 * Q] = {};
    float4 ra[V], rb[V];
    fp32_load<!TA, T>(ra, A, lda, M, m0, kb, ke);
    fp32_load<TB, T>(rb, B, ldb, N, n0, kb, ke);
    for (int k0 = kb, buf = 0; k0 < ke; k0 += FK, buf ^= 1) {
        fp32_store<!TA, T>(As[buf], ra);
        fp32_store<TB, T>(Bs[buf], rb);
        __syncthreads();
        if (k0 + FK < ke) {
            fp32_load<!TA, T>(ra, A, lda, M, m0, k0 + FK, ke);
            fp32_load<TB, T>(rb, B, ldb, N, n0, k0 + FK, ke);
        }
#pragma unroll
        for (int kk = 0; kk < FK; ++kk) {
            float a[4 * Q], b[4 * Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                *(float4 *)&a[4 * q] = *(const float4 *)&As[buf][kk][tr + 64 * q];
                *(float4 *)&b[4 * q] = *(const float4 *)&Bs[buf][kk][tc + 64 * q];
            }
#pragma unroll
            for (int i = 0; i < 4 * Q; ++i)
#pragma unroll
                for (int j = 0; j < 4 * Q; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4 * Q; ++i)
#pragma unroll
        for (int j = 0; j < 4 * Q; ++j) {
            const int row = m0 + tr + 64 * (i / 4) + i % 4, col = n0 + tc + 64 * (j / 4) + j % 4;
            if (row < M && col < N) {
                float o = acc[i][j];
                if (gridDim.z == 1) {
                    if (bias) o += bias[col];
                    if (relu && o < 0.0f) o = 0.0f;
                }
                Cout[(size_t)row * ldc + col] = o;
            }
        }
}

// Output tile of an FP32 product: 128 from four such workgroups to a CU on (a
// product in parts stays below that, see splits_for).
// Measured (us, 64 / 128): 4096^3, 1024 tiles of 128, 1860 / 1768; 2048^3, 256
// of them, 271 / 398; 1000 x 3001 x 777 114 / 178.
inline int fp32_tile(int M, int N, int splits)
{
    return (int64_t)((M + 127) / 128) * ((N + 127) / 128) * splits >= 1024 ? 128 : 64;
}
template <bool TA, bool TB>
void launch_fp32(const float *A, int lda, const float *B, int ldb, float *C, int ldc, int M, int N, int K, int kps, int splits,
                 const float *bias, int relu, hipStream_t st)
{
    const int T = fp32_tile(M, N, splits);
    const dim3 grid((N + T - 1) / T, (M + T - 1) / T, splits);
    if (T == 128)
        hipLaunchKernelGGL((k_gemm_fp32<TA, TB, 128>), grid, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, kps, bias, relu);
    else
        hipLaunchKernelGGL((k_gemm_fp32<TA, TB, 64>), grid, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, kps, bias, relu);
}

// ----------------------------------------------------------------------------
// BF16 GEMM on MFMA
// ----------------------------------------------------------------------------

// One workgroup of four wave64 (2 x 2) makes a (64 WM) x (64 WN) tile of C,
// each wave (32 WM) x (32 WN) of it as WM x WN v_mfma_f32_32x32x16_bf16
// tiles.  K goes in stages of 64 through two LDS buffers: while one stage is
// multiplied, the next is written to the other buffer and the one after it
// is on its way from memory in registers, so there is one barrier per stage.
//
// What bounds it.  Per 64 of K a tile of T x T costs T^2 / 32 clocks of the
// CU's four matrix cores, and the waves read their operands from LDS at 128
// bytes a clock: with 64 x 64 to a wave (T = 128) that alone takes as long as
// the MFMAs.  The 256 tile gives each of its eight waves 128 x 64: 4096^3 in
// 138 us, host call included (the kernel 127 to 143 us, 134 on average, 1.0
// PFLOP/s), where 128 x 128 tiles with scattered LDS writes took 255; four waves
// of 128 x 128 spilled registers (200 us).  A small product is a chain of stages
// instead: the kernel of 256 x 1024 x 1024 went from 71 us (scalar staging, one
// stage at a time) to 10.
//
// An operand is staged as it lies in memory, in 16-byte vectors with no
// alignment asked of them (a global load takes any address; an odd leading
// dimension then costs one more cache line per row piece, not a load per
// element).  Stored with k contiguous (KC) it sits in LDS as [row][k], rows
// padded to 144 bytes, and an operand fragment (8 consecutive k of one row
// per lane) is one 16-byte read.  Stored with the other index contiguous it
// sits as [k][row] and the fragment is two transposing reads
// (ds_read_b64_tr_b16: within 16 lanes, lane i gets element i of the four
// k rows the lanes' addresses point at), where it used to be scattered over
// eight LDS rows by 2-byte writes.  Rows there are padded by 64 bytes, which
// puts the four k rows of a read on disjoint quarters of the banks.
constexpr int BK = 64;   // K per stage

// LDS elements of one staged operand of ROWS rows, its row pitch, and the
// 16-byte vectors that each of NT threads moves
template <bool KC, int ROWS, int NT>
struct Stage {
    static constexpr int pitch = KC ? BK + 8 : ROWS + 32;
    static constexpr int size = KC ? ROWS * pitch : BK * pitch;
    static constexpr int vecs = ROWS * BK / 8 / NT;
    static_assert(ROWS * BK % (8 * NT) == 0, "whole vectors");
    // vector v holds 8 elements from (row, k) on: along k, or along the rows
    static __device__ __forceinline__ int row(int v) { return KC ? v / (BK / 8) : (v % (ROWS / 8)) * 8; }
    static __device__ __forceinline__ int k(int v) { return KC ? (v % (BK / 8)) * 8 : v / (ROWS / 8); }
    static __device__ __forceinline__ int lds(int v) { return KC ? row(v) * pitch + k(v) : k(v) * pitch + row(v); }
};

// 8 elements moved down by n places (n < 8)
__device__ __forceinline__ uint4 shift_down(uint4 w, int n)
{
    uint64_t lo = (uint64_t)w.x | (uint64_t)w.y << 32, hi = (uint64_t)w.z | (uint64_t)w.w << 32;
    const int b = 16 * (n & 3);
    if (n >= 4) {
        lo = hi;
        hi = 0;
    }
    if (b) {
        lo = lo >> b | hi << (64 - b);
        hi >>= b;
    }
    return make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
}

// This thread's vectors of the whole stage of k from k0 on: rows r0.. of
// op(X), which has R rows.  A row past R belongs to outputs that are not
// stored, so KC reads row R - 1 in its place.  Across the rows (not KC) a
// tile that reaches past R (EDGE) reads the last 8 rows there are (R >= 8)
// and moves down those it wants.  No branch, so that the loads of a stage
// stay in flight while the stage before is multiplied.
template <bool KC, int ROWS, int NT, bool EDGE>
__device__ __forceinline__ void stage_load(uint4 *out, const uint16_t *X, int ld, int R, int r0, int k0)
{
    using S = Stage<KC, ROWS, NT>;
#pragma unroll
    for (int h = 0; h < S::vecs; ++h) {
        const int v = (int)threadIdx.x + NT * h;
        const int r = r0 + S::row(v), k = k0 + S::k(v);
        const uint16_t *p;
        if (KC) p = X + (size_t)min(r, R - 1) * ld + k;
        else p = X + (size_t)k * ld + (EDGE ? min(r, R - 8) : r);
        __builtin_memcpy(&out[h], p, 16);
    }
}

// the same for a stage that ends before its 64th k (at ke), or of an operand
// of fewer than 8 rows: element by element, zero past the ends
template <bool KC, int ROWS, int NT>
__device__ __forceinline__ void stage_load_part(uint4 *out, const uint16_t *X, int ld, int R, int r0, int k0, int ke)
{
    using S = Stage<KC, ROWS, NT>;
#pragma unroll
    for (int h = 0; h < S::vecs; ++h) {
        const int v = (int)threadIdx.x + NT * h;
        const int r = r0 + S::row(v), k = k0 + S::k(v);
        uint16_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int ri = KC ? r : r + i, ki = KC ? k + i : k;
            const bool in = ri < R && ki < ke;
            const size_t at = KC ? (size_t)(in ? ri : 0) * ld + (in ? ki : 0) : (size_t)(in ? ki : 0) * ld + (in ? ri : 0);
            e[i] = in ? X[at] : (uint16_t)0;
        }
        __builtin_memcpy(&out[h], e, 16);
    }
}

// EDGE: as stage_load read them
template <bool KC, int ROWS, int NT, bool EDGE>
__device__ __forceinline__ void stage_store(uint16_t *lds, const uint4 *val, int R, int r0)
{
    using S = Stage<KC, ROWS, NT>;
#pragma unroll
    for (int h = 0; h < S::vecs; ++h) {
        const int v = (int)threadIdx.x + NT * h;
        uint4 w = val[h];
        if (EDGE && !KC) {
            const int past = r0 + S::row(v) - (R - 8);
            if (past > 0) w = shift_down(w, min(past, 7));
        }
        *(uint4 *)(lds + S::lds(v)) = w;
    }
}

// the fragment of rows r..r+31 at k kk..kk+15 of a stage: lane l holds row
// r + l % 32, k kk + 8 (l / 32) .. + 7
template <bool KC, int P>
__device__ __forceinline__ bf16x8 stage_frag(const uint16_t *S, int r, int kk)
{
    const int lane = (int)threadIdx.x & 63;
    bf16x8 f;
    if (KC) {
        __builtin_memcpy(&f, S + (r + (lane & 31)) * P + kk + 8 * (lane >> 5), 16);
    } else {
        typedef __attribute__((address_space(3))) s16x4 lds4;
        const uint16_t *p = S + (kk + 8 * (lane >> 5) + ((lane >> 2) & 3)) * P + r + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)(p + 4 * P));
        const s16x8 w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        __builtin_memcpy(&f, &w, 16);
    }
    return f;
}

struct GemmArgs {
    const uint16_t *A, *B;
    int lda, ldb, M, N, K;
    int kps;               // K per split (blockIdx.y)
    float *C;              // split z at C + z M ldc; may be null when Cb is set
    int ldc;
    const float *bias;     // with one split: + bias[N], ReLU, bfloat16 copy Cb
    int relu;
    uint16_t *Cb;
};

// The wave tiles of one stage: 64 of K in four steps
template <bool AK, bool BKC, int WM, int WN, int PA, int PB>
__device__ __forceinline__ void stage_step(f32x16 (&acc)[WM][WN], const uint16_t *As, const uint16_t *Bs, int wm, int wn,
                                           int kk)
{
    bf16x8 a[WM], b[WN];
#pragma unroll
    for (int i = 0; i < WM; ++i) a[i] = stage_frag<AK, PA>(As, wm + 32 * i, kk);
#pragma unroll
    for (int j = 0; j < WN; ++j) b[j] = stage_frag<BKC, PB>(Bs, wn + 32 * j, kk);
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
}

// All stages of K [kb, ke) of one output tile; EDGE: an operand stored across
// its rows (not KC) reaches past its last row in this tile.  D stages are on
// their way from memory in registers.
template <bool AK, bool BKC, int WR, int WC, int WM, int WN, int D, bool EDGE>
__device__ __forceinline__ void gemm_stages(f32x16 (&acc)[WM][WN], const GemmArgs &g, uint16_t *smem, int m0, int n0, int kb,
                                            int ke, int wm, int wn)
{
    constexpr int NT = 64 * WR * WC, BM = 32 * WM * WR, BN = 32 * WN * WC;
    using SA = Stage<AK, BM, NT>;
    using SB = Stage<BKC, BN, NT>;
    uint16_t *As = smem, *Bs = smem + 2 * SA::size;   // two buffers each
    uint4 ra[D][SA::vecs], rb[D][SB::vecs];
    const bool tiny = (!AK && g.M < 8) || (!BKC && g.N < 8);   // no vector of 8 rows to read
    const int full = tiny ? 0 : (ke - kb) / BK;
    if (full > 0) {
        // past the last stage the same one is read and stored again, to no
        // use and no harm, so that the loads of a stage have no branch
        const int last = kb + (full - 1) * BK;
        auto load = [&](int d, int stage) {
            const int k0 = min(kb + stage * BK, last);
            stage_load<AK, BM, NT, EDGE>(ra[d], g.A, g.lda, g.M, m0, k0);
            stage_load<BKC, BN, NT, EDGE>(rb[d], g.B, g.ldb, g.N, n0, k0);
        };
        auto store = [&](int d, int buf) {
            stage_store<AK, BM, NT, EDGE>(As + buf * SA::size, ra[d], g.M, m0);
            stage_store<BKC, BN, NT, EDGE>(Bs + buf * SB::size, rb[d], g.N, n0);
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, d);
        store(0, 0);
        load(0, D);
        __syncthreads();
        for (int t0 = 0;; t0 += 2 * D) {   // stage t waits in registers t % D, then in buffer t % 2
#pragma unroll
            for (int u = 0; u < 2 * D; ++u) {
                const int t = t0 + u;
                const uint16_t *Ac = As + (u & 1) * SA::size, *Bc = Bs + (u & 1) * SB::size;
                stage_step<AK, BKC, WM, WN, SA::pitch, SB::pitch>(acc, Ac, Bc, wm, wn, 0);
                stage_step<AK, BKC, WM, WN, SA::pitch, SB::pitch>(acc, Ac, Bc, wm, wn, 16);
                store((u + 1) % D, (u + 1) & 1);
                load((u + 1) % D, t + 1 + D);
                stage_step<AK, BKC, WM, WN, SA::pitch, SB::pitch>(acc, Ac, Bc, wm, wn, 32);
                stage_step<AK, BKC, WM, WN, SA::pitch, SB::pitch>(acc, Ac, Bc, wm, wn, 48);
                __syncthreads();
                if (t + 1 >= full) goto done;   // the same for the whole workgroup
            }
        }
    }
done:
    for (int k0 = kb + full * BK; k0 < ke; k0 += BK) {   // what is left, if anything
        stage_load_part<AK, BM, NT>(ra[0], g.A, g.lda, g.M, m0, k0, ke);
        stage_load_part<BKC, BN, NT>(rb[0], g.B, g.ldb, g.N, n0, k0, ke);
        stage_store<AK, BM, NT, false>(As, ra[0], g.M, m0);
        stage_store<BKC, BN, NT, false>(Bs, rb[0], g.N, n0);
        __syncthreads();
        for (int kk = 0; kk < BK; kk += 16) stage_step<AK, BKC, WM, WN, SA::pitch, SB::pitch>(acc, As, Bs, wm, wn, kk);
        __syncthreads();
    }
}

// WR x WC waves of WM x WN MFMA tiles each: a (32 WM WR) x (32 WN WC) tile of C
template <bool AK, bool BKC, int WR, int WC, int WM, int WN, int D>
__global__ __launch_bounds__(64 * WR * WC, WM * WN > 8 ? 1 : 2) void k_gemm_mfma(GemmArgs g)
{
    constexpr int BM = 32 * WM * WR, BN = 32 * WN * WC;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    // Workgroups go to the 8 XCDs in turn: each XCD takes one contiguous run
    // of tiles, in column panels of up to 8 tile rows, so that the tiles in
    // flight on it share their operands in its L2.
    const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN, tiles = tm * tn;
    const int per = (tiles + 7) / 8, tile = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (tile >= tiles) return;
    const int gm = min(tm, 8), panel = tile / (gm * tn), in = tile - panel * gm * tn;
    const int rows = min(gm, tm - panel * gm);   // tile rows of this panel
    const int m0 = (panel * gm + in % rows) * BM, n0 = (in / rows) * BN;
    const int kb = (int)blockIdx.y * g.kps, ke = min(g.K, kb + g.kps);
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int wm = (wave / WC) * 32 * WM, wn = (wave % WC) * 32 * WN;
    f32x16 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    if ((!AK && m0 + BM > g.M) || (!BKC && n0 + BN > g.N))
        gemm_stages<AK, BKC, WR, WC, WM, WN, D, true>(acc, g, smem, m0, n0, kb, ke, wm, wn);
    else
        gemm_stages<AK, BKC, WR, WC, WM, WN, D, false>(acc, g, smem, m0, n0, kb, ke, wm, wn);
    float *Cout = g.C ? g.C + (size_t)blockIdx.y * (size_t)g.M * g.ldc : nullptr;
    const bool plain = gridDim.y > 1 || (!g.bias && !g.relu && !g.Cb);
#pragma unroll
    for (int j = 0; j < WN; ++j) {
        const int col = n0 + wn + 32 * j + (lane & 31);
        const bool in = col < g.N;
        const float add = !plain && g.bias && in ? g.bias[col] : 0.0f;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int row0 = m0 + wm + 32 * i + 4 * (lane >> 5);
            if (plain) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = row0 + 8 * (v >> 2) + (v & 3);
                    if (row < g.M && in) Cout[(size_t)row * g.ldc + col] = acc[i][j][v];
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = row0 + 8 * (v >> 2) + (v & 3);
                    float o = acc[i][j][v];
                    if (g.bias) o += add;
                    if (g.relu && o < 0.0f) o = 0.0f;
                    if (row < g.M && in) {
                        if (g.Cb) g.Cb[(size_t)row * g.ldc + col] = f2bf(o);
                        if (Cout) Cout[(size_t)row * g.ldc + col] = o;
                    }
                }
            }
        }
    }
}

// Output tile of a BF16 product with M x N outputs in `splits` parts of kps of K
// each: the one with the least time as fitted to measurements of each tile (34
// shapes of 64 x 30001 to 6000 x 6000, K 64 to 4096, all four forms): a part of
// the call, one per wave of 256 workgroups (one to a CU), one per k and one per
// k and wave.  A smaller tile costs a call less, a larger one an output.  A CU
// holds one 256-tile, so those come in whole waves; of the smaller ones it runs
// several at once, and a part of a wave costs less than a whole one (fill).
// Measured (us, 64 / 128 / 256, host call included): 4096^3 234 / 173 / 138,
// 3000 x 3000 x 4096 158 / 136 / 117, 4200 x 4100 x 1500 161 / 118 / 126, 2000 x
// 3000 x 1500 67 / 57 / 66, 1000 x 3001 x 777 39 / 38 / 52, 256 x 1024 x 777 25 /
// 35 / 48.
inline int mfma_tile(int M, int N, int kps, int splits)
{
    const struct {
        int side;
        double fill, call, wave, k, wave_k;   // the last four in us
    } tiles[3] = {{64, 0.75, 21.0, 0.66, 0.0004, 0.00404},
                  {128, 0.5, 21.2, 3.18, 0.0013, 0.01017},
                  {256, 1.0, 18.9, 10.7, -0.0061, 0.03015}};
    int best = 0;
    double cost = 0.0;
    for (const auto &t : tiles) {
        const int64_t n = (int64_t)((M + t.side - 1) / t.side) * ((N + t.side - 1) / t.side) * splits;
        const double even = (double)n / 256.0, waves = std::max(1.0, even + t.fill * (std::ceil(even) - even));
        const double c = t.call + t.wave * waves + (t.k + t.wave_k * waves) * kps;
        if (best == 0 || c < cost) {
            cost = c;
            best = t.side;
        }
    }
    return best;
}

template <bool AK, bool BKC, int WR, int WC, int WM, int WN, int D>
void launch_mfma_tile(const GemmArgs &g, int splits, hipStream_t st)
{
    constexpr int NT = 64 * WR * WC, BM = 32 * WM * WR, BN = 32 * WN * WC;
    const int64_t tiles = (int64_t)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    const int lds = 2 * (int)sizeof(uint16_t) * (Stage<AK, BM, NT>::size + Stage<BKC, BN, NT>::size);
    const auto kernel = &k_gemm_mfma<AK, BKC, WR, WC, WM, WN, D>;
    if (lds > 65536)
        HIPT(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles + 7) / 8 * 8), splits), dim3(NT), lds, st, g);
    HIPT(hipGetLastError());
}

template <bool AK, bool BKC>
void launch_mfma(const GemmArgs &g, int splits, hipStream_t st)
{
    switch (mfma_tile(g.M, g.N, std::min(g.kps, g.K), splits)) {
    case 256: launch_mfma_tile<AK, BKC, 2, 4, 4, 2, 1>(g, splits, st); break;
    case 128: launch_mfma_tile<AK, BKC, 2, 2, 2, 2, 2>(g, splits, st); break;
    default:
        if (g.kps > 2 * BK) launch_mfma_tile<AK, BKC, 2, 2, 1, 1, 2>(g, splits, st);
        else launch_mfma_tile<AK, BKC, 2, 2, 1, 1, 1>(g, splits, st);
        break;
    }
}

// ----------------------------------------------------------------------------
// the output layer
// ----------------------------------------------------------------------------

// op(A) op(B) + bias for few rows (a batch), few k (the rank, at most 64) and
// very many columns: 256 x 300001 x 64 reads 38 MB and writes 307 MB, so it
// is a stream of stores.  As tiles of a general product each workgroup spent
// its life waiting for its one stage of K (157 us at best; 285 before, with
// scalar loads and a bfloat16 copy of the output that nothing read).  Now 124
// us, and 82 at 300,032 columns, where every row is whole cache lines.  Of the
// difference the output's partial lines are only a part: storing whole lines,
// the results turned between lanes, took 112 (and 88 to 99 where rows are whole
// lines anyway, so it was left out); the weights' rows are odd too.  Here a
// workgroup keeps its 256 rows of A in registers (64 rows to a wave) and walks
// the column tiles, 64 wide (MSE: 32), with the next tile's weights on their way
// while it stores this one's results.  Tiles go to XCDs in contiguous runs:
// neighbours share the cache lines at their seam (rows of an odd length are not
// aligned), which one L2 then completes.
//
// MSE (a training step): the predictions z are not stored; of d = z - target
// come dz = 2 d / (M N) as bfloat16 (Cb), the sum of d^2 over the workgroup's
// tiles (loss, one per workgroup) and the column sums of dz (colsum, one row
// of N per 256 rows).
constexpr int kOutRows = 256;   // rows of A per workgroup

struct OutArgs {
    const uint16_t *A, *B;   // A [M x K], B [K x N], rows contiguous; K <= 64, N >= 8
    int M, N, K;
    const float *bias;       // [N]
    float *C;                // [M x N]
    uint16_t *Cb;            // MSE: dz
    const float *target;     // MSE: [M x N]
    double *loss;            // MSE: [gridDim.y * gridDim.x]
    float *colsum;           // MSE: [gridDim.y][N]
};

template <bool MSE>
__global__ __launch_bounds__(256, 2) void k_out_layer(OutArgs g)
{
    constexpr int WN = MSE ? 1 : 2, TC = 32 * WN;   // MFMA tiles across, columns per tile
    using SB = Stage<false, TC, 256>;
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][SB::size];
    __shared__ float csum[2][4][TC];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int m0 = (int)blockIdx.y * kOutRows + wave * 64, N = g.N;
    bf16x8 a[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = min(m0 + 32 * i + (lane & 31), g.M - 1), k = 16 * q + 8 * (lane >> 5);
            const uint16_t *p = g.A + (size_t)row * g.K + k;
            uint16_t e[8];
            if (g.K == BK) {
                __builtin_memcpy(e, p, 16);
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) e[u] = k + u < g.K ? p[u] : (uint16_t)0;
            }
            __builtin_memcpy(&a[i][q], e, 16);
        }
    const int tn = (N + TC - 1) / TC, per = (tn + 7) / 8;
    const int first = ((int)blockIdx.x & 7) * per, last = min(tn, first + per), step = (int)gridDim.x >> 3;
    const float len = (float)((int64_t)g.M * N);
    // a result is at (wave's row block + 8 (v / 4) + v % 4) N + tile's column,
    // the same for the wavefront, plus `at`
    const unsigned at = (unsigned)(4 * (lane >> 5)) * (unsigned)N + (unsigned)(lane & 31);
    auto row_of = [](int i, int v) { return 32 * i + 8 * (v >> 2) + (v & 3); };
    // What a tile reads: its weights, biases and (MSE) targets.  All of it is
    // loaded a tile ahead, before this tile's stores: vector memory completes
    // in order, so a load after them would wait for them all.
    uint4 rb[SB::vecs];
    float bias[WN], z[MSE ? 2 : 1][16];
    auto load = [&](int tile) {   // past the run's end: its last tile again
        const int n0 = min(tile, last - 1) * TC;
        if (g.K == BK) stage_load<false, TC, 256, true>(rb, g.B, N, N, n0, 0);
        else stage_load_part<false, TC, 256>(rb, g.B, N, N, n0, 0, g.K);
#pragma unroll
        for (int j = 0; j < WN; ++j) bias[j] = g.bias[min(n0 + 32 * j + (lane & 31), N - 1)];
        if constexpr (MSE) {
            const bool in = n0 + TC <= N && m0 + 64 <= g.M;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float *p = g.target + (size_t)(m0 + row_of(i, v)) * N + n0;
                    if (!in) {
                        const int row = m0 + row_of(i, v) + 4 * (lane >> 5), col = n0 + (lane & 31);
                        z[i][v] = g.target[(size_t)min(row, g.M - 1) * N + min(col, N - 1)];
                    } else {
                        z[i][v] = p[at];
                    }
                }
        }
    };
    const int tile0 = first + ((int)blockIdx.x >> 3);
    double s = 0.0;
    if (tile0 < last) load(tile0);
    int buf = 0;
    for (int tile = tile0; tile < last; tile += step, buf ^= 1) {
        const int n0 = tile * TC;
        if (g.K == BK) stage_store<false, TC, 256, true>(Bs[buf], rb, N, n0);
        else stage_store<false, TC, 256, false>(Bs[buf], rb, N, n0);
        float add[WN], zc[MSE ? 2 : 1][16];
#pragma unroll
        for (int j = 0; j < WN; ++j) add[j] = bias[j];
        if constexpr (MSE) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) zc[i][v] = z[i][v];
        }
        __syncthreads();
        load(tile + step);
        f32x16 acc[2][WN];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const bf16x8 b = stage_frag<false, SB::pitch>(Bs[buf], 32 * j, 16 * q);
#pragma unroll
                for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][q], b, acc[i][j], 0, 0, 0);
            }
        if (MSE && tile > tile0 && t < TC)   // the tile before: its four waves' column sums
            g.colsum[(size_t)blockIdx.y * N + (n0 - step * TC) + t] =
                ((csum[buf ^ 1][0][t] + csum[buf ^ 1][1][t]) + csum[buf ^ 1][2][t]) + csum[buf ^ 1][3][t];
        const bool whole = n0 + TC <= N && m0 + 64 <= g.M;
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            float cs = 0.0f;
            const bool in = n0 + 32 * j + (lane & 31) < N;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const size_t base = (size_t)(m0 + row_of(i, v)) * N + (n0 + 32 * j);
                    const bool mine = whole || (in && m0 + row_of(i, v) + 4 * (lane >> 5) < g.M);
                    if constexpr (MSE) {
                        const float d = (acc[i][j][v] + add[j]) - zc[i][v];
                        const float dz = 2.0f * d / len;
                        if (mine) {
                            s += (double)d * (double)d;
                            cs += dz;
                            (g.Cb + base)[at] = f2bf(dz);
                        }
                    } else if (mine) {
                        (g.C + base)[at] = acc[i][j][v] + add[j];
                    }
                }
            if constexpr (MSE) {
                cs += __shfl_xor(cs, 32);
                if (lane < 32) csum[buf][wave][32 * j + lane] = cs;
            }
        }
    }
    if constexpr (MSE) {
        __shared__ double lsum[4];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) lsum[wave] = s;
        __syncthreads();
        if (tile0 < last) {
            const int n0 = (tile0 + (last - 1 - tile0) / step * step) * TC;   // the last tile
            if (t < TC && n0 + t < N)
                g.colsum[(size_t)blockIdx.y * N + n0 + t] =
                    ((csum[buf ^ 1][0][t] + csum[buf ^ 1][1][t]) + csum[buf ^ 1][2][t]) + csum[buf ^ 1][3][t];
        }
        if (t == 0)
            g.loss[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = ((lsum[0] + lsum[1]) + lsum[2]) + lsum[3];
    }
}

// two workgroups to a CU, fewer when the tiles are fewer; a multiple of the 8 XCDs
inline int out_grid(int N) { return std::min(512, ((N + 31) / 32 + 7) / 8 * 8); }

// the shapes k_out_layer is for: enough columns for its workgroups to walk
// several tiles (below, the tiled product spreads over the GPU as well)
inline bool out_layer_shape(int N, int K) { return K <= BK && N >= 8192 && N < (1 << 28); }

template <bool MSE>
void launch_out_layer(const OutArgs &g, hipStream_t st)
{
    hipLaunchKernelGGL(k_out_layer<MSE>, dim3(out_grid(g.N), (g.M + kOutRows - 1) / kOutRows), dim3(256), 0, st, g);
    HIPT(hipGetLastError());
}

__global__ void k_to_bf16(const float *x, uint16_t *y, int64_t len)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < len) y[i] = f2bf(x[i]);
}

// (x - mu) / sigma per feature, rows of width d; also as bfloat16 when yb is set
__global__ void k_standardize(const float *x, const float *mu, const float *sig, float *y, uint16_t *yb, int64_t len,
                              int d)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    const float v = (x[i] - mu[i % d]) / sig[i % d];
    y[i] = v;
    if (yb) yb[i] = f2bf(v);
}

// loss partials and dZ = 2 (Z - Z*) / (B * D)
__global__ void k_mse(const float *Z, const float *Zs, float *dZ, int64_t len, double *part)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double s = 0.0;
    if (i < len) {
        const float d = Z[i] - Zs[i];
        s = (double)d * (double)d;
        dZ[i] = 2.0f * d / (float)len;
    }
    __shared__ double sh[256];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// What follows a layer's input gradient [rows x cols], in one pass over it:
// its parts added in order (one part: as it is), zeroed where H <= 0 (H null:
// not), stored as T (FP32, where dY may be the one part itself, or bfloat16),
// and its column sums over each `chunk` rows (the bias gradient of the layer
// below, which k_grad_finish completes).  A workgroup takes 64 columns of one
// chunk, four threads to a column, each adding every fourth row in order.  These
// were four launches, the column sums alone 50 us on 256 x 1024 values (a thread
// per column, four workgroups).
template <typename T>
__global__ __launch_bounds__(256) void k_dy(const float *part, int parts, const float *__restrict__ H, T *dY,
                                            float *__restrict__ cpart, int rows, int cols, int chunk)
{
    __shared__ float sh[4][64];
    const int tc = (int)threadIdx.x & 63, tr = (int)threadIdx.x >> 6;
    const int c = (int)blockIdx.x * 64 + tc;
    const int r1 = min(rows, ((int)blockIdx.y + 1) * chunk);
    float sum = 0.0f;
    if (c < cols) {
        const size_t len = (size_t)rows * cols;
        for (int r = (int)blockIdx.y * chunk + tr; r < r1; r += 4) {
            const size_t i = (size_t)r * cols + c;
            float v = part[i];
#pragma unroll 16
            for (int z = 1; z < parts; ++z) v += part[z * len + i];
            if (H && !(H[i] > 0.0f)) v = 0.0f;
            if constexpr (sizeof(T) == sizeof(float)) dY[i] = v;
            else dY[i] = f2bf(v);
            sum += v;
        }
    }
    sh[tr][tc] = sum;
    __syncthreads();
    if (tr == 0 && c < cols) cpart[(size_t)blockIdx.y * cols + c] = ((sh[0][tc] + sh[1][tc]) + sh[2][tc]) + sh[3][tc];
}

// One layer's bias gradient in the making: column sums of its output gradient
// per `chunk` rows, [ceil(B / chunk)][cols] at cpart, to go to grad.
struct BiasPart {
    const float *cpart;
    float *grad;
    int cols, chunk;
};

// The end of a step's gradient, all layers in one launch (blockIdx.y: the
// layer): the chunks' column sums added in order; and the loss (its np
// partials added, over len values).
__global__ __launch_bounds__(256) void k_grad_finish(const BiasPart *parts, int B, const double *lpart, int np, int64_t len,
                                                     double *loss)
{
    if (blockIdx.x > 0) {
        const BiasPart p = parts[blockIdx.y];
        const int c = ((int)blockIdx.x - 1) * 256 + (int)threadIdx.x, n = (B + p.chunk - 1) / p.chunk;
        if (c >= p.cols) return;
        float s = p.cpart[c];
#pragma unroll 8
        for (int k = 1; k < n; ++k) s += p.cpart[(size_t)k * p.cols + c];
        p.grad[c] = s;
        return;
    }
    if (blockIdx.y > 0) return;
    __shared__ double sh[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < np; i += 256) s += lpart[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = sh[0] / (double)len;
}

__global__ void k_adam(float *p, float *m, float *v, const float *g, uint16_t *pb, int64_t len, float lr, float b1,
                       float b2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    if (pb) pb[i] = f2bf(pi);
}

// out[b][s] = sum_j S[s][j] * D[b][j]   (S: CSR, rows x cols; D: [B x cols])
__global__ void k_sketch(const int *rp, const int *ci, const float *v, const float *D, int cols, float *out, int rows)
{
    const int s = blockIdx.x, b = blockIdx.y;
    double acc = 0.0;
    for (int p = rp[s] + threadIdx.x; p < rp[s + 1]; p += 256) acc += (double)v[p] * (double)D[(size_t)b * cols + ci[p]];
    __shared__ double sh[256];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[(size_t)b * rows + s] = (float)sh[0];
}

inline int nblk(int64_t len) { return (int)((len + 255) / 256); }

// K per part when a product's K is contracted in `splits` parts, and how many
// parts that makes
inline int k_per_split(int K, int &splits)
{
    if (splits < 1) splits = 1;
    const int kps = ((K + splits - 1) / splits + GK - 1) / GK * GK;
    splits = std::max(1, (K + kps - 1) / kps);
    return kps;
}

// C = op(A) op(B) with optional epilogue; splits > 1 (only with ldc == N)
// contracts K in parts, no epilogue then, left in `scratch` (parts x M x N)
// for the caller to add.  Returns the number of parts.
int gemm(hipStream_t st, bool bf, bool ta, bool tb, int M, int N, int K, const void *A, int lda, const void *B,
         int ldb, float *C, int ldc, const float *bias, bool relu, uint16_t *Cb, int splits, float *scratch)
{
    if (M <= 0 || N <= 0) return 1;
    const int kps = k_per_split(K, splits);
    float *out = splits > 1 ? scratch : C;
    const int ldo = splits > 1 ? N : ldc;
    const float *bs = splits > 1 ? nullptr : bias;
    const int rl = splits > 1 ? 0 : (int)relu;
    if (bf && !ta && !tb && splits == 1 && bias && !relu && !Cb && lda == K && ldb == N && ldc == N && out_layer_shape(N, K)) {
        OutArgs g{};
        g.A = (const uint16_t *)A; g.B = (const uint16_t *)B;
        g.M = M; g.N = N; g.K = K; g.bias = bias; g.C = C;
        launch_out_layer<false>(g, st);
        return 1;
    }
    if (bf) {
        GemmArgs g{};
        g.A = (const uint16_t *)A; g.B = (const uint16_t *)B;
        g.lda = lda; g.ldb = ldb; g.M = M; g.N = N; g.K = K; g.kps = kps;
        g.C = out; g.ldc = ldo; g.bias = bs; g.relu = rl; g.Cb = splits > 1 ? nullptr : Cb;
        if (!ta && !tb) launch_mfma<true, false>(g, splits, st);
        else if (ta && !tb) launch_mfma<false, false>(g, splits, st);
        else if (!ta && tb) launch_mfma<true, true>(g, splits, st);
        else launch_mfma<false, true>(g, splits, st);
        return splits;
    }
    const float *Af = (const float *)A, *Bf = (const float *)B;
    if (!ta && !tb) launch_fp32<false, false>(Af, lda, Bf, ldb, out, ldo, M, N, K, kps, splits, bs, rl, st);
    else if (ta && !tb) launch_fp32<true, false>(Af, lda, Bf, ldb, out, ldo, M, N, K, kps, splits, bs, rl, st);
    else if (!ta && tb) launch_fp32<false, true>(Af, lda, Bf, ldb, out, ldo, M, N, K, kps, splits, bs, rl, st);
    else launch_fp32<true, true>(Af, lda, Bf, ldb, out, ldo, M, N, K, kps, splits, bs, rl, st);
    HIPT(hipGetLastError());
    return splits;
}

}  // namespace pdlp

using namespace pdlp;

struct lpw_net {
    lpw_config cfg{};
    hipStream_t st = nullptr;
    Arena arena;
    int L = 0;                                   // linear layers = layers + 2
    std::vector<int> din, dout;                  // per layer
    std::vector<int64_t> woff, boff;             // offsets into the flat parameter vector
    int64_t nparam = 0;
    float *P = nullptr, *G = nullptr, *Mm = nullptr, *Vv = nullptr;   // params, grads, Adam moments
    uint16_t *Pb = nullptr;                      // bf16 copy of the params
    float *mu = nullptr, *sig = nullptr;
    // activations for up to cfg.max_batch rows: A[0] = standardized input, A[l+1] = output of layer l
    std::vector<float *> Act, dAct;
    std::vector<uint16_t *> Actb, dActb;
    float *scratch = nullptr;
    int64_t scratch_len = 0;
    double *lpart = nullptr, *lout = nullptr;   // loss partials and the loss
    bool fused_out = false;                      // a training step's output layer is k_out_layer<true>
    // per layer: column sums of its output gradient over every `chunk` rows
    // (of a fused output layer: every kOutRows)
    std::vector<float *> cpart;
    std::vector<int> chunk;
    BiasPart *bias_parts = nullptr;
    int64_t step = 0;
    std::string err;
};

namespace {

int net_fail(lpw_net *N, const HipError &h)
{
    char buf[512];
    snprintf(buf, sizeof(buf), "%s failed: %s", h.what, hipGetErrorString(h.e));
    if (N) N->err = buf;
    return h.e == hipErrorOutOfMemory ? LP_ERR_NOMEM : LP_ERR_HIP;
}

bool use_bf(const lpw_net *N) { return N->cfg.precision == LPW_BF16; }

// splits for the long contraction of layer l's input gradient
int splits_for(int K, int tiles)
{
    int s = 1;
    while (tiles * s < 512 && K / (s * 2) >= 256) s *= 2;
    return s;
}

// the layers up to (not including) `layers`, the output layer's product to
// Z when it is among them
void forward(lpw_net *N, const float *X, int B, int layers, float *Z)
{
    hipStream_t st = N->st;
    const bool bf = use_bf(N);
    const int d0 = N->din[0];
    hipLaunchKernelGGL(k_standardize, dim3(nblk((int64_t)B * d0)), dim3(256), 0, st, X, (const float *)N->mu,
                       (const float *)N->sig, N->Act[0], bf ? N->Actb[0] : nullptr, (int64_t)B * d0, d0);
    for (int l = 0; l < layers; ++l) {
        const int K = N->din[l], Nn = N->dout[l];
        const bool relu = l < N->L - 2, last = l == N->L - 1;
        const void *A = bf ? (const void *)N->Actb[l] : (const void *)N->Act[l];
        const void *W = bf ? (const void *)(N->Pb + N->woff[l]) : (const void *)(N->P + N->woff[l]);
        gemm(st, bf, false, false, B, Nn, K, A, K, W, Nn, last ? Z : N->Act[l + 1], Nn, N->P + N->boff[l], relu,
             bf && !last ? N->Actb[l + 1] : nullptr, 1, nullptr);
    }
}

// k_dy on the gradient of layer l's output [B x dout], in `parts` parts
void launch_dy(lpw_net *N, int l, const float *part, int parts, const float *H, int B)
{
    const int cols = N->dout[l], chunk = N->chunk[l];
    const dim3 grid((cols + 63) / 64, (B + chunk - 1) / chunk);
    if (use_bf(N))
        hipLaunchKernelGGL(k_dy<uint16_t>, grid, dim3(256), 0, N->st, part, parts, H, N->dActb[l + 1], N->cpart[l], B, cols,
                           chunk);
    else
        hipLaunchKernelGGL(k_dy<float>, grid, dim3(256), 0, N->st, part, parts, H, N->dAct[l + 1], N->cpart[l], B, cols,
                           chunk);
    HIPT(hipGetLastError());
}

// The output layer, the mean squared error against Zstar (its
// partials to lpart), its gradient dZ (in dAct[L], BF16 mode: dActb[L])
// and its column sums.  In BF16 mode, at the ranks k_out_layer takes, the
// product's epilogue does it all, so the predictions and FP32 gradients of
// the batch never go to memory.
void output_loss(lpw_net *N, const float *Zstar, int B)
{
    hipStream_t st = N->st;
    const int l = N->L - 1, K = N->din[l], Nn = N->dout[l];
    const int64_t len = (int64_t)B * Nn;
    if (N->fused_out) {
        OutArgs g{};
        g.A = N->Actb[l]; g.B = N->Pb + N->woff[l];
        g.M = B; g.N = Nn; g.K = K; g.bias = N->P + N->boff[l]; g.Cb = N->dActb[N->L];
        g.target = Zstar; g.loss = N->lpart; g.colsum = N->cpart[l];
        launch_out_layer<true>(g, st);
        return;
    }
    const bool bf = use_bf(N);
    gemm(st, bf, false, false, B, Nn, K, bf ? (const void *)N->Actb[l] : (const void *)N->Act[l], K,
         bf ? (const void *)(N->Pb + N->woff[l]) : (const void *)(N->P + N->woff[l]), Nn, N->Act[N->L], Nn,
         N->P + N->boff[l], false, nullptr, 1, nullptr);
    hipLaunchKernelGGL(k_mse, dim3(nblk(len)), dim3(256), 0, st, (const float *)N->Act[N->L], Zstar, N->dAct[N->L], len,
                       N->lpart);
    launch_dy(N, l, N->dAct[N->L], 1, nullptr, B);
}

// backward from dZ (output_loss); fills G and the loss
void backward(lpw_net *N, int B)
{
    hipStream_t st = N->st;
    const bool bf = use_bf(N);
    for (int l = N->L - 1; l >= 0; --l) {
        const int K = N->din[l], Nn = N->dout[l];
        const void *dYo = bf ? (const void *)N->dActb[l + 1] : (const void *)N->dAct[l + 1];
        const void *Xo = bf ? (const void *)N->Actb[l] : (const void *)N->Act[l];
        // dW = X' dY  [K x Nn], contraction over the batch
        gemm(st, bf, true, false, K, Nn, B, Xo, K, dYo, Nn, N->G + N->woff[l], Nn, nullptr, false, nullptr, 1,
             nullptr);
        if (l > 0) {
            // dX = dY W'  [B x K], contraction over Nn (long for the output
            // layer); it is the gradient of the layer below's output, through
            // its ReLU if it has one
            const void *Wo = bf ? (const void *)(N->Pb + N->woff[l]) : (const void *)(N->P + N->woff[l]);
            const int tiles = ((B + GT - 1) / GT) * ((K + GT - 1) / GT);
            int splits = splits_for(Nn, tiles);
            while (splits > 1 && (int64_t)splits * B * K > N->scratch_len) splits /= 2;
            splits = gemm(st, bf, false, true, B, K, Nn, dYo, Nn, Wo, Nn, N->dAct[l], K, nullptr, false, nullptr, splits,
                          N->scratch);
            launch_dy(N, l - 1, splits > 1 ? N->scratch : N->dAct[l], splits, l - 1 < N->L - 2 ? N->Act[l] : nullptr, B);
        }
    }
    // the bias gradients and the loss
    const int64_t len = (int64_t)B * N->cfg.out_dim;
    const int np = N->fused_out ? out_grid(N->cfg.out_dim) * ((B + kOutRows - 1) / kOutRows) : nblk(len);
    const int widest = *std::max_element(N->dout.begin(), N->dout.end());
    hipLaunchKernelGGL(k_grad_finish, dim3(1 + nblk(widest), N->L), dim3(256), 0, st, (const BiasPart *)N->bias_parts, B,
                       (const double *)N->lpart, np, len, N->lout);
    HIPT(hipGetLastError());
}

}  // namespace

extern "C" {

void lpw_default_config(lpw_config *c)
{
    if (!c) return;
    std::memset(c, 0, sizeof(*c));
    c->in_dim = 256;
    c->hidden = 1024;
    c->layers = 3;
    c->rank = 64;
    c->out_dim = 0;
    c->max_batch = 256;
    c->precision = LPW_BF16;
    c->stream = nullptr;
}

int lpw_create(lpw_net **out, const lpw_config *cfg)
{
    if (!out || !cfg) return LP_ERR_ARG;
    *out = nullptr;
    if (cfg->in_dim <= 0 || cfg->hidden <= 0 || cfg->layers < 1 || cfg->rank <= 0 || cfg->out_dim <= 0 ||
        cfg->max_batch <= 0 || (cfg->precision != LPW_BF16 && cfg->precision != LPW_FP32))
        return LP_ERR_ARG;
    std::unique_ptr<lpw_net> N(new lpw_net());
    N->cfg = *cfg;
    N->st = (hipStream_t)cfg->stream;
    N->L = cfg->layers + 2;
    N->din.push_back(cfg->in_dim);
    for (int l = 0; l < cfg->layers; ++l) {
        N->dout.push_back(cfg->hidden);
        N->din.push_back(cfg->hidden);
    }
    N->dout.push_back(cfg->rank);
    N->din.push_back(cfg->rank);
    N->dout.push_back(cfg->out_dim);
    int64_t off = 0;
    for (int l = 0; l < N->L; ++l) {
        N->woff.push_back(off);
        off += (int64_t)N->din[l] * N->dout[l];
        N->boff.push_back(off);
        off += N->dout[l];
    }
    N->nparam = off;
    try {
        Arena &A = N->arena;
        N->P = A.make<float>(off);
        N->G = A.make<float>(off);
        N->Mm = A.make<float>(off);
        N->Vv = A.make<float>(off);
        N->Pb = A.make<uint16_t>(off);
        HIPT(hipMemsetAsync(N->Mm, 0, sizeof(float) * (size_t)off, N->st));
        HIPT(hipMemsetAsync(N->Vv, 0, sizeof(float) * (size_t)off, N->st));
        HIPT(hipMemsetAsync(N->G, 0, sizeof(float) * (size_t)off, N->st));
        N->mu = A.make<float>(cfg->in_dim);
        N->sig = A.make<float>(cfg->in_dim);
        std::vector<float> zeros(cfg->in_dim, 0.0f), ones(cfg->in_dim, 1.0f);
        h2d(N->st, N->mu, zeros.data(), cfg->in_dim);
        h2d(N->st, N->sig, ones.data(), cfg->in_dim);
        const int64_t Bm = cfg->max_batch;
        const bool bf = cfg->precision == LPW_BF16;
        N->fused_out = bf && cfg->rank <= BK && cfg->out_dim >= 8 && cfg->out_dim < (1 << 28);
        for (int l = 0; l <= N->L; ++l) {
            const int w = l == 0 ? N->din[0] : N->dout[l - 1];
            // the predictions go to the caller, and a fused output layer
            // makes its gradient in bfloat16: no FP32 ones then
            const bool fp = !N->fused_out || l < N->L;
            N->Act.push_back(fp ? A.make<float>(Bm * w) : nullptr);
            N->dAct.push_back(fp ? A.make<float>(Bm * w) : nullptr);
            N->Actb.push_back(bf && l < N->L ? A.make<uint16_t>(Bm * w) : nullptr);
            N->dActb.push_back(bf ? A.make<uint16_t>(Bm * w) : nullptr);
        }
        N->scratch_len = 64 * Bm * std::max(cfg->hidden, cfg->rank);
        N->scratch = A.make<float>(N->scratch_len);
        // one loss partial per 256 values, or per workgroup of k_out_layer
        N->lpart = A.make<double>(N->fused_out ? out_grid(cfg->out_dim) * ((Bm + kOutRows - 1) / kOutRows)
                                               : nblk(Bm * (int64_t)cfg->out_dim));
        int64_t sums = 0;
        for (int l = 0; l < N->L; ++l) {
            // few enough rows to a chunk that a full batch makes about 256
            // workgroups of a wide layer and 64 of a narrow one
            N->chunk.push_back(N->fused_out && l == N->L - 1 ? kOutRows : N->dout[l] >= 512 ? 16 : 4);
            sums += (Bm + N->chunk[l] - 1) / N->chunk[l] * N->dout[l];
        }
        float *cpart = A.make<float>(sums);
        std::vector<BiasPart> bp;
        for (int l = 0; l < N->L; ++l) {
            N->cpart.push_back(cpart);
            bp.push_back({cpart, N->G + N->boff[l], N->dout[l], N->chunk[l]});
            cpart += (Bm + N->chunk[l] - 1) / N->chunk[l] * N->dout[l];
        }
        N->bias_parts = A.make<BiasPart>(N->L);
        h2d(N->st, N->bias_parts, bp.data(), N->L);
        N->lout = A.make<double>(1);
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N.get(), h);
    }
    *out = N.release();
    return LP_OK;
}

int64_t lpw_param_count(const lpw_net *N) { return N ? N->nparam : 0; }

int lpw_set_params(lpw_net *N, const float *host)
{
    if (!N || !host) return LP_ERR_ARG;
    try {
        h2d(N->st, N->P, host, N->nparam);
        hipLaunchKernelGGL(k_to_bf16, dim3(nblk(N->nparam)), dim3(256), 0, N->st, (const float *)N->P, N->Pb,
                           N->nparam);
        HIPT(hipMemsetAsync(N->Mm, 0, sizeof(float) * (size_t)N->nparam, N->st));
        HIPT(hipMemsetAsync(N->Vv, 0, sizeof(float) * (size_t)N->nparam, N->st));
        N->step = 0;
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N, h);
    }
    return LP_OK;
}

int lpw_get_params(const lpw_net *Nc, float *host)
{
    lpw_net *N = const_cast<lpw_net *>(Nc);
    if (!N || !host) return LP_ERR_ARG;
    try {
        d2h(N->st, host, (const float *)N->P, N->nparam);
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N, h);
    }
    return LP_OK;
}

int lpw_set_norm(lpw_net *N, const float *mu, const float *sigma)
{
    if (!N || !mu || !sigma) return LP_ERR_ARG;
    for (int i = 0; i < N->cfg.in_dim; ++i)
        if (!(sigma[i] > 0.0f)) return LP_ERR_ARG;
    try {
        h2d(N->st, N->mu, mu, N->cfg.in_dim);
        h2d(N->st, N->sig, sigma, N->cfg.in_dim);
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N, h);
    }
    return LP_OK;
}

int lpw_forward(lpw_net *N, const float *X, int B, float *Z)
{
    if (!N || !X || !Z || B <= 0 || B > N->cfg.max_batch) return LP_ERR_ARG;
    try {
        forward(N, X, B, N->L, Z);
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N, h);
    }
    return LP_OK;
}

int lpw_loss_grad(lpw_net *N, const float *X, const float *Zstar, int B, double *loss)
{
    if (!N || !X || !Zstar || B <= 0 || B > N->cfg.max_batch) return LP_ERR_ARG;
    try {
        forward(N, X, B, N->L - 1, nullptr);
        output_loss(N, Zstar, B);
        backward(N, B);
        if (loss) d2h(N->st, loss, (const double *)N->lout, 1);
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N, h);
    }
    return LP_OK;
}

int lpw_get_grads(const lpw_net *Nc, float *host)
{
    lpw_net *N = const_cast<lpw_net *>(Nc);
    if (!N || !host) return LP_ERR_ARG;
    try {
        d2h(N->st, host, (const float *)N->G, N->nparam);
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N, h);
    }
    return LP_OK;
}

int lpw_adam_step(lpw_net *N, float lr, float beta1, float beta2, float eps)
{
    if (!N || !(lr > 0.0f)) return LP_ERR_ARG;
    try {
        N->step += 1;
        const float c1 = 1.0f - std::pow(beta1, (float)N->step), c2 = 1.0f - std::pow(beta2, (float)N->step);
        hipLaunchKernelGGL(k_adam, dim3(nblk(N->nparam)), dim3(256), 0, N->st, N->P, N->Mm, N->Vv, (const float *)N->G,
                           N->Pb, N->nparam, lr, beta1, beta2, eps, c1, c2);
        HIPT(hipGetLastError());
        HIPT(hipStreamSynchronize(N->st));
    } catch (const HipError &h) {
        return net_fail(N, h);
    }
    return LP_OK;
}

int lpw_train_step(lpw_net *N, const float *X, const float *Zstar, int B, float lr, double *loss)
{
    const int rc = lpw_loss_grad(N, X, Zstar, B, loss);
    if (rc != LP_OK) return rc;
    return lpw_adam_step(N, lr, 0.9f, 0.999f, 1e-8f);
}

int lpw_gemm(int precision, int trans_a, int trans_b, int M, int N, int K, const void *A, int lda, const void *B,
             int ldb, float *C, int ldc, void *stream)
{
    if (!A || !B || !C || M <= 0 || N <= 0 || K <= 0) return LP_ERR_ARG;
    try {
        gemm((hipStream_t)stream, precision == LPW_BF16, trans_a != 0, trans_b != 0, M, N, K, A, lda, B, ldb, C, ldc,
             nullptr, false, nullptr, 1, nullptr);
        HIPT(hipStreamSynchronize((hipStream_t)stream));
    } catch (const HipError &) {
        return LP_ERR_HIP;
    }
    return LP_OK;
}

int lpw_sketch(const int *rp, const int *ci, const float *v, int rows, const float *D, int cols, int B, float *out,
               void *stream)
{
    if (!rp || !ci || !v || !D || !out || rows <= 0 || cols <= 0 || B <= 0) return LP_ERR_ARG;
    try {
        hipLaunchKernelGGL(k_sketch, dim3(rows, B), dim3(256), 0, (hipStream_t)stream, rp, ci, v, D, cols, out, rows);
        HIPT(hipGetLastError());
        HIPT(hipStreamSynchronize((hipStream_t)stream));
    } catch (const HipError &) {
        return LP_ERR_HIP;
    }
    return LP_OK;
}

void lpw_free(lpw_net *N)
{
    if (!N) return;
    (void)hipStreamSynchronize(N->st);
    delete N;
}

const char *lpw_last_error(const lpw_net *N) { return N ? N->err.c_str() : ""; }

}  // extern "C"
