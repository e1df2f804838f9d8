// Tiled GEMMs for two or more activation rows (chunked prefill, batched decode,
// verification passes): Y[m][n] (+)= sum_k X[m][k] * W[n][k]; X fp32 [M][ldx], W row-major
// [N][K], Y fp32 [M][ldy].  Both operands are contiguous along K ("NT" form).
//   * fp32 weights: plain VALU tile kernel (the tiny configuration only).
//   * bf16 weights: MFMA kernels.  An fp32 activation x enters as two bf16 numbers,
//     hi = bf16(x) and lo = bf16(x - hi) (split_rows_kernel, or the producing kernel
//     writes the halves itself), and every weight tile is multiplied with both
//     (W.hi + W.lo, fp32 accumulation): the activations keep 16 mantissa bits, which
//     the bit-for-bit agreement of the bf16 KV-cache entries with an exact evaluation
//     needs; one bf16 pass would leave 8.
//       2..128 rows, gate/up with SwiGLU and heads of 160..256 row blocks: gemm_stream_kernel
//       2..64 rows, the rest: gemm_rows_kernel with K slices (gemm_rows64_kernel for small matrices,
//         gemm_rows_sk_kernel, work dealt evenly, for those of 200 row blocks and more)
//       more rows: gemm_tile_kernel, five block tiles from 128 x 128 to 256 x 256
// Requirements checked by the caller: K % 64 == 0; N, M arbitrary.
#pragma once
#include <algorithm>
#include <atomic>
#include "common.h"
#include "gemv.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// ---------------------------------------------------------------- fp32 tiles
// 64x64 output tile, 16x16 threads, 4x4 outputs per thread, BK = 16.
template <int EPI>
__global__ __launch_bounds__(256) void sgemm_nt_kernel(const float* __restrict__ W, int N, int K,
                                                       const float* __restrict__ X, int ldx,
                                                       float* __restrict__ Y, int ldy, int M) {
    __shared__ float As[16][64 + 4];
    __shared__ float Bs[16][64 + 4];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += 16) {
        // 64 rows x 16 k = 1024 elements per operand: 4 per thread
        {
            const int row = tid >> 2, kq = (tid & 3) * 4;
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
            if (m0 + row < M) a = *reinterpret_cast<const float4*>(X + (size_t)(m0 + row) * ldx + k0 + kq);
            if (n0 + row < N) b = *reinterpret_cast<const float4*>(W + (size_t)(n0 + row) * K + k0 + kq);
            As[kq + 0][row] = a.x; As[kq + 1][row] = a.y; As[kq + 2][row] = a.z; As[kq + 3][row] = a.w;
            Bs[kq + 0][row] = b.x; Bs[kq + 1][row] = b.y; Bs[kq + 2][row] = b.z; Bs[kq + 3][row] = b.w;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = As[k][ty * 4 + i]; b[i] = Bs[k][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + ty * 4 + i;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + tx * 4 + j;
            if (n < N) {
                float* yp = Y + (size_t)m * ldy + n;
                *yp = (EPI == EPI_RESID) ? (*yp + acc[i][j]) : acc[i][j];
            }
        }
    }
}

// The same for products whose 64x64 tiles would leave most of the chip idle (the tiny configuration: 128 rows of 128..1024
// columns are 4 to 32 of them): 32x32 tiles, K in blocks of 64 with the next block requested while the present one is multiplied.
// Every wave multiplies the whole tile on its quarter of a K block, 4x4 outputs per lane (eight 16-byte LDS reads for 64
// multiply-adds), and the quarters are added at the end.  Bound by the latency of the K steps and, within one, by the FMAs.
// 128 rows x 256 columns, K = 256 and 1024 in turn: 27.0 -> 16.6 us on average against 2x2 outputs per thread and all of K (two LDS
// reads for every four multiply-adds); 128 columns, K = 128 and 512, 15.2 -> 9.3.
template <int EPI>
__global__ __launch_bounds__(256) void sgemm32_nt_kernel(const float* __restrict__ W, int N, int K,
                                                         const float* __restrict__ X, int ldx,
                                                         float* __restrict__ Y, int ldy, int M) {
    constexpr int BK = 64, LD = BK + 4;                      // row stride 68: eight rows of 16 bytes touch all 32 banks
    __shared__ __attribute__((aligned(16))) float sm[2 * 32 * LD];
    float *Xs = sm, *Ws = sm + 32 * LD;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tx = lane & 7, ty = lane >> 3;
    const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    // copies: 16 threads per row of 64 k, rows tid / 16 and tid / 16 + 16
    const int row = tid >> 4, kq = (tid & 15) * 4;
    const float* xa[2] = {X + (size_t)min(m0 + row, M - 1) * ldx + kq, X + (size_t)min(m0 + row + 16, M - 1) * ldx + kq};
    const float* wb[2] = {W + (size_t)min(n0 + row, N - 1) * K + kq, W + (size_t)min(n0 + row + 16, N - 1) * K + kq};
    float acc[4][4] = {};
    f32x4_t a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) { a[i] = *reinterpret_cast<const f32x4_t*>(xa[i]); b[i] = *reinterpret_cast<const f32x4_t*>(wb[i]); }
    for (int k0 = 0; k0 < K; k0 += BK) {                     // (K is a multiple of 64)
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *reinterpret_cast<f32x4_t*>(Xs + (row + 16 * i) * LD + kq) = a[i];
            *reinterpret_cast<f32x4_t*>(Ws + (row + 16 * i) * LD + kq) = b[i];
        }
        __syncthreads();
        const int kn = min(k0 + BK, K - BK);
#pragma unroll
        for (int i = 0; i < 2; ++i) { a[i] = *reinterpret_cast<const f32x4_t*>(xa[i] + kn); b[i] = *reinterpret_cast<const f32x4_t*>(wb[i] + kn); }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int k = wave * 16 + kk * 4;
            f32x4_t x[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[i] = *reinterpret_cast<const f32x4_t*>(Xs + (ty + 8 * i) * LD + k);
                w[i] = *reinterpret_cast<const f32x4_t*>(Ws + (tx + 8 * i) * LD + k);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += x[i].x * w[j].x + x[i].y * w[j].y + x[i].z * w[j].z + x[i].w * w[j].w;
        }
    }
    // wave i takes row part i of all four quarters
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) sm[((wave * 4 + i) * 4 + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    const int m = m0 + ty + 8 * wave;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + tx + 8 * j;
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) v += sm[((q * 4 + wave) * 4 + j) * 64 + lane];
        if (m < M && n < N) {
            float* yp = Y + (size_t)m * ldy + n;
            *yp = (EPI == EPI_RESID) ? (*yp + v) : v;
        }
    }
}

// ---------------------------------------------------------------- bf16 MFMA, 2..64 rows, pre-split activations
// The activations arrive as two bf16 matrices Xh + Xl = x (hi and lo halves, [MT*32][K]; rows beyond M
// may hold anything: a row of x only ever meets its own row of the result).  A block of eight waves owns
// 256 rows of W and one K slice.  Every wave reads its 32 rows of W in whole 128-byte lines (8 lanes per
// row), two K blocks of 64 ahead in registers, and passes them through a private LDS tile into the MFMA
// operand layout (a lane of an MFMA operand holds 16 bytes of ONE row, so loading operands directly would
// touch every line with four separate instructions).  The activation tile of a K block (hi and lo) is
// copied as it is into LDS, double buffered, and shared by the eight waves.  LDS tiles are [row][64 k]
// with the eight 16-byte chunks of a row permuted by (row / 2) % 8, which makes both the line-wise
// writes and the operand reads conflict-free without padding.  No load in the loop is conditional
// (addresses past the end are clamped and never used), so the loads stay in flight across iterations.
// Partial results go to part[z][m][n]; a finish kernel adds the slices and applies the epilogue.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));    // native vector: stays in registers across LDS stores

// 16 bytes of a weight matrix that is read exactly once per launch: marked non-temporal, so that the stream of
// weights does not push the activation tiles (re-read by every block) out of L2
#ifndef RSD_W_NT
#define RSD_W_NT 1
#endif
__device__ __forceinline__ u32x4_t load_w16(const bf16_t* p) {
#if RSD_W_NT
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
#else
    return *reinterpret_cast<const u32x4_t*>(p);
#endif
}

// Thread blocks are handed to the eight XCDs round-robin by their linear index, and every XCD has an L2 of
// its own.  Blocks of one K slice read the same slice of the activations, so a K-sliced launch is renumbered:
// XCD k takes the logical indices [start(k), start(k + 1)), i.e. consecutive row blocks of few K slices, and
// fetches only those slices of the activations instead of all of them (7B down projection at 64 rows: the
// launch fetched 181 MB for 136 MB of weights, the 4.85 MB of activation halves once per XCD; 34.2 -> 32.1 us
// renumbered).  Done only where the activations weigh at least a tenth of the weights when fetched eight times
// (32 M >= 0.2 N): launches with small activations lose a little instead (72B output projection at 16 rows:
// 24.8 -> 26.9 us).  Results do not depend on the numbering.
__device__ __forceinline__ int xcd_major(int id, int nb, int M, int N) {
    if (160 * M < N) return id;
    constexpr int X = 8;
    const int k = id % X, j = id / X, q = nb / X, r = nb % X;
    return k * q + min(k, r) + j;
}

template <int MT>
__global__ __launch_bounds__(512, 2) void gemm_rows_kernel(const bf16_t* __restrict__ W, int N, int K,
                                                           const uint16_t* __restrict__ Xh,
                                                           const uint16_t* __restrict__ Xl,
                                                           float* __restrict__ part, int M) {
    constexpr int BK = 64, NWV = 8;
    constexpr int ROWS = 32 * MT;
    __shared__ __attribute__((aligned(16))) uint16_t Ah[2][ROWS * BK];
    __shared__ __attribute__((aligned(16))) uint16_t Al[2][ROWS * BK];
    __shared__ __attribute__((aligned(16))) uint16_t Ws[NWV][32 * BK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lin = xcd_major(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y, M, N);
    const int bx = lin % gridDim.x, by = lin / gridDim.x;     // row block, K slice
    const int nw = bx * (32 * NWV) + wave * 32;  // first W row of this wave
    const int kg = lane >> 5, l32 = lane & 31;
    const int nkb = K / BK;
    const int per = (nkb + gridDim.y - 1) / gridDim.y;
    const int kb0 = by * per, kb1 = min(nkb, kb0 + per);
    const int nk = kb1 - kb0;                            // K blocks of this slice (may be <= 0)
    const int kb_last = max(kb1 - 1, 0);
    // loads: lane -> row lane / 8 (+ 8 p), 16-byte chunk lane % 8 of the row's 128 bytes
    const int lrow = lane >> 3, lchunk = lane & 7;
    const bf16_t* wr0 = W + (size_t)min(nw + lrow, N - 1) * K + lchunk * 8;
    const bf16_t* wr1 = W + (size_t)min(nw + lrow + 8, N - 1) * K + lchunk * 8;
    const bf16_t* wr2 = W + (size_t)min(nw + lrow + 16, N - 1) * K + lchunk * 8;
    const bf16_t* wr3 = W + (size_t)min(nw + lrow + 24, N - 1) * K + lchunk * 8;
    uint16_t* ws = Ws[wave];
    // LDS offset (in bf16) of chunk c of row r
    auto sw = [](int r, int c) { return r * BK + ((c ^ ((r >> 1) & 7)) << 3); };
    const int ws_st0 = sw(lrow, lchunk), ws_st1 = sw(lrow + 8, lchunk), ws_st2 = sw(lrow + 16, lchunk), ws_st3 = sw(lrow + 24, lchunk);
    // activation tile: MT = 2: thread -> (row tid / 8, chunk tid % 8) of both halves; MT = 1: threads 0..255 the hi half, the rest lo
    const int xrow = (MT == 2) ? (tid >> 3) : ((tid & 255) >> 3);
    const int xsrc = min(xrow, M - 1);      // tile rows beyond M are never used: they repeat row M - 1 instead of fetching more of L2
    const uint16_t* xp0 = ((MT == 2 || tid < 256) ? Xh : Xl) + (size_t)xsrc * K + lchunk * 8;
    const uint16_t* xp1 = Xl + (size_t)xsrc * K + lchunk * 8;      // MT = 2 only
    const int x_st = sw(xrow, lchunk);

    f32x16_t acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;

    // register sets named member by member (arrays indexed in loops end up in scratch memory)
    struct WRegs { u32x4_t w0, w1, w2, w3; };
    WRegs wa, wb;
    u32x4_t x0, x1;
#define RSD_FETCH_W(kb, R)                                                                       \
    {                                                                                            \
        const size_t k0_ = (size_t)min((kb), kb_last) * BK;                                      \
        R.w0 = load_w16(wr0 + k0_);                                     \
        R.w1 = load_w16(wr1 + k0_);                                     \
        R.w2 = load_w16(wr2 + k0_);                                     \
        R.w3 = load_w16(wr3 + k0_);                                     \
    }
#define RSD_FETCH_X(kb)                                                                          \
    {                                                                                            \
        const size_t k0_ = (size_t)min((kb), kb_last) * BK;                                      \
        x0 = *reinterpret_cast<const u32x4_t*>(xp0 + k0_);                                       \
        if (MT == 2) x1 = *reinterpret_cast<const u32x4_t*>(xp1 + k0_);                          \
    }
#define RSD_STAGE_W(R)                                                                           \
    {                                                                                            \
        *reinterpret_cast<u32x4_t*>(ws + ws_st0) = R.w0;                                         \
        *reinterpret_cast<u32x4_t*>(ws + ws_st1) = R.w1;                                         \
        *reinterpret_cast<u32x4_t*>(ws + ws_st2) = R.w2;                                         \
        *reinterpret_cast<u32x4_t*>(ws + ws_st3) = R.w3;                                         \
    }
#define RSD_STAGE_X(buf)                                                                         \
    {                                                                                            \
        if (MT == 2) {                                                                           \
            *reinterpret_cast<u32x4_t*>(&Ah[(buf)][x_st]) = x0;                                  \
            *reinterpret_cast<u32x4_t*>(&Al[(buf)][x_st]) = x1;                                  \
        } else {                                                                                 \
            *reinterpret_cast<u32x4_t*>((tid < 256 ? &Ah[(buf)][0] : &Al[(buf)][0]) + x_st) = x0; \
        }                                                                                        \
    }
    // one K block: W tile of this wave in ws, activation tile in LDS buffer `buf`
#define RSD_COMPUTE(buf)                                                                         \
    {                                                                                            \
        _Pragma("unroll") for (int j_ = 0; j_ < 4; ++j_) {                                       \
            const bf16x8_t b_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(ws + sw(l32, kg * 4 + j_))); \
            _Pragma("unroll") for (int t_ = 0; t_ < MT; ++t_) {                                  \
                const int off_ = sw(t_ * 32 + l32, kg * 4 + j_);                                 \
                const bf16x8_t ah_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(&Ah[(buf)][off_])); \
                const bf16x8_t al_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(&Al[(buf)][off_])); \
                acc[t_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al_, b_, acc[t_], 0, 0, 0);    \
                acc[t_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah_, b_, acc[t_], 0, 0, 0);    \
            }                                                                                    \
        }                                                                                        \
    }
    // step i: the activation tile of block i + 1 moves into the LDS buffer that block i - 1 has left and
    // its registers at once take the request of block i + 2; block i is multiplied while W of block i + 2
    // is requested into the free set F; then W of block i + 1 (set S) replaces the wave's W tile
#define RSD_STEP(i_step, F, S)                                                                   \
    {                                                                                            \
        RSD_STAGE_X(((i_step) + 1) & 1)                                                          \
        RSD_FETCH_X(kb0 + (i_step) + 2)                                                          \
        RSD_FETCH_W(kb0 + (i_step) + 2, F)                                                       \
        RSD_COMPUTE((i_step) & 1)                                                                \
        RSD_STAGE_W(S)                                                                           \
        __syncthreads();                                                                         \
    }
    RSD_FETCH_W(kb0, wa)
    RSD_FETCH_X(kb0)
    RSD_FETCH_W(kb0 + 1, wb)
    RSD_STAGE_W(wa)
    RSD_STAGE_X(0)
    RSD_FETCH_X(kb0 + 1)
    __syncthreads();
    int i = 0;
    for (; i + 1 < nk; i += 2) {
        RSD_STEP(i, wa, wb)
        RSD_STEP(i + 1, wb, wa)
    }
    if (i < nk) RSD_STEP(i, wa, wb)
#undef RSD_STEP
#undef RSD_COMPUTE
#undef RSD_STAGE_W
#undef RSD_STAGE_X
#undef RSD_FETCH_W
#undef RSD_FETCH_X

    const int n = nw + l32;
    if (n < N) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = t * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (m < M) part[((size_t)by * ROWS + m) * N + n] = acc[t][v];      // rows beyond M are never read
            }
    }
}

// The same kernel with the work dealt evenly: the (256-row block of W) x (K block of 64) units of the product,
// numbered row block by row block, are cut into gridDim.x equal runs, one per thread block, whatever N and K
// are.  A run crosses at most a few row blocks; each stretch inside one row block is computed like a K slice
// above and written as a partial tile.  The partial tiles of row block rb come from the consecutive thread
// blocks first(rb) .. last(rb); thread block g writes its tile of rb into slice z = g - first(rb), so the slices
// of a row block are in ascending K order and the finish kernels add them in that fixed order.  D = 2 or 4 W
// register sets (K blocks requested ahead of their use).
struct SkGeom {
    int nkb;            // K blocks of 64
    int units;          // row blocks x K blocks
    int G;              // thread blocks the units are dealt to
    int zmax;           // most partial tiles any row block receives (slices of the partial buffer)
};
__host__ __device__ __forceinline__ long long sk_start(const SkGeom& g, int b) { return (long long)b * g.units / g.G; }
// first / last thread block whose run holds units of row block rb
__host__ __device__ __forceinline__ int sk_first(const SkGeom& g, int rb) {
    const long long x = (long long)rb * g.nkb;                       // largest b with start(b) <= x
    return (int)(((x + 1) * g.G + g.units - 1) / g.units) - 1;
}
__host__ __device__ __forceinline__ int sk_last(const SkGeom& g, int rb) {
    const long long y = (long long)(rb + 1) * g.nkb;                 // largest b with start(b) < y
    return (int)((y * g.G + g.units - 1) / g.units) - 1;
}

template <int MT, int D>
__global__ __launch_bounds__(512, D == 2 ? 2 : 1) void gemm_rows_sk_kernel(const bf16_t* __restrict__ W, int N, int K,
                                                                        const uint16_t* __restrict__ Xh,
                                                                        const uint16_t* __restrict__ Xl,
                                                                        float* __restrict__ part, SkGeom geo, int M) {
    constexpr int BK = 64, NWV = 8;
    constexpr int ROWS = 32 * MT;
    __shared__ __attribute__((aligned(16))) uint16_t Ah[2][ROWS * BK];
    __shared__ __attribute__((aligned(16))) uint16_t Al[2][ROWS * BK];
    __shared__ __attribute__((aligned(16))) uint16_t Ws[NWV][32 * BK];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kg = lane >> 5, l32 = lane & 31;
    const int lrow = lane >> 3, lchunk = lane & 7;
    uint16_t* ws = Ws[wave];
    auto sw = [](int r, int c) { return r * BK + ((c ^ ((r >> 1) & 7)) << 3); };
    const int ws_st0 = sw(lrow, lchunk), ws_st1 = sw(lrow + 8, lchunk), ws_st2 = sw(lrow + 16, lchunk), ws_st3 = sw(lrow + 24, lchunk);
    const int xrow = (MT == 2) ? (tid >> 3) : ((tid & 255) >> 3);
    const int xsrc = min(xrow, M - 1);      // tile rows beyond M are never used: they repeat row M - 1 instead of fetching more of L2
    const uint16_t* xp0 = ((MT == 2 || tid < 256) ? Xh : Xl) + (size_t)xsrc * K + lchunk * 8;
    const uint16_t* xp1 = Xl + (size_t)xsrc * K + lchunk * 8;      // MT = 2 only
    const int x_st = sw(xrow, lchunk);

    long long u = sk_start(geo, blockIdx.x);
    const long long u_end = sk_start(geo, blockIdx.x + 1);
    while (u < u_end) {
        const int rb = (int)(u / geo.nkb);
        const int kb0 = (int)(u - (long long)rb * geo.nkb);
        const int kb1 = (int)min((long long)geo.nkb, kb0 + (u_end - u));
        const int nk = kb1 - kb0, kb_last = kb1 - 1;
        u += nk;
        const int nw = rb * (32 * NWV) + wave * 32;      // first W row of this wave
        const bf16_t* wr0 = W + (size_t)min(nw + lrow, N - 1) * K + lchunk * 8;
        const bf16_t* wr1 = W + (size_t)min(nw + lrow + 8, N - 1) * K + lchunk * 8;
        const bf16_t* wr2 = W + (size_t)min(nw + lrow + 16, N - 1) * K + lchunk * 8;
        const bf16_t* wr3 = W + (size_t)min(nw + lrow + 24, N - 1) * K + lchunk * 8;

        f32x16_t acc[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;

        struct WRegs { u32x4_t w0, w1, w2, w3; };
        WRegs wa, wb, wc, wd;
        u32x4_t x0, x1;
#define SK_FETCH_W(kb, R)                                                                        \
    {                                                                                            \
        const size_t k0_ = (size_t)min((kb), kb_last) * BK;                                      \
        R.w0 = load_w16(wr0 + k0_);                                     \
        R.w1 = load_w16(wr1 + k0_);                                     \
        R.w2 = load_w16(wr2 + k0_);                                     \
        R.w3 = load_w16(wr3 + k0_);                                     \
    }
#define SK_FETCH_X(kb)                                                                           \
    {                                                                                            \
        const size_t k0_ = (size_t)min((kb), kb_last) * BK;                                      \
        x0 = *reinterpret_cast<const u32x4_t*>(xp0 + k0_);                                       \
        if (MT == 2) x1 = *reinterpret_cast<const u32x4_t*>(xp1 + k0_);                          \
    }
#define SK_STAGE_W(R)                                                                            \
    {                                                                                            \
        *reinterpret_cast<u32x4_t*>(ws + ws_st0) = R.w0;                                         \
        *reinterpret_cast<u32x4_t*>(ws + ws_st1) = R.w1;                                         \
        *reinterpret_cast<u32x4_t*>(ws + ws_st2) = R.w2;                                         \
        *reinterpret_cast<u32x4_t*>(ws + ws_st3) = R.w3;                                         \
    }
#define SK_STAGE_X(buf)                                                                          \
    {                                                                                            \
        if (MT == 2) {                                                                           \
            *reinterpret_cast<u32x4_t*>(&Ah[(buf)][x_st]) = x0;                                  \
            *reinterpret_cast<u32x4_t*>(&Al[(buf)][x_st]) = x1;                                  \
        } else {                                                                                 \
            *reinterpret_cast<u32x4_t*>((tid < 256 ? &Ah[(buf)][0] : &Al[(buf)][0]) + x_st) = x0; \
        }                                                                                        \
    }
#define SK_COMPUTE(buf)                                                                          \
    {                                                                                            \
        _Pragma("unroll") for (int j_ = 0; j_ < 4; ++j_) {                                       \
            const bf16x8_t b_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(ws + sw(l32, kg * 4 + j_))); \
            _Pragma("unroll") for (int t_ = 0; t_ < MT; ++t_) {                                  \
                const int off_ = sw(t_ * 32 + l32, kg * 4 + j_);                                 \
                const bf16x8_t ah_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(&Ah[(buf)][off_])); \
                const bf16x8_t al_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(&Al[(buf)][off_])); \
                acc[t_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al_, b_, acc[t_], 0, 0, 0);    \
                acc[t_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah_, b_, acc[t_], 0, 0, 0);    \
            }                                                                                    \
        }                                                                                        \
    }
        // step i: the activation tile of block i + 1 moves into the LDS buffer that block i - 1 has left and its
        // registers take the request of block i + 2; W of block i + D is requested into the set F that block i
        // came from; block i is multiplied; W of block i + 1 (set S) replaces the wave's W tile
#define SK_STEP(i_step, F, S)                                                                    \
    {                                                                                            \
        SK_STAGE_X(((i_step) + 1) & 1)                                                           \
        SK_FETCH_X(kb0 + (i_step) + 2)                                                           \
        SK_FETCH_W(kb0 + (i_step) + D, F)                                                        \
        SK_COMPUTE((i_step) & 1)                                                                 \
        SK_STAGE_W(S)                                                                            \
        __syncthreads();                                                                         \
    }
        SK_FETCH_W(kb0, wa)
        SK_FETCH_X(kb0)
        SK_FETCH_W(kb0 + 1, wb)
        if (D == 4) {
            SK_FETCH_W(kb0 + 2, wc)
            SK_FETCH_W(kb0 + 3, wd)
        }
        SK_STAGE_W(wa)
        SK_STAGE_X(0)
        SK_FETCH_X(kb0 + 1)
        __syncthreads();
        int i = 0;
        if (D == 2) {
            for (; i + 1 < nk; i += 2) {
                SK_STEP(i, wa, wb)
                SK_STEP(i + 1, wb, wa)
            }
            if (i < nk) SK_STEP(i, wa, wb)
        } else {
            for (; i + 3 < nk; i += 4) {
                SK_STEP(i, wa, wb)
                SK_STEP(i + 1, wb, wc)
                SK_STEP(i + 2, wc, wd)
                SK_STEP(i + 3, wd, wa)
            }
            if (i < nk) { SK_STEP(i, wa, wb) ++i; }
            if (i < nk) { SK_STEP(i, wb, wc) ++i; }
            if (i < nk) { SK_STEP(i, wc, wd) }
        }
#undef SK_STEP
#undef SK_COMPUTE
#undef SK_STAGE_W
#undef SK_STAGE_X
#undef SK_FETCH_W
#undef SK_FETCH_X
        const int z = (int)blockIdx.x - sk_first(geo, rb);
        const int n = nw + l32;
        if (n < N) {
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = t * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                    if (m < M) part[((size_t)z * ROWS + m) * N + n] = acc[t][v];
                }
        }
    }
}

// The same product for small weight matrices (attention projections, the draft's MLP): with 256 rows of W
// per block such a matrix gives few blocks, the K slices needed to fill the chip get short (two K blocks
// for the 7B output projection) and their partial results weigh as much as the weights.  Here a block of
// eight waves owns 64 rows of W and one K slice; the W tile and the activation tile of a K block are
// shared through LDS (double buffered; W requested four K blocks ahead), the waves divide the
// 64 x ROWS x 64 product of a K block among themselves by (W half, activation half, K part) and add their
// K parts in a fixed order through LDS at the end.  Same partial-result layout and finish kernels.
// Measured at 64 rows (kernel alone, against the 256-row kernel): 7B output projection 17.0 -> 11.7 us,
// 7B QKV 16.7 -> 14.1, 1.5B down 16.4 -> 13.6, 1.5B QKV 7.8 -> 4.8; large matrices (7B down) lose.
template <int MT, bool LONG>
__global__ __launch_bounds__(512, 2) void gemm_rows64_kernel(const bf16_t* __restrict__ W, int N, int K,
                                                             const uint16_t* __restrict__ Xh,
                                                             const uint16_t* __restrict__ Xl,
                                                             float* __restrict__ part, int M) {
    constexpr int BK = 64, ROWS = 32 * MT, KH = 4 / MT, JS = 4 / KH;   // K parts per K block; operand steps per wave
    constexpr int WS_E = 64 * BK, XS_E = ROWS * BK;
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * WS_E + 4 * XS_E];
    uint16_t* Ws = smem;                       // [2][64 * 64]
    uint16_t* Ah = smem + 2 * WS_E;            // [2][ROWS * 64]
    uint16_t* Al = Ah + 2 * XS_E;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = wave & 1;                                   // W rows wi * 32 ..
    const int xj = (MT == 2) ? ((wave >> 1) & 1) : 0;          // activation rows xj * 32 ..
    const int kh = (MT == 2) ? (wave >> 2) : (wave >> 1);      // K part
    const int kg = lane >> 5, l32 = lane & 31;
    const int lin = xcd_major(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y, M, N);
    const int bx = lin % gridDim.x, by = lin / gridDim.x;     // row block, K slice
    const int n0 = bx * 64;
    const int nkb = K / BK;
    const int per = (nkb + gridDim.y - 1) / gridDim.y;
    const int kb0 = by * per, kb1 = min(nkb, kb0 + per);
    const int nk = kb1 - kb0;
    const int kb_last = max(kb1 - 1, 0);
    auto sw = [](int r, int c) { return r * BK + ((c ^ ((r >> 1) & 7)) << 3); };
    // copies: thread -> 16-byte chunk tid % 8 of row tid / 8 of the W tile; the same of the activation halves
    const int lrow = tid >> 3, lchunk = tid & 7;
    const bf16_t* wr = W + (size_t)min(n0 + lrow, N - 1) * K + lchunk * 8;
    const int w_st = sw(lrow, lchunk);
    const int xrow = (MT == 2) ? lrow : ((tid & 255) >> 3);
    const int xsrc = min(xrow, M - 1);      // as above: rows beyond M repeat row M - 1
    const uint16_t* xp0 = ((MT == 2 || tid < 256) ? Xh : Xl) + (size_t)xsrc * K + lchunk * 8;
    const uint16_t* xp1 = Xl + (size_t)xsrc * K + lchunk * 8;      // MT = 2 only
    const int x_st = sw(xrow, lchunk);

    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;

    // requested ahead: W four K blocks, the thread's activation chunks x, y as far in long slices, else one block (set 0)
    u32x4_t w0, w1, w2, w3, x0, x1, x2, x3, y0, y1, y2, y3;
#define R64_FETCH_W(kb, S) { w##S = load_w16(wr + (size_t)min((kb), kb_last) * BK); }
#define R64_FETCH_X(kb, S)                                                                       \
    {                                                                                            \
        const size_t k0_ = (size_t)min((kb), kb_last) * BK;                                      \
        x##S = *reinterpret_cast<const u32x4_t*>(xp0 + k0_);                                     \
        if (MT == 2) y##S = *reinterpret_cast<const u32x4_t*>(xp1 + k0_);                        \
    }
#define R64_FETCH(kb, S) R64_FETCH_W(kb, S) R64_FETCH_X(kb, S)
#define R64_STAGE(buf, S, X)                                                                     \
    {                                                                                            \
        *reinterpret_cast<u32x4_t*>(Ws + (buf) * WS_E + w_st) = w##S;                            \
        if (MT == 2) {                                                                           \
            *reinterpret_cast<u32x4_t*>(Ah + (buf) * XS_E + x_st) = x##X;                        \
            *reinterpret_cast<u32x4_t*>(Al + (buf) * XS_E + x_st) = y##X;                        \
        } else {                                                                                 \
            *reinterpret_cast<u32x4_t*>((tid < 256 ? Ah : Al) + (buf) * XS_E + x_st) = x##X;     \
        }                                                                                        \
    }
#define R64_COMPUTE(buf)                                                                         \
    {                                                                                            \
        _Pragma("unroll") for (int s_ = 0; s_ < JS; ++s_) {                                      \
            const int c_ = kg * 4 + kh * JS + s_;                                                \
            const bf16x8_t b_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(Ws + (buf) * WS_E + sw(wi * 32 + l32, c_))); \
            const int off_ = sw(xj * 32 + l32, c_);                                              \
            const bf16x8_t ah_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(Ah + (buf) * XS_E + off_)); \
            const bf16x8_t al_ = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(Al + (buf) * XS_E + off_)); \
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al_, b_, acc, 0, 0, 0);                \
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah_, b_, acc, 0, 0, 0);                \
        }                                                                                        \
    }
    // step i: block i + 1 (W in set S) moves into the LDS buffer that block i - 1 has left; S at once takes the request of W block
    // i + 5, the activation set that has become free that of block i + 5 or i + 2; block i is multiplied
#define R64_STEP(i_step, S)                                                                      \
    {                                                                                        \
        if (LONG) {                                                              \
            R64_STAGE(((i_step) + 1) & 1, S, S)                                              \
            R64_FETCH(kb0 + (i_step) + 5, S)                                                 \
        } else {                                                                             \
            R64_STAGE(((i_step) + 1) & 1, S, 0)                                              \
            R64_FETCH_W(kb0 + (i_step) + 5, S)                                               \
            R64_FETCH_X(kb0 + (i_step) + 2, 0)                                               \
        }                                                                                    \
        R64_COMPUTE((i_step) & 1)                                                            \
        __syncthreads();                                                                     \
    }
    R64_FETCH(kb0, 0)
    if (LONG) {
        R64_FETCH(kb0 + 1, 1)
        R64_FETCH(kb0 + 2, 2)
        R64_FETCH(kb0 + 3, 3)
    } else {
        R64_FETCH_W(kb0 + 1, 1)
        R64_FETCH_W(kb0 + 2, 2)
        R64_FETCH_W(kb0 + 3, 3)
    }
    R64_STAGE(0, 0, 0)
    R64_FETCH_W(kb0 + 4, 0)
    if (LONG) R64_FETCH_X(kb0 + 4, 0) else R64_FETCH_X(kb0 + 1, 0)
    __syncthreads();
    int i = 0;
    for (; i + 3 < nk; i += 4) {
        R64_STEP(i, 1)
        R64_STEP(i + 1, 2)
        R64_STEP(i + 2, 3)
        R64_STEP(i + 3, 0)
    }
    if (i < nk) { R64_STEP(i, 1) ++i; }
    if (i < nk) { R64_STEP(i, 2) ++i; }
    if (i < nk) { R64_STEP(i, 3) }
#undef R64_STEP
#undef R64_COMPUTE
#undef R64_STAGE
#undef R64_FETCH
#undef R64_FETCH_W
#undef R64_FETCH_X

    // add the K parts in ascending order through LDS (the tiles are dead: every wave is past the last barrier)
    float* red = reinterpret_cast<float*>(smem);
    const int pair = wi + 2 * xj;                       // waves with equal (wi, xj) hold parts of one 32 x 32 result
    if (kh > 0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) red[(((kh - 1) * (2 * MT) + pair) * 16 + v) * 64 + lane] = acc[v];
    }
    __syncthreads();
    if (kh == 0) {
#pragma unroll
        for (int p = 0; p < KH - 1; ++p)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] += red[((p * (2 * MT) + pair) * 16 + v) * 64 + lane];
        const int n = n0 + wi * 32 + l32;
        if (n < N) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = xj * 32 + 8 * (v >> 2) + 4 * kg + (v & 3);
                if (m < M) part[((size_t)by * ROWS + m) * N + n] = acc[v];
            }
        }
    }
}

// x[4] as hi + lo bf16 halves
__device__ __forceinline__ void store_halves(uint16_t* __restrict__ h, uint16_t* __restrict__ l, const float4& x) {
    uint2 hi, lo;
    split2(x.x, x.y, hi.x, lo.x);
    split2(x.z, x.w, hi.y, lo.y);
    *reinterpret_cast<uint2*>(h) = hi;
    *reinterpret_cast<uint2*>(l) = lo;
}

// fp32 rows -> hi + lo bf16 rows, optionally through RMSNorm (gain != nullptr).  One block per row.  EMBED: the rows are token
// embeddings gathered here and also left in X (one launch instead of two at the start of a pass; rows without a token
// are skipped).  A row is requested once, whole and with its gains, and kept in registers: few rows are bound by latency (four
// columns per thread; 7B, 32 rows: gather and split 3.8 + 5.0 us in two launches, 4.6 in one), many by traffic (sixteen columns
// per thread, small blocks; 6001 rows: split 33.6 -> 28 us, gather and split 67 -> 47).
template <typename WT, bool EMBED>
__global__ __launch_bounds__(1024) void split_rows_kernel(float* __restrict__ X, int ldx, int K, const WT* __restrict__ gain, float eps,
                                                          uint16_t* __restrict__ Xh, uint16_t* __restrict__ Xl,
                                                          const WT* __restrict__ E, const int* __restrict__ tokens, int max_ctx,
                                                          RowMap rm) {
    __shared__ float red[16];
    constexpr int NI = 4;
    const int tid = threadIdx.x, step = blockDim.x * 4;
    float* xr = X + (size_t)blockIdx.x * ldx;
    uint16_t* xh = Xh + (size_t)blockIdx.x * K;
    uint16_t* xl = Xl + (size_t)blockIdx.x * K;
    Raw4<WT> gv[NI];
    if (gain) {
#pragma unroll
        for (int i = 0; i < NI; ++i) if (i * step < K) gv[i].load(gain + min(tid * 4 + i * step, K - 4));
    }
    const WT* er = nullptr;
    if (EMBED) {
        int seq, pos;
        if (!row_lookup(rm, blockIdx.x, seq, pos)) return;
        er = E + (size_t)tokens[(size_t)seq * max_ctx + pos] * K;
    }
    auto load = [&](int k) {
        if (!EMBED) return *reinterpret_cast<const float4*>(xr + k);
        Raw4<WT> e;
        e.load(er + k);
        return e.get();
    };
    float4 v[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) if (i * step < K) v[i] = load(min(tid * 4 + i * step, K - 4));
    float rs = 1.0f;
    if (gain) {
        float ss = 0.0f;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (tid * 4 + i * step < K) ss += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
        for (int k = tid * 4 + NI * step; k < K; k += step) {
            const float4 w = load(k);
            ss += w.x * w.x + w.y * w.y + w.z * w.z + w.w * w.w;
        }
        ss = wave_sum(ss);
        if ((tid & 63) == 0) red[tid >> 6] = ss;
        __syncthreads();
        float tot = 0.0f;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) tot += red[w];
        rs = 1.0f / sqrtf(tot / (float)K + eps);
    }
    auto finish = [&](int k, float4 x, const Raw4<WT>& gr) {
        if (EMBED) *reinterpret_cast<float4*>(xr + k) = x;
        if (gain) {
            const float4 g = gr.get();
            x.x *= rs * g.x; x.y *= rs * g.y; x.z *= rs * g.z; x.w *= rs * g.w;
        }
        store_halves(xh + k, xl + k, x);
    };
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int k = tid * 4 + i * step;
        if (k < K) finish(k, v[i], gv[i]);
    }
    for (int k = tid * 4 + NI * step; k < K; k += step) {
        Raw4<WT> g;
        if (gain) g.load(gain + k);
        finish(k, load(k), g);
    }
}

// sum over z (ascending) of the float4 at p + z * stride; eight loads are requested at a time, the last
// batch with clamped addresses (one round trip for the remainder instead of one per slice)
__device__ __forceinline__ float4 sum_slices(const float* __restrict__ p, size_t stride, int KS) {
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    int z = 0;
    for (; z + 8 <= KS; z += 8) {
        float4 b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = *reinterpret_cast<const float4*>(p + (size_t)(z + i) * stride);
#pragma unroll
        for (int i = 0; i < 8; ++i) { a.x += b[i].x; a.y += b[i].y; a.z += b[i].z; a.w += b[i].w; }
    }
    if (z < KS) {
        float4 b[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = *reinterpret_cast<const float4*>(p + (size_t)min(z + i, KS - 1) * stride);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (z + i < KS) { a.x += b[i].x; a.y += b[i].y; a.z += b[i].z; a.w += b[i].w; }
    }
    return a;
}

// Adds the K slices of gemm_rows_kernel (ascending z) and finishes:
//   EPI_STORE   Y[m][n]  = sum
//   EPI_RESID   Y[m][n] += sum
//   EPI_SWIGLU  N = 2F columns [gate ; up]: act = silu(gate) * up, written as hi + lo bf16 rows [m][F]
// geo.G > 0: the slices come from gemm_rows_sk_kernel, and a column of row block rb = n / 256 has
// sk_last(rb) - sk_first(rb) + 1 of them (KS is ignored).
template <int EPI>
__global__ void rows_finish_kernel(const float* __restrict__ part, int KS, int ROWS, int M, int N,
                                   float* __restrict__ Y, int ldy, uint16_t* __restrict__ Oh, uint16_t* __restrict__ Ol,
                                   SkGeom geo) {
    const int NO = (EPI == EPI_SWIGLU) ? N / 2 : N;
    const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i >= (size_t)M * NO) return;
    const size_t m = i / NO, n = i - m * NO;           // NO is a multiple of 4
    auto sum = [&](size_t col) {
        int ks = KS;
        if (geo.G > 0) { const int rb = (int)(col >> 8); ks = sk_last(geo, rb) - sk_first(geo, rb) + 1; }
        return sum_slices(part + m * N + col, (size_t)ROWS * N, ks);
    };
    float4 a = sum(n);
    if (EPI == EPI_SWIGLU) {
        const float4 u = sum(NO + n);
        store_halves(Oh + m * NO + n, Ol + m * NO + n,
                     make_float4(a.x / (1.0f + expf(-a.x)) * u.x, a.y / (1.0f + expf(-a.y)) * u.y,
                                 a.z / (1.0f + expf(-a.z)) * u.z, a.w / (1.0f + expf(-a.w)) * u.w));
    } else {
        float4* yp = reinterpret_cast<float4*>(Y + m * ldy + n);
        if (EPI == EPI_RESID) { const float4 y = *yp; a.x += y.x; a.y += y.y; a.z += y.z; a.w += y.w; }
        *yp = a;
    }
}

// EPI_RESID finish for a whole row per block, with the RMSNorm of the NEXT projection folded in: adds the K
// slices (ascending z) and the residual, stores the new residual stream H, and writes
// RMSNorm(H row) * gain as hi + lo bf16 halves.  N <= 8192, N % 4 == 0.
template <typename WT>
__global__ __launch_bounds__(1024) void rows_finish_norm_kernel(const float* __restrict__ part, int KS, int ROWS, int N,
                                                                float* __restrict__ H, int ldh,
                                                                const WT* __restrict__ gain, float eps,
                                                                uint16_t* __restrict__ Xh, uint16_t* __restrict__ Xl,
                                                                SkGeom geo) {
    __shared__ float red[16];
    const int m = blockIdx.x, tid = threadIdx.x;
    float4 v[2];
    float ss = 0.0f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = tid * 4 + i * 4096;
        v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (n < N) {
            int ks = KS;
            if (geo.G > 0) { const int rb = n >> 8; ks = sk_last(geo, rb) - sk_first(geo, rb) + 1; }
            float4 a = sum_slices(part + (size_t)m * N + n, (size_t)ROWS * N, ks);
            float4* hp = reinterpret_cast<float4*>(H + (size_t)m * ldh + n);
            const float4 y = *hp;
            a.x += y.x; a.y += y.y; a.z += y.z; a.w += y.w;
            *hp = a;
            v[i] = a;
            ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
        }
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    float tot = 0.0f;
#pragma unroll
    for (int w = 0; w < 16; ++w) tot += red[w];
    const float rs = 1.0f / sqrtf(tot / (float)N + eps);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = tid * 4 + i * 4096;
        if (n < N) {
            store_halves(Xh + (size_t)m * N + n, Xl + (size_t)m * N + n,
                         make_float4(v[i].x * (rs * ld1(gain + n)), v[i].y * (rs * ld1(gain + n + 1)),
                                     v[i].z * (rs * ld1(gain + n + 2)), v[i].w * (rs * ld1(gain + n + 3))));
        }
    }
}

// K slices for gemm_rows_kernel.  Measured (K-slice sweeps over the 1.5B / 7B / 72B shapes at 16 and 64 rows):
// the kernel is fastest when the grid has at most one block per compute unit and covers most of them
// (7B down: 252 or 224 blocks 32 us, 280 blocks 45 us, 462 blocks 35 us); two co-resident blocks only
// pay when one per unit would leave the chip half empty (148 row blocks of K = 3584: x 3 slices 59 us, x 1 86 us; the 7B gate/up pair
// has that shape, but goes to gemm_stream_kernel).
// So: the largest count with rows-of-blocks x slices <= 256 if that fills 200 units or more; otherwise the
// count that minimises (rounds of 512 resident blocks) x (K blocks per slice) plus the traffic of the
// partial results, in units of one K block over 256 rows of W.
static int gemm_rows64_slices(int N, int K, int rows, size_t part_floats);
static bool gemm_rows_small(int N, int K);
static int gemm_rows_slices(int N, int K, int rows, size_t part_floats) {
    if (gemm_rows_small(N, K)) return gemm_rows64_slices(N, K, rows, part_floats);
    const int nb = (N + 255) / 256, nkb = K / 64;
    {
        int ks = std::min(256 / nb, nkb / 2);
        while (ks > 1 && ((size_t)ks * rows * N > part_floats || (ks - 1) * ((nkb + ks - 1) / ks) >= nkb)) --ks;
        if (ks >= 1 && nb * ks >= 200 && (size_t)ks * rows * N <= part_floats) return ks;
    }
    int best = 1;
    double best_cost = 1e30;
    for (int ks = 1; ks <= 64 && ks <= nkb; ++ks) {
        if ((size_t)ks * rows * N > part_floats) break;
        const int per = (nkb + ks - 1) / ks;
        if ((ks - 1) * per >= nkb) continue;                 // would leave a slice empty
        const int rounds = (nb * ks + 511) / 512;
        const double cost = (double)rounds * per * 512 * 256 * 128 + (double)ks * rows * N * 8;
        if (cost < best_cost) { best_cost = cost; best = ks; }
    }
    return best;
}

// Small matrices (at most 17 M weights: the 7B QKV and output projections, the 1.5B down and attention
// projections) go to the 64-row kernel, with as many K slices as bring the grid to about 450 blocks (4..8, and
// at least two K blocks each).  The 7B QKV (16.5 M) is the largest of them: 16.5 us there against 18.0 us on
// 256-row blocks at 64 rows, and its 6 instead of 14 K slices make the attention kernel that adds them
// 2 us faster.
static bool gemm_rows_small(int N, int K) { return (size_t)N * K <= ((size_t)17 << 20); }
static int gemm_rows64_slices(int N, int K, int rows, size_t part_floats) {
    const int nb = (N + 63) / 64, nkb = K / 64;
    int ks = std::max(4, std::min(8, (448 + nb / 2) / nb));
    while (ks > 1 && (ks * 2 > nkb || (size_t)ks * rows * N > part_floats || (ks - 1) * ((nkb + ks - 1) / ks) >= nkb)) --ks;
    return ks;
}

// Geometry of the evenly dealt kernel for an [N][K] matrix on G thread blocks (G is lowered to the number of
// units when there are fewer).
static SkGeom sk_geometry(int N, int K, int G) {
    SkGeom g;
    const int nb = (N + 255) / 256;
    g.nkb = K / 64;
    g.units = nb * g.nkb;
    g.G = std::max(1, std::min(G, g.units));
    g.zmax = 1;
    for (int rb = 0; rb < nb; ++rb) g.zmax = std::max(g.zmax, sk_last(g, rb) - sk_first(g, rb) + 1);
    return g;
}
// Which few-row products take the evenly dealt kernel: those with 200 or more 256-row blocks, which uniform K
// slices cannot spread evenly over 256 compute units (measured at 16 rows: [59136][8192] 190 -> 183 us,
// [151936][8192] 526 -> 457 us, [151936][1536] 112 -> 106 us; with fewer row blocks uniform slices at two
// co-resident blocks per unit are as fast or faster: [37888][3584] 52 against 58 us).  One thread block per
// compute unit and two W register sets: 512 thread blocks or four sets were slower or equal.
constexpr int kSkBlocks = 256, kSkDepth = 2;
static bool gemm_rows_even(int N, int K) { (void)K; return (N + 255) / 256 >= 200; }
template <int D>
static void gemm_rows_sk_launch(hipStream_t st, const bf16_t* W, int N, int K, const uint16_t* Xh, const uint16_t* Xl,
                                int M, float* part, const SkGeom& g) {
    if (M <= 32) hipLaunchKernelGGL((gemm_rows_sk_kernel<1, D>), dim3(g.G), dim3(512), 0, st, W, N, K, Xh, Xl, part, g, M);
    else         hipLaunchKernelGGL((gemm_rows_sk_kernel<2, D>), dim3(g.G), dim3(512), 0, st, W, N, K, Xh, Xl, part, g, M);
}

// K blocks per slice from which gemm_rows64_kernel requests the activations as far ahead as the weights: a step of one block ahead lasts as
// long as an L2 read, which a long slice pays many times (1536 x 8960, 18 blocks: 4 rows 10.9 -> 8.2 us, 16 rows 11.0 -> 9.0, 32 rows
// 11.4 -> 10.2, 64 rows 14.1 -> 13.4); short ones re-read their last block for the requests beyond it, at 64 rows (7 blocks, 3584 x 3584:
// 14.9 -> 15.9; 10 blocks, 4608 x 3584: 17.3 -> 18.4) as at fewer (4 / 16 / 32 rows: 8.8 -> 8.5, 9.6 -> 9.7, 11.0 -> 11.3 and 10.3 -> 10.1,
// 11.2 -> 11.4, 13.0 -> 13.3; within whole passes).  No matrix with slices of 11 to 17 blocks has been measured: the line lies between.
constexpr int kLongSlice = 14;
static void gemm_rows_launch(hipStream_t st, const bf16_t* W, int N, int K, const uint16_t* Xh, const uint16_t* Xl,
                             int M, float* part, int ks) {
    if (gemm_rows_small(N, K)) {
        const dim3 grid((N + 63) / 64, ks), block(512);
#define RSD_R64(LONG)                                                                                                \
    if (M <= 32) hipLaunchKernelGGL((gemm_rows64_kernel<1, LONG>), grid, block, 0, st, W, N, K, Xh, Xl, part, M);     \
    else         hipLaunchKernelGGL((gemm_rows64_kernel<2, LONG>), grid, block, 0, st, W, N, K, Xh, Xl, part, M);
        if ((K / 64 + ks - 1) / ks >= kLongSlice) { RSD_R64(true) } else { RSD_R64(false) }
#undef RSD_R64
        return;
    }
    const dim3 grid((N + 255) / 256, ks), block(512);
    if (M <= 32) hipLaunchKernelGGL((gemm_rows_kernel<1>), grid, block, 0, st, W, N, K, Xh, Xl, part, M);
    else         hipLaunchKernelGGL((gemm_rows_kernel<2>), grid, block, 0, st, W, N, K, Xh, Xl, part, M);
}

// ---------------------------------------------------------------- dispatch
static void gemm_launch(hipStream_t st, int epi, const float* W, int N, int K, const float* X, int ldx,
                        float* Y, int ldy, int M, float* part, size_t part_floats) {
    (void)part; (void)part_floats;
    if (M <= 8) { gemv_launch<float>(st, PRO_NONE, epi, W, N, K, X, ldx, nullptr, 0.f, Y, ldy, M); return; }
    const dim3 grid((N + 63) / 64, (M + 63) / 64), block(256);
    if (grid.x * grid.y < 256) {                             // fewer 64x64 tiles than compute units: see sgemm32_nt_kernel
        const dim3 grid32((N + 31) / 32, (M + 31) / 32);
        if (epi == EPI_RESID) hipLaunchKernelGGL((sgemm32_nt_kernel<EPI_RESID>), grid32, block, 0, st, W, N, K, X, ldx, Y, ldy, M);
        else                  hipLaunchKernelGGL((sgemm32_nt_kernel<EPI_STORE>), grid32, block, 0, st, W, N, K, X, ldx, Y, ldy, M);
        return;
    }
    if (epi == EPI_RESID) hipLaunchKernelGGL((sgemm_nt_kernel<EPI_RESID>), grid, block, 0, st, W, N, K, X, ldx, Y, ldy, M);
    else                  hipLaunchKernelGGL((sgemm_nt_kernel<EPI_STORE>), grid, block, 0, st, W, N, K, X, ldx, Y, ldy, M);
}

// silu(g) * u as accurate as g / (1 + expf(-g)) * u (largest relative error against 64 bits 1.8e-7 in both, rms 4e-8), in 14 vector
// instructions instead of 27.  e = exp(-g) is 2^n times the hardware's exponential of an exactly reduced argument (n an integer,
// |t| <= 1/2 with the low part of log2 e); n is rounded and shifted into the exponent by one addition each (as long as e / 4 is a
// normal number, hence the upper limit: beyond 60 it vanishes in the sum); the quotient is a reciprocal with one correction.  Sum and
// numerator are kept a factor of 4 smaller than they are: the reciprocal of (1 + e) / 4 is a normal number as long as e is finite, and
// beyond that (g < -88.72) zero.
// Together with the conversions of common.h (30 -> 18 vector instructions per value in the epilogue, which no product overlaps):
// 8192 x 17920 x 1536 683 -> 674 us, 2048 x 37888 x 3584 763 -> 759.
// (exp2(-g log2 e) unreduced with the bare reciprocal, six instructions, has an error that grows with |g|: 1e-6 at -20, 3.9e-6 at -87.)
__device__ __forceinline__ float silu_mul(float g, float u) {
    constexpr float R = 12582910.0f;                         // 1.5 x 2^23 - 2: the sum's low bits are n - 2
    const float c = __builtin_amdgcn_fmed3f(g, -89.0f, 60.0f), m = fmaf(-1.4426950408889634f, c, R), n = m - R;
    const float t = fmaf(-1.9259629911e-8f, c, fmaf(-1.4426950408889634f, c, -n));
    const float e = __uint_as_float((__float_as_uint(m) << 23) + __float_as_uint(__builtin_amdgcn_exp2f(t)));
    const float s = 0.25f + e, r = __builtin_amdgcn_rcpf(s);
    const float h = 0.25f * g, q = h * r;
    return fmaf(fmaf(-s, q, h), r, q) * u;
}

// ---------------------------------------------------------------- bf16 MFMA, many rows, pre-split activations
// Y[m][n] (+)= sum_k (Xh + Xl)[m][k] * W[n][k] for more than 64 rows (prefill chunks, large decode batches).
// Block tile BM rows of X x BN rows of W on eight waves, MFMA tiles of 16x16x32, lo half of X first, then hi.
//
// What bounds it: the power the chip may draw, and with it the energy of a product.  Three choices follow from that:
//   * 16x16x32 MFMAs instead of 32x32x16: the same products with half as much accumulator traffic.  A register-only loop on
//     normally distributed operands sustains 2.04 PFLOP/s at 2.0 GHz with them, 1.81 at 1.77 GHz with 32x32x16; in this
//     kernel 8192 x 37888 x 3584 3340 -> 3178 us, 8192 x 4608 x 3584 424 -> 393.  W is the first operand: a lane then holds
//     four consecutive columns of a row and stores them at once;
//   * K blocks of 64, so that every request of the copies covers whole 128-byte lines: with blocks of 32 each line was asked
//     for in two halves, twice the requests at L2 (8192 x 3584 x 18944: 2.08e8 -> 1.06e8).  With the copies taken
//     out altogether the loop runs 14-24 % faster: what moves through L2 costs both issue slots and power.
//     8192 x 37888 x 3584 3178 -> 3118 us, 8192 x 3584 x 18944 1642 -> 1557, 8192 x 1536 x 8960 367 -> 331;
//   * operands stay in registers as long as they are used: a tile of W is overwritten by its successor right behind its
//     last product, the X operands of the next pass are read while this one multiplies.
// A K block is four passes of 32 k: lo half of X first and second 32 k, hi half first and second.  LDS holds a ring of three
// X units (the lo and the hi half of a block in turn) and two W units, [rows][64 k] with chunks of 16 bytes permuted by
// (row / 2) % 8, which makes the operand reads conflict-free without padding.  The copies go straight from global memory
// into LDS (global_load_lds, 1 KB per wave request, the permutation applied to the source address), a whole K block before
// they are used.  One barrier in the second pass of either half, two tiles of W into it, while the products have all their
// operands: before it every wave has the unit that is read next landed (vmcnt) and has read the one that becomes free
// (lgkmcnt).  The order inside a pass is pinned with sched_barrier; the requests are inline assembly because the compiler
// would otherwise drain them (vmcnt(0)) in front of every LDS read.  They write no registers.
// Measured against the kernel of 32x32x16 MFMAs and blocks of 32 k (one card): 8192 x 37888 x 3584 3340 -> 3118 us (1.33 -> 1.43
// PFLOP/s executed), 2048 rows of it 843 -> 788, 8192 x 3584 x 18944 1705 -> 1557, 8192 x 4608 x 3584 424 -> 373, 8192 x 17920 x
// 1536 735 -> 704, 8192 x 1536 x 8960 384 -> 331; 2400 shader cycles per 32 k (2048 of MFMA issue) at 1.82 GHz, 2270 at 1.60
// before; no LDS bank conflicts.  Fewer, larger waves (four of 128 x 128) leave the barrier exposed.
// Thread blocks go to the XCDs round-robin by index; they are renumbered so that an XCD works on consecutive tiles in
// groups of four row tiles (32 resident blocks = 4 x 8 tiles share their operands in that XCD's L2): 3.50 -> 3.23 ms.
// gridDim.z > 1 cuts K into slices whose partial tiles go to part[z][M][N] (finished by rows_finish_kernel).
__device__ __forceinline__ void copy16_to_lds(uint32_t lds_off, uint32_t voff, const char* base) {
    // lane l: 16 bytes at base + voff -> LDS byte lds_off + 16 l  (M0 holds the wave's LDS address; one wait state behind its write)
    // (M0 is not named as clobbered: it is a reserved register, in which the compiler keeps no value from one statement to the next -
    // naming it draws a warning - and in these kernels no instruction of the compiler's own reads it)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_off), "v"(voff), "s"(base) : "memory");
}
template <int BM, int BN>
struct TileCfg {
    static constexpr int BK = 64;
    static constexpr int WN = 2, WM = 4;                                 // waves along the columns / rows of the tile
    static constexpr int TM = BM / 16 / WM, TN = BN / 16 / WN;           // MFMA tiles of a wave
    static constexpr int XU = BM * BK, WU = BN * BK;                     // bf16 elements of a ring unit
    static constexpr int LDS = (3 * XU + 2 * WU) * 2;
    static constexpr int NA = BM / 64, NB = BN / 64;                     // requests of a wave per X half / per W unit
};
template <int EPI, int BM, int BN>
__global__ __launch_bounds__(512, 2) void gemm_tile_kernel(const bf16_t* __restrict__ W, int N, int K,
                                                           const uint16_t* __restrict__ Xh,
                                                           const uint16_t* __restrict__ Xl, int M,
                                                           float* __restrict__ Y, int ldy,
                                                           float* __restrict__ part,
                                                           uint16_t* __restrict__ Oh, uint16_t* __restrict__ Ol,
                                                           unsigned long long* __restrict__ clk) {
    // clk != nullptr (a timing probe is armed): the block in the middle of the grid reports how many shader clock
    // ticks and how many ticks of the constant 100 MHz counter its K loop took: {shader ticks, reference ticks,
    // launches} are added to clk[0..2], which gives the clock the chip sustains while this kernel runs
    long long clk_c0 = 0, clk_w0 = 0;
    if (clk) { clk_c0 = clock64(); clk_w0 = wall_clock64(); }
    using C = TileCfg<BM, BN>;
    constexpr int BK = C::BK, TM = C::TM, TN = C::TN, XU = C::XU, WU = C::WU, NA = C::NA, NB = C::NB;
    extern __shared__ __attribute__((aligned(16))) uint16_t tile_sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    int bx, by, bz;
    {
        constexpr int GM = 4;
        const int nxy = gridDim.x * gridDim.y, nb = nxy * gridDim.z;
        const int id = blockIdx.x + gridDim.x * blockIdx.y + nxy * blockIdx.z;
        const int k = id % 8, j = id / 8, q = nb / 8, r = nb % 8;
        int lin = k * q + min(k, r) + j;
        bz = lin / nxy; lin -= bz * nxy;
        const int per = GM * gridDim.x, g = lin / per, rem = lin - g * per;
        const int gm = min(GM, (int)gridDim.y - g * GM);
        by = g * GM + rem % gm; bx = rem / gm;
        // (the divisions leave them in vector registers; the copies below need their base addresses in scalar ones)
        bx = __builtin_amdgcn_readfirstlane(bx); by = __builtin_amdgcn_readfirstlane(by); bz = __builtin_amdgcn_readfirstlane(bz);
    }
    const int m0 = by * BM, n0 = bx * BN;
    const int nkb_all = K / BK;
    const int per = __builtin_amdgcn_readfirstlane((nkb_all + gridDim.z - 1) / gridDim.z);
    const int nk = min(nkb_all, bz * per + per) - bz * per, kb0 = min(bz * per, nkb_all - 1);     // K blocks of this slice (an empty one: nk <= 0, zeros)

    // copies: a request covers eight rows of 128 bytes; lane -> row lane / 8, LDS chunk lane % 8, which holds source chunk
    // (lane % 8) ^ ((row / 2) % 8); request i of a wave: rows 8 (wave + 8 i) .. + 7 of a unit
    const int lrow = lane >> 3, lch = (lane & 7) ^ ((((wave & 1) * 4 + (lane >> 4))) & 7);
    // W row behind tile row r.  EPI_SWIGLU (W = [gate | up], N = 2F, never K-sliced): a 32-row group is 16 gate rows and the
    // 16 up rows of the same units
    const int F = N / 2;
    auto wrow = [&](int r) { return EPI == EPI_SWIGLU ? ((r >> 4) & 1) * F + min(bx * (BN / 2) + (r >> 5) * 16 + (r & 15), F - 1) : min(n0 + r, N - 1); };
    const char *pa_h[NA], *pa_l[NA], *pb[NB];
    uint32_t va[NA], vb[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int r = m0 + (i * 8 + wave) * 8, b = min(r, M - 1);
        va[i] = (uint32_t)(min(r + lrow, M - 1) - b) * (uint32_t)K * 2u + lch * 16u;
        pa_h[i] = reinterpret_cast<const char*>(Xh + (size_t)b * K + (size_t)kb0 * BK);
        pa_l[i] = reinterpret_cast<const char*>(Xl + (size_t)b * K + (size_t)kb0 * BK);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int r = (i * 8 + wave) * 8, b = wrow(r);
        vb[i] = (uint32_t)(wrow(r + lrow) - b) * (uint32_t)K * 2u + lch * 16u;
        pb[i] = reinterpret_cast<const char*>(W + (size_t)b * K + (size_t)kb0 * BK);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)tile_sm + wave * 1024;
    auto request_x = [&](const char* const* p, int kb, int s, int d) { copy16_to_lds(lds0 + s * (XU * 2) + d * 8192, va[d], p[d] + (size_t)kb * (BK * 2)); };
    auto request_w = [&](int kb, int s, int d) { copy16_to_lds(lds0 + 3 * XU * 2 + s * (WU * 2) + d * 8192, vb[d], pb[d] + (size_t)kb * (BK * 2)); };

    f32x4_t acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[j][i][v] = 0.0f;
    const int l16 = lane & 15, kg = lane >> 4;
    // operand reads: rows of a wave's tiles start at multiples of 16, so the permutation depends on the lane alone
    const int o0 = l16 * BK + ((kg ^ (l16 >> 1)) << 3), o1 = l16 * BK + (((4 + kg) ^ (l16 >> 1)) << 3);      // first / second 32 k of a block
    const uint16_t* A = tile_sm + wm * TM * 16 * BK;
    const uint16_t* B = tile_sm + 3 * XU + wn * TN * 16 * BK;
    u32x4_t w[TN], x[2][TM];
    auto lds16 = [](const uint16_t* p) { return *reinterpret_cast<const u32x4_t*>(p); };
    constexpr int T = TM * TN, TB = 2 * TM;
    // product t of a pass: tiles of W in ascending order, the rows of X up and down in turn (one operand is always the one before)
    auto mfma = [&](const u32x4_t* xs, int t) {
        const int j = t / TM, i = j & 1 ? TM - 1 - t % TM : t % TM;
        acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[j]), __builtin_bit_cast(bf16x8_t, xs[i]), acc[j][i], 0, 0, 0);
    };
    // a pass: the products of 32 k of one half; the X operands of the next pass are read from a, and W tile by tile, behind its last use, from b
    auto pass = [&](const u32x4_t* xs, u32x4_t* xn, const uint16_t* a, const uint16_t* b) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            mfma(xs, t);
            if (t < TM) xn[t] = lds16(a + t * 16 * BK);
            if (t % TM == TM - 1) w[t / TM] = lds16(b + t / TM * 16 * BK);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // the same with the barrier behind its first two tiles of W: only behind it may a and b be read
    auto pass_bar = [&](const u32x4_t* xs, u32x4_t* xn, const uint16_t* a, const uint16_t* b, auto wait, auto req, int nreq) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (t == TB) { wait(); __builtin_amdgcn_sched_barrier(0); }
            mfma(xs, t);
            if (t >= TB && t < TB + TM) xn[t - TB] = lds16(a + (t - TB) * 16 * BK);
            if (t == TB) w[0] = lds16(b);
            if (t == TB + 1) w[1] = lds16(b + 16 * BK);
            if (t >= TB && t % TM == TM - 1) w[t / TM] = lds16(b + t / TM * 16 * BK);
#pragma unroll
            for (int d = 0; d < nreq; ++d) if (t == TB + 1 + d * (T - TB - 1) / nreq) req(d);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    {
        const int last = max(nk - 1, 0), k1 = min(1, last);
#pragma unroll
        for (int d = 0; d < NA; ++d) request_x(pa_l, 0, 0, d);
#pragma unroll
        for (int d = 0; d < NB; ++d) request_w(0, 0, d);
#pragma unroll
        for (int d = 0; d < NA; ++d) request_x(pa_h, 0, 1, d);
#pragma unroll
        for (int d = 0; d < NA; ++d) request_x(pa_l, k1, 2, d);
#pragma unroll
        for (int d = 0; d < NB; ++d) request_w(k1, 1, d);
    }
    // the lo half and W of the first block have landed when at most the requests behind them are outstanding
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * NA + NB) : "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i) x[0][i] = lds16(A + o0 + i * 16 * BK);
#pragma unroll
    for (int j = 0; j < TN; ++j) {                           // (in the order of the loop, so that the first product need not wait for the last of them)
        __builtin_amdgcn_sched_barrier(0);
        w[j] = lds16(B + o0 + j * 16 * BK);
    }
    __builtin_amdgcn_sched_barrier(0);
    int sl = 0, sh = 1, sn = 2;                              // ring units of this block's lo half, its hi half and the next block's lo half
    for (int kb = 0; kb < nk; ++kb) {
        const uint16_t *b = B + (kb & 1) * WU, *bn = B + ((kb & 1) ^ 1) * WU;
        const int k1 = min(kb + 1, nk - 1), k2 = min(kb + 2, nk - 1);
        pass(x[0], x[1], A + sl * XU + o1, b + o1);                                     // lo half, first 32 k
        pass_bar(x[1], x[0], A + sh * XU + o0, b + o0,                                  // lo half, second 32 k; behind the barrier the lo half's unit is free and the hi half has landed
                 [&] { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NA + NB) : "memory"); },
                 [&](int d) { request_x(pa_h, k1, sl, d); }, NA);
        pass(x[0], x[1], A + sh * XU + o1, b + o1);                                     // hi half, first 32 k
        pass_bar(x[1], x[0], A + sn * XU + o0, bn + o0,                                 // hi half, second 32 k; behind the barrier its unit and W's are free and the next block's lo half and W have landed
                 [&] { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NA) : "memory"); },
                 [&](int d) { if (d < NA) request_x(pa_l, k2, sh, d); else request_w(k2, kb & 1, d - NA); }, NA + NB);
        const int f = sl;
        sl = sn; sn = sh; sh = f;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");      // nothing is in flight into LDS when the block ends
    if (clk && tid == 0 && blockIdx.x == gridDim.x / 2 && blockIdx.y == gridDim.y / 2 && blockIdx.z == 0) {
        atomicAdd(&clk[0], (unsigned long long)(clock64() - clk_c0));
        atomicAdd(&clk[1], (unsigned long long)(wall_clock64() - clk_w0));
        atomicAdd(&clk[2], 1ull);
    }

    // a lane's accumulator of tile (j, i): columns (wn TN + j) 16 + 4 (lane / 16) .. + 3 of row (wm TM + i) 16 + lane % 16
    if (EPI == EPI_SWIGLU) {
        // silu(gate) * up straight into the hi / lo halves the down projection reads; tiles 2 p and 2 p + 1 are gate and up of the same units
#pragma unroll
        for (int p = 0; p < TN / 2; ++p)
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int col = bx * (BN / 2) + (wn * (TN / 2) + p) * 16 + 4 * kg, m = m0 + (wm * TM + i) * 16 + l16;
                if (m < M && col < F) {                      // (F is a multiple of 64: it is the K of the down projection)
                    const f32x4_t g = acc[2 * p][i], u = acc[2 * p + 1][i];
                    store_halves(Oh + (size_t)m * F + col, Ol + (size_t)m * F + col,
                                 make_float4(silu_mul(g[0], u[0]), silu_mul(g[1], u[1]), silu_mul(g[2], u[2]), silu_mul(g[3], u[3])));
                }
            }
        return;
    }
    const bool sliced = gridDim.z > 1;
    float* out = sliced ? part + (size_t)bz * M * N : Y;
    const size_t ldo = sliced ? N : ldy;
    const bool add = EPI == EPI_RESID && !sliced;
    if (((N | (int)ldo) & 3) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
        float4 res[2][TM];   // EPI_RESID: the residual values of a column of tiles are requested while the one before it is stored
        auto at = [&](int j, int i) { return out + (size_t)min(m0 + (wm * TM + i) * 16 + l16, M - 1) * ldo + min(n0 + (wn * TN + j) * 16 + 4 * kg, N - 4); };
        if (add) {
#pragma unroll
            for (int i = 0; i < TM; ++i) res[0][i] = *reinterpret_cast<const float4*>(at(0, i));
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (add && j + 1 < TN) {
#pragma unroll
                for (int i = 0; i < TM; ++i) res[(j + 1) & 1][i] = *reinterpret_cast<const float4*>(at(j + 1, i));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (m0 + (wm * TM + i) * 16 + l16 >= M || n0 + (wn * TN + j) * 16 + 4 * kg >= N) continue;
                float4 y = make_float4(acc[j][i][0], acc[j][i][1], acc[j][i][2], acc[j][i][3]);
                if (add) { const float4 r = res[j & 1][i]; y.x += r.x; y.y += r.y; y.z += r.z; y.w += r.w; }
                *reinterpret_cast<float4*>(at(j, i)) = y;
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + (wm * TM + i) * 16 + l16, n = n0 + (wn * TN + j) * 16 + 4 * kg + v;
                if (m < M && n < N) {
                    float* y = out + (size_t)m * ldo + n;
                    *y = add ? *y + acc[j][i][v] : acc[j][i][v];
                }
            }
}

// Block tile and K slices of a many-row product: the plan for which a cost model is smallest.  The model was fitted to
// 3385 timings (12 projection shapes of the 1.5B / 7B / 72B models x 14 row counts from 70 to 8192 x all tiles and slice
// counts; rms error 8 %, the plans it picks are 1.0 % slower than the best measured ones on average and 16 % at worst; with the
// constants fitted to the kernel's predecessor 2.2 % and 46 %): a round of thread
// blocks that fills the chip costs `full` per 32 k, one that occupies the share x of it `light` + x (`full` -
// `light`) (fewer busy units clock higher) but not less than `least` (the latency of a block's own loop), and every round `over` for
// filling the ring and storing the tile.  K slices
// pay a finish kernel that reads their partial sums back; a residual product without slices pays the separate kernel
// that leaves the normalised halves for the next projection.
struct TilePlan { int bm, bn, ks; };
struct TileCost { int bm, bn, per_cu; float full, light, least, over; };        // microseconds
static constexpr TileCost kTileCosts[] = {
    {256, 256, 1, 1.399f, 0.921f, 0.979f, 8.8f}, {256, 192, 1, 1.108f, 0.740f, 0.667f, 5.6f}, {128, 256, 1, 0.809f, 0.537f, 0.483f, 4.0f},
    {128, 192, 1, 0.619f, 0.386f, 0.488f, 4.0f}, {128, 128, 2, 0.951f, 0.148f, 0.305f, 3.4f}};
static TilePlan gemm_tile_plan(int epi, int N, int K, int M, size_t part_floats) {
    const int nkb = K / 64;
    const float mn = 1e-6f * (float)M * (float)N;
    TilePlan best{256, 256, 1};
    float best_us = 1e30f;
    for (const TileCost& c : kTileCosts)
        for (int ks : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
            const int per = (nkb + ks - 1) / ks, kb = 2 * per;
            // slices: whole columns of four (finish kernels), at least three K blocks each, none empty, room for the partial sums
            if (ks > 1 && (N % 4 || per < 3 || (ks - 1) * per >= nkb || (size_t)ks * M * N > part_floats)) continue;
            const long long blocks = (long long)((N + c.bn - 1) / c.bn) * ((M + c.bm - 1) / c.bm) * ks, cap = 256 * c.per_cu;
            const float part = (float)(blocks % cap) / (float)cap;
            float us = (float)(blocks / cap) * (kb * c.full + c.over);
            if (part > 0.0f) us += kb * std::max(c.least, c.light + part * (c.full - c.light)) + c.over;
            if (ks > 1) us += 5.7f + 1.10f * ks * mn;
            else if (epi == EPI_RESID) us += 7.2f + 0.82f * mn;
            if (us < best_us) { best_us = us; best = TilePlan{c.bm, c.bn, ks}; }
        }
    return best;
}

// ---------------------------------------------------------------- bf16 MFMA, 2..128 rows, the whole of K in one block
// The gate/up projection with its SwiGLU, and the output head, without K slices: a block owns BN rows of W (the gate and the up
// rows of BN / 2 units) over all of K, so there are no partial sums to write and read back and no finish kernel.  BN is
// chosen so that the blocks make one round on 256 compute units (stream_bn).  X and W tiles of 64 k go straight into a ring
// of up to six LDS stages, all but one of them in flight; the waves divide a K block among themselves and add their K parts
// through LDS at the end.  Bound by what the copies pull through L2: W once and, per block, all of X (217 MB beside
// 272 MB at 64 rows of the 7B shape, 435 at 128: 8.5 to 9 TB/s together).  Above 32 rows a wave takes all columns, half of the rows and a
// quarter of the K block: an operand is read from LDS by one or two waves only (72 KB a K block at 128 rows and 160 columns; 180 with 32
// columns and half of K per wave).  128 rows 80.7 -> 76.4, 27.9 -> 26.6, head 25.7 -> 23.6 us; 64 rows 56.7 / 56.8, 19.7 / 19.8, 17.7 ->
// 17.0.  Measured against K slices plus their finish kernel (us; 7B gate/up, 1.5B gate/up, a
// head of 16384 x 1536): 16 rows 48.4 / 51.6, 14.8 / 18.3, 12.1 / 17.4; 32 rows 50.2 / 55.6, 16.7 / 20.3, 13.7 / 19.5; 64 rows 58.8 /
// 68.6, 21.3 / 24.7, 19.2 / 25.8; 128 rows (against the tile kernel) 84.6 / 93.1, 30.3 / 35.6, 30.3 / 34.9.  Matrices that give no
// single round of blocks stay with the slices: [59136][8192] at 16 rows 182 against 159.
template <int MT, int BN> struct StreamCfg {
    static constexpr int BK = 64;
    // up to 32 rows: a wave per 32 columns and half (quarter) of the K block; more: all columns, half of the rows, a quarter of K
    static constexpr int TN = MT == 1 ? 1 : BN / 32, WN = BN / 32 / TN, WM = MT == 1 ? 1 : 2, KW = MT > 1 || BN == 64 ? 4 : 2;
    static constexpr int TM = MT / WM, NW = WN * WM * KW;             // row tiles of a wave; waves
    static constexpr int XREQ = MT * 8, REQ = XREQ + BN / 8;          // 1 KB requests of a K block: X hi, X lo, W
    static constexpr int NS = (160 * 1024) / (REQ * 1024) > 6 ? 6 : (160 * 1024) / (REQ * 1024);
    static constexpr int CNT = REQ / NW, EXTRA = REQ % NW;
    static constexpr int LDS = NS * REQ * 1024;
    static_assert(NS >= 2 && (KW - 1) * WN * WM * TN * 4096 <= LDS, "");
};
template <int EPI, int MT, int BN>
__global__ __launch_bounds__((StreamCfg<MT, BN>::NW * 64)) void gemm_stream_kernel(const bf16_t* __restrict__ W, int N, int K,
                                                             const uint16_t* __restrict__ Xh, const uint16_t* __restrict__ Xl, int M,
                                                             float* __restrict__ Y, int ldy,
                                                             uint16_t* __restrict__ Oh, uint16_t* __restrict__ Ol) {
    using C = StreamCfg<MT, BN>;
    constexpr int BK = C::BK, TM = C::TM, TN = C::TN, WN = C::WN, WM = C::WM, KW = C::KW, NW = C::NW, NS = C::NS, CNT = C::CNT, EXTRA = C::EXTRA;
    constexpr int STAGE = C::REQ * 512;                       // bf16 elements of a stage
    extern __shared__ __attribute__((aligned(16))) uint16_t tile_sm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wm = wave / WN % WM, kw = wave / (WN * WM);
    const int bx = blockIdx.x, n0 = bx * BN, nk = K / BK;
    const int F = N / 2;
    auto wrow = [&](int r) { return EPI == EPI_SWIGLU ? ((r >> 4) & 1) * F + min(bx * (BN / 2) + (r >> 5) * 16 + (r & 15), F - 1) : min(n0 + r, N - 1); };
    // copies (as in gemm_tile_kernel): request id = wave + NW i covers eight rows of 128 bytes; lane -> row lane / 8, LDS chunk
    // lane % 8, which holds source chunk (lane % 8) ^ ((row / 2) % 8)
    const char* base[CNT + 1];
    uint32_t voff[CNT + 1];
#pragma unroll
    for (int i = 0; i <= CNT; ++i) {
        const int id = min(wave + NW * i, C::REQ - 1);
        const int x = id < MT * 4 ? id : id - MT * 4;         // 8-row group of an X half
        const bool isx = id < C::XREQ;
        const int g8 = isx ? x : id - C::XREQ;
        const int rl = g8 * 8 + (lane >> 3);
        const uint32_t ch = ((lane & 7) ^ (((g8 & 1) * 4 + (lane >> 4)) & 7)) * 16;
        const int b = isx ? min(g8 * 8, M - 1) : wrow(g8 * 8), r = isx ? min(rl, M - 1) : wrow(rl);
        base[i] = reinterpret_cast<const char*>((isx ? (id < MT * 4 ? Xh : Xl) : reinterpret_cast<const uint16_t*>(W)) + (size_t)b * K);
        voff[i] = (uint32_t)(r - b) * (uint32_t)K * 2u + ch;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)tile_sm + wave * 1024;
    const bool extra = EXTRA > 0 && wave < EXTRA;
    auto request = [&](int kb, int s) {
        const size_t ko = (size_t)min(kb, nk - 1) * (BK * 2);
#pragma unroll
        for (int i = 0; i < CNT; ++i) copy16_to_lds(lds0 + s * (STAGE * 2) + i * (NW * 1024), voff[i], base[i] + ko);
        if (extra) copy16_to_lds(lds0 + s * (STAGE * 2) + CNT * (NW * 1024), voff[CNT], base[CNT] + ko);
    };
    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    const int l32 = lane & 31, kg = lane >> 5, swz = (l32 >> 1) & 7;
    const uint16_t* B = tile_sm + C::XREQ * 512 + wn * TN * 32 * BK;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) request(s, s);
    int cur = 0, prev = NS - 1;
    // block kb has landed when at most the requests of the NS - 2 blocks behind it are outstanding; behind the barrier that holds
    // for every wave, and everybody has read block kb - 1, whose stage takes block kb + NS - 1
    for (int kb = 0; kb < nk; ++kb) {
        if (extra) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * (CNT + 1)) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * CNT) : "memory");
        request(kb + NS - 1, prev);
        const uint16_t *a = tile_sm + cur * STAGE, *b = B + cur * STAGE;
#pragma unroll
        for (int q = 0; q < 4 / KW; ++q) {
            const int off = l32 * BK + (((2 * (kw * (4 / KW) + q) + kg) ^ swz) << 3);
            bf16x8_t w[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) w[j] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(b + j * 32 * BK + off));
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const bf16x8_t xl = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(a + (MT + wm * TM + i) * 32 * BK + off));
                const bf16x8_t xh = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(a + (wm * TM + i) * 32 * BK + off));
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xl, w[j], acc[i][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh, w[j], acc[i][j], 0, 0, 0);
            }
        }
        prev = cur;
        cur = cur == NS - 1 ? 0 : cur + 1;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // Add the K parts through LDS: the waves of one (row, column) part share the 16 values a lane has of a tile, 8 / KW pairs
    // (v, v + 8) each.  Whoever adds a value adds the parts in ascending order: every row of a product is the same sum, wherever it
    // stands in the tile.  One row tile of every wave at a time.
    constexpr int PV = 8 / KW;                                // pairs per wave
    float2* red = reinterpret_cast<float2*>(tile_sm);        // [owner][source][wn, wm][j][pair][lane]
    auto at = [&](int owner, int src, int j, int p) {
        return red + ((((owner * (KW - 1) + (src < owner ? src : src - 1)) * (WN * WM) + wave % (WN * WM)) * TN + j) * PV + p) * 64 + lane;
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i > 0) __syncthreads();
#pragma unroll
        for (int o = 0; o < KW; ++o)
            if (o != kw)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int p = 0; p < PV; ++p) *at(o, kw, j, p) = make_float2(acc[i][j][o * PV + p], acc[i][j][o * PV + p + 8]);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int p = 0; p < PV; ++p) {
                // (scalars, chosen between with constant indices: float2 structs would be chosen by address, in scratch memory)
                float xo = 0.0f, yo = 0.0f, xq[KW - 1], yq[KW - 1];      // the wave's own pair, the others'
#pragma unroll
                for (int o = 0; o < KW; ++o) {
                    xo = o == kw ? acc[i][j][o * PV + p] : xo;
                    yo = o == kw ? acc[i][j][o * PV + p + 8] : yo;
                }
#pragma unroll
                for (int q = 0; q < KW - 1; ++q) {
                    const float2 y = *at(kw, q < kw ? q : q + 1, j, p);
                    xq[q] = y.x; yq[q] = y.y;
                }
                float2 x = make_float2(kw == 0 ? xo : xq[0], kw == 0 ? yo : yq[0]);
#pragma unroll
                for (int q = 1; q < KW; ++q) {
                    x.x += q == kw ? xo : q < kw ? xq[q < KW - 1 ? q : 0] : xq[q - 1];
                    x.y += q == kw ? yo : q < kw ? yq[q < KW - 1 ? q : 0] : yq[q - 1];
                }
                const int v = kw * PV + p, m0 = (wm * TM + i) * 32 + 8 * (v >> 2) + 4 * kg + (v & 3);       // x.y: row m0 + 16
                if (EPI == EPI_SWIGLU) {
                    const int col = bx * (BN / 2) + (wn * TN + j) * 16 + (lane & 15);
                    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x.x), __float_as_uint(x.y), false, false);
                    const float g = __uint_as_float(s[0]), u = __uint_as_float(s[1]);
                    const int m = m0 + ((lane & 16) ? 16 : 0);
                    if (m < M && col < F) {
                        const float z = silu_mul(g, u);
                        const uint16_t hi = f2bf(z);
                        Oh[(size_t)m * F + col] = hi;
                        Ol[(size_t)m * F + col] = f2bf(z - bf2f(hi));
                    }
                } else {
                    const int n = n0 + (wn * TN + j) * 32 + l32;
                    if (m0 < M && n < N) Y[(size_t)m0 * ldy + n] = x.x;
                    if (m0 + 16 < M && n < N) Y[(size_t)(m0 + 16) * ldy + n] = x.y;
                }
            }
    }
}

// BN for which an [N][K] matrix gives 160..256 blocks, as many as possible; 0: none
static int stream_bn(int N) {
    for (int bn : {64, 96, 160}) {
        const int blocks = (N + bn - 1) / bn;
        if (blocks >= 160 && blocks <= 256) return bn;
    }
    return 0;
}
#define RSD_STREAM_SIZES(X) X(1, 64) X(1, 96) X(1, 160) X(2, 64) X(2, 96) X(2, 160) X(4, 64) X(4, 96) X(4, 160)
static void gemm_stream_launch(hipStream_t st, int epi, int bn, const bf16_t* W, int N, int K, const uint16_t* Xh, const uint16_t* Xl, int M,
                               float* Y, int ldy, uint16_t* Oh, uint16_t* Ol) {
    const int mt = M <= 32 ? 1 : M <= 64 ? 2 : 4;
    const dim3 grid((N + bn - 1) / bn);
#define RSD_STREAM_CASE(MT, BN)                                                                                              \
    if (mt == MT && bn == BN) {                                                                                              \
        constexpr size_t lds = StreamCfg<MT, BN>::LDS;                                                                       \
        const dim3 block(StreamCfg<MT, BN>::NW * 64);                                                                        \
        if (epi == EPI_SWIGLU) hipLaunchKernelGGL((gemm_stream_kernel<EPI_SWIGLU, MT, BN>), grid, block, lds, st, W, N, K, Xh, Xl, M, Y, ldy, Oh, Ol); \
        else                   hipLaunchKernelGGL((gemm_stream_kernel<EPI_STORE, MT, BN>), grid, block, lds, st, W, N, K, Xh, Xl, M, Y, ldy, Oh, Ol);  \
        return;                                                                                                              \
    }
    RSD_STREAM_SIZES(RSD_STREAM_CASE)
#undef RSD_STREAM_CASE
}

#define RSD_TILE_SIZES(X) X(256, 256) X(256, 192) X(128, 256) X(128, 192) X(128, 128)

// These kernels need more than 64 KB of LDS: allowed once per context on its device (never from inside a launch, which may
// be recording a graph).
static hipError_t gemm_tile_raise() {
    hipError_t e = hipSuccess;
#define RSD_TILE_RAISE(BM, BN)                                                                                               \
    for (const void* f : {reinterpret_cast<const void*>(gemm_tile_kernel<EPI_STORE, BM, BN>),                                \
                          reinterpret_cast<const void*>(gemm_tile_kernel<EPI_RESID, BM, BN>),                                \
                          reinterpret_cast<const void*>(gemm_tile_kernel<EPI_SWIGLU, BM, BN>)})                              \
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, TileCfg<BM, BN>::LDS);
    RSD_TILE_SIZES(RSD_TILE_RAISE)
#undef RSD_TILE_RAISE
#define RSD_STREAM_RAISE(MT, BN)                                                                                             \
    for (const void* f : {reinterpret_cast<const void*>(gemm_stream_kernel<EPI_STORE, MT, BN>),                              \
                          reinterpret_cast<const void*>(gemm_stream_kernel<EPI_SWIGLU, MT, BN>)})                            \
        if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, StreamCfg<MT, BN>::LDS);
    RSD_STREAM_SIZES(RSD_STREAM_RAISE)
#undef RSD_STREAM_RAISE
    return e;
}

// epi == EPI_SWIGLU (W = [gate | up], ks = 1): the activated values go to Oh / Ol [M][N / 2] as hi / lo halves
static void gemm_tile_launch(hipStream_t st, int epi, TilePlan pl, const bf16_t* W, int N, int K, const uint16_t* Xh,
                             const uint16_t* Xl, int M, float* Y, int ldy, float* part,
                             uint16_t* Oh = nullptr, uint16_t* Ol = nullptr, unsigned long long* clk = nullptr) {
    const dim3 grid((N + pl.bn - 1) / pl.bn, (M + pl.bm - 1) / pl.bm, pl.ks), block(512);
#define RSD_TILE_CASE(BM, BN)                                                                                                \
    if (pl.bm == BM && pl.bn == BN) {                                                                                        \
        constexpr size_t lds = TileCfg<BM, BN>::LDS;                                                                         \
        if (epi == EPI_SWIGLU)     hipLaunchKernelGGL((gemm_tile_kernel<EPI_SWIGLU, BM, BN>), grid, block, lds, st, W, N, K, Xh, Xl, M, Y, ldy, part, Oh, Ol, clk); \
        else if (epi == EPI_RESID) hipLaunchKernelGGL((gemm_tile_kernel<EPI_RESID, BM, BN>), grid, block, lds, st, W, N, K, Xh, Xl, M, Y, ldy, part, Oh, Ol, clk);  \
        else                       hipLaunchKernelGGL((gemm_tile_kernel<EPI_STORE, BM, BN>), grid, block, lds, st, W, N, K, Xh, Xl, M, Y, ldy, part, Oh, Ol, clk);  \
        return;                                                                                                              \
    }
    RSD_TILE_SIZES(RSD_TILE_CASE)
#undef RSD_TILE_CASE
}
