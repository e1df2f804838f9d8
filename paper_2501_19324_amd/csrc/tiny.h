// Single-token decode of small fp32 models (the tiny configuration): two launches a layer and one for the output head, instead of
// five and two.
//
// Nothing in such a layer is bound by bandwidth (0.5 to 4 MB of weights in L2); an iteration is a chain of dependent launches of
// 2.5 to 5 us each, whatever they compute.  So the chain is shortened: a launch does everything up to the next product that needs
// a whole row.  The products that would need one more launch to be added up are left as partial sums that the next launch adds while it
// stages its input, each block for itself:
//   tiny_attn_kernel, block (row, head): x = h + sum of the MLP's partials (or the token's embedding); RMSNorm; q, k, v of the head;
//     rotary embedding; cache write (the first head of a group); attention; the head's share of the output projection -> partials
//   tiny_mlp_kernel, block (row, 32 hidden units): x = h + sum of the heads' partials; RMSNorm; gate and up; SiLU; the units' share of
//     the down projection -> partials
//   tiny_head_kernel, block (row, 64 tokens): x = h + sum of the MLP's partials; RMSNorm; logits; greedy: the arg max as well, chosen
//     and appended by the block that finishes a row, as in sample_max_kernel
// One block of a row writes the new residual stream, into the other of two buffers (every block of the launch reads the old one).
// Everything a block reads that does not depend on the launch before it - its weights - is requested first and kept in registers.
// Partials are added in a fixed order: results do not depend on timing.
// Measured, four rows, contexts up to 96 (rocprofv3, launch to launch): a layer of d_model 256 18.9 -> 9.6 us, of 128 18.5 -> 8.4; head and
// arg max 8.7 -> 6.1; the whole tiny configuration (four steps of 16 tokens, draft, score, target) 11.8 -> 7.5 ms with the faster fp32 tiles.
#pragma once
#include "attn.h"
#include "common.h"
#include "sample.h"

constexpr int kTinyT = 512;                  // threads of a block: 32 groups of 16 lanes, or 64 of 8
constexpr int kTinyPos = 128;                // positions a block holds in registers (two a lane group)
constexpr int kTinyUnits = 32;               // hidden units of an MLP block
constexpr int kTinyVocab = 64;               // tokens of a head block

// sums over the 8 or 16 lanes of a group; every lane gets the result
template <int CTRL> __device__ __forceinline__ float dpp_plus(float x) { return x + __uint_as_float(dpp_move<CTRL>(__float_as_uint(x))); }
__device__ __forceinline__ float sum8(float v) { return dpp_plus<0x141>(dpp_plus<0x4E>(dpp_plus<0xB1>(v))); }   // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror
__device__ __forceinline__ float sum16(float v) { return dpp_plus<0x140>(sum8(v)); }                            // row_mirror
// over the eight groups of 8 lanes: row_ror by 8, then the four rows
__device__ __forceinline__ float sum_groups(float v) { return rows4_sum(dpp_plus<0x128>(v)); }
__device__ __forceinline__ float max_groups(float v) { return rows4_max(fmaxf(v, __uint_as_float(dpp_move<0x128>(__float_as_uint(v))))); }
__device__ __forceinline__ float dot4(const float4& a, const float4& b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }

struct TinyIn {
    const float* h;          // [M][D] residual stream; the first layer: the embedding table
    const float* part;       // [M][ns][D] partial sums to add to it
    int ns;
    const float* gain;
    float eps;
    float* h_out;            // [M][D] where the sum goes (nullptr: nowhere)
};
// (LDS arrays that are read or written 16 bytes at a time say so: a float array alone need only be aligned to 4)
template <int D> struct TinyLds {
    alignas(16) float xs[D];                                // the staged row times the gain, before 1 / rms
    alignas(16) float part[kTinyT / (D / 4)][D];
    float red[kTinyT / 64];
};
static_assert(alignof(TinyLds<128>) == 16 && alignof(TinyLds<256>) == 16, "");
// What a thread holds of the row to be staged: one column and its gain, four columns of the partials i = g, g + GR, ...
// Requested before the weights: loads return in order, and staging would otherwise wait for all of them.
template <int D> struct TinyRow {
    static constexpr int C4 = D / 4, GR = kTinyT / C4, NP = 4;               // float4 columns; groups of threads that share the partials
    static constexpr int kMaxParts = GR * NP;
    float old, gn;
    float4 p[NP];
    // src: the row of in.h
    __device__ __forceinline__ void request(const TinyIn& in, int r, const float* src) {
        const int tid = threadIdx.x, c = tid % C4, g = tid / C4;
        old = src[tid % D];
        gn = in.gain[tid % D];
        const float* q = in.part + (size_t)r * in.ns * D + c * 4;
#pragma unroll
        for (int i = 0; i < NP; ++i) p[i] = *reinterpret_cast<const float4*>(q + (size_t)min(g + i * GR, max(in.ns - 1, 0)) * D);
    }
    // all threads: the sum to s.xs times the gain (and to h_out); returns 1 / rms
    __device__ __forceinline__ float stage(const TinyIn& in, int r, bool write, TinyLds<D>& s) {
        const int tid = threadIdx.x, c = tid % C4, g = tid / C4;
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (g + i * GR < in.ns) { a.x += p[i].x; a.y += p[i].y; a.z += p[i].z; a.w += p[i].w; }
        *reinterpret_cast<float4*>(&s.part[g][c * 4]) = a;
        __syncthreads();
        float ss = 0.0f;
        if (tid < D) {
            float x = old;
#pragma unroll
            for (int i = 0; i < GR; ++i) x += s.part[i][tid];
            if (write && in.h_out) in.h_out[(size_t)r * D + tid] = x;
            s.xs[tid] = x * gn;
            ss = wave_sum(x * x);
        }
        if ((tid & 63) == 0) s.red[tid >> 6] = ss;
        __syncthreads();
        float t = 0.0f;
#pragma unroll
        for (int i = 0; i < D / 64; ++i) t += s.red[i];
        return 1.0f / sqrtf(t / (float)D + in.eps);
    }
};
__device__ __forceinline__ float4 pick(bool first, const float4& a, const float4& b) {
    return make_float4(first ? a.x : b.x, first ? a.y : b.y, first ? a.z : b.z, first ? a.w : b.w);
}

// wqkv: [(H + 2 Hkv) * 32][D], wo: [D][H * 32], out: [M][H][D] partials of the output projection.  head_dim 32, contexts of at
// most kTinyPos positions.
template <int D>
__global__ __launch_bounds__(kTinyT) void tiny_attn_kernel(TinyIn in, const float* __restrict__ wqkv, const float* __restrict__ wo,
                                                           float* __restrict__ pool_layer, const int* __restrict__ block_table,
                                                           int max_pages, RowMap rm, const int* __restrict__ tokens, int max_ctx,
                                                           const float2* __restrict__ rope, int H, int Hkv, float scale,
                                                           float* __restrict__ out) {
    constexpr int HD = 32, NX = D / 64, NO = D / 64;         // float4s per lane of a weight row (16 lanes); passes of 64 rows of wo
    __shared__ TinyLds<D> s;
    __shared__ __attribute__((aligned(16))) float s_q[3][HD], s_att[HD], s_acc[kTinyT / 64][HD];
    __shared__ float s_m[kTinyT / 64], s_l[kTinyT / 64];
    const int r = blockIdx.x, h = blockIdx.y, G = H / Hkv, hk = h / G, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub16 = tid & 15, row16 = tid >> 4, sub8 = tid & 7, row8 = tid >> 3;
    int seq, pos;
    if (!row_lookup(rm, r, seq, pos)) return;
    const int* bt = block_table + (size_t)seq * max_pages;
    int page[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) page[i] = bt[min(row8 + 64 * i, max(pos - 1, 0)) / RSD_PAGE];
    TinyRow<D> row;
    row.request(in, r, in.h + (size_t)(tokens ? tokens[(size_t)seq * max_ctx + pos] : r) * D);
    __builtin_amdgcn_sched_barrier(0);
    float4 w[3][NX], o[NO];
    {
        const int rows[3] = {h * HD, (H + hk) * HD, (H + Hkv + hk) * HD};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int i = 0; i < NX; ++i)
                w[a][i] = *reinterpret_cast<const float4*>(wqkv + (size_t)(rows[a] + row16) * D + (i * 16 + sub16) * 4);
    }
    const size_t page_elts = (size_t)2 * Hkv * RSD_PAGE * HD, head_off = (size_t)hk * RSD_PAGE * HD, v_off = (size_t)Hkv * RSD_PAGE * HD;
    float4 kx[2], vx[2];                                     // (past the cached positions: the last one again, not counted)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = min(row8 + 64 * i, max(pos - 1, 0));
        const float* kb = pool_layer + (size_t)page[i] * page_elts + head_off + (p % RSD_PAGE) * HD + sub8 * 4;
        kx[i] = *reinterpret_cast<const float4*>(kb);
        vx[i] = *reinterpret_cast<const float4*>(kb + v_off);
    }
    const int j4 = (sub8 & 3) * 4;                           // rotary index of this lane's first dim
    const float4 c0 = *reinterpret_cast<const float4*>(rope + (size_t)pos * (HD / 2) + j4);
    const float4 c1 = *reinterpret_cast<const float4*>(rope + (size_t)pos * (HD / 2) + j4 + 2);
#pragma unroll
    for (int i = 0; i < NO; ++i) o[i] = *reinterpret_cast<const float4*>(wo + (size_t)(i * 64 + row8) * (H * HD) + h * HD + sub8 * 4);

    __builtin_amdgcn_sched_barrier(0);
    const float rs = row.stage(in, r, h == 0, s);
    float q3[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const float4 x = *reinterpret_cast<const float4*>(s.xs + (i * 16 + sub16) * 4);
#pragma unroll
        for (int a = 0; a < 3; ++a) q3[a] += dot4(w[a][i], x);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        q3[a] = sum16(q3[a]) * rs;
        if (sub16 == 0) s_q[a][row16] = q3[a];
    }
    __syncthreads();
    auto rotated = [&](const float* v) {                     // dims 4 sub8 .. + 3 of a rotated head
        const float4 a = *reinterpret_cast<const float4*>(v + sub8 * 4), b = *reinterpret_cast<const float4*>(v + (sub8 ^ 4) * 4);
        const float f = sub8 < 4 ? -1.0f : 1.0f;
        return make_float4(a.x * c0.x + f * b.x * c0.y, a.y * c0.z + f * b.y * c0.w, a.z * c1.x + f * b.z * c1.y, a.w * c1.z + f * b.w * c1.w);
    };
    float4 q = rotated(s_q[0]);
    q.x *= scale; q.y *= scale; q.z *= scale; q.w *= scale;
    const float4 kn = rotated(s_q[1]), vn = *reinterpret_cast<const float4*>(s_q[2] + sub8 * 4);
    if (row8 == 0 && h == hk * G) {                          // the first head of the group writes the new token's entry
        float* kb = pool_layer + (size_t)bt[pos / RSD_PAGE] * page_elts + head_off + (pos % RSD_PAGE) * HD + sub8 * 4;
        *reinterpret_cast<float4*>(kb) = kn;
        *reinterpret_cast<float4*>(kb + v_off) = vn;
    }
    float sc[2], mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int p = row8 + 64 * i;
        sc[i] = sum8(dot4(q, pick(p == pos, kn, kx[i])));
        if (p > pos) sc[i] = -INFINITY;
        mx = fmaxf(mx, sc[i]);
    }
    mx = max_groups(mx);
    float l = 0.0f;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float p = sc[i] == -INFINITY ? 0.0f : __expf(sc[i] - mx);
        const float4 v = pick(row8 + 64 * i > pos, make_float4(0.f, 0.f, 0.f, 0.f), pick(row8 + 64 * i == pos, vn, vx[i]));
        l += p;
        a.x += p * v.x; a.y += p * v.y; a.z += p * v.z; a.w += p * v.w;
    }
    l = sum_groups(l);
    a = make_float4(sum_groups(a.x), sum_groups(a.y), sum_groups(a.z), sum_groups(a.w));
    if (lane < 8) *reinterpret_cast<float4*>(&s_acc[wave][lane * 4]) = a;
    if (lane == 0) { s_m[wave] = mx; s_l[wave] = l; }
    __syncthreads();
    if (tid < HD) {
        float mn = -INFINITY, acc = 0.0f, ll = 0.0f;
#pragma unroll
        for (int i = 0; i < kTinyT / 64; ++i) mn = fmaxf(mn, s_m[i]);
#pragma unroll
        for (int i = 0; i < kTinyT / 64; ++i) {
            const float c = s_m[i] == -INFINITY ? 0.0f : __expf(s_m[i] - mn);
            acc += s_acc[i][tid] * c;
            ll += s_l[i] * c;
        }
        s_att[tid] = acc / ll;
    }
    __syncthreads();
    const float4 x = *reinterpret_cast<const float4*>(s_att + sub8 * 4);
    float* op = out + ((size_t)r * H + h) * D;
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const float y = sum8(dot4(o[i], x));
        if (sub8 == 0) op[i * 64 + row8] = y;
    }
}

// wgu: [2 F][D] (gate, then up), wdown: [D][F], out: [M][F / 32][D] partials of the down projection
template <int D>
__global__ __launch_bounds__(kTinyT) void tiny_mlp_kernel(TinyIn in, const float* __restrict__ wgu, const float* __restrict__ wdown, int F,
                                                          RowMap rm, float* __restrict__ out) {
    constexpr int NX = D / 64, NO = D / 64;
    __shared__ TinyLds<D> s;
    __shared__ __attribute__((aligned(16))) float s_act[kTinyUnits];
    const int r = blockIdx.x, u0 = blockIdx.y * kTinyUnits, tid = threadIdx.x;
    const int sub16 = tid & 15, row16 = tid >> 4, sub8 = tid & 7, row8 = tid >> 3;
    int seq, pos;
    if (!row_lookup(rm, r, seq, pos)) return;
    TinyRow<D> row;
    row.request(in, r, in.h + (size_t)r * D);
    __builtin_amdgcn_sched_barrier(0);
    float4 wg[NX], wu[NX], o[NO];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        wg[i] = *reinterpret_cast<const float4*>(wgu + (size_t)(u0 + row16) * D + (i * 16 + sub16) * 4);
        wu[i] = *reinterpret_cast<const float4*>(wgu + (size_t)(F + u0 + row16) * D + (i * 16 + sub16) * 4);
    }
#pragma unroll
    for (int i = 0; i < NO; ++i) o[i] = *reinterpret_cast<const float4*>(wdown + (size_t)(i * 64 + row8) * F + u0 + sub8 * 4);
    __builtin_amdgcn_sched_barrier(0);
    const float rs = row.stage(in, r, u0 == 0, s);
    float g = 0.0f, u = 0.0f;
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const float4 x = *reinterpret_cast<const float4*>(s.xs + (i * 16 + sub16) * 4);
        g += dot4(wg[i], x);
        u += dot4(wu[i], x);
    }
    g = sum16(g) * rs;
    u = sum16(u) * rs;
    if (sub16 == 0) s_act[row16] = g / (1.0f + expf(-g)) * u;
    __syncthreads();
    const float4 x = *reinterpret_cast<const float4*>(s_act + sub8 * 4);
    float* op = out + ((size_t)r * (F / kTinyUnits) + blockIdx.y) * D;
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const float y = sum8(dot4(o[i], x));
        if (sub8 == 0) op[i * 64 + row8] = y;
    }
}

// W: [V][D]; logits [M][V].  CHOOSE (at most SMP_NB blocks a row): the sampler's phase A with a block as a span; its workspace and counter
// are used as sample_max_kernel uses them (64 more on the row's counter with every call)
template <int D, bool CHOOSE>
__global__ __launch_bounds__(kTinyT) void tiny_head_kernel(TinyIn in, const float* __restrict__ W, int V, RowMap rm, float* __restrict__ logits,
                                                           SampleArgs sa, AppendArgs ap) {
    constexpr int NX = D / 64, NV = kTinyVocab / 32;
    __shared__ TinyLds<D> s;
    const int r = blockIdx.x, tid = threadIdx.x, sub16 = tid & 15, row16 = tid >> 4;
    int seq, pos;
    if (!row_lookup(rm, r, seq, pos)) return;
    TinyRow<D> row;
    row.request(in, r, in.h + (size_t)r * D);
    __builtin_amdgcn_sched_barrier(0);
    float4 w[NV][NX];
#pragma unroll
    for (int a = 0; a < NV; ++a)
#pragma unroll
        for (int i = 0; i < NX; ++i)
            w[a][i] = *reinterpret_cast<const float4*>(W + (size_t)min((int)blockIdx.y * kTinyVocab + a * 32 + row16, V - 1) * D + (i * 16 + sub16) * 4);
    __builtin_amdgcn_sched_barrier(0);
    const float rs = row.stage(in, r, false, s);
    float y[NV] = {};
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const float4 x = *reinterpret_cast<const float4*>(s.xs + (i * 16 + sub16) * 4);
#pragma unroll
        for (int a = 0; a < NV; ++a) y[a] += dot4(w[a][i], x);
    }
    float bv = -INFINITY; int bi = 0x7FFFFFFF;
#pragma unroll
    for (int a = 0; a < NV; ++a) {
        const int n = blockIdx.y * kTinyVocab + a * 32 + row16;
        float z = sum16(y[a]) * rs;
        if (sub16 == 0 && n < V) logits[(size_t)r * V + n] = z;
        if (n == sa.sep_id) z += sa.sep_bias;
        if (n < V && z > bv) { bv = z; bi = n; }
    }
    if constexpr (!CHOOSE) return;
    __shared__ float fred[kTinyT / 64];
    __shared__ int ired[kTinyT / 64];
    wave_argmax_rows(bv, bi);                                // (a row of 16 lanes has one token at a time)
    if ((tid & 63) == 0) { fred[tid >> 6] = bv; ired[tid >> 6] = bi; }
    __syncthreads();
    if (tid >= 64) return;
    if (tid == 0) {
#pragma unroll
        for (int i = 1; i < kTinyT / 64; ++i) take_better(bv, bi, fred[i], ired[i]);
        __hip_atomic_store(&sa.pmax[(size_t)r * SMP_NB + blockIdx.y], bv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&sa.pidx[(size_t)r * SMP_NB + blockIdx.y], bi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int last = 0;
    if (tid == 0) {
        const unsigned mine = blockIdx.y ? 1u : SMP_NB + 1u - gridDim.y;
        last = (__hip_atomic_fetch_add(reinterpret_cast<unsigned*>(sa.sel + (size_t)r * SMP_SEL + 8), mine, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) + mine) % SMP_NB == 0;
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    bv = -INFINITY; bi = 0x7FFFFFFF;
    if (tid < (int)gridDim.y) {
        bv = __hip_atomic_load(&sa.pmax[(size_t)r * SMP_NB + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bi = __hip_atomic_load(&sa.pidx[(size_t)r * SMP_NB + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    wave_argmax(bv, bi);
    if (tid == 0) smp_append(sa, ap, r, seq, bi);
}
