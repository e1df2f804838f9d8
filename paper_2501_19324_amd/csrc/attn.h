// Grouped-query attention of one query token per row over a paged KV cache,
// plus the rotary-embedding / cache-write kernel that feeds it.
//
// KV pool of one model: [layer][page][K|V][kv_head][16 tokens][head_dim], so
// the keys (or values) of one page and KV head are 16*head_dim contiguous
// elements (in which order inside that block depends on the cache type, see
// KvTraits / KvTiled below).  Token at position p of a sequence lives in logical
// page p / 16, slot p % 16; block_table[seq][logical page] gives the physical page.
#pragma once
#include "common.h"
#include "gemm.h"

#define RSD_PAGE 16

// bf16 caches keep the values of a page transposed, [head_dim][16 tokens], so that
// the token axis (the contraction axis of P.V) is contiguous for the MFMA
// operands; fp32 caches (tiny configuration, VALU kernels only) keep [16][head_dim].
template <typename KT> struct KvTraits { static constexpr bool v_transposed = false; };
template <> struct KvTraits<bf16_t> { static constexpr bool v_transposed = true; };

// bf16 caches with head_dim 128 (the MFMA kernels) go one step further: inside the 4 KB key block and the
// 4 KB value block of a (page, KV head) the elements are stored in the order the MFMA operands are loaded,
// so that every operand load of a wave (lane l takes 16 bytes) reads 1 KB of consecutive memory:
//   keys:   chunk j (elements 32 j .. 32 j + 31) of the 16 tokens is 1 KB; lane l = 16 c + t holds
//           elements 32 j + 8 c .. + 7 of token t            -> offset ((4 j + c) * 16 + t) * 8 + i
//   values: head dims 32 m .. 32 m + 31 are 1 KB; lane l = 16 c + (d % 16) holds tokens 4 c .. 4 c + 3 of
//           dims 32 m + d % 16 and 32 m + 16 + d % 16        -> offset ((64 m + l) * 2 + (d / 16) % 2) * 4 + t % 4
template <typename KT, int HD> struct KvTiled { static constexpr bool value = false; };
template <> struct KvTiled<bf16_t, 128> { static constexpr bool value = true; };
__device__ __forceinline__ int kv_tiled_k(int t, int e) { return ((((e >> 5) * 4 + ((e >> 3) & 3)) * 16) + t) * 8 + (e & 7); }
__device__ __forceinline__ int kv_tiled_v(int t, int d) {
    return ((((d >> 5) * 64 + ((t >> 2) * 16 + (d & 15))) * 2 + ((d >> 4) & 1)) * 4) + (t & 3);
}
// offset of elements [e0, e0 + 8) (e0 a multiple of 8: they are contiguous in either layout) of token `slot` in a key block
template <typename KT, int HD>
__device__ __forceinline__ int k_off8(int slot, int e0) { return KvTiled<KT, HD>::value ? kv_tiled_k(slot, e0) : slot * HD + e0; }

// 8 consecutive head-dim elements [e0, e0+8) of token `slot` from one head's value page
template <typename KT, int HD>
__device__ __forceinline__ void load_v8(const KT* __restrict__ vhead, int slot, int e0, float o[8]) {
    if (KvTiled<KT, HD>::value) {
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = ld1(vhead + kv_tiled_v(slot, e0 + e));
    } else if (KvTraits<KT>::v_transposed) {
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = ld1(vhead + (e0 + e) * RSD_PAGE + slot);
    } else {
        load8(vhead + slot * HD + e0, o);
    }
}
template <typename KT, int HD>
__device__ __forceinline__ KT* v_addr(KT* vhead, int slot, int e) {
    if (KvTiled<KT, HD>::value) return vhead + kv_tiled_v(slot, e);
    return KvTraits<KT>::v_transposed ? vhead + e * RSD_PAGE + slot : vhead + slot * HD + e;
}

// One block per (row, kv head, split).  The G query heads of the group share
// every key/value load.  A "lane group" of HD/8 lanes covers one token (16
// bytes of bf16 per lane); each lane group runs its own online softmax over
// the tokens it sees, and the streams are merged at the end (lane groups by
// shuffles, waves through LDS, splits by attn_combine_kernel).
template <typename KT, int HD, int G>
__global__ __launch_bounds__(256) void attn_rows_kernel(const float* __restrict__ qkv, int ldq,
                                                        const KT* __restrict__ pool_layer,
                                                        const int* __restrict__ block_table, int max_pages,
                                                        RowMap rm, int H, int Hkv, int S, float scale,
                                                        float* __restrict__ out, int ldo,
                                                        float* __restrict__ part_acc,
                                                        float* __restrict__ part_ml) {
    constexpr int LPT = HD / 8;          // lanes per token
    constexpr int TPW = 64 / LPT;        // tokens per wave-wide load
    constexpr int ITERS = RSD_PAGE / TPW > 0 ? RSD_PAGE / TPW : 1;   // wave loads per page
    constexpr int PPW = TPW / RSD_PAGE > 0 ? TPW / RSD_PAGE : 1;     // pages per wave load (HD = 32: 1)
    static_assert(PPW == 1, "a wave load covers at most one page");
    const int r = blockIdx.x, hk = blockIdx.y, sp = blockIdx.z;
    int seq, pos;
    if (!row_lookup(rm, r, seq, pos)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = lane % LPT, tsub = lane / LPT;

    float q[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        load8(qkv + (size_t)r * ldq + (hk * G + g) * HD + part * 8, q[g]);
#pragma unroll
        for (int e = 0; e < 8; ++e) q[g][e] *= scale;
    }
    float mx[G], l[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        mx[g] = -INFINITY; l[g] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.0f;
    }

    const int n_keys = pos + 1;
    const int n_pages = (n_keys + RSD_PAGE - 1) / RSD_PAGE;
    const int pps = (n_pages + S - 1) / S;
    const int p_begin = sp * pps, p_end = min(n_pages, p_begin + pps);
    const int* bt = block_table + (size_t)seq * max_pages;
    const size_t page_elts = (size_t)2 * Hkv * RSD_PAGE * HD;

    for (int pg = p_begin + wave; pg < p_end; pg += 4) {
        const KT* kbase = pool_layer + (size_t)bt[pg] * page_elts + (size_t)hk * RSD_PAGE * HD;
        const KT* vbase = kbase + (size_t)Hkv * RSD_PAGE * HD;
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            const int slot = it * TPW + tsub;
            const int t = pg * RSD_PAGE + slot;
            float kx[8], vx[8];
            load8(kbase + k_off8<KT, HD>(slot, part * 8), kx);
            load_v8<KT, HD>(vbase, slot, part * 8, vx);
            float s[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float d = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) d += q[g][e] * kx[e];
#pragma unroll
                for (int off = 1; off < LPT; off <<= 1) d += __shfl_xor(d, off, RSD_WAVE);
                s[g] = d;
            }
            if (t < n_keys) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float mn = fmaxf(mx[g], s[g]);
                    const float corr = __expf(mx[g] - mn);      // exp(-inf) = 0 on the first token
                    const float p = __expf(s[g] - mn);
                    l[g] = l[g] * corr + p;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[g][e] = acc[g][e] * corr + p * vx[e];
                    mx[g] = mn;
                }
            }
        }
    }

    // merge the lane groups of the wave
#pragma unroll
    for (int off = LPT; off < 64; off <<= 1) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float mo = __shfl_xor(mx[g], off, RSD_WAVE);
            const float lo = __shfl_xor(l[g], off, RSD_WAVE);
            const float mn = fmaxf(mx[g], mo);
            const float ca = (mx[g] == -INFINITY) ? 0.0f : __expf(mx[g] - mn);
            const float cb = (mo == -INFINITY) ? 0.0f : __expf(mo - mn);
            l[g] = l[g] * ca + lo * cb;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float ao = __shfl_xor(acc[g][e], off, RSD_WAVE);
                acc[g][e] = acc[g][e] * ca + ao * cb;
            }
            mx[g] = mn;
        }
    }
    // merge the four waves through LDS
    __shared__ float s_acc[4][G][HD];
    __shared__ float s_m[4][G], s_l[4][G];
    if (lane < LPT) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s_acc[wave][g][part * 8 + e] = acc[g][e];
            if (lane == 0) { s_m[wave][g] = mx[g]; s_l[wave][g] = l[g]; }
        }
    }
    __syncthreads();
    const int H_ = H;
    for (int idx = tid; idx < G * HD; idx += 256) {
        const int g = idx / HD, e = idx - g * HD;
        float mn = fmaxf(fmaxf(s_m[0][g], s_m[1][g]), fmaxf(s_m[2][g], s_m[3][g]));
        float a = 0.0f, ll = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float c = (s_m[w][g] == -INFINITY) ? 0.0f : __expf(s_m[w][g] - mn);
            a += s_acc[w][g][e] * c;
            ll += s_l[w][g] * c;
        }
        const int h = hk * G + g;
        if (S == 1) {
            out[(size_t)r * ldo + h * HD + e] = a / ll;
        } else {
            const size_t pi = ((size_t)r * H_ + h) * S + sp;
            part_acc[pi * HD + e] = a;
            if (e == 0) { part_ml[pi * 2] = mn; part_ml[pi * 2 + 1] = ll; }
        }
    }
}

// Merge the S partial results of every (row, head).  LOG2: their maxima are in units of log2 (chunked prefill) - merged as they
// are, since a conversion would round them and with that move a split's weight by up to 2^-24 of its maximum.
template <int HD, bool LOG2 = false>
__global__ void attn_combine_kernel(const float* __restrict__ part_acc, const float* __restrict__ part_ml,
                                    RowMap rm, int H, int S, float* __restrict__ out, int ldo,
                                    uint16_t* __restrict__ out_h = nullptr, uint16_t* __restrict__ out_l = nullptr) {
    const int r = blockIdx.x, h = blockIdx.y, e = threadIdx.x;
    int seq, pos;
    if (!row_lookup(rm, r, seq, pos)) return;
    const size_t base = ((size_t)r * H + h) * S;
    float mn = -INFINITY;
    for (int s = 0; s < S; ++s) mn = fmaxf(mn, part_ml[(base + s) * 2]);
    float a = 0.0f, ll = 0.0f;
    for (int s = 0; s < S; ++s) {
        const float m = part_ml[(base + s) * 2];
        const float c = (m == -INFINITY) ? 0.0f : (LOG2 ? __builtin_amdgcn_exp2f(m - mn) : __expf(m - mn));
        a += part_acc[(base + s) * HD + e] * c;
        ll += part_ml[(base + s) * 2 + 1] * c;
    }
    const float y = a / ll;
    if (out_h) {                // as hi + lo bf16 halves, for the MFMA projection that follows
        const uint16_t hi = f2bf(y);
        out_h[(size_t)r * ldo + h * HD + e] = hi;
        out_l[(size_t)r * ldo + h * HD + e] = f2bf(y - bf2f(hi));
    } else {
        out[(size_t)r * ldo + h * HD + e] = y;
    }
}

// Where the projected q, k, v of the rows come from when the projection's K slices have not been added up yet:
// part[z][row][col], z < ks, slices `stride` floats apart (the layout the few-row and the tile GEMM leave).
struct QkvParts { const float* part; int ks; size_t stride; };

__device__ __forceinline__ void store4(float* p, const float4& v) { *reinterpret_cast<float4*>(p) = v; }
__device__ __forceinline__ void store4(bf16_t* p, const float4& v) {
    *reinterpret_cast<uint2*>(p) = make_uint2(f2bf2(v.x, v.y), f2bf2(v.z, v.w));
}

// Rotate q (in place, fp32) and k with the precomputed table rope[pos][i] =
// (cos, sin)(pos * theta^(-2i/HD)), pairing element i with i + HD/2; write the
// rotated k and v of the row's token into its cache slot.  PARTS: q, k, v are still the K slices of their projection, which
// are added up here (ascending) instead of by a finish kernel; only q goes to `qkv` then.
// A thread takes four element pairs (or four elements of v) and requests them before the row's position is known; walking
// a row element by element with 256 threads, each round waited for the stores of the one before it.
// 7B, 32 rows: finish and rotation 4.3 + 5.8 us in two launches, 5.2 in one (6001 rows, no slices: 44 us both ways).
template <typename KT, int HD, bool PARTS>
__global__ __launch_bounds__(1024) void rope_kv_kernel(float* __restrict__ qkv, int ldq,
                                                      KT* __restrict__ pool_layer,
                                                      const int* __restrict__ block_table, int max_pages,
                                                      RowMap rm, const float2* __restrict__ rope,
                                                      int H, int Hkv, QkvParts qp) {
    constexpr int HALF = HD / 2, QH = HALF / 4;
    const int r = blockIdx.x;
    float* row = qkv + (size_t)r * ldq;
    const float* src = PARTS ? qp.part + (size_t)r * ldq : row;
    const int nqk = (H + Hkv) * QH, total = nqk + Hkv * (HD / 4);
    float4 x, y;
    auto fetch = [&](int idx) {
        const bool qk = idx < nqk;
        const int at = qk ? (idx / QH) * HD + (idx % QH) * 4 : (H + Hkv) * HD + (idx - nqk) * 4;
        const int at2 = at + (qk ? HALF : 0);
        if (PARTS) {
            x = sum_slices(src + at, qp.stride, qp.ks);
            y = sum_slices(src + at2, qp.stride, qp.ks);
        } else {
            x = *reinterpret_cast<const float4*>(src + at);
            y = *reinterpret_cast<const float4*>(src + at2);
        }
    };
    fetch(min((int)threadIdx.x, total - 1));
    int seq, pos;
    if (!row_lookup(rm, r, seq, pos)) return;
    const float* cs = reinterpret_cast<const float*>(rope + (size_t)pos * HALF);
    const int page = block_table[(size_t)seq * max_pages + pos / RSD_PAGE], slot = pos % RSD_PAGE;
    const size_t page_elts = (size_t)2 * Hkv * RSD_PAGE * HD;
    KT* kpage = pool_layer + (size_t)page * page_elts;
    KT* vpage = kpage + (size_t)Hkv * RSD_PAGE * HD;
    for (int idx = threadIdx.x; idx < total;) {
        if (idx < nqk) {
            const int h = idx / QH, i = (idx % QH) * 4;                 // heads H.. are the key heads
            const float4 c0 = *reinterpret_cast<const float4*>(cs + 2 * i), c1 = *reinterpret_cast<const float4*>(cs + 2 * i + 4);
            const float4 ra = make_float4(x.x * c0.x - y.x * c0.y, x.y * c0.z - y.y * c0.w, x.z * c1.x - y.z * c1.y, x.w * c1.z - y.w * c1.w);
            const float4 rb = make_float4(y.x * c0.x + x.x * c0.y, y.y * c0.z + x.y * c0.w, y.z * c1.x + x.z * c1.y, y.w * c1.z + x.w * c1.w);
            if (h < H) {
                *reinterpret_cast<float4*>(row + h * HD + i) = ra;
                *reinterpret_cast<float4*>(row + h * HD + i + HALF) = rb;
            } else {
                KT* khead = kpage + (size_t)(h - H) * RSD_PAGE * HD;
                store4(khead + k_off8<KT, HD>(slot, i & ~7) + (i & 7), ra);
                store4(khead + k_off8<KT, HD>(slot, (i + HALF) & ~7) + (i & 7), rb);
            }
        } else {
            const int j = (idx - nqk) * 4, hk = j / HD, e = j - hk * HD;
            KT* vhead = vpage + (size_t)hk * RSD_PAGE * HD;
            st1(v_addr<KT, HD>(vhead, slot, e), x.x);     st1(v_addr<KT, HD>(vhead, slot, e + 1), x.y);
            st1(v_addr<KT, HD>(vhead, slot, e + 2), x.z); st1(v_addr<KT, HD>(vhead, slot, e + 3), x.w);
        }
        idx += blockDim.x;
        if (idx < total) fetch(idx);
    }
}

// ---------------------------------------------------------------------------
// Single-token decode: rotary embedding, cache write and attention in one
// launch.  grid = (sequences, kv heads, S).  Every block rotates the group's
// queries itself; the cached positions 0..pos-1 are cut into S page ranges, one
// per block, and the new token (position pos) is added by the block of the
// last range straight from registers, after rounding its key and value to the
// cache's storage type, and written to the cache by that block.  With S > 1
// each block leaves a partial (max, sum, accumulator) for attn_combine_kernel.
// (Merging inside this kernel would need device-scope fences between blocks,
// which on this multi-die part write back and invalidate L2 and cost far more
// than a second launch.)
template <typename KT> __device__ __forceinline__ float round_store(float v);
template <> __device__ __forceinline__ float round_store<float>(float v) { return v; }
template <> __device__ __forceinline__ float round_store<bf16_t>(float v) { return bf2f(f2bf(v)); }

__device__ __forceinline__ void store8(float* p, const float v[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16_t* p, const float v[8]) {
    uint4 r;
    r.x = f2bf2(v[0], v[1]);
    r.y = f2bf2(v[2], v[3]);
    r.z = f2bf2(v[4], v[5]);
    r.w = f2bf2(v[6], v[7]);
    *reinterpret_cast<uint4*>(p) = r;
}

template <typename KT, int HD, int G>
__global__ __launch_bounds__(256) void attn_decode_kernel(const float* __restrict__ qkv, int ldq,
                                                          KT* __restrict__ pool_layer,
                                                          const int* __restrict__ block_table, int max_pages,
                                                          const int* __restrict__ kv_len,
                                                          const int* __restrict__ active,
                                                          const float2* __restrict__ rope, int H, int Hkv, int S,
                                                          float scale, float* __restrict__ out, int ldo,
                                                          float* __restrict__ part_acc, float* __restrict__ part_ml,
                                                          const int* __restrict__ row_seq) {
    constexpr int LPT = HD / 8, TPW = 64 / LPT;
    constexpr int ITERS = RSD_PAGE / TPW > 0 ? RSD_PAGE / TPW : 1;
    constexpr bool AHEAD = ITERS == 1;              // the next page is requested before the present one is used (registers)
    const int r = blockIdx.x, hk = blockIdx.y, sp = blockIdx.z;
    const int seq = row_seq ? row_seq[r] : r;       // packed rows: the sequence this row stands for (< 0: none)
    if (seq < 0) return;
    const int pos = kv_len[seq], is_active = active[seq];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = lane % LPT, tsub = lane / LPT;
    const float* row = qkv + (size_t)r * ldq;
    const int* bt = block_table + (size_t)seq * max_pages;
    // A short context is a chain of loads (position, pages and rotary table, keys and values), so what does not depend on the
    // position is requested with it: q, the new token's k and v and, without splits, this wave's pages (lane i: its i-th).  With the
    // shared maximum and the halving sums below: head_dim 32, 8 pages, four heads per KV head 6.9 -> 4.9 us, two 5.2 -> 4.0.
    const bool first = part * 8 < HD / 2;
    const int e_oth = first ? part * 8 + HD / 2 : part * 8 - HD / 2;
    float q[G][8], q_oth[G][8], kn[8], k_oth[8], vn[8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        load8(row + (hk * G + g) * HD + part * 8, q[g]);
        load8(row + (hk * G + g) * HD + e_oth, q_oth[g]);
    }
    load8(row + (H + hk) * HD + part * 8, kn);
    load8(row + (H + hk) * HD + e_oth, k_oth);
    load8(row + (H + Hkv + hk) * HD + part * 8, vn);
    int bt_mine = bt[min(wave + 4 * lane, max_pages - 1)];
    if (!is_active) return;

    const int n_pages = (pos + RSD_PAGE - 1) / RSD_PAGE;      // pages holding cached positions 0..pos-1
    const int pps = (n_pages + S - 1) / S;
    const int p_begin = sp * pps, p_end = min(n_pages, p_begin + pps);
    const int n_mine = max(0, (p_end - p_begin - wave + 3) >> 2);               // pages p_begin + wave, + 4, ...
    if (p_begin > 0) bt_mine = bt[min(p_begin + wave + 4 * lane, max_pages - 1)];
    float2 cs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cs[e] = rope[(size_t)pos * (HD / 2) + (first ? part * 8 : e_oth) + e];
    const int bt_new = bt[pos / RSD_PAGE];
    const size_t page_elts = (size_t)2 * Hkv * RSD_PAGE * HD;
    const size_t head_off = (size_t)hk * RSD_PAGE * HD, v_off = (size_t)Hkv * RSD_PAGE * HD;
    float kx[ITERS][8], vx[ITERS][8];
    auto fetch = [&](int i) {
        const int id = i < 64 ? __shfl(bt_mine, i, RSD_WAVE) : bt[p_begin + wave + 4 * i];
        const KT* kbase = pool_layer + (size_t)id * page_elts + head_off;
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            const int slot = it * TPW + tsub;
            load8(kbase + k_off8<KT, HD>(slot, part * 8), kx[it]);
            load_v8<KT, HD>(kbase + v_off, slot, part * 8, vx[it]);
        }
    };
    if (n_mine > 0) fetch(0);
    auto rotate = [&](float (&own)[8], const float (&oth)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) own[e] = first ? (own[e] * cs[e].x - oth[e] * cs[e].y) : (own[e] * cs[e].x + oth[e] * cs[e].y);
    };
#pragma unroll
    for (int g = 0; g < G; ++g) {
        rotate(q[g], q_oth[g]);
#pragma unroll
        for (int e = 0; e < 8; ++e) q[g][e] *= scale;
    }
    float mx[G], l[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        mx[g] = -INFINITY; l[g] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.0f;
    }
    auto absorb = [&](const float kx[8], const float vx[8], bool valid) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float d = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) d += q[g][e] * kx[e];
#pragma unroll
            for (int off = 1; off < LPT; off <<= 1) d += __shfl_xor(d, off, RSD_WAVE);
            if (valid) {
                const float mn = fmaxf(mx[g], d);
                const float corr = __expf(mx[g] - mn);
                const float p = __expf(d - mn);
                l[g] = l[g] * corr + p;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[g][e] = acc[g][e] * corr + p * vx[e];
                mx[g] = mn;
            }
        }
    };

    for (int i = 0; i < n_mine; ++i) {
        float kc[ITERS][8], vc[ITERS][8];
#pragma unroll
        for (int it = 0; it < ITERS; ++it)
#pragma unroll
            for (int e = 0; e < 8; ++e) { kc[it][e] = kx[it][e]; vc[it][e] = vx[it][e]; }
        if (AHEAD && i + 1 < n_mine) fetch(i + 1);
#pragma unroll
        for (int it = 0; it < ITERS; ++it) absorb(kc[it], vc[it], (p_begin + wave + 4 * i) * RSD_PAGE + it * TPW + tsub < pos);
        if (!AHEAD && i + 1 < n_mine) fetch(i + 1);
    }
    if (sp == S - 1 && wave == (max(p_end - p_begin, 0) & 3)) {       // (a wave with the fewest pages)
        // the new token: rotate its key, round key and value as the cache stores them, write, attend
        rotate(kn, k_oth);
#pragma unroll
        for (int e = 0; e < 8; ++e) { kn[e] = round_store<KT>(kn[e]); vn[e] = round_store<KT>(vn[e]); }
        if (tsub == 0) {
            KT* khead = pool_layer + (size_t)bt_new * page_elts + head_off;
            store8(khead + k_off8<KT, HD>(pos % RSD_PAGE, part * 8), kn);
#pragma unroll
            for (int e = 0; e < 8; ++e) st1(v_addr<KT, HD>(khead + v_off, pos % RSD_PAGE, part * 8 + e), vn[e]);
        }
        absorb(kn, vn, tsub == 0);
    }

    // the wave's token lanes: common maximum first, then plain sums.  A step of the sums halves the elements a lane carries
    // (8 -> 4 -> 2 -> 1) as long as there are any to halve; lane bits LPT, 2 LPT, 4 LPT select element bits 2, 1, 0.
    int e0 = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float mn = mx[g];
#pragma unroll
        for (int off = LPT; off < 64; off <<= 1) mn = fmaxf(mn, __shfl_xor(mn, off, RSD_WAVE));
        const float c = (mx[g] == -INFINITY) ? 0.0f : __expf(mx[g] - mn);
        mx[g] = mn;
        l[g] *= c;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] *= c;
        e0 = 0;
        int n = 4;
#pragma unroll
        for (int off = LPT; off < 64; off <<= 1) {
            l[g] += __shfl_xor(l[g], off, RSD_WAVE);
            if (n > 0) {
                const bool up = lane & off;
                e0 += up ? n : 0;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < n) {
                        const float keep = up ? acc[g][j + n] : acc[g][j], send = up ? acc[g][j] : acc[g][j + n];
                        acc[g][j] = keep + __shfl_xor(send, off, RSD_WAVE);
                    }
                n >>= 1;
            } else acc[g][0] += __shfl_xor(acc[g][0], off, RSD_WAVE);
        }
    }
    constexpr int NL = TPW >= 8 ? 1 : 8 / TPW;                           // elements left in a lane
    __shared__ float s_acc[4][G][HD];
    __shared__ float s_m[4][G], s_l[4][G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int j = 0; j < NL; ++j)
            if (lane < 8 * LPT) s_acc[wave][g][part * 8 + e0 + j] = acc[g][j];      // (lanes above hold copies)
        if (lane == 0) { s_m[wave][g] = mx[g]; s_l[wave][g] = l[g]; }
    }
    __syncthreads();
    for (int idx = tid; idx < G * HD; idx += 256) {
        const int g = idx / HD, e = idx - g * HD;
        const float mn = fmaxf(fmaxf(s_m[0][g], s_m[1][g]), fmaxf(s_m[2][g], s_m[3][g]));
        float a = 0.0f, ll = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float c = (s_m[w][g] == -INFINITY) ? 0.0f : __expf(s_m[w][g] - mn);
            a += s_acc[w][g][e] * c;
            ll += s_l[w][g] * c;
        }
        const int h = hk * G + g;
        if (S == 1) {
            out[(size_t)r * ldo + h * HD + e] = a / ll;
        } else {
            const size_t pi = ((size_t)r * H + h) * S + sp;
            part_acc[pi * HD + e] = a;
            if (e == 0) { part_ml[pi * 2] = mn; part_ml[pi * 2 + 1] = ll; }
        }
    }
}

// ---------------------------------------------------------------------------
// MFMA single-token decode attention for bf16 caches, head_dim 128.
//
// One block per (sequence, kv head, split); each of its NW waves takes pages
// round-robin.  Per page (16 tokens) and wave:
//   S^T[token][head] = K . Q^T      v_mfma_f32_16x16x32_bf16, 4 steps over head_dim;
//                                   K straight from HBM (64 contiguous bytes per lane),
//                                   Q^T of the group's G heads padded to 16 columns
//   online softmax per head (column), in the accumulator layout
//   O[head][col]   += P . V         v_mfma_f32_16x16x16bf16_1k, 8 column blocks; the
//                                   softmax output already sits in the A-operand layout,
//                                   V^T pages give 8 contiguous bytes per lane
// The fp32 operands (rotated, scaled q and the probabilities) enter as hi + lo
// bf16 pairs, two MFMAs each, so they keep 16 significant bits; K and V are
// bf16 in the cache and enter exactly.  The new token is added from registers
// by wave 0 of the last split, which also writes it to the cache.  With S > 1
// the partials are merged by attn_combine_kernel.
typedef __attribute__((ext_vector_type(8))) __bf16 abf16x8_t;
typedef __attribute__((ext_vector_type(4))) short as16x4_t;
typedef __attribute__((ext_vector_type(4))) float af32x4_t;

__device__ __forceinline__ void split_hi_lo8(const float x[8], abf16x8_t& hi, abf16x8_t& lo) {
    uint4 h, l;
    split2(x[0], x[1], h.x, l.x);
    split2(x[2], x[3], h.y, l.y);
    split2(x[4], x[5], h.z, l.z);
    split2(x[6], x[7], h.w, l.w);
    hi = __builtin_bit_cast(abf16x8_t, h);
    lo = __builtin_bit_cast(abf16x8_t, l);
}

// PARTS: the kernel adds the K slices of the QKV projection itself (ascending, like the finish kernels) while
// its first pages are in flight, which saves the launch of a finish kernel per layer; `qkv` is then unused.
// What bounds short contexts and few rows is the chain of dependent loads (position, pages and rotary table, q / k / v, new
// token): everything that does not depend on the position is requested with it, everything else right behind it.  Per layer,
// against asking for each when it is needed: 1.5B one row 7.2 -> 5.4 us, 16 rows 13.5 -> 12.2, 64 ragged rows 18.8 -> 17.3; 7B 64 rows
// 21.6 -> 19.2; 72B 16 rows 15.7 -> 12.8.
// 16 bytes of a cache page in the decode kernel: every page is read once per launch, so the loads are marked
// non-temporal and leave the caches to what is used again (batch 256 at 4096 tokens: 392 -> 367 us per 7B
// layer, 200 -> 180 us per 1.5B layer; the 7B iteration at batch 64: 5.27 -> 4.94 ms)
#ifndef RSD_KV_NT
#define RSD_KV_NT 1
#endif
__device__ __forceinline__ uint4 load_kv16(const bf16_t* p) {
#if RSD_KV_NT
    typedef uint32_t nt_u32x4 __attribute__((ext_vector_type(4)));
    const nt_u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4*>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
#else
    return *reinterpret_cast<const uint4*>(p);
#endif
}
template <int G, int NW, bool PARTS>
__global__ __launch_bounds__(NW * 64, NW == 4 ? 2 : 1) void attn_decode_mfma_kernel(const float* __restrict__ qkv, int ldq,
                                                                   bf16_t* __restrict__ pool_layer,
                                                                   const int* __restrict__ block_table, int max_pages,
                                                                   const int* __restrict__ kv_len,
                                                                   const int* __restrict__ active,
                                                                   const float2* __restrict__ rope, int H, int Hkv,
                                                                   int S, float scale, float* __restrict__ out, int ldo,
                                                                   float* __restrict__ part_acc, float* __restrict__ part_ml,
                                                                   uint16_t* __restrict__ out_h, uint16_t* __restrict__ out_l,
                                                                   const int* __restrict__ row_seq, QkvParts qp) {
    constexpr int HD = 128;
    const int r = blockIdx.x, hk = blockIdx.y, sp = blockIdx.z;
    const int seq_raw = row_seq ? row_seq[r] : r;   // packed rows: the sequence this row stands for (< 0: none)
    const int seq = max(seq_raw, 0);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // Pages are dealt round-robin: the i-th page of (split sp, wave w) is sp + S * (w + NW * i), whatever
    // the position turns out to be.  So the table entries (lane i holds the i-th; entries beyond the
    // sequence are never used) are requested together with the position, not after it.
    const int is_active = seq_raw >= 0 && active[seq];
    const int pos = kv_len[seq];
    const int pg0 = sp + S * wave, pg_step = S * NW;
    int bt_mine = -1;
    if (pg0 + pg_step * lane < max_pages) bt_mine = block_table[(size_t)seq * max_pages + pg0 + pg_step * lane];
    const int l16 = lane & 15, c = lane >> 4;
    const float* row = qkv + (size_t)r * ldq;
    // q of the group's heads, k and v of this KV head for the row (PARTS: their K slices) do not depend on the position
    // either: they are requested before anything waits for it.  The new token is the business of wave 0 of the last split.
    const bool owns_new = (sp == S - 1 && wave == 0);
    __shared__ float s_row[PARTS ? (G + 2) * HD : 1];
    constexpr int NQ = 16 * (HD / 2) / (NW * 64);
    float qa[NQ], qb[NQ], kx[4][8], vx[8];
    constexpr int NE = (G + 2) * HD, NI = (NE + NW * 64 - 1) / (NW * 64);
    float pb[PARTS ? NI : 1][8];                              // PARTS: the first eight slices of this thread's elements
    auto part_at = [&](int ii) {
        const int i = min(tid + ii * NW * 64, NE - 1);
        const int col = i < G * HD ? hk * G * HD + i : (i < (G + 1) * HD ? (H + hk) * HD + (i - G * HD) : (H + Hkv + hk) * HD + (i - (G + 1) * HD));
        return qp.part + (size_t)r * ldq + col;
    };
    if constexpr (PARTS) {
#pragma unroll
        for (int ii = 0; ii < NI; ++ii) {
            const float* p = part_at(ii);
#pragma unroll
            for (int u = 0; u < 8; ++u) pb[ii][u] = p[(size_t)min(u, qp.ks - 1) * qp.stride];
        }
    } else {
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int idx = tid + i * NW * 64, g = min(idx / (HD / 2), G - 1), e = idx & (HD / 2 - 1);
            qa[i] = row[(hk * G + g) * HD + e]; qb[i] = row[(hk * G + g) * HD + e + HD / 2];
        }
        if (owns_new) {
#pragma unroll
            for (int j = 0; j < 4; ++j) load8(row + (H + hk) * HD + j * 32 + c * 8, kx[j]);
#pragma unroll
            for (int m = 0; m < 8; ++m) vx[m] = row[(H + Hkv + hk) * HD + m * 16 + l16];
        }
    }
    if (!is_active) return;
    const float2* cs = rope + (size_t)pos * (HD / 2);
    float2 cq[NQ], cn[2][8];
#pragma unroll
    for (int i = 0; i < NQ; ++i) cq[i] = cs[(tid + i * NW * 64) & (HD / 2 - 1)];
    if (owns_new) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 8; ++e) cn[j][e] = cs[j * 32 + c * 8 + e];
    }

    const int n_pages = (pos + RSD_PAGE - 1) / RSD_PAGE;      // pages holding cached positions 0..pos-1
    const int* bt = block_table + (size_t)seq * max_pages;
    const size_t page_elts = (size_t)2 * Hkv * RSD_PAGE * HD;
    const size_t head_off = (size_t)hk * RSD_PAGE * HD, v_off = (size_t)Hkv * RSD_PAGE * HD;

    // operands of one page (tiled page layout, see KvTiled): K chunk j of token l16 = K[l16][j*32 + c*8 ..+8] is
    // the lane's 16 bytes of the j-th KB of the key block; the lane's 16 bytes of the m-th KB of the value
    // block hold V^T[(2m)*16 + l16][c*4 ..+4] (.x, .y) and V^T[(2m+1)*16 + l16][c*4 ..+4] (.z, .w)
    uint4 kc[4], kn[4];
    uint4 vc[4], vn[4];
    auto fetch_phys = [&](int phys, uint4 k[4], uint4 v[4]) {
        const bf16_t* kb = pool_layer + (size_t)phys * page_elts + head_off;
#pragma unroll
        for (int j = 0; j < 4; ++j) k[j] = load_kv16(kb + (j * 64 + lane) * 8);
#pragma unroll
        for (int m = 0; m < 4; ++m) v[m] = load_kv16(kb + v_off + (m * 64 + lane) * 8);
    };
    // i-th page of this wave (i < 64: a wave never holds more than 64 pages)
    auto fetch = [&](int i, uint4 k[4], uint4 v[4]) { fetch_phys(__shfl(bt_mine, i, RSD_WAVE), k, v); };
    uint4 k2[4];
    uint4 v2[4];                 // two pages in flight ahead of the one being used
    int pg = pg0, it = 0;
    if (pg < n_pages) fetch(0, kc, vc);
    if (pg + pg_step < n_pages) fetch(1, kn, vn);

    if constexpr (PARTS) {
#pragma unroll
        for (int ii = 0; ii < NI; ++ii) {
            float a = 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) if (u < qp.ks) a += pb[ii][u];
            const float* p = part_at(ii);
            for (int z = 8; z < qp.ks; z += 8) {              // (clamped addresses: one round trip per eight slices)
                float b[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) b[u] = p[(size_t)min(z + u, qp.ks - 1) * qp.stride];
#pragma unroll
                for (int u = 0; u < 8; ++u) if (z + u < qp.ks) a += b[u];
            }
            if (tid + ii * NW * 64 < NE) s_row[tid + ii * NW * 64] = a;
        }
        __syncthreads();
    }
    // rotated, scaled queries of the group, computed once per block and kept in LDS as hi + lo bf16
    // (rows >= G stay zero); the waves read their MFMA operands from there for every page
    __shared__ __attribute__((aligned(16))) uint16_t s_qh[16][HD + 8];
    __shared__ __attribute__((aligned(16))) uint16_t s_ql[16][HD + 8];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int idx = tid + i * NW * 64, g = idx / (HD / 2), e = idx & (HD / 2 - 1);
        float ra = 0.0f, rb = 0.0f;
        if (g < G) {
            const float a = PARTS ? s_row[g * HD + e] : qa[i], b = PARTS ? s_row[g * HD + e + HD / 2] : qb[i];
            ra = (a * cq[i].x - b * cq[i].y) * scale;
            rb = (b * cq[i].x + a * cq[i].y) * scale;
        }
        const uint16_t ha = f2bf(ra), hb = f2bf(rb);
        s_qh[g][e] = ha; s_qh[g][e + HD / 2] = hb;
        s_ql[g][e] = f2bf(ra - bf2f(ha)); s_ql[g][e + HD / 2] = f2bf(rb - bf2f(hb));
    }
    __syncthreads();

    // the new token as a pseudo page whose only valid token is row 0 (wave 0 of the last split):
    // rotate its key, round key and value to bf16 as the cache stores them, write them to the cache.
    // Done before the page loop so that its loads overlap the first page fetches.
    uint4 k1[4];
    uint4 v1[4];
    if (owns_new) {
        if constexpr (PARTS) {
#pragma unroll
            for (int j = 0; j < 4; ++j) load8(s_row + G * HD + j * 32 + c * 8, kx[j]);
#pragma unroll
            for (int m = 0; m < 8; ++m) vx[m] = s_row[(G + 1) * HD + m * 16 + l16];
        }
        bf16_t* kb = pool_layer + (size_t)bt[pos / RSD_PAGE] * page_elts + head_off;
        const int slot = pos % RSD_PAGE;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {                    // elements 2 i, 2 i + 1: chunk j is rotated with chunk j +- 2
                float k2[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int e = 2 * i + u;
                    const float2 t = cn[j & 1][e];
                    k2[u] = j < 2 ? kx[j][e] * t.x - kx[j + 2 < 4 ? j + 2 : 0][e] * t.y : kx[j][e] * t.x + kx[j >= 2 ? j - 2 : 0][e] * t.y;
                }
                w[i] = f2bf2(k2[0], k2[1]);
            }
            const uint4 pk = make_uint4(w[0], w[1], w[2], w[3]);
            if (l16 == 0) *reinterpret_cast<uint4*>(kb + kv_tiled_k(slot, j * 32 + c * 8)) = pk;
            k1[j] = (l16 == 0) ? pk : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint16_t va = f2bf(vx[2 * m]);
            const uint16_t vb = f2bf(vx[2 * m + 1]);
            if (c == 0) {
                kb[v_off + kv_tiled_v(slot, (2 * m) * 16 + l16)].v = va;
                kb[v_off + kv_tiled_v(slot, (2 * m + 1) * 16 + l16)].v = vb;
            }
            v1[m] = make_uint4(c == 0 ? (uint32_t)va : 0u, 0u, c == 0 ? (uint32_t)vb : 0u, 0u);
        }
    }

    // Scores come out transposed, S^T[token c*4+i][head l16], which is at once the layout of P^T as the
    // B operand of O^T = V^T P^T.  So every lane works for ONE head (l16): its running maximum, sum and
    // rescaling factor are its own, and sums over tokens run over i and over the four 16-lane rows.
    float m_run = -INFINITY, l_run = 0.0f;
    af32x4_t o[8];                                          // o[nb][i] = O[head l16][nb*16 + c*4 + i]
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) o[nb] = af32x4_t{0.f, 0.f, 0.f, 0.f};

    // one page: tokens c*4+i of it are valid iff (vmask >> i) & 1
    auto process = [&](const uint4 k[4], const uint4 v[4], int vmask) {
        af32x4_t s = {0.f, 0.f, 0.f, 0.f}, s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const abf16x8_t ka = __builtin_bit_cast(abf16x8_t, k[j]);
            const abf16x8_t qlo = __builtin_bit_cast(abf16x8_t, *reinterpret_cast<const uint4*>(&s_ql[l16][j * 32 + c * 8]));
            const abf16x8_t qhi = __builtin_bit_cast(abf16x8_t, *reinterpret_cast<const uint4*>(&s_qh[l16][j * 32 + c * 8]));
            s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qlo, s2, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qhi, s, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] += s2[i];
        float mloc = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) if ((vmask >> i) & 1) mloc = fmaxf(mloc, s[i]);
        mloc = rows4_max(mloc);
        const float m_new = fmaxf(m_run, mloc);
        const float corr = (m_run == -INFINITY) ? 0.0f : __expf(m_run - m_new);
        float p[4], lsum = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = (((vmask >> i) & 1) && m_new > -INFINITY) ? __expf(s[i] - m_new) : 0.0f;
            lsum += p[i];
        }
        lsum = rows4_sum(lsum);
        l_run = l_run * corr + lsum;
        m_run = m_new;
        uint2 ph, pl;
        split2(p[0], p[1], ph.x, pl.x);
        split2(p[2], p[3], ph.y, pl.y);
        const as16x4_t pa = __builtin_bit_cast(as16x4_t, ph), pb = __builtin_bit_cast(as16x4_t, pl);
        // slots past the sequence hold whatever the pool held: zero them (0 * NaN would poison the sum)
        const uint32_t mk0 = ((vmask & 1) ? 0xFFFFu : 0u) | ((vmask & 2) ? 0xFFFF0000u : 0u);
        const uint32_t mk1 = ((vmask & 4) ? 0xFFFFu : 0u) | ((vmask & 8) ? 0xFFFF0000u : 0u);
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[nb][i] *= corr;
            const uint32_t vx = (nb & 1) ? v[nb >> 1].z : v[nb >> 1].x, vy = (nb & 1) ? v[nb >> 1].w : v[nb >> 1].y;
            const as16x4_t vb = __builtin_bit_cast(as16x4_t, make_uint2(vx & mk0, vy & mk1));
            o[nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vb, pb, o[nb], 0, 0, 0);
            o[nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vb, pa, o[nb], 0, 0, 0);
        }
    };

    if (owns_new) process(k1, v1, c == 0 ? 1 : 0);          // order of accumulation is free
    // Three register buffers take fixed turns (no copies between them: a copy would have to wait for
    // the load it copies): while page i is used, pages i+1 and i+2 are in flight.
    auto page_mask = [&](int page) {
        int vm = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) vm |= (page * RSD_PAGE + c * 4 + i < pos) ? (1 << i) : 0;
        return vm;
    };
    while (pg < n_pages) {
        if (pg + 2 * pg_step < n_pages) fetch(it + 2, k2, v2);
        process(kc, vc, page_mask(pg));
        pg += pg_step; ++it;
        if (pg >= n_pages) break;
        if (pg + 2 * pg_step < n_pages) fetch(it + 2, kc, vc);
        process(kn, vn, page_mask(pg));
        pg += pg_step; ++it;
        if (pg >= n_pages) break;
        if (pg + 2 * pg_step < n_pages) fetch(it + 2, kn, vn);
        process(k2, v2, page_mask(pg));
        pg += pg_step; ++it;
    }

    // ---- merge the waves of the block through LDS
    __shared__ __attribute__((aligned(16))) float s_o[NW][G][HD];
    __shared__ float s_m[NW][16], s_l[NW][16];
    if (c == 0) { s_m[wave][l16] = m_run; s_l[wave][l16] = l_run; }
    if (l16 < G) {
#pragma unroll
        for (int nb = 0; nb < 8; ++nb)
            *reinterpret_cast<float4*>(&s_o[wave][l16][nb * 16 + c * 4]) = make_float4(o[nb][0], o[nb][1], o[nb][2], o[nb][3]);
    }
    __syncthreads();
    for (int idx = tid; idx < G * HD; idx += NW * 64) {
        const int g = idx / HD, e = idx - g * HD;
        float mn = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) mn = fmaxf(mn, s_m[w][g]);
        float a = 0.0f, ll = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float cc = (s_m[w][g] == -INFINITY) ? 0.0f : __expf(s_m[w][g] - mn);
            a += s_o[w][g][e] * cc;
            ll += s_l[w][g] * cc;
        }
        const int h = hk * G + g;
        if (S == 1) {
            const float y = a / ll;
            if (out_h) {            // as hi + lo bf16 halves, for the MFMA projection that follows
                const uint16_t hi = f2bf(y);
                out_h[(size_t)r * ldo + h * HD + e] = hi;
                out_l[(size_t)r * ldo + h * HD + e] = f2bf(y - bf2f(hi));
            } else {
                out[(size_t)r * ldo + h * HD + e] = y;
            }
        } else {
            const size_t pi = ((size_t)r * H + h) * S + sp;
            part_acc[pi * HD + e] = a;
            if (e == 0) { part_ml[pi * 2] = mn; part_ml[pi * 2 + 1] = ll; }
        }
    }
}

// ---------------------------------------------------------------------------
// MFMA chunked-prefill attention for bf16 caches, head_dim 128.
//
// Runs after rope_kv_kernel has rotated q in place and written the chunk's keys/values to the cache.  One block of four
// waves per work item = up to 16 consecutive rows (query tokens) of one sequence and one kv head; a wave takes four rows =
// 32 columns, a column being (row, head of the group), and keeps their rotated, scaled q as hi + lo bf16 operands in
// registers.  The item's pages are walked once, two pages (32 tokens) per step, through a ring of three LDS stages that the
// waves share: a page's key and value blocks of one head are 4 KB each of consecutive memory, copied straight into LDS more
// than two steps ahead.  The one barrier per step stands in its middle, when the step's operands are all in registers; the
// next step's keys are read between the MFMAs behind it.  Per step and wave:
//   S^T[token][column] = K . Q^T       v_mfma_f32_32x32x16_bf16, 8 steps over head_dim, hi and lo of q
//   online softmax per column in the accumulator layout (a lane holds 16 of its column's 32 tokens, the lane 32 further on
//   the others: one register swap per maximum); masks are formed only where a step reaches past a row's own position
//   O^T[dim][column] += V^T . P^T      16 tokens per MFMA, P as hi + lo; a lane's probabilities are already the operand
// Scores are kept in units of log2 (log2 e is folded into the scaling of q).
// What bounds it: the chain QK, softmax, PV of a step (1024 cycles of MFMA issue and about 700 of vector instructions per
// wave; two waves per SIMD, of different blocks, overlap them: matrix cores busy 56 % of the time at 6001 rows of one context).  The
// values' 8-byte operand reads cost four bank-conflict cycles per LDS instruction.  Its predecessor (every wave on its
// own pages and 16-column tiles, values at half the MFMA rate) spent its time in vector instructions and read each page
// through L2 once per four rows.
// Measured per layer: 8192 rows of 1024-token prompts 7B 382 -> 187 us, 1.5B 215 -> 107 us; 6001 rows of one context 7B
// 1315 -> 582 us.
// gridDim.z = S > 1 (few rows over a long context): split sp walks its share of the steps and leaves a partial (max in units of
// log2, sum, accumulator) per (row, head) for attn_combine_kernel, in the layout of the decode kernels.
// The result is written as hi + lo bf16 halves, the input of the output projection (out: as fp32, a pass of a single row).
constexpr int kPfItemRows = 16;
template <int G>
__global__ __launch_bounds__(256, 2) void attn_prefill_mfma_kernel(const float* __restrict__ qkv, int ldq,
                                                                const bf16_t* __restrict__ pool_layer,
                                                                const int* __restrict__ block_table, int max_pages,
                                                                const int* __restrict__ row_seq,
                                                                const int* __restrict__ row_pos,
                                                                const int* __restrict__ item_row0,
                                                                const int* __restrict__ item_n,
                                                                int H, int Hkv, float scale,
                                                                float* __restrict__ out, int ldo,
                                                                uint16_t* __restrict__ out_h, uint16_t* __restrict__ out_l,
                                                                float* __restrict__ part_acc,
                                                                float* __restrict__ part_ml) {
    constexpr int HD = 128, STEP = 2 * RSD_PAGE, STAGE = 2 * STEP * HD;      // bf16 elements of a stage: K and V of 32 tokens
    __shared__ __attribute__((aligned(16))) uint16_t s_kv[3 * STAGE];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = gridDim.x - 1 - blockIdx.x;             // (later items have the longer contexts: they go first)
    const int hk = blockIdx.y, sp = blockIdx.z, S = gridDim.z;
    const int r0 = item_row0[item], n = item_n[item];
    const int seq = row_seq[r0], p0 = row_pos[r0];
    const int* bt = block_table + (size_t)seq * max_pages;
    const size_t page_elts = (size_t)2 * Hkv * RSD_PAGE * HD;
    const size_t head_off = (size_t)hk * RSD_PAGE * HD, v_off = (size_t)Hkv * RSD_PAGE * HD;
    const int p_last = p0 + n - 1, n_pages = p_last / RSD_PAGE + 1, n_steps = p_last / STEP + 1;
    const int per = (n_steps + S - 1) / S;
    const int s_lo = min(n_steps, sp * per), s_hi = min(n_steps, s_lo + per);        // this split's steps

    const int col = lane & 31, h = lane >> 5;
    const int n_w = min(max(n - 4 * wave, 0), 4);            // rows of this wave (0: it only copies)
    const int ri = col >> 3, g = col & 7;
    const bool live = ri < n_w && g < G;
    const int pw = p0 + 4 * wave, pw_last = pw + n_w - 1;    // positions of its first and last row
    const int pos_col = min(pw + ri, p_last);                // (columns without a row compute something finite that nobody reads)
    const int row = r0 + 4 * wave + ri;

    // wave w copies K (w = 0, 1) or V (w = 2, 3) of page w % 2 of a step; past the end the last page is copied again
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)s_kv + wave * (RSD_PAGE * HD * 2);
    // (lane i holds the table entry of this wave's page of step bt_base + i; looked up afresh every 64 steps)
    int bt_base = s_lo, bt_mine = bt[min(2 * (s_lo + lane) + (wave & 1), n_pages - 1)];
    auto request = [&](int step, int stg) {
        step = min(step, max(s_hi - 1, s_lo));
        if (step - bt_base >= 64) {
            bt_base = step;
            bt_mine = bt[min(2 * (step + lane) + (wave & 1), n_pages - 1)];
            asm volatile("" : "+v"(bt_mine));                // (waited for here: at the branch's end every step would wait, for the copies too)
        }
        const int phys = __builtin_amdgcn_readlane(bt_mine, step - bt_base);
        const char* src = reinterpret_cast<const char*>(pool_layer + (size_t)phys * page_elts + head_off + (wave >> 1) * v_off);
#pragma unroll
        for (int i = 0; i < 4; ++i) copy16_to_lds(lds0 + stg * (STAGE * 2) + i * 1024, (uint32_t)(i * 1024 + lane * 16), src);
    };
#pragma unroll
    for (int i = 0; i < 3; ++i) request(s_lo + i, i);

    // q of this lane's column: dims 16 j + 8 h .. + 7
    abf16x8_t qh[8], ql[8];
    {
        const float* q = qkv + (size_t)(live ? row : r0) * ldq + (hk * G + (live ? g : 0)) * HD + h * 8;
        const float sc_q = live ? scale : 0.0f;
        float qv[8][8];
#pragma unroll
        for (int j = 0; j < 8; ++j) load8(q + j * 16, qv[j]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
#pragma unroll
            for (int e = 0; e < 8; ++e) qv[j][e] = live ? qv[j][e] * sc_q : 0.0f;
            split_hi_lo8(qv[j], qh[j], ql[j]);
        }
    }
    float m_run = -INFINITY, l_run = 0.0f;
    f32x16_t o[4];                                           // o[m][v] = O[column][32 m + 8 (v / 4) + 4 h + v % 4]
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[m][v] = 0.0f;

    // operand addresses inside a stage.  K: token col of the step, dims 16 j + 8 h .. : 16 bytes (tiled page layout, KvTiled)
    const int k_addr = (col >> 4) * (RSD_PAGE * HD) + (h * 16 + (col & 15)) * 8;              // + j * 256
    // V: dim 32 m + col, tokens 4 h .. + 3 and 8 + 4 h .. + 3 of page a: 8 bytes each
    const int v_addr_ = 2 * RSD_PAGE * HD + h * 128 + (col & 15) * 8 + (col >> 4) * 4;        // + a * 2048 + m * 512 (+ 256)
    uint4 kf[8], vf[8];                                      // operands: K chunk j; V of page a, dims 32 m (vf[4 a + m])
    auto read_k = [&](const uint16_t* kv, int j) { kf[j] = *reinterpret_cast<const uint4*>(kv + k_addr + j * 256); };
    auto read_v = [&](const uint16_t* kv, int i) {
        const uint16_t* p = kv + v_addr_ + (i >> 2) * 2048 + (i & 3) * 512;
        const uint2 x = *reinterpret_cast<const uint2*>(p), y = *reinterpret_cast<const uint2*>(p + 256);
        vf[i] = make_uint4(x.x, x.y, y.x, y.y);
    };
    // the first step has landed when at most the requests of the two others are outstanding
    asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int j = 0; j < 8; ++j) read_k(s_kv, j);
    int stg = 0;
    // in the middle of a step: the next one's copies have landed and this one's operands are all in registers, so behind the
    // barrier the next step may be read and this one's stage overwritten
    auto turn = [&](int s) {
        asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        request(s + 3, stg);
        stg = stg == 2 ? 0 : stg + 1;
    };
    const int s_w = n_w ? min(s_hi, pw_last / STEP + 1) : s_lo;         // steps of which some row of this wave sees a token
    int s = s_lo;
    for (; s < s_w; ++s) {
        const uint16_t* kv = s_kv + stg * STAGE;
        f32x16_t sc, s2;                                     // scores: hi part, lo part
#pragma unroll
        for (int v = 0; v < 16; ++v) { sc[v] = 0.0f; s2[v] = 0.0f; }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const abf16x8_t k = __builtin_bit_cast(abf16x8_t, kf[j]);
            s2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, ql[j], s2, 0, 0, 0);
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, qh[j], sc, 0, 0, 0);
            read_v(kv, j);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) sc[v] += s2[v];
        if (s * STEP + STEP - 1 > pw) {                      // some row of the wave does not see all tokens
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (s * STEP + 8 * (v >> 2) + 4 * h + (v & 3) > pos_col) sc[v] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, sc[v]);
        {
            const auto w2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(w2[0]), __uint_as_float(w2[1]));
        }
        // the reference m_run only moves when a score exceeds it by more than 2^6: weights stay below 2^6 (no precision is
        // lost, they are floating point) and the accumulators are rarely rescaled
        if (__any(mx > m_run + 6.0f)) {
            const float m_new = mx > m_run + 6.0f ? mx : m_run;
            const float corr = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= corr;
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[m][v] *= corr;
        }
        const float m_use = m_run == -INFINITY ? 0.0f : m_run;         // (no token of the column seen yet: all weights 0)
        float lsum = 0.0f;
        uint32_t ph[8], pl[8];                               // probabilities of tokens v = 2 i, 2 i + 1
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float a = __builtin_amdgcn_exp2f(sc[2 * i] - m_use), b = __builtin_amdgcn_exp2f(sc[2 * i + 1] - m_use);
            lsum += a + b;
            split2(a, b, ph[i], pl[i]);
        }
        l_run += lsum;                                       // (each half of the wave sums its own tokens; added up at the end)
        if (s * STEP + STEP - 1 > p_last) {                  // slots behind the last row hold whatever the pool held: zero those values
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                uint32_t mk[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = s * STEP + a * RSD_PAGE + 4 * h + (i >> 1) * 8 + (i & 1) * 2;
                    mk[i] = (t <= p_last ? 0xFFFFu : 0u) | (t + 1 <= p_last ? 0xFFFF0000u : 0u);
                }
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    vf[4 * a + m].x &= mk[0]; vf[4 * a + m].y &= mk[1]; vf[4 * a + m].z &= mk[2]; vf[4 * a + m].w &= mk[3];
                }
            }
        }
        turn(s);
        kv = s_kv + stg * STAGE;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {                       // page a, lo then hi, dims 32 m; the next step's K in between
            const int a = i >> 3, hi = (i >> 2) & 1, m = i & 3;
            const uint32_t* p = hi ? ph : pl;
            const abf16x8_t pa = __builtin_bit_cast(abf16x8_t, make_uint4(p[4 * a], p[4 * a + 1], p[4 * a + 2], p[4 * a + 3]));
            o[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(abf16x8_t, vf[4 * a + m]), pa, o[m], 0, 0, 0);
            if (i & 1) read_k(kv, i >> 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    for (; s < s_hi; ++s) turn(s);                           // (the other waves still need this one's copies)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // nothing is in flight into LDS when the block ends
    {
        const auto w2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
        l_run = __uint_as_float(w2[0]) + __uint_as_float(w2[1]);
    }
    if (!live) return;
    if (S == 1) {
        const float inv = 1.0f / l_run;
        const size_t at = (size_t)row * ldo + (hk * G + g) * HD + 4 * h;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (out) {
                    *reinterpret_cast<float4*>(out + at + 32 * m + 8 * q) =
                        make_float4(o[m][4 * q] * inv, o[m][4 * q + 1] * inv, o[m][4 * q + 2] * inv, o[m][4 * q + 3] * inv);
                    continue;
                }
                uint2 hi, lo;
                split2(o[m][4 * q] * inv, o[m][4 * q + 1] * inv, hi.x, lo.x);
                split2(o[m][4 * q + 2] * inv, o[m][4 * q + 3] * inv, hi.y, lo.y);
                *reinterpret_cast<uint2*>(out_h + at + 32 * m + 8 * q) = hi;
                *reinterpret_cast<uint2*>(out_l + at + 32 * m + 8 * q) = lo;
            }
    } else {
        const size_t pi = ((size_t)row * H + hk * G + g) * S + sp;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(part_acc + pi * HD + 32 * m + 8 * q + 4 * h) =
                    make_float4(o[m][4 * q], o[m][4 * q + 1], o[m][4 * q + 2], o[m][4 * q + 3]);
        if (h == 0) { part_ml[pi * 2] = m_run; part_ml[pi * 2 + 1] = l_run; }
    }
}
