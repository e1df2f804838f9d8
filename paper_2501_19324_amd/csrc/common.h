// Shared device helpers: bf16 storage type, 8-element loads, wave reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#define RSD_WAVE 64

struct bf16_t { uint16_t v; };

__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// fp32 -> bf16, round to nearest even: one conversion instruction for two values, with the results of the integer form
// (u + 0x7FFF + bit 16) >> 16 for every number and infinity.  That form was 10 of the 30 vector instructions per value of the SwiGLU
// epilogue of the many-row products.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f2bf2(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t)); }
// a, b as hi + lo bf16 pairs
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& lo) {
    hi = f2bf2(a, b);
    lo = f2bf2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u));
}

__device__ __forceinline__ void load8(const float* __restrict__ p, float o[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}

__device__ __forceinline__ void unpack8(const uint4 r, float o[8]) {
    o[0] = __uint_as_float(r.x << 16); o[1] = __uint_as_float(r.x & 0xFFFF0000u);
    o[2] = __uint_as_float(r.y << 16); o[3] = __uint_as_float(r.y & 0xFFFF0000u);
    o[4] = __uint_as_float(r.z << 16); o[5] = __uint_as_float(r.z & 0xFFFF0000u);
    o[6] = __uint_as_float(r.w << 16); o[7] = __uint_as_float(r.w & 0xFFFF0000u);
}

__device__ __forceinline__ void load8(const bf16_t* __restrict__ p, float o[8]) {
    unpack8(*reinterpret_cast<const uint4*>(p), o);
}

__device__ __forceinline__ float ld1(const float* p) { return *p; }
__device__ __forceinline__ float ld1(const bf16_t* p) { return bf2f(p->v); }
__device__ __forceinline__ void st1(float* p, float v) { *p = v; }
__device__ __forceinline__ void st1(bf16_t* p, float v) { p->v = f2bf(v); }

// ---- Reductions over a wave by cross-lane register moves.  A shuffle (ds_bpermute) is a trip through the LDS, and the six of a
// reduction wait for one another, in launches of 4 to 10 us: the tiny target's MLP launch 4.7 -> 3.8, a token of the 1.5B model 1.06 -> 1.04 ms.
// All 64 lanes must be active; every lane gets the result.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_move(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
// f(ctrl) for the four moves that bring together the 16 lanes of a row: quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror
template <typename F> __device__ __forceinline__ void row16_moves(F f) {
    f(std::integral_constant<int, 0xB1>{});
    f(std::integral_constant<int, 0x4E>{});
    f(std::integral_constant<int, 0x141>{});
    f(std::integral_constant<int, 0x140>{});
}
// Lanes 32, 16, 8, 4, 2, 1 apart in turn, the order of wave_sums (gemv.h): a bf16 cache entry near the middle between two numbers is
// rounded one way or the other with the last bit of a sum, so the order is part of the result and does not depend on how lanes exchange.
// (After the steps over 32, 16 and 8 lanes a value repeats every 8 lanes: the rotation by 4 brings the lane 4 apart.)
__device__ __forceinline__ float wave_sum(float v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    v += __uint_as_float(dpp_move<0x128>(__float_as_uint(v)));       // row_ror by 8
    v += __uint_as_float(dpp_move<0x124>(__float_as_uint(v)));       // row_ror by 4
    v += __uint_as_float(dpp_move<0x4E>(__float_as_uint(v)));        // quad_perm [2,3,0,1]
    v += __uint_as_float(dpp_move<0xB1>(__float_as_uint(v)));        // quad_perm [1,0,3,2]
    return v;
}
// Neighbours first: the order gemv_flat_kernel has
__device__ __forceinline__ float wave_sum_near(float v) {
    row16_moves([&](auto c) { v += __uint_as_float(dpp_move<decltype(c)::value>(__float_as_uint(v))); });
    const int bits = __float_as_int(v);                     // each row of 16 lanes holds its sum
    return (__int_as_float(__builtin_amdgcn_readlane(bits, 0)) + __int_as_float(__builtin_amdgcn_readlane(bits, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(bits, 32)) + __int_as_float(__builtin_amdgcn_readlane(bits, 48)));
}

// Reductions over the four 16-lane rows of a wave (lanes l, l+16, l+32, l+48), register moves only:
// a swap of odd/even rows, then of the two wave halves.  Every lane gets the result.
__device__ __forceinline__ float rows4_max(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows4_sum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ float wave_max(float v) {
    row16_moves([&](auto c) { v = fmaxf(v, __uint_as_float(dpp_move<decltype(c)::value>(__float_as_uint(v)))); });
    return rows4_max(v);
}
// arg max: the largest value, on ties the lowest index.  wave_argmax_rows: lanes that agree within the 16-lane rows already
__device__ __forceinline__ void take_better(float& v, int& i, float ov, int oi) { if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; } }
__device__ __forceinline__ void wave_argmax_rows(float& v, int& i) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const auto b = __builtin_amdgcn_permlane16_swap((uint32_t)i, (uint32_t)i, false, false);
    v = __uint_as_float(a[0]); i = (int)b[0];
    take_better(v, i, __uint_as_float(a[1]), (int)b[1]);
    const auto c = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const auto d = __builtin_amdgcn_permlane32_swap((uint32_t)i, (uint32_t)i, false, false);
    v = __uint_as_float(c[0]); i = (int)d[0];
    take_better(v, i, __uint_as_float(c[1]), (int)d[1]);
}
__device__ __forceinline__ void wave_argmax(float& v, int& i) {
    row16_moves([&](auto c) {
        constexpr int C = decltype(c)::value;
        const float ov = __uint_as_float(dpp_move<C>(__float_as_uint(v)));
        take_better(v, i, ov, (int)dpp_move<C>((uint32_t)i));
    });
    wave_argmax_rows(v, i);
}
// 64-bit sums
typedef unsigned long long u64_t;
__device__ __forceinline__ u64_t u64_of(uint32_t lo, uint32_t hi) { return ((u64_t)hi << 32) | lo; }
__device__ __forceinline__ u64_t wave_sum_u64(u64_t v) {
    row16_moves([&](auto c) {
        constexpr int C = decltype(c)::value;
        v += u64_of(dpp_move<C>((uint32_t)v), dpp_move<C>((uint32_t)(v >> 32)));
    });
    u64_t s = 0;
#pragma unroll
    for (int r = 0; r < 64; r += 16)
        s += u64_of((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, r), (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), r));
    return s;
}

// Sum over a 256-thread block; `red` is 4 floats of LDS. All threads get the result.
__device__ __forceinline__ float block256_sum(float v, float* red) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}

// Row descriptor shared by the per-row kernels.  Chunked prefill passes give
// explicit (sequence, position) arrays; single-token decode passes leave them
// null: row r is sequence r, fed at position kv_len[r], skipped when inactive.
// Which sequence and which position a row of a pass stands for.
//   chunked pass:   row_seq[r], row_pos[r] (every row is in use)
//   decode, dense:  row r is sequence r at position kv_len[r], in use while active[r]
//   decode, packed: row r is sequence row_seq[r] (< 0: unused row) at kv_len[seq], in use while active[seq]
struct RowMap {
    const int* row_seq;
    const int* row_pos;
    const int* kv_len;
    const int* active;
};
__device__ __forceinline__ bool row_lookup(const RowMap& rm, int r, int& seq, int& pos) {
    if (rm.row_seq) {
        seq = rm.row_seq[r];
        if (rm.row_pos) { pos = rm.row_pos[r]; return true; }
        if (seq < 0) return false;
        pos = rm.kv_len[seq];
        return rm.active[seq] != 0;
    }
    seq = r; pos = rm.kv_len[r];
    return rm.active[r] != 0;
}
