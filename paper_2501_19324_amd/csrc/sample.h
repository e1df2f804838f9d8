// Next-token choice from a row of fp32 logits: arg max (lowest id on ties), or
// temperature / nucleus (top-p) sampling by inverse CDF from a supplied uniform.
//
// Nucleus definition implemented here: with e_t = exp(x_t - max x), x = logit /
// temperature, the nucleus S is {t : e_t >= tau} for the largest tau whose set
// still holds at least top_p of the total mass (all ties at tau included); the
// draw walks S in ascending token id and returns the first token whose running
// mass exceeds u * mass(S).
//
// No sort: tau is found by selection over the bit patterns of the non-negative floats e_t.  Masses are summed as
// 64-bit fixed point (e * 2^40), so every sum is exact, order-independent and reproducible from run to run, whatever
// the path to tau.  A row is cut into SMP_NB spans of the vocabulary; the phases are separate launches:
//   A  max of every span; clears what B and C add to.  Greedy: arg max of every span, and the block that finishes a row's last
//      span chooses among them and appends the token
//   B  histogram of masses over 1792 bins of 1/32 and 1/64 octave (exponent and five or six mantissa bits, 2^-40 .. 1); tokens so
//      light that the threshold cannot lie among them are only added up
//   C  every block finds the bin tau lies in, sums what lies above it per span and lists the keys inside it (a bin is
//      1 or 2 % wide: mostly a few hundred keys).  (B and C each have a plain form for short spans: sample_launch_spans)
//   D  one block per row resolves tau among the listed keys (10 + 9 bits), forms the nucleus mass of every span, locates
//      the draw and appends the token to its sequence.
// So the logits are read three times and everything after C works on a few hundred keys.  (Three radix levels over the
// whole row and a fifth pass for the masses, with a 2048-bin histogram cleared and flushed for every 2400 tokens, took
// 109 us on 64 rows of 151936 logits and 36 on one.)  What bounds it on many rows: in B the vector instructions (1530 a wave on 64 rows; the
// vector units are busy 46 % of the counted cycles, the start and end of the launch among them, and 17 % in A and C), in A and C the
// reading of the logits, on few rows the chain of block scans in D.  Launches of 64 rows with logits as a trained model gives them, not read before,
// A to D: 11.6 / 15.3 / 10.4 / 6.9 us (D 8.9 with block-wide searches); with a bin for every token, a full division and expf for each in B and C 11.0 / 18.3 / 17.0 / 9.3.
// A bin that may hold more keys than there is room for (nearly equal logits; the bin's mass tells in advance) makes the row
// "dense": C then adds up sub-bins of 256 keys instead of listing, and D is SMP_FB blocks, which count the keys of the deciding
// sub-bin span by span; the last of them to finish resolves tau from these counts and goes on alone.  A call on 64 rows
// of 151936 equal logits takes 115 us (1055 when the one block of D searched the row by itself, 190 with the three radix levels), on
// one row 58 (650, 57); 16 rows of a few tied values 71 (668, 67).
// top_p >= 1 needs no selection: the nucleus is every token whose mass is not zero, e >= 2^-40.
#pragma once
#include "common.h"
#include "misc.h"

constexpr int SMP_NB = 64;      // spans a row is cut into
constexpr int SMP_T = 256;      // threads per block
constexpr uint32_t SMP_UNIT = 0x2B800000u;                // key of 2^-40, the smallest e with a mass
// histogram bins of a row: 32 per octave (2^18 keys each) from 2^-40 to 2^-16, behind these (from bin SMP_FINE on) 64 per octave to 1;
// e = 1 itself joins the last one
constexpr int SMP_FINE = 768, SMP_BINS = 1792, SMP_BIN0 = (int)(SMP_UNIT >> 18);
static_assert((0x3F800000 >> 17) - 2 * SMP_BIN0 - SMP_FINE == SMP_BINS && (SMP_UNIT & 0x3FFFFu) == 0, "");
// Workspace of a row, u64 entries: the histogram, behind it the lists of keys (u32: span << 19 | key - first key of the bin), one for
// every span and one for what these have no room for.  Dense rows: sub-bins of 256 keys at the end, and, when the histogram has
// been read, counts [span][256] (u32) at the front.
constexpr int SMP_SUB = 1280;                             // sub-bins: 2^18 / 256, one for e = 1, rounded up to whole threads
constexpr int SMP_WS = SMP_NB * 256 / 2 + SMP_SUB;
constexpr int SMP_LIST = 128;                             // words of a span's list
constexpr int SMP_DENSE = (SMP_WS - SMP_BINS) * 2 - SMP_NB * SMP_LIST;   // of the shared one: a bin that may hold more keys makes the row dense
static_assert(SMP_DENSE > 0 && SMP_BINS + SMP_SUB <= SMP_WS, "");
constexpr int SMP_SEL = 9;                                // words of a row's `sel`
constexpr int SMP_FB = SMP_NB / 4;                        // blocks of phase D of a dense row: a span per wave

__device__ __forceinline__ u64_t shfl_xor_u64(u64_t v, int d) {
    const unsigned lo = __shfl_xor((unsigned)v, d, RSD_WAVE), hi = __shfl_xor((unsigned)(v >> 32), d, RSD_WAVE);
    return ((u64_t)hi << 32) | lo;
}
// Inclusive scans over the lanes in vector instructions: shifts inside the rows of 16 lanes, then the last lane of a row to the rows behind it
// (phase D on one row with shuffles 9.1 us, this way 7.7)
__device__ __forceinline__ u64_t wave_incl_scan_u64(u64_t x) {
    using std::integral_constant;
    auto add = [&](auto ctrl, auto rows) {
        constexpr int C = decltype(ctrl)::value, R = decltype(rows)::value;
        x += u64_of((uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, C, R, 0xF, false),
                    (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), C, R, 0xF, false));
    };
    add(integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});       // row_shr by 1, 2, 4, 8
    add(integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
    add(integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
    add(integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
    add(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});       // row_bcast 15 into rows 1 and 3
    add(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});       // row_bcast 31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ int wave_incl_scan(int x) {
    using std::integral_constant;
    auto add = [&](auto ctrl, auto rows) { x += __builtin_amdgcn_update_dpp(0, x, decltype(ctrl)::value, decltype(rows)::value, 0xF, false); };
    add(integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});       // row_shr by 1, 2, 4, 8
    add(integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
    add(integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
    add(integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
    add(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});       // row_bcast 15 into rows 1 and 3
    add(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});       // row_bcast 31 into rows 2 and 3
    return x;
}
// inclusive scan over the 256 threads of a block; wtot is 4 u64 of LDS
__device__ __forceinline__ u64_t block256_incl_scan_u64(u64_t v, u64_t* wtot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u64_t incl = wave_incl_scan_u64(v);
    __syncthreads();
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    u64_t base = 0;
    for (int w = 0; w < wave; ++w) base += wtot[w];
    return incl + base;
}

struct SampleArgs {
    const float* logits; int ld; int V;
    const float* u; const int* u_index; int u_stride;   // uniform of row r: u[r * u_stride + (u_index ? u_index[r] : 0)]
    float temperature, top_p;
    int sep_id; float sep_bias;                          // logit[sep_id] += sep_bias before anything else
    const int* active;                                   // nullable: rows with active[r] == 0 are skipped
    int* out;                                            // nullable when the result is appended
    // workspace, per row: pmax[SMP_NB], pidx[SMP_NB], hist[SMP_WS], psum[SMP_NB] and sel[SMP_SEL]: [0] mass the nucleus must reach, [1] mass
    // above the deciding bin, [2] that bin (-1: none), [3] keys in the shared list, [4] dense, [5] tau, [6] point of the draw, [7] blocks done,
    // [8] spans whose arg max is known: 64 more with every greedy call, zero at first
    float* pmax; int* pidx; u64_t* hist; u64_t* psum; u64_t* sel;
    // nullable: packed rows.  Row r then stands for sequence row_seq[r] (< 0: unused row); u, u_index, active and
    // the appended state are indexed by the sequence, logits, out and the workspace by the row
    const int* row_seq;
};
// the sequence of a row, or -1 when the row is unused or its sequence is not active
__device__ __forceinline__ int smp_seq(const SampleArgs& a, int row) {
    const int s = a.row_seq ? a.row_seq[row] : row;
    if (s < 0 || (a.active && !a.active[s])) return -1;
    return s;
}

// what phase D does with the chosen token besides (or instead of) storing it
struct AppendArgs {
    int enabled;                 // 0: off; 1: a token of a reasoning step; 2: a proposal of speculative regeneration
    SeqState st; int B, max_ctx, model;
    const int* forced; int sep_id, eos_id, step_cap, max_steps;
    int prop_stride;             // proposals recorded per step (mode 2): step_cap * proposals per round
};

__device__ __forceinline__ float smp_x(const SampleArgs& a, const float* lg, int i) {
    return (lg[i] + (i == a.sep_id ? a.sep_bias : 0.0f)) / a.temperature;
}
// x of U biased logits.  The division is by the same number for every token: a product with its reciprocal r (rounded to nearest) and two
// corrections give the correctly rounded quotient in five instructions instead of twelve - the first leaves an error below
// an ulp, from which the second, by Markstein's theorem, gets the rounded quotient - where nothing in between leaves the normal
// range: T within 2^-20 .. 2^20 and no |v| above 2^60 (a tiny |v| may come out a tiny bit off, which the difference to
// the maximum does not show).  Otherwise, infinities among them, it is the plain division.  (NaN, also what an infinity would
// become, has no mass.)
template <int U>
__device__ __forceinline__ void smp_divide(const float (&v)[U], float (&x)[U], float T, float r) {
    float m = 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) m = fmaxf(m, fabsf(v[u]));
    if (T >= 0x1p-20f && T <= 0x1p20f && !__any(m > 0x1p60f)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float q = v[u] * r;
            q = fmaf(fmaf(-q, T, v[u]), r, q);
            x[u] = fmaf(fmaf(-q, T, v[u]), r, q);
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = v[u] / T;
    }
}
// f(i, v) for the biased logits v[u] of tokens i + u * step of [s0, s1), `fill` past the end, i = s0 + lane + multiples of U * step.
// AHEAD: the next batch is requested before the present one is worked on (two register sets in turn: a copy would wait for the load)
template <int U, bool AHEAD, typename F>
__device__ __forceinline__ void smp_scan(const SampleArgs& a, const float* lg, int s0, int s1, int lane, int step, float fill, F f) {
    auto load = [&](float (&v)[U], int base) {
        const float* p = lg + base + lane;
        if (base + U * step <= s1) {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = p[u * step];
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = lg[min(base + lane + u * step, s1 - 1)];
        }
    };
    auto use = [&](float (&v)[U], int base) {
        if (a.sep_id >= base && a.sep_id < base + U * step) {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] += base + lane + u * step == a.sep_id ? a.sep_bias : 0.0f;
        }
        if (base + U * step > s1) {
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = base + lane + u * step < s1 ? v[u] : fill;
        }
        f(base + lane, v);
    };
    if (!AHEAD || s1 - s0 <= U * step) {
        for (int base = s0; base < s1; base += U * step) {
            float v[U];
            load(v, base);
            use(v, base);
        }
    } else {
        float p[U], q[U];
        load(p, s0);
        for (int base = s0;;) {
            load(q, base + U * step);
            use(p, base);
            if ((base += U * step) >= s1) break;
            load(p, base + U * step);
            use(q, base);
            if ((base += U * step) >= s1) break;
        }
    }
}
// exp(d) of a difference to the maximum, d <= 0: 2^n times the hardware's exponential of the rest of d log2 e, which is known to more than
// a float's digits (product, its rounding error and the low part of log2 e); n is rounded and shifted into the exponent by one
// addition each.  Below -80 (no mass; NaN as well) 2^-115.  Three instructions fewer than expf, which also looks after the ends of its range,
// and as accurate (largest relative error 8.32e-8, rms 2.10e-8 over all floats of -28 .. -1e-6 for both; they differ in five of them).
// No contraction: y stands for the rounded product in both of its places.  (Fused into y - n, the product would bring in there the
// rounding error that the other term adds: 1.4e-6 off at -28, 7e-7 at -15.)
__device__ __forceinline__ float smp_exp(float d) {
#pragma clang fp contract(off)
    const float c = fmaxf(d, -80.0f), y = 1.44269502f * c, m = y + 12582912.0f, n = m - 12582912.0f;
    const float t = (y - n) + fmaf(1.92596303e-8f, c, fmaf(1.44269502f, c, -y));
    return __uint_as_float((__float_as_uint(m) << 23) + __float_as_uint(__builtin_amdgcn_exp2f(t)));
}
__device__ __forceinline__ u64_t smp_fix(float e) { return (u64_t)(e * 1099511627776.0f); }   // e * 2^40, e in [0, 1]

__device__ __forceinline__ float smp_row_max(const SampleArgs& a, int row, float* fred) {
    float m = -INFINITY;
    if (threadIdx.x < SMP_NB) m = a.pmax[(size_t)row * SMP_NB + threadIdx.x];
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) fred[threadIdx.x >> 6] = m;
    __syncthreads();
    return fmaxf(fmaxf(fred[0], fred[1]), fmaxf(fred[2], fred[3]));
}

// The bin (searching from the top) in which the running mass first reaches thr.
// hist has n_bins = 256 * P entries; `above` is the mass above this histogram on
// entry and the mass strictly above the chosen bin on exit.  Whole block calls.
template <int P>
__device__ __forceinline__ int smp_find_bin(const u64_t* hist, u64_t thr, u64_t& above, u64_t* wtot, int* s_bin,
                                            u64_t* s_above) {
    const int tid = threadIdx.x, top = 256 * P - 1 - tid * P;   // thread t owns bins top, top-1, ..., top-P+1
    u64_t h[P], loc = 0;
#pragma unroll
    for (int j = 0; j < P; ++j) { h[j] = hist[top - j]; loc += h[j]; }
    const u64_t incl = block256_incl_scan_u64(loc, wtot);
    u64_t run = above + (incl - loc);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < P; ++j) {
        if (run < thr && run + h[j] >= thr) { *s_bin = top - j; *s_above = run; }
        run += h[j];
    }
    __syncthreads();
    above = *s_above;
    return *s_bin;
}

__device__ __forceinline__ u64_t readlane_u64(u64_t v, int lane) {
    return u64_of((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane), (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane));
}
// The same on n_bins = 64 * P bins by one wave (every wave of a block for itself: no barriers); 0 where there is no such bin
template <int P>
__device__ __forceinline__ int smp_find_bin_wave(const u64_t* hist, u64_t thr, u64_t& above) {
    const int lane = threadIdx.x & 63, top = 64 * P - 1 - lane * P;
    u64_t h[P], loc = 0;
#pragma unroll
    for (int j = 0; j < P; ++j) { h[j] = hist[top - j]; loc += h[j]; }
    u64_t run = above + (wave_incl_scan_u64(loc) - loc), at = 0;
    int bin = -1;
#pragma unroll
    for (int j = 0; j < P; ++j) {
        if (run < thr && run + h[j] >= thr) { bin = top - j; at = run; }
        run += h[j];
    }
    const u64_t hit = __ballot(bin >= 0);
    if (!hit) return 0;
    const int l = __builtin_ctzll(hit);
    above = readlane_u64(at, l);
    return __builtin_amdgcn_readlane(bin, l);
}

// bin of the key of an e with a mass
__device__ __forceinline__ int smp_bin(uint32_t key) {      // (2 i - SMP_FINE overtakes i at i = SMP_FINE)
    return min(max((int)(key >> 18) - SMP_BIN0, (int)(key >> 17) - 2 * SMP_BIN0 - SMP_FINE), SMP_BINS - 1);
}
// keys of a bin: [smp_lo, smp_hi)
__device__ __forceinline__ uint32_t smp_lo(int bin) {
    return bin < SMP_FINE ? (uint32_t)(bin + SMP_BIN0) << 18 : (uint32_t)(bin + SMP_FINE + 2 * SMP_BIN0) << 17;
}
__device__ __forceinline__ uint32_t smp_hi(int bin) { return bin == SMP_BINS - 1 ? 0x3F800001u : smp_lo(bin + 1); }
// Adds m to *p for every active lane, where lanes often agree on the key (tied logits): one addition for those that agree with
// the first
template <typename M>
__device__ __forceinline__ void smp_add_tied(M* p, uint32_t key, M m) {
    const u64_t same = __ballot(key == (uint32_t)__builtin_amdgcn_readfirstlane((int)key));
    if (!((same >> (threadIdx.x & 63)) & 1)) atomicAdd(p, m);
    else if ((int)(threadIdx.x & 63) == __builtin_ctzll(same)) atomicAdd(p, m * (M)__popcll(same));
}
// span of block blockIdx.x: with WPS = 4 waves per span the block's only one, with WPS = 1 one per wave; lane smp_lane() of
// its threads works on it
template <int WPS> __device__ __forceinline__ int smp_span() { return WPS == 4 ? blockIdx.x : blockIdx.x * 4 + (threadIdx.x >> 6); }
template <int WPS> __device__ __forceinline__ int smp_lane() { return WPS == 4 ? threadIdx.x : threadIdx.x & 63; }

// tokens a thread requests together: two batches cover a span of 2374 with 256 threads, five with 64
template <int WPS> constexpr int SMP_U = WPS == 4 ? 5 : 8;

// One thread: stores the chosen token of a row and appends it to its sequence
__device__ void smp_append(const SampleArgs& a, const AppendArgs& ap, int row, int seq, int token) {
    // a row without any finite logit (or with an infinite one) has no arg max and no member to draw: token 0, never an id outside
    // the vocabulary, which the next pass would look up in the embedding
    if (token < 0 || token >= a.V) token = 0;
    if (a.out) a.out[row] = token;
    if (!ap.enabled) return;
    // append the token and decide whether the step of this sequence goes on
    const SeqState& st = ap.st;
    const int b = seq;
    const int pos = st.ctx_len[b];
    if (ap.enabled == 2) {
        // a proposal: written behind the committed tokens and recorded as the n-th proposal of the
        // step (a place of the step can be proposed for in several rounds); the step's own length
        // and records wait for the target's decision
        const size_t rec = ((size_t)b * ap.max_steps + st.cur_step[0]) * ap.prop_stride + st.sd_nprop[b] + (pos - st.sd_base[b]);
        st.sampled[2][rec] = token;
        int tok = token;
        if (ap.forced) { const int f = ap.forced[rec]; if (f >= 0) tok = f; }
        st.tokens[(size_t)b * ap.max_ctx + pos] = tok;
        st.ctx_len[b] = pos + 1;
        st.kv_len[ap.model * ap.B + b] = pos;
        if (tok == ap.sep_id || tok == ap.eos_id || pos + 1 >= st.sd_lim[b]) {
            st.active[b] = 0;
            atomicSub(st.n_active, 1);
        }
        return;
    }
    const size_t rec = ((size_t)b * ap.max_steps + st.cur_step[0]) * ap.step_cap + st.step_len[b];
    st.sampled[ap.model][rec] = token;
    int tok = token;
    if (ap.forced) { const int f = ap.forced[rec]; if (f >= 0) tok = f; }
    st.tokens[(size_t)b * ap.max_ctx + pos] = tok;
    st.ctx_len[b] = pos + 1;
    st.kv_len[ap.model * ap.B + b] = pos;          // every token before the new one has been fed
    const int sl = st.step_len[b] + 1;
    st.step_len[b] = sl;
    if (tok == ap.sep_id || tok == ap.eos_id || sl >= ap.step_cap || pos + 1 >= ap.max_ctx) {
        st.active[b] = 0;
        atomicSub(st.n_active, 1);
    }
}

// ---- phase A: max of every span of x (sampling) or arg max of the biased logits (greedy).  x = logit / temperature
// grows with the logit, so the division is done once per span
template <int WPS, bool GREEDY>
__global__ __launch_bounds__(SMP_T) void sample_max_kernel(SampleArgs a, AppendArgs ap) {
    const int row = blockIdx.y, j = smp_span<WPS>(), tid = smp_lane<WPS>(), wave = threadIdx.x >> 6;
    const int seq = smp_seq(a, row);
    if (seq < 0) return;
    const float* lg = a.logits + (size_t)row * a.ld;
    const int span = (a.V + SMP_NB - 1) / SMP_NB, s0 = min(j * span, a.V), s1 = min(a.V, s0 + span);
    constexpr int T = WPS * 64, U = SMP_U<WPS>;
    if constexpr (!GREEDY) {                               // for phases B and C
        constexpr int NH = SMP_BINS / SMP_NB, NS = SMP_SUB / SMP_NB;
        u64_t* hist = a.hist + (size_t)row * SMP_WS;
        if (tid < NH + NS) hist[tid < NH ? j * NH + tid : SMP_WS - SMP_SUB + j * NS + tid - NH] = 0;
        if (tid == 0 && j == 0) { a.sel[(size_t)row * SMP_SEL + 3] = 0; a.sel[(size_t)row * SMP_SEL + 7] = 0; }
    }
    float bv = -INFINITY; int bi = 0x7FFFFFFF;
    for (int i0 = s0 + tid; i0 < s1; i0 += T * U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = lg[min(i0 + u * T, s1 - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + u * T, s1 - 1);
            if (i == a.sep_id) v[u] += a.sep_bias;
            if (v[u] > bv) { bv = v[u]; bi = i; }
        }
    }
    wave_argmax(bv, bi);
    if (WPS == 4) {
        __shared__ float fred[4];
        __shared__ int ired[4];
        if ((tid & 63) == 0) { fred[wave] = bv; ired[wave] = bi; }
        __syncthreads();
        if (tid == 0)
            for (int w = 1; w < 4; ++w)
                if (fred[w] > bv || (fred[w] == bv && ired[w] < bi)) { bv = fred[w]; bi = ired[w]; }
    }
    if constexpr (!GREEDY) {
        if (tid == 0) a.pmax[(size_t)row * SMP_NB + j] = bv / a.temperature;
        return;
    }
    // Greedy: the block that finishes a row's last span chooses among the spans and appends the token, instead of a launch of its
    // own (one row of 151936 logits, kernels alone: 5.8 -> 5.2 us, 6.4 -> 5.8 when the logits have not been read before; a call 10.2 -> 7.3 us,
    // the gap between the launches included).  Results go past the L2 of this XCD and have arrived before they are counted,
    // as in smp_dense.  The count only ever grows, by 64 a call, so that it needs no clearing.
    __shared__ int s_last;
    if (tid == 0) {
        __hip_atomic_store(&a.pmax[(size_t)row * SMP_NB + j], bv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.pidx[(size_t)row * SMP_NB + j], bi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        constexpr unsigned mine = WPS == 4 ? 1u : 4u;
        s_last = (__hip_atomic_fetch_add(reinterpret_cast<unsigned*>(a.sel + (size_t)row * SMP_SEL + 8), mine, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT) + mine) % SMP_NB == 0;
    }
    __syncthreads();
    if (!s_last || threadIdx.x >= SMP_NB) return;
    bv = __hip_atomic_load(&a.pmax[(size_t)row * SMP_NB + threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bi = __hip_atomic_load(&a.pidx[(size_t)row * SMP_NB + threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wave_argmax(bv, bi);
    if (threadIdx.x == 0) smp_append(a, ap, row, seq, bi);
}

// ---- phase B: the histogram of masses
template <int WPS, bool PLAIN>
__global__ __launch_bounds__(SMP_T) void sample_hist_kernel(SampleArgs a) {
    const int row = blockIdx.y, j = smp_span<WPS>(), tid = smp_lane<WPS>();
    if (smp_seq(a, row) < 0) return;
    const float* lg = a.logits + (size_t)row * a.ld;
    const int span = (a.V + SMP_NB - 1) / SMP_NB, s0 = min(j * span, a.V), s1 = min(a.V, s0 + span);
    __shared__ u64_t lh[SMP_BINS];
    __shared__ float fred[4];
    u64_t* hist = a.hist + (size_t)row * SMP_WS;
    for (int b = threadIdx.x; b < SMP_BINS; b += SMP_T) lh[b] = 0;
    const float mx = smp_row_max(a, row, fred);           // (holds a barrier)
    constexpr int T = WPS * 64, U = SMP_U<WPS>;
    // The mass reached from the top is at least top_p of a total of at least 1 (the maximum's own e), so tokens that even all together
    // have less than 1 - top_p need no bin of their own: those below `tail` are only added up, in registers (exactly: less than
    // 2^28 + 2^26 units a lane) and at the end in the lowest bin.  For 151936 tokens and 0.95 that is e < 2^-22: nearly all of them
    const float rest = 0.99f * (1.0f - a.top_p) / (float)a.V;
    const uint32_t tail = min(max(__float_as_uint(rest) & 0x7F800000u, SMP_UNIT), 0x38800000u);      // (2^-14)
    uint32_t low = 0;
    auto add = [&](uint32_t key) { atomicAdd(&lh[smp_bin(key)], smp_fix(__uint_as_float(key))); };
    if constexpr (PLAIN) {
        for (int i0 = s0 + tid; i0 < s1; i0 += T * U) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = smp_x(a, lg, min(i0 + u * T, s1 - 1));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u * T >= s1) continue;
                const float e = smp_exp(x[u] - mx);
                if (__float_as_uint(e) >= tail) add(__float_as_uint(e));
                else low += (uint32_t)(e * 1099511627776.0f);
            }
        }
    } else {
        // the others are few, then, in most waves: a batch's are listed, without a branch (lanes with nothing to list write to a slot
        // nobody reads), and added to the histogram 64 at a time; where half of a batch is above the tail, at once
        // (few rows are bound by latency, which the sum over the lanes adds to: there, and where there is no tail, all are added at once)
        const float rT = 1.0f / a.temperature;
        constexpr int LIST = WPS == 1 ? 64 + 32 * U : 0;
        const bool lists = WPS == 1 && tail > SMP_UNIT;
        __shared__ uint32_t s_list[4][LIST + 64];
        uint32_t* list = s_list[threadIdx.x >> 6];
        const int lane = threadIdx.x & 63;
        int n = 0;
        // the list is exchanged between the lanes of a wave, whose LDS operations stay in order: this keeps the compiler's (no instruction)
        auto order = [] {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        smp_scan<U, false>(a, lg, s0, s1, tid, T, __builtin_nanf(""), [&](int i, const float (&v)[U]) {
            if (s1 - (i - tid) <= U / 2 * T) {                  // (a short end: only what is there, as it comes)
#pragma unroll
                for (int u = 0; u < U / 2; ++u) {
                    if (s1 - (i - tid) <= u * T) break;
                    const uint32_t key = __float_as_uint(smp_exp(v[u] / a.temperature - mx));
                    low += key >= tail ? 0u : (uint32_t)(__uint_as_float(key) * 1099511627776.0f);
                    if (key >= tail) add(key);
                }
                return;
            }
            float x[U];
            uint32_t key[U];
            int above = 0;
            smp_divide<U>(v, x, a.temperature, rT);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float e = smp_exp(x[u] - mx);
                key[u] = __float_as_uint(e);
                above += key[u] >= tail;
                low += key[u] >= tail ? 0u : (uint32_t)(e * 1099511627776.0f);
            }
            if (!lists) {
#pragma unroll
                for (int u = 0; u < U; ++u) if (key[u] >= tail) add(key[u]);
                return;
            }
            int at = wave_incl_scan(above);
            const int k = __builtin_amdgcn_readlane(at, 63);
            if (k == 0) return;
            if (k > 32 * U) {
#pragma unroll
                for (int u = 0; u < U; ++u) if (key[u] >= tail) add(key[u]);
                return;
            }
            at += n - above;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = key[u] >= tail;
                list[in ? at : LIST + lane] = key[u];
                at += in;
            }
            n += k;
            order();                                           // other lanes' entries are read below ...
            while (n >= 64) {
                n -= 64;
                add(list[n + lane]);
            }
            order();                                           // ... and written over by the next batch
        });
        if (lists && lane < n) add(list[lane]);
    }
    // (eight lanes at a time: less than 2^32)
    auto dpp = [](uint32_t x, auto ctrl) { return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xF, 0xF, true); };
    low = dpp(low, std::integral_constant<int, 0xB1>{});       // quad_perm [1,0,3,2]
    low = dpp(low, std::integral_constant<int, 0x4E>{});       // quad_perm [2,3,0,1]
    low = dpp(low, std::integral_constant<int, 0x141>{});      // row_half_mirror
    if ((threadIdx.x & 7) == 0 && low) atomicAdd(&lh[0], (u64_t)low);
    __syncthreads();
    for (int b = threadIdx.x; b < SMP_BINS; b += SMP_T)
        if (lh[b]) atomicAdd(&hist[b], lh[b]);
}

// ---- phase C: the bin in which the mass reaches top_p of the total; per span the mass above it, and the keys inside it (dense
// rows: their masses by sub-bin)
template <int WPS, bool PLAIN>
__global__ __launch_bounds__(SMP_T) void sample_select_kernel(SampleArgs a) {
    const int row = blockIdx.y, j = smp_span<WPS>(), tid = smp_lane<WPS>(), wave = threadIdx.x >> 6;
    if (smp_seq(a, row) < 0) return;
    const float* lg = a.logits + (size_t)row * a.ld;
    const int span = (a.V + SMP_NB - 1) / SMP_NB, s0 = min(j * span, a.V), s1 = min(a.V, s0 + span);
    __shared__ u64_t lds[SMP_SUB];                        // dense rows: the sub-bins
    __shared__ u64_t wtot[4];
    __shared__ float fred[4];
    __shared__ int s_bin, s_cnt[4];
    __shared__ u64_t s_above, s_mass;
    u64_t* hist = a.hist + (size_t)row * SMP_WS;
    u64_t* sel = a.sel + (size_t)row * SMP_SEL;
    const float mx = smp_row_max(a, row, fred);
    if (threadIdx.x == 0) { s_bin = 0; s_above = 0; s_mass = 0; }
    if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0;
    // (every block repeats the deterministic search)
    constexpr int P = SMP_BINS / SMP_T;
    const int top = SMP_BINS - 1 - threadIdx.x * P;       // this thread's bins: top, top - 1, ...
    u64_t h[P], loc = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) { h[i] = hist[top - i]; loc += h[i]; }
    const u64_t incl = block256_incl_scan_u64(loc, wtot);
    const u64_t z = wtot[0] + wtot[1] + wtot[2] + wtot[3];
    u64_t thr = (u64_t)ceil((double)a.top_p * (double)z);
    if (thr < 1) thr = 1;
    if (thr > z) thr = z;
    u64_t run = incl - loc;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        if (run < thr && run + h[i] >= thr) { s_bin = top - i; s_above = run; s_mass = h[i]; }
        run += h[i];
    }
    __syncthreads();
    const int bin = thr == z ? -1 : s_bin;                // -1: the nucleus is every token with a mass
    // keys below lo are outside, from hi on inside the nucleus; those between are listed
    const uint32_t lo = bin < 0 ? SMP_UNIT : smp_lo(bin), hi = bin < 0 ? SMP_UNIT : smp_hi(bin);
    // no key of the bin has less than the mass of lo, which bounds their number: those of a row that is not dense fit the shared list
    const bool dense = bin >= 0 && s_mass > SMP_DENSE * smp_fix(__uint_as_float(lo));
    if (blockIdx.x == 0 && threadIdx.x == 0) { sel[0] = thr; sel[1] = s_above; sel[2] = (u64_t)(long long)bin; sel[4] = dense; }
    if (dense) {
        for (int b = threadIdx.x; b < SMP_SUB; b += SMP_T) lds[b] = 0;
        __syncthreads();
    }
    // A logit below cut is outside for certain: the margin is far above the rounding of quotient, difference, exponential and of cut
    // itself.  Most tokens are (a nucleus of top_p 0.95 is some hundred of 151936), so that a wave seldom has to form one's key.
    // (Not a number, from an infinite maximum: nothing is below it.)
    const float x_lo = mx + __logf(__uint_as_float(lo)), cut = (x_lo - (1e-3f + 1e-5f * (fabsf(mx) + fabsf(x_lo)))) * a.temperature;
    uint32_t* lists = reinterpret_cast<uint32_t*>(hist + SMP_BINS);
    uint32_t* list = lists + j * SMP_LIST;
    int* cnt = &s_cnt[WPS == 4 ? 0 : wave];
    u64_t acc = 0;
    constexpr int T = WPS * 64, U = WPS == 4 ? SMP_U<4> : 6;        // (eight spill)
    auto scan = [&](auto inside) {
        auto take = [&](float x) {
            const float e = smp_exp(x - mx);
            const uint32_t key = __float_as_uint(e);
            if (key >= hi) acc += smp_fix(e);
            else if (key >= lo) inside(key);
        };
        if constexpr (PLAIN) {
            for (int i0 = s0 + tid; i0 < s1; i0 += T * U) {
                float x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = smp_x(a, lg, min(i0 + u * T, s1 - 1));
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (i0 + u * T < s1) take(x[u]);
            }
        } else {
            smp_scan<U, true>(a, lg, s0, s1, tid, T, -INFINITY, [&](int, const float (&v)[U]) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (__any(!(v[u] < cut))) take(v[u] / a.temperature);
            });
        }
    };
    if (dense)
        scan([&](uint32_t key) { smp_add_tied(&lds[(key - lo) >> 8], key, smp_fix(__uint_as_float(key))); });
    else
        scan([&](uint32_t key) {
            const uint32_t w = ((uint32_t)j << 19) | (key - lo);
            const int at = atomicAdd(cnt, 1);
            if (at < SMP_LIST) list[at] = w;
            else lists[SMP_NB * SMP_LIST + atomicAdd(reinterpret_cast<unsigned*>(sel + 3), 1u)] = w;
        });
    acc = wave_sum_u64(acc);
    __syncthreads();
    if (dense) {                                          // (the masses of the spans are added up in phase D)
        for (int b = threadIdx.x; b < SMP_SUB; b += SMP_T)
            if (lds[b]) atomicAdd(&hist[SMP_WS - SMP_SUB + b], lds[b]);
        return;
    }
    if (WPS == 4) {
        if ((tid & 63) == 0) wtot[wave] = acc;
        __syncthreads();
        acc = wtot[0] + wtot[1] + wtot[2] + wtot[3];
    }
    if (tid == 0) {
        a.psum[(size_t)row * SMP_NB + j] = acc;
        a.pidx[(size_t)row * SMP_NB + j] = min(*cnt, SMP_LIST);
    }
}

// First part of phase D of a dense row, SMP_FB blocks: every wave counts the keys of the deciding sub-bin in its span and adds up
// what lies above.  Returns true in the block that is the last to finish, which then holds tau and the mass of every span
// (s_mass).  Whole block calls; lh: 512 entries of LDS, s_flag: one int
__device__ bool smp_dense(const SampleArgs& a, int row, float mx, u64_t* lh, u64_t* wtot, int* s_flag, u64_t* s_above, u64_t* s_mass, uint32_t& tau) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* lg = a.logits + (size_t)row * a.ld;
    u64_t* hist = a.hist + (size_t)row * SMP_WS;
    u64_t* sel = a.sel + (size_t)row * SMP_SEL;
    u64_t* counts = hist;                                  // [span][128]: two keys each
    const u64_t thr = sel[0];
    u64_t run = sel[1];
    if (tid == 0) { *s_flag = 0; *s_above = run; }
    const int sub = smp_find_bin<SMP_SUB / SMP_T>(hist + SMP_WS - SMP_SUB, thr, run, wtot, s_flag, s_above);
    const uint32_t lo = smp_lo((int)(long long)sel[2]) + ((uint32_t)sub << 8), hi = lo + 256;
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lh) + wave * 256;
#pragma unroll
    for (int i = 0; i < 4; ++i) cnt[lane + 64 * i] = 0;
    __syncthreads();                                       // (also: s_flag has been read)
    const int span = (a.V + SMP_NB - 1) / SMP_NB, j = blockIdx.y * 4 + wave, s0 = min(j * span, a.V), s1 = min(a.V, s0 + span);
    u64_t acc = 0;
    for (int i0 = s0; i0 < s1; i0 += 64 * 8) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = smp_x(a, lg, min(i0 + lane + u * 64, s1 - 1));
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float e = smp_exp(x[u] - mx);
            const uint32_t key = __float_as_uint(e);
            if (i0 + lane + u * 64 < s1) {
                if (key >= hi) acc += smp_fix(e);
                else if (key >= lo) smp_add_tied(&cnt[key - lo], key, 1u);
            }
        }
    }
    acc = wave_sum_u64(acc);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // Counts and masses go past the L2 of this XCD (agent-scope stores), each wave waits until its own have arrived and the
    // barrier until all have, so the block that then finds itself the last one may read everybody's, past its L2 too.  (Fences
    // at device scope write back and invalidate the whole L2 of the XCD: 110 us for this kernel on 64 rows.)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int v = lane + 64 * i;
        __hip_atomic_store(&counts[j * 128 + v], ((u64_t)cnt[v * 2 + 1] << 32) | cnt[v * 2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) __hip_atomic_store(&a.psum[(size_t)row * SMP_NB + j], acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) *s_flag = __hip_atomic_fetch_add(reinterpret_cast<unsigned*>(sel + 7), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == SMP_FB - 1;
    __syncthreads();
    if (!*s_flag) return false;
    auto from_all = [](const u64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // key lo + v stands for (number of them) x (its mass); every thread adds up 32 of the 64 spans of two keys
    lh[tid] = 0;
    if (tid < SMP_NB) s_mass[tid] = from_all(&a.psum[(size_t)row * SMP_NB + tid]);
    auto mass = [&](int v, u64_t c) { return c * smp_fix(__uint_as_float(lo + v)); };
    __syncthreads();
    const int pair = tid & 127;
    u64_t c0 = 0, c1 = 0;
#pragma unroll
    for (int q = 0; q < SMP_NB / 2; ++q) {
        const u64_t c = from_all(&counts[(2 * q + (tid >> 7)) * 128 + pair]);
        c0 += (uint32_t)c; c1 += c >> 32;
    }
    if (c0) atomicAdd(&lh[pair * 2], mass(pair * 2, c0));
    if (c1) atomicAdd(&lh[pair * 2 + 1], mass(pair * 2 + 1, c1));
    if (tid == 0) { *s_flag = 0; *s_above = run; }
    __syncthreads();
    const int low = smp_find_bin<1>(lh, thr, run, wtot, s_flag, s_above);
    tau = lo + low;
    u64_t m = 0;                                           // four threads per span
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const int v = 2 * (4 * q + (tid & 3));
        const u64_t c = from_all(&counts[(tid >> 2) * 128 + v / 2]);
        if (v >= low) m += mass(v, (uint32_t)c);
        if (v + 1 >= low) m += mass(v + 1, c >> 32);
    }
    m += shfl_xor_u64(m, 1);
    m += shfl_xor_u64(m, 2);
    if ((tid & 3) == 0) s_mass[tid >> 2] += m;
    return true;
}

// ---- phase D: one block per row (dense rows: SMP_FB of which one goes on): tau, the nucleus mass of every span, the token;
// appends it
__global__ __launch_bounds__(SMP_T) void sample_finish_kernel(SampleArgs a, AppendArgs ap) {
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int seq = smp_seq(a, row);
    if (seq < 0) return;
    __shared__ u64_t wtot[4];
    __shared__ float fred[4];
    __shared__ int s_tok, s_bin;
    __shared__ u64_t s_above;
    int token;
    {
        u64_t* sel = a.sel + (size_t)row * SMP_SEL;
        const float* lg = a.logits + (size_t)row * a.ld;
        const u64_t* hist = a.hist + (size_t)row * SMP_WS;
        __shared__ u64_t lh[768 + 512];
        __shared__ u64_t s_mass[SMP_NB];
        // what a row that is not dense needs is requested together with the word that says so: four threads per span hold the keys
        // of its list; the first 16 (mostly all) are kept
        constexpr int NK = 4;
        const uint32_t* lists = reinterpret_cast<const uint32_t*>(hist + SMP_BINS);
        const uint32_t* list = lists + (tid >> 2) * SMP_LIST;
        int n_list = 0;
        uint32_t kept[NK];
        u64_t mass_above = 0;
        if (blockIdx.y == 0) {
            n_list = a.pidx[(size_t)row * SMP_NB + (tid >> 2)];
#pragma unroll
            for (int i = 0; i < NK; ++i) kept[i] = list[(tid & 3) + 4 * i];
            mass_above = a.psum[(size_t)row * SMP_NB + (tid & (SMP_NB - 1))];
        }
        const u64_t thr = sel[0], above = sel[1];
        const int bin = (int)(long long)sel[2], n_over = (int)sel[3];
        const bool dense = sel[4] != 0;
        if (!dense && blockIdx.y > 0) return;
        const float uu = a.u[(size_t)seq * a.u_stride + (a.u_index ? a.u_index[seq] : 0)];
        const int span = (a.V + SMP_NB - 1) / SMP_NB;
        uint32_t tau = SMP_UNIT;
        float mx;
        if (dense) {
            mx = smp_row_max(a, row, fred);
            if (!smp_dense(a, row, mx, lh, wtot, &s_bin, &s_above, s_mass, tau)) return;
        } else {
            auto rest = [&](const uint32_t* p, int i0, int step, int n, auto f) {
                for (; i0 < n; i0 += step * NK) {
                    uint32_t w[NK];
#pragma unroll
                    for (int i = 0; i < NK; ++i) w[i] = p[min(i0 + step * i, n - 1)];
#pragma unroll
                    for (int i = 0; i < NK; ++i) if (i0 + step * i < n) f(w[i]);
                }
            };
            auto each_key = [&](auto f) {
#pragma unroll
                for (int i = 0; i < NK; ++i) if ((tid & 3) + 4 * i < n_list) f(kept[i]);
                rest(list, (tid & 3) + 4 * NK, 4, n_list, f);
                rest(lists + SMP_NB * SMP_LIST, tid, SMP_T, n_over, f);
            };
            if (tid < SMP_NB) s_mass[tid] = mass_above;
            for (int b = tid; b < 768 + 512; b += SMP_T) lh[b] = 0;
            mx = smp_row_max(a, row, fred);                // (holds a barrier)
            if (bin >= 0) {
                const uint32_t lo = smp_lo(bin);
                auto off = [](uint32_t w) { return w & 0x7FFFFu; };
                auto mass = [&](uint32_t w) { return smp_fix(__uint_as_float(lo + off(w))); };
                u64_t run = above;
                // bits 9..18, then 0..8 of the keys' distance from the bin's first
                each_key([&](uint32_t w) { atomicAdd(&lh[off(w) >> 9], mass(w)); });
                __syncthreads();
                const uint32_t up = (uint32_t)smp_find_bin_wave<12>(lh, thr, run);
                each_key([&](uint32_t w) { if (off(w) >> 9 == up) atomicAdd(&lh[768 + (off(w) & 0x1FFu)], mass(w)); });
                __syncthreads();
                const uint32_t rel = (up << 9) | (uint32_t)smp_find_bin_wave<8>(lh + 768, thr, run);
                tau = lo + rel;
                each_key([&](uint32_t w) { if (off(w) >= rel) atomicAdd(&s_mass[w >> 19], mass(w)); });
            }
        }
        if (tid == 0) s_tok = -1;
        __syncthreads();
        // (every wave finds the span for itself)
        const u64_t pv = s_mass[lane], pincl = wave_incl_scan_u64(pv), zs = readlane_u64(pincl, 63);
        const u64_t target = (u64_t)floor((double)uu * (double)zs);      // running > u * Z  <=>  running > floor(u * Z)
        if (wave == 0) a.psum[(size_t)row * SMP_NB + lane] = pv;
        if (tid == 0) { sel[5] = tau; sel[6] = target; }
        // if rounding of u * Z left no crossing, the draw is the last member: of the last span with a mass
        u64_t at = __ballot(pincl > target && pincl - pv <= target);
        if (!at) at = __ballot(pv != 0);
        const int blk = at ? 63 - __builtin_clzll(at) : 0;
        const u64_t base = at ? readlane_u64(pincl - pv, blk) : 0;
        // every thread takes a run of consecutive tokens of the span; the one whose run holds the crossing walks it
        const int s0 = min(blk * span, a.V), s1 = min(a.V, s0 + span);
        const int per = (s1 - s0 + SMP_T - 1) / SMP_T, t0 = min(s1, s0 + tid * per), t1 = min(s1, t0 + per);
        u64_t mine = 0;
        int last_member = -1;
        constexpr int NB = 10;                                 // (spans of 2374: one batch, which is kept)
        float kept_e[NB];
        for (int i0 = t0; i0 < t1; i0 += NB) {
            float x[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) x[u] = smp_x(a, lg, min(i0 + u, t1 - 1));
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                const float e = smp_exp(x[u] - mx);
                const bool in = i0 + u < t1 && __float_as_uint(e) >= tau;
                kept_e[u] = in ? e : 0.0f;
                if (in) { mine += smp_fix(e); last_member = i0 + u; }
            }
        }
        const u64_t incl = base + block256_incl_scan_u64(mine, wtot);
        if (mine && incl > target && incl - mine <= target) {
            u64_t run = incl - mine;
            if (per <= NB) {
                int tok = -1;
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    run += smp_fix(kept_e[u]);
                    if (tok < 0 && run > target) tok = t0 + u;
                }
                s_tok = tok;
            } else {
                for (int i = t0; i < t1; ++i) {
                    const float e = smp_exp(smp_x(a, lg, i) - mx);
                    if (__float_as_uint(e) >= tau) { run += smp_fix(e); if (run > target) { s_tok = i; break; } }
                }
            }
        }
        __syncthreads();
        if (s_tok < 0) {
            // no crossing (u * Z rounded up to the full mass): the last member of the nucleus
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) last_member = max(last_member, __shfl_xor(last_member, off, RSD_WAVE));
            __shared__ int lred[4];
            if (lane == 0) lred[wave] = last_member;
            __syncthreads();
            if (tid == 0) s_tok = max(max(lred[0], lred[1]), max(lred[2], lred[3]));
            __syncthreads();
        }
        token = s_tok;
    }
    if (tid == 0) smp_append(a, ap, row, seq, token);
}

// Few rows of a large vocabulary: a span per block of four waves, to have many blocks.  Otherwise a span per wave: a block then works
// on four spans, which spreads the cost of its histogram (clearing and flushing 1792 bins) over four times as many tokens.  The
// line: us of the four launches, span per block / per wave: 151936 tokens, 16 rows 32.7 / 33.8, 24 rows 38.1 / 36.8; 100000, 8 rows 25.5 /
// 28.2, 15 rows 31.2 / 29.4; 50257, 4 rows 20.9 / 21.9, 8 rows 22.9 / 22.6; 32000, 1 row 19.0 / 19.4, 4 rows 20.4 / 19.6; 16384, 1 row
// 18.5 / 18.3, 15 rows 24.9 / 20.1.
// Short spans take plain passes over the tokens, without the steps that only pay where a wave has many: a histogram pass of up to two
// batches without lists and the division by reciprocal, a selection of up to 1280 tokens without skipping.  64 rows of 32000, a third
// of the tokens not masked: 28.0 us, 30.3 with the long spans' passes (27.8 before there were such passes); 16 rows 21.4, 22.3 (21.2); 64
// rows of 1000 normal logits 21.1, 22.4 (23.4); the logits of a trained model, 17 rows of 151936: 28.3, 28.4 (33.1); 64 of 32000: 25.2, 26.1 (27.9).
template <int WPS>
static void sample_launch_spans(hipStream_t st, const SampleArgs& a, const AppendArgs& ap, int rows) {
    const dim3 grid(SMP_NB * WPS / 4, rows), block(SMP_T);
    if (a.temperature == 0.0f) {
        hipLaunchKernelGGL((sample_max_kernel<WPS, true>), grid, block, 0, st, a, ap);
        return;
    }
    const int span = (a.V + SMP_NB - 1) / SMP_NB;
    hipLaunchKernelGGL((sample_max_kernel<WPS, false>), grid, block, 0, st, a, ap);
    if (span <= 2 * SMP_U<WPS> * WPS * 64) hipLaunchKernelGGL((sample_hist_kernel<WPS, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((sample_hist_kernel<WPS, false>), grid, block, 0, st, a);
    if (span <= 1280) hipLaunchKernelGGL((sample_select_kernel<WPS, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((sample_select_kernel<WPS, false>), grid, block, 0, st, a);
}
static void sample_launch(hipStream_t st, const SampleArgs& a, const AppendArgs& ap, int rows) {
    if (rows * 8192LL < a.V) sample_launch_spans<4>(st, a, ap, rows);
    else sample_launch_spans<1>(st, a, ap, rows);
    if (a.temperature != 0.0f) hipLaunchKernelGGL(sample_finish_kernel, dim3(rows, SMP_FB), dim3(SMP_T), 0, st, a, ap);
}
